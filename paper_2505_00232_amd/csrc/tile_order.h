// In which order the product kernels walk over their tiles (also compiled for the host, by a test).
#pragma once

namespace qfc {

// Tile of workgroup `b` of a product, in an order whose neighbours run on one XCD (workgroups are dealt to the 8
// XCDs round robin, each with its own L2): XCD x takes the x-th eighth of the tiles, the first total % 8
// XCDs one more, channel tile by channel tile or (by_tokens) token tile by token tile, in bands of kBand tiles of the other operand.
// (Tile counts that 8 does not divide: int8 x int8, 9216 x 4096 at 400 rows 46.7 us in launch order, 27.3 like
// this; 4352 x 4096 at 900 rows 31.3 / 21.3; int8 x int4 9472 x 4096 at 400 rows 34.7 / 27.6; the fp16 kernels are level.)
// Bands: an XCD works on 32 or 64 tiles at a time, and what they read of both operands together has to come through its L2 of 4 MB.  Walking all
// token tiles of a channel tile, 64 tiles in flight share one or two channel tiles and no token tile; in bands of eight they are eight by
// eight.  us, before / in bands: int4 codes, binary16, 28672 x 4096 6000 rows 1043 / 990, 18432 x 2304 (groups) 4096 rows 298 / 281; int8 14336 x 4096 4096 rows 390 / 375;
// int8 activations 28672 x 4096 int8 4096 rows 428 / 406, int4 381 / 355; 4096 x 14336 6000 rows 340 / 325.  Up to 1000 rows level; the worst 2304 x 9216 int8
// activations 4096 rows 118 / 122, 18432 x 512 1308 rows 30.0 / 30.7.
constexpr int kBand = 8;
__host__ __device__ __forceinline__ void banded_tile(int i, int inner, int outer, int &o, int &r) {
    const int band = i / (kBand * outer), first = band * kBand, j = i - first * outer, width = inner - first < kBand ? inner - first : kBand;
    o = j / width, r = first + j % width;
}
__host__ __device__ __forceinline__ void xcd_tile(int b, int n_tiles, int m_tiles, int by_tokens, int &nt, int &mt) {
    const int total = n_tiles * m_tiles, xcd = b % 8;
    const int i = xcd * (total / 8) + (xcd < total % 8 ? xcd : total % 8) + b / 8;
    int o, r;
    banded_tile(i, by_tokens ? n_tiles : m_tiles, by_tokens ? m_tiles : n_tiles, o, r);
    nt = by_tokens ? r : o;
    mt = by_tokens ? o : r;
}
// The order for which an XCD pulls fewer bytes: its eighth of the tiles covers a band of one operand (several, if it is more than one) and
// tiles of the other.  (w_bytes, x_bytes: of a channel tile and of a token tile, per k.)
inline int walk_by_tokens(int n_tiles, int m_tiles, float w_bytes, float x_bytes) {
    const int share = (n_tiles * m_tiles + 7) / 8;
    auto covered = [&](int inner, int outer, float inner_bytes, float outer_bytes) {
        const int width = inner < kBand ? inner : kBand, bands = (share + width * outer - 1) / (width * outer);
        const int across = bands > 1 ? outer : (share + width - 1) / width;
        return (float)(bands * width < inner ? bands * width : inner) * inner_bytes + (float)(bands * across) * outer_bytes;
    };
    return covered(n_tiles, m_tiles, w_bytes, x_bytes) < covered(m_tiles, n_tiles, x_bytes, w_bytes) ? 1 : 0;
}

}  // namespace qfc
