// In which order the product kernels walk over their tiles (also compiled for the host, by a test).
#pragma once

namespace qfc {

// Tile of workgroup `b` of a product, in an order whose neighbours run on one XCD (workgroups are dealt to the 8
// XCDs round robin, each with its own L2): XCD x takes the x-th eighth of the tiles, the first total % 8
// XCDs one more, channel tile by channel tile or (by_tokens) token tile by token tile, in bands of tiles of the other operand.
// (Tile counts that 8 does not divide: int8 x int8, 9216 x 4096 at 400 rows 46.7 us in launch order, 27.3 like
// this; 4352 x 4096 at 900 rows 31.3 / 21.3; int8 x int4 9472 x 4096 at 400 rows 34.7 / 27.6; the fp16 kernels are level.)
// Bands: an XCD works on 32 or 64 tiles at a time, and what they read of both operands together has to come through its L2 of 4 MB.  Walking all
// token tiles of a channel tile, 64 tiles in flight share one or two channel tiles and no token tile; in bands of about eight they are eight by
// eight.  us, without / with: int4 codes, binary16, 28672 x 4096 6000 rows 1011 / 951, 18432 x 2304 (groups) 4096 rows 291 / 275; int8 14336 x 4096 4096 rows 379 / 361;
// int8 activations 28672 x 4096 int8 4096 rows 444 / 388, int4 387 / 353.
// The bands of a product are of equal width: tiles of a last band of one or two share nothing (int8 activations, us, without bands / eights and
// the rest / equal: 6720 x 7424 518 rows, nine token tiles, 56.2 / 96.9 / 56.3; 1849 x 8448 1084 rows 38.3 / 45.9 / 37.3; 18432 x 512 1308 rows 28.1 / 28.9 / 28.1).
constexpr int kBand = 8;
inline int band_count(int inner) { return inner < kBand + kBand / 2 ? 1 : (inner + kBand / 2) / kBand; }
inline int band_width(int inner) { return (inner + band_count(inner) - 1) / band_count(inner); }
__host__ __device__ __forceinline__ void banded_tile(int i, int inner, int outer, int band, int &o, int &r) {
    const int first = i / (band * outer) * band, j = i - first * outer, width = inner - first < band ? inner - first : band;
    o = j / width, r = first + j % width;
}
// How a product walks over its tiles: token tile by token tile (or channel tile by channel tile), in bands of that many tiles of the other operand
struct TileWalk {
    int by_tokens, band;
};
__host__ __device__ __forceinline__ void xcd_tile(int b, int n_tiles, int m_tiles, TileWalk walk, int &nt, int &mt) {
    const int total = n_tiles * m_tiles, xcd = b % 8;
    const int i = xcd * (total / 8) + (xcd < total % 8 ? xcd : total % 8) + b / 8;
    int o, r;
    banded_tile(i, walk.by_tokens ? n_tiles : m_tiles, walk.by_tokens ? m_tiles : n_tiles, walk.band, o, r);
    nt = walk.by_tokens ? r : o;
    mt = walk.by_tokens ? o : r;
}
// The order for which an XCD pulls fewer bytes: its eighth of the tiles covers a band of one operand (several, if it is more than one; without bands: all
// tiles) and tiles of the other.  w_bytes, x_bytes: of a channel tile and of a token tile, per k.
inline TileWalk fewest_bytes_walk(int n_tiles, int m_tiles, float w_bytes, float x_bytes, bool banded) {
    const int share = (n_tiles * m_tiles + 7) / 8;
    auto covered = [&](int inner, int outer, float inner_bytes, float outer_bytes) {
        const int width = banded ? band_width(inner) : inner, bands = (share + width * outer - 1) / (width * outer);
        const int across = bands > 1 ? outer : (share + width - 1) / width;
        return (float)(bands * width < inner ? bands * width : inner) * inner_bytes + (float)(bands * across) * outer_bytes;
    };
    const int by_tokens = covered(n_tiles, m_tiles, w_bytes, x_bytes) < covered(m_tiles, n_tiles, x_bytes, w_bytes) ? 1 : 0, inner = by_tokens ? n_tiles : m_tiles;
    return {by_tokens, banded ? band_width(inner) : inner};
}
// Put to measured times over 841 shapes of 704 to 60000 channels, K of 256 to 14336 and
// 300 to 6000 rows, all formats, against walks without bands and in bands of eight in either direction.  Over 816 others 1.4 % faster than without bands, 27 of them
// more than 2 % slower (eights and the rest: 0.7 %, 74); the worst int8 6336 x 6144 1481 rows 77 / 84, 51008 x 3328 1125 rows 176 / 188.
inline TileWalk tile_walk(int n_tiles, int m_tiles, int K, bool int8_activations, float w_bytes, float x_bytes) {
    const int share = (n_tiles * m_tiles + 7) / 8;
    // Int8 activations, one band of channel tiles and far more token tiles: the rows, which the quantization has just written, go to one XCD each and the
    // outputs leave it as whole rows (us, by channels / by tokens: int4 1664 x 3072 1508 rows 21.0 / 19.0, int8 1587 x 1280 2516 rows 28.9 / 26.5, 2304 x 9216 4096 rows
    // 122.5 / 116; with fewer token tiles the early touch of the weights has too few to share it, 2304 x 9216 3000 rows, 24 token tiles, 73.2 / 80.7)
    if (int8_activations && band_count(n_tiles) == 1 && m_tiles >= (K <= 4096 ? 2 : 3) * n_tiles) return {1, n_tiles};
    // More tiles than an XCD has in flight, several bands: token tile by token tile, which asks for a band's weights in one go and for the rows again with
    // each band (int8 55128 x 1280 2399 rows 240 / 194, 53398 x 1792 2397 rows 407 / 351).  Weights that the memory-side cache (256 MB) does not hold are to be
    // read once (33866 x 13568 5312 rows, by tokens in bands / all token tiles of a channel tile 2256 / 2076; 40498 x 12032 2881 rows 1320 / 1246).
    if (share > 64 && band_count(n_tiles) > 1 && m_tiles > kBand) {
        if ((float)n_tiles * w_bytes * (float)K > 256e6f) return {0, m_tiles};
        return {1, band_width(n_tiles)};
    }
    return fewest_bytes_walk(n_tiles, m_tiles, w_bytes, x_bytes, true);
}

// Tiles of 128 x 128 that stage both operands, two to a compute unit: bands from 1024 tiles on (us, without / with: int8 x int4 1600 x 1152 4173 rows, 429 tiles, 23.7 /
// 27.0, 2432 x 1152 2018 rows 18.1 / 20.2, binary16 activations, int4 groups 2880 x 4000 4015 rows, 736 tiles, 127 / 142, int8 137 / 123; up to 1024 tiles binary16 gains 0.2 % by
// bands, above 0.6 to 3 %).
inline TileWalk staged_tile_walk(int n_tiles, int m_tiles, int K, bool int8_activations, float w_bytes, float x_bytes) {
    return n_tiles * m_tiles > 1024 ? tile_walk(n_tiles, m_tiles, K, int8_activations, w_bytes, x_bytes) : fewest_bytes_walk(n_tiles, m_tiles, w_bytes, x_bytes, false);
}

}  // namespace qfc
