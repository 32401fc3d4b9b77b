// Which token rows the tiles of gemm_f16_tile_kernel copy (also compiled for the host, by a test).
#pragma once

namespace qfc {

// Rows in front of a tile that its copies may read too: the tile before, where there is one.
__host__ __device__ __forceinline__ int rows_in_front(int m0, int rows) { return m0 > 0 ? rows : 0; }

// Row that is copied to row 32 i + 8 wave + r (r < 8) of the tile of `rows` rows at m0, counted from the rows in front.  Rows past the last
// (their products are never stored) take others' data so that no wavefront copies one line over and over (many copies of the same lines
// in flight have been seen to land after the counter said they were done): rows of the tile before, or, in the first tile (9 rows at least),
// piece i + wave of eight rows, starting over behind the last of `pieces`.  With 32 rows and more a wavefront copies a line twice at most.
__host__ __device__ __forceinline__ int source_row(int i, int wave, int r, int m0, int M, int rows) {
    const int at = 32 * i + 8 * wave + r;
    const int pieces = M >= 64 ? 8 : M >= 32 ? 4 : M >= 16 ? 2 : 1;  // whole pieces, a power of two of them
    const int instead = m0 > 0 ? 32 * i + 8 * wave : 8 * ((i + wave) & (pieces - 1));
    return m0 + at < M ? rows_in_front(m0, rows) + at : instead + r;
}

}  // namespace qfc
