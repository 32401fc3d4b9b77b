// Prefill product with binary16 activations on the fp16 matrix cores:
//   y[m,n] = sum_k x[m,k] * (s * Wq[n,k]),  fp32 accumulation,
// with s = s[n, k/32] (group scales) or s[n] (per-channel scales), int4 or int8 codes.
// FP16 activations with quantized weights (section 4.2 of the paper), computed
// on matrix units as the compute-bound prefill stage wants (section 3.7).
//
// Two kernels.  The main one (K a multiple of 128, int8 codes: of 64; described in front of it)
// never writes dequantized weights anywhere: packed tiles are copied verbatim
// into LDS, a lane reads the codes of its MFMA operand, converts them in
// registers and feeds the matrix core.  Int4 weights are a quarter of the
// activation bytes, so LDS carries far fewer bytes per MFMA than with a
// dequantized weight tile.  The second kernel is the general fallback (any K
// that is a multiple of 32):
//
// Per K stage of 128 (one packed weight tile per 16 rows): every thread loads
// 16-byte vectors of packed codes (four octets, one per quantization group of
// the tile) plus the four group scales of its row, dequantizes in registers
// (exact int -> binary16, then one binary16 multiply by the scale) and writes
// 16-byte binary16 vectors to LDS.  Activations are copied to LDS as they are.
// LDS holds both tiles octet-major ([k/8][row], 16 B each), so an MFMA fragment
// (32 rows x 16 k, lane = row + 32 * (k/8)) is two runs of 512 contiguous
// bytes; the activation tile has a one-vector pad per octet so that its
// transposing writes are conflict free as well.
#include <type_traits>

#include "qfc_internal.h"
#include "tile_rows.h"

namespace qfc {
namespace {

typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int BN = 128, BM = 128, BK = 128;
constexpr int OCT = BK / 8;      // 16-byte octets (8 binary16) per row per stage
constexpr int LDW = BN;          // vectors per octet, weights
constexpr int LDX = BM + 1;      // vectors per octet, activations (padded)
constexpr size_t kLdsBytes = (size_t)OCT * (LDW + LDX) * 16;

struct GemmF16Args {
    const uint4 *w;   // packed int4 row tiles (W4G32 or W4C)
    const uint4 *x;   // binary16 [M, K] viewed as 16-byte vectors
    _Float16 *y;
    const _Float16 *res;  // [M, N] residual added before the rounding, or null
    const float *sw;  // W4C: fp32 scale per output channel [Np]
    int M, N, K, KT, rt_stride, n_tiles, m_tiles;
    TileWalk walk;  // order of the tiles (see xcd_tile)
    int gated_act = -1;  // QFC_ACT_*: the layer is packed in pairs and y [M, N/2] = fp16(act(gate) * other)
};

__device__ __forceinline__ h2 as_h2(uint32_t u) { return __builtin_bit_cast(h2, u); }
__device__ __forceinline__ uint32_t as_u32(h2 h) { return __builtin_bit_cast(uint32_t, h); }

// eight biased codes -> eight scaled binary16 values, k ascending
__device__ __forceinline__ uint4 dequant8_scaled(uint32_t w, uint32_t scale_bits) {
    const h2 c1032 = {(_Float16)1032.0f, (_Float16)1032.0f};
    const h2 c72 = {(_Float16)72.0f, (_Float16)72.0f};
    const h2 c16th = {(_Float16)0.0625f, (_Float16)0.0625f};
    const _Float16 sh = __builtin_bit_cast(_Float16, (uint16_t)scale_bits);
    const h2 s = {sh, sh};
    const uint32_t lo = w & 0x0F0F0F0Fu, hi = w & 0xF0F0F0F0u;
    const h2 p0 = (as_h2(__builtin_amdgcn_perm(0x64646464u, lo, 0x04010400u)) - c1032) * s;
    const h2 p1 = (as_h2(__builtin_amdgcn_perm(0x64646464u, lo, 0x04030402u)) - c1032) * s;
    const h2 p2 = (as_h2(__builtin_amdgcn_perm(0x64646464u, hi, 0x04010400u)) * c16th - c72) * s;
    const h2 p3 = (as_h2(__builtin_amdgcn_perm(0x64646464u, hi, 0x04030402u)) * c16th - c72) * s;
    return make_uint4(as_u32(p0), as_u32(p1), as_u32(p2), as_u32(p3));
}

// eight int8 codes (two dwords) -> eight binary16 values, exactly (sign bit flipped: b + 128 under the
// exponent byte 0x64 is 1024 + b + 128)
__device__ __forceinline__ uint4 dequant_i8x8(uint32_t lo, uint32_t hi) {
    const h2 c1152 = {(_Float16)1152.0f, (_Float16)1152.0f};
    const uint32_t a = lo ^ 0x80808080u, b = hi ^ 0x80808080u;
    const h2 p0 = as_h2(__builtin_amdgcn_perm(0x64646464u, a, 0x04010400u)) - c1152;
    const h2 p1 = as_h2(__builtin_amdgcn_perm(0x64646464u, a, 0x04030402u)) - c1152;
    const h2 p2 = as_h2(__builtin_amdgcn_perm(0x64646464u, b, 0x04010400u)) - c1152;
    const h2 p3 = as_h2(__builtin_amdgcn_perm(0x64646464u, b, 0x04030402u)) - c1152;
    return make_uint4(as_u32(p0), as_u32(p1), as_u32(p2), as_u32(p3));
}

// PC = per-channel scales (W4C): unscaled integer weights in the MFMA, fp32 scale in the epilogue.
// W8 (with PC) = int8 per-channel weights with binary16 activations (the "q8" scheme of section 4.2
// with FP16 activations at M > 8): two packed KiB tiles of 64 k per row tile and stage, converted
// exactly to binary16 on their way into LDS, fp32 scale in the epilogue.
template <bool PC, bool W8 = false>
__global__ __launch_bounds__(256) void gemm_f16_w4_kernel(GemmF16Args a) {
    static_assert(!W8 || PC, "int8 weights carry per-channel scales");
    extern __shared__ uint4 lds[];
    uint4 *lds_w = lds;
    uint4 *lds_x = lds + OCT * LDW;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wn = wave & 1, wm = wave >> 1;

    int nt, mt;
    xcd_tile(blockIdx.x, a.n_tiles, a.m_tiles, a.walk, nt, mt);

    // weights: thread -> two packed vectors per stage: row tile (tid / 64) and (tid / 64 + 4)
    const int c = lane & 15, q = lane >> 4;
    const uint4 *w_rt[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
        w_rt[i] = a.w + (size_t)(nt * (BN / 16) + wave + 4 * i) * a.rt_stride * 64;
    const int K8 = a.K / 8;

    v16f acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    uint4 wreg[2], wreg2[W8 ? 2 : 1], xreg[8];
    uint2 sreg[2];
    auto load_stage = [&](int kt) {
        const int u = kt >> 3;
        const int wpos = W8 ? 2 * kt : PC ? kt : kt + u;       // weight tile kt of the row tile (int8: tiles 2 kt, 2 kt + 1)
        const int spos = min(8 * u + 8, a.KT) + u;             // scale tile of its unit
        const int soff = (((kt & 7) >> 1) * 16 + c) * 2 + (kt & 1);  // 8-byte index inside it
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            wreg[i] = w_rt[i][(size_t)wpos * 64 + lane];
            if (W8) wreg2[i] = w_rt[i][(size_t)(wpos + 1) * 64 + lane];
            sreg[i] = PC ? make_uint2(0x3C003C00u, 0x3C003C00u)  // 1.0: the multiply is exact
                         : reinterpret_cast<const uint2 *>(w_rt[i] + (size_t)spos * 64)[soff];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int v = tid + 256 * i;
            const int row = mt * BM + (v >> 4);
            const int o = kt * OCT + (v & 15);
            xreg[i] = (row < a.M && o < K8) ? a.x[(size_t)row * K8 + o] : make_uint4(0, 0, 0, 0);
        }
    };

    const int stages = W8 ? a.KT / 2 : a.KT;  // (int8 rows are padded to a multiple of 256 k: an even number of tiles)
    load_stage(0);
    for (int kt = 0; kt < stages; ++kt) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int row = (wave + 4 * i) * 16 + c;
            if (W8) {
                // lane (c, q) of tile h holds the codes k = 64 h + 16 q .. + 15: octets 8 h + 2 q and + 1 of the stage
                lds_w[(2 * q) * LDW + row] = dequant_i8x8(wreg[i].x, wreg[i].y);
                lds_w[(2 * q + 1) * LDW + row] = dequant_i8x8(wreg[i].z, wreg[i].w);
                lds_w[(8 + 2 * q) * LDW + row] = dequant_i8x8(wreg2[i].x, wreg2[i].y);
                lds_w[(8 + 2 * q + 1) * LDW + row] = dequant_i8x8(wreg2[i].z, wreg2[i].w);
                continue;
            }
            const uint32_t wd[4] = {wreg[i].x, wreg[i].y, wreg[i].z, wreg[i].w};
            const uint32_t sc[4] = {sreg[i].x & 0xFFFFu, sreg[i].x >> 16, sreg[i].y & 0xFFFFu, sreg[i].y >> 16};
#pragma unroll
            for (int j = 0; j < 4; ++j) lds_w[(j * 4 + q) * LDW + row] = dequant8_scaled(wd[j], sc[j]);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int v = tid + 256 * i;
            lds_x[(v & 15) * LDX + (v >> 4)] = xreg[i];
        }
        __syncthreads();
        if (kt + 1 < stages) load_stage(kt + 1);
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            const int o = 2 * ks + (lane >> 5);
            v8h fa[2], fb[2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
                fa[i] = __builtin_bit_cast(v8h, lds_w[o * LDW + wn * 64 + i * 32 + (lane & 31)]);
#pragma unroll
            for (int j = 0; j < 2; ++j)
                fb[j] = __builtin_bit_cast(v8h, lds_x[o * LDX + wm * 64 + j * 32 + (lane & 31)]);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fa[i], fb[j], acc[i][j], 0, 0, 0);
        }
    }

    // Epilogue.  A lane holds one token row (lane % 32) and groups of four
    // consecutive n; stored directly, every store instruction would touch 32 rows
    // of y with 8 bytes each.  The binary16 values go through LDS (32 token rows x
    // 64 channels per wavefront at a time) and leave as 16-byte stores along n.
    __syncthreads();  // all wavefronts are done with the tiles in LDS
    if ((a.N % 8) == 0) {
        constexpr int PITCH = (64 + 8) * 2;  // bytes per staged row
        char *region = reinterpret_cast<char *>(lds) + wave * (32 * PITCH);
        const int n0 = nt * BN + wn * 64;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int mrow0 = mt * BM + wm * 64 + j * 32;
            const bool has_res = a.res != nullptr;
            if (has_res) stage_residual_block<8, PITCH>(region, a.res, mrow0, n0, a.M, a.N, lane);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
#pragma unroll
                for (int qq = 0; qq < 4; ++qq) {
                    const int nl = i * 32 + 8 * qq + 4 * (lane >> 5);
                    typedef _Float16 h4 __attribute__((ext_vector_type(4)));
                    float4 sc = make_float4(1.0f, 1.0f, 1.0f, 1.0f);
                    if (PC) sc = *reinterpret_cast<const float4 *>(a.sw + n0 + nl);
                    float v[4] = {acc[i][j][4 * qq + 0] * sc.x, acc[i][j][4 * qq + 1] * sc.y,
                                  acc[i][j][4 * qq + 2] * sc.z, acc[i][j][4 * qq + 3] * sc.w};
                    if (has_res) {
                        float rv[4];
                        staged_residual4(region, (lane & 31) * PITCH + nl * 2, rv);
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] += rv[e];
                    }
                    const h4 hv = {(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]};
                    *reinterpret_cast<h4 *>(region + (lane & 31) * PITCH + nl * 2) = hv;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int it = 0; it < 4; ++it) {  // 32 rows x 8 chunks of 16 bytes
                const int idx = it * 64 + lane;
                const int row = idx >> 3, ch = idx & 7;
                const uint4 v = *reinterpret_cast<const uint4 *>(region + row * PITCH + ch * 16);
                const int mm = mrow0 + row, nn = n0 + ch * 8;
                if (mm < a.M && nn < a.N) *reinterpret_cast<uint4 *>(a.y + (size_t)mm * a.N + nn) = v;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        return;
    }
    const bool vec_ok = (a.N % 4) == 0;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int m = mt * BM + wm * 64 + j * 32 + (lane & 31);
        if (m >= a.M) continue;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
#pragma unroll
            for (int qq = 0; qq < 4; ++qq) {
                const int n = nt * BN + wn * 64 + i * 32 + 8 * qq + 4 * (lane >> 5);
                if (n >= a.N) continue;
                _Float16 *y = a.y + (size_t)m * a.N + n;
                _Float16 h[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float v = PC ? acc[i][j][4 * qq + e] * a.sw[n + e] : acc[i][j][4 * qq + e];
                    if (a.res && n + e < a.N) v += (float)a.res[(size_t)m * a.N + n + e];
                    h[e] = (_Float16)v;
                }
                if (vec_ok) {
                    typedef _Float16 h4 __attribute__((ext_vector_type(4)));
                    *reinterpret_cast<h4 *>(y) = h4{h[0], h[1], h[2], h[3]};
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (n + e < a.N) y[e] = h[e];
                }
            }
        }
    }
}


typedef __attribute__((address_space(3))) void *lptr_t;

constexpr int TN = 256;                    // output channels of a workgroup
constexpr int kStorePitch = (64 + 8) * 2;  // bytes per staged row of the store phase

// Half of an MFMA operand, as two dwords of binary16 values (k ascending): of eight biased int4 codes the low (HI = 0) or the high nibbles,
// exactly, times the group scale if there is one; of four int8 codes, exactly.
template <bool HI, bool SC>
__device__ __forceinline__ uint2 dequant4_half(uint32_t w, h2 s) {
    const h2 c1032 = {(_Float16)1032.0f, (_Float16)1032.0f};
    const h2 c72 = {(_Float16)72.0f, (_Float16)72.0f};
    const h2 c16th = {(_Float16)0.0625f, (_Float16)0.0625f};
    const uint32_t v = w & (HI ? 0xF0F0F0F0u : 0x0F0F0F0Fu);
    h2 p0 = as_h2(__builtin_amdgcn_perm(0x64646464u, v, 0x04010400u)), p1 = as_h2(__builtin_amdgcn_perm(0x64646464u, v, 0x04030402u));
    if (HI)
        p0 = p0 * c16th - c72, p1 = p1 * c16th - c72;
    else
        p0 -= c1032, p1 -= c1032;
    if (SC) p0 *= s, p1 *= s;
    return make_uint2(as_u32(p0), as_u32(p1));
}
__device__ __forceinline__ uint2 dequant8_half(uint32_t w) {
    const h2 c1152 = {(_Float16)1152.0f, (_Float16)1152.0f};
    const uint32_t v = w ^ 0x80808080u;
    return make_uint2(as_u32(as_h2(__builtin_amdgcn_perm(0x64646464u, v, 0x04010400u)) - c1152),
                      as_u32(as_h2(__builtin_amdgcn_perm(0x64646464u, v, 0x04030402u)) - c1152));
}

// ---------------------------------------------------------------------------
// Main kernel: weights never dequantized into LDS, activations through an LDS ring.
//
// A workgroup is four wavefronts (KS = 1) over 256 output channels x 32 JP token rows.  A wavefront owns 64 channels (four
// packed row tiles) and all the rows, 4 x 2 JP tiles of v_mfma_f32_16x16x32_f16 over all of K: it converts its weights once for
// 32 JP rows, its codes are wanted by no other wavefront, and nothing is exchanged at the end.  Weights are the row operand, so a
// lane ends up with four consecutive n of one token row of each tile.
//
// What bounds it: power on real data, then what a wavefront does before its first and after its last MFMA.  Hence two workgroups of JP
// = 4 per compute unit, with everything within half its registers and 80 KiB of LDS: one stores or starts while the other
// multiplies, and a barrier stops one wavefront of a SIMD, not both.  Hence also the 16 x 16 shape: register-only loops (probe.hip; int4 codes
// and normal activations; one / two wavefronts per SIMD) hold 2.07 / 2.11 PFLOP/s with it, 1.67 / 1.68 with
// v_mfma_f32_32x32x16_f16, whose MFMAs take more power for the same products.
// us, one workgroup of eight wavefronts and 32 x 32 MFMAs per compute unit / this, in one session: int4 in groups of 32 18432 x 2304 gated
// 2048 rows 188 / 151, 9216 x 768 1000 rows 29.3 / 20.5; int4 codes 28672 x 4096 gated 6000 rows 1239 / 1011, 6144 x 4096 279 / 221, 4096 x 14336
// 548 / 467; int8 codes (then dequantized into LDS) 14336 x 4096 1000 rows 147 / 99, 4096 x 4096 2048 rows 80 / 58.
//
// KS = 2: eight wavefronts, two groups of four over the same outputs, each with half of K and rings of its own; they
// swap halves of their sums through LDS at the end.  For launches of about one workgroup per compute unit, whose SIMDs would
// hold one wavefront.  Which JP and KS: tile_us.
//
// Everything arrives by direct global -> LDS copies (16 bytes per lane, one KiB per wavefront instruction), which complete in
// issue order, so that waits are counts of the copies issued later.  A half stage is 64 k of the token rows: rows of 128 bytes, the
// 16-byte octet o of row r at position o ^ ((r >> 1) & 7), which makes the operand reads conflict free while a copy still
// reads whole 128-byte row pieces.  Three half stages, copied two ahead; one barrier per half stage.  Codes of 128 k (int8: of 64 k, two in
// turn) and, for group scales, the vectors of 8 groups of the wavefront's 64 rows are copied after the tile before has been
// read into registers.  No copy is issued past the end of K.
//
// Inside a wavefront: a k step of 32 multiplies row tiles 0 and 1 with all blocks of 16 token rows, then 2 and 3; the weights of 2 and 3 are
// converted during the first pass, those of 0 and 1 of the next step during the second, in which each block of token rows is
// replaced by the next step's as soon as it has been multiplied.  (Converting a whole step ahead needs 16 registers more: with group
// scales the loop then spills.)  An MFMA operand is 16 rows x 32 k, lane = (row c, octet q): with 4-bit codes dword g of the
// lane's vector of a packed tile for group g; with int8 codes half of it, and the token rows are read in the same order of octets.
//
// FMT: packed format; JP: blocks of 32 token rows.
template <int FMT, int JP>
struct TileLds {
    static constexpr int kX = JP * 4096;                       // half stage: 32 JP rows x 64 k
    static constexpr int kW = FMT == kW8C ? 2 * 16384 : 16384;  // codes of 128 k
    static constexpr int kS = FMT == kW4G32 ? 4096 : 0;         // scales of 8 groups
    static constexpr int kStaging = 4 * 32 * kStorePitch;
    static constexpr int kRings = 3 * kX + kW + kS;
    static constexpr int kBytes = kRings > kStaging ? kRings : kStaging;
};

// Eight binary16 values, wherever they lie in memory (one 16-byte access; rows of N not a multiple of 8 are not aligned to it).
struct __attribute__((packed, aligned(2))) Octet {
    uint32_t v[4];
};

// Calls f for the octets of a staged block of 32 token rows x 64 channels that lie inside [M, N], or part(..., values) for the one
// that holds a row's last `values` < 8.  (8917 x 256 int4, 2713 rows: 86 us with single values of 32 rows per store instruction, 21.7 like this.)
template <typename F, typename P>
__device__ __forceinline__ void block_rows(const GemmF16Args &a, char *region, int mrow0, int n0, int lane, F &&f, P &&part) {
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int idx = it * 64 + lane, row = idx >> 3, ch = idx & 7;
        const int m = mrow0 + row, n = n0 + ch * 8;
        char *staged = region + row * kStorePitch + ch * 16;
        if (m < a.M && n + 8 <= a.N)
            f(staged, (size_t)m * a.N + n);
        else if (m < a.M && n < a.N)
            part(reinterpret_cast<_Float16 *>(staged), (size_t)m * a.N + n, a.N - n);
    }
}

// Store phase of a wavefront's 64 channels x 16 NJ token rows.  A lane holds one token row (lane % 16) of a block of 16 and four
// consecutive n (4 (lane / 16) + e) of each row tile; the binary16 values go through a block of LDS of the wavefront's own (32 token rows x 64
// channels) and leave as 16-byte stores along n.
template <bool PC, int NJ>
__device__ __forceinline__ void store_tile(const GemmF16Args &a, v4f (&acc)[4][NJ], int n0, int m0, char *region, int lane) {
    typedef _Float16 h4 __attribute__((ext_vector_type(4)));
    const int c = lane & 15, q = lane >> 4;
    if (PC) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const v4f sc = *reinterpret_cast<const v4f *>(a.sw + n0 + 16 * i + 4 * q);
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[i][j] *= sc;
        }
    }
    auto wave_sync = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    if (a.gated_act >= 0) {
        // Layer packed in pairs (operator fusion, section 3.6 of the paper): row tiles 2 t and 2 t + 1 are the gate's and the other
        // branch's rows of the same 16 channels.  32 output channels per wavefront, rows of N / 2 values.
        const GateCoeffs gc = gate_coeffs(a.gated_act);
        const int halfn = a.N / 2, o0 = n0 / 2;
#pragma unroll
        for (int jp = 0; jp < NJ; jp += 2) {
#pragma unroll
            for (int jj = 0; jj < 2; ++jj)
#pragma unroll
                for (int i = 0; i < 4; i += 2) {
                    h4 hv;
#pragma unroll
                    for (int e = 0; e < 4; ++e) hv[e] = (_Float16)(gate_activation(acc[i][jp + jj][e], gc) * acc[i + 1][jp + jj][e]);
                    *reinterpret_cast<h4 *>(region + (16 * jj + c) * kStorePitch + (8 * i + 4 * q) * 2) = hv;
                }
            wave_sync();
#pragma unroll
            for (int it = 0; it < 2; ++it) {  // 32 rows x 4 chunks of 16 bytes
                const int idx = it * 64 + lane;
                const int row = idx >> 2, ch = idx & 3;
                const uint4 v = *reinterpret_cast<const uint4 *>(region + row * kStorePitch + ch * 16);
                const int mm = m0 + jp * 16 + row, nn = o0 + ch * 8;
                if (mm < a.M && nn < halfn) *reinterpret_cast<uint4 *>(a.y + (size_t)mm * halfn + nn) = v;
            }
            wave_sync();
        }
        return;
    }
    const bool has_res = a.res != nullptr;
#pragma unroll
    for (int jp = 0; jp < NJ; jp += 2) {
        const int mrow0 = m0 + jp * 16;
        if (has_res) {
            block_rows(a, region, mrow0, n0, lane,
                       [&](char *staged, size_t at) { *reinterpret_cast<uint4 *>(staged) = __builtin_bit_cast(uint4, *reinterpret_cast<const Octet *>(a.res + at)); },
                       [&](_Float16 *staged, size_t at, int values) { for (int e = 0; e < values; ++e) staged[e] = a.res[at + e]; });
            wave_sync();
        }
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int at = (16 * jj + c) * kStorePitch + (16 * i + 4 * q) * 2;
                v4f v = acc[i][jp + jj];
                if (has_res) {
                    float rv[4];
                    staged_residual4(region, at, rv);
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] += rv[e];
                }
                *reinterpret_cast<h4 *>(region + at) = h4{(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]};
            }
        wave_sync();
        block_rows(a, region, mrow0, n0, lane,
                   [&](char *staged, size_t at) { *reinterpret_cast<Octet *>(a.y + at) = __builtin_bit_cast(Octet, *reinterpret_cast<const uint4 *>(staged)); },
                   [&](_Float16 *staged, size_t at, int values) { for (int e = 0; e < values; ++e) a.y[at + e] = staged[e]; });
        wave_sync();
    }
}

template <int FMT, int JP, int KS>
__global__ __launch_bounds__(256 * KS, KS == 2 ? 2 : JP == 1 ? 4 : JP == 2 ? 3 : 2) void gemm_f16_tile_kernel(GemmF16Args a) {
    using L = TileLds<FMT, JP>;
    constexpr bool W8 = FMT == kW8C, G32 = FMT == kW4G32;
    constexpr int ROWS = 32 * JP;
    constexpr int W_OFF = 3 * L::kX, S_OFF = W_OFF + L::kW;
    constexpr int XC = JP, WC = G32 ? 5 : 4;  // copies per wavefront: of a half stage; of 128 k (int8: 64 k) of codes
    extern __shared__ uint4 lds[];
    char *lds_all = reinterpret_cast<char *>(lds);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) & 3);
    const int group = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);  // part of K
    char *lds_b = lds_all + group * L::kBytes;
    const int c = lane & 15, q = lane >> 4;
    int nt, mt;
    xcd_tile(blockIdx.x, a.n_tiles, a.m_tiles, a.walk, nt, mt);
    const int m0 = mt * ROWS;
    // half stages of this group (4-bit codes: an even number); the first group has the odd step
    constexpr int kStep = W8 ? 1 : 2;
    const int nst_all = a.K / 64, first = KS == 1 ? nst_all : (nst_all / kStep + 1) / 2 * kStep;
    const int nst = group ? nst_all - first : first, i0 = group ? first : 0;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)lds + group * L::kBytes;

    const char *xbase = reinterpret_cast<const char *>(a.x) + (size_t)(m0 - rows_in_front(m0, ROWS)) * a.K * 2;
    uint32_t xlane[XC];
#pragma unroll
    for (int i = 0; i < XC; ++i) {
        const int rl = 32 * i + 8 * wave + (lane >> 3);
        const int oct = (lane & 7) ^ ((rl >> 1) & 7);
        xlane[i] = (uint32_t)source_row(i, wave, lane >> 3, m0, a.M, ROWS) * (uint32_t)a.K * 2u + oct * 16;
    }
    const size_t rt_bytes = (size_t)a.rt_stride * 1024;
    const char *wbase = reinterpret_cast<const char *>(a.w) + (size_t)(nt * 16 + wave * 4) * rt_bytes;
    const uint32_t wlane = lane * 16;
    const uint32_t slane = (uint32_t)q * a.rt_stride * 1024u + c * 16;

    auto issue_x = [&](int i, int blk) __attribute__((always_inline)) {  // half stage i
        copy16_to_lds(xbase + (size_t)(i0 + i) * 128, xlane[blk], lds0 + (i % 3) * L::kX + blk * 4096 + wave * 1024);
    };
    // codes of tile t (int8: of half stage t), row tile k of the wavefront; k = 4: its scales
    auto issue_w = [&](int t, int k) __attribute__((always_inline)) {
        const int ta = i0 / kStep + t, u = ta >> 3;
        if (k < 4)
            copy16_to_lds(wbase + k * rt_bytes + (size_t)(G32 ? ta + u : ta) * 1024, wlane, lds0 + W_OFF + (W8 ? (t & 1) * 16384 : 0) + (wave * 4 + k) * 1024);
        else
            copy16_to_lds(wbase + (size_t)(min(8 * u + 8, a.KT) + u) * 1024 + (size_t)((ta & 7) >> 1) * 256, slane, lds0 + S_OFF + wave * 1024);
    };

    constexpr int NJ = 2 * JP;  // blocks of 16 token rows
    v4f acc[4][NJ];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = v4f{0.0f, 0.0f, 0.0f, 0.0f};

    int xoff[2];  // k step s of a half stage: octet of this lane
#pragma unroll
    for (int s = 0; s < 2; ++s) xoff[s] = c * 128 + (((W8 ? 2 * q + s : 4 * s + q) ^ ((c >> 1) & 7)) << 4);
    const char *wread = lds_b + W_OFF + wave * 4096 + lane * 16;
    const char *sread = lds_b + S_OFF + wave * 1024 + c * 16;

    uint4 xv[NJ];     // token rows of a k step of 32; each block is replaced by the next step's once it has been multiplied
    uint2 fa[4][2];   // converted weights: [row tile][half], of a step's first two row tiles ahead of it, of the others during it
    uint4 wv[4];      // codes: of 128 k, one dword per k step (int8: of 64 k, half of it per k step)
    uint2 sv[4];
    auto read_x = [&](int i, int s, int j) __attribute__((always_inline)) {
        xv[j] = *reinterpret_cast<const uint4 *>(lds_b + (i % 3) * L::kX + xoff[s] + j * 2048);
    };
    auto read_ws = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            wv[i] = *reinterpret_cast<const uint4 *>(wread + (W8 ? (t & 1) * 16384 : 0) + i * 1024);
            if (G32) sv[i] = *reinterpret_cast<const uint2 *>(sread + i * 256 + ((i0 / kStep + t) & 1) * 8);
        }
    };
    // half p of the operand of row tile i, k step s of half h
    auto convert = [&](int i, int p, int h, int s) __attribute__((always_inline)) {
        const uint4 &v = wv[i];
        if (W8) {
            fa[i][p] = dequant8_half(s ? (p ? v.w : v.z) : p ? v.y : v.x);
            return;
        }
        const int g = 2 * h + s;
        const uint32_t w = g == 0 ? v.x : g == 1 ? v.y : g == 2 ? v.z : v.w;
        h2 sc = {(_Float16)1.0f, (_Float16)1.0f};
        if (G32) sc = as_h2(__builtin_amdgcn_perm(0u, g & 2 ? sv[i].y : sv[i].x, g & 1 ? 0x03020302u : 0x01000100u));
        fa[i][p] = p ? dequant4_half<true, G32>(w, sc) : dequant4_half<false, G32>(w, sc);
    };
    auto multiply = [&](int pair, int j) __attribute__((always_inline)) {  // row tiles 2 pair, 2 pair + 1
#pragma unroll
        for (int i = 2 * pair; i < 2 * pair + 2; ++i) {
            const uint4 f = make_uint4(fa[i][0].x, fa[i][0].y, fa[i][1].x, fa[i][1].y);
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, f), __builtin_bit_cast(v8h, xv[j]), acc[i][j], 0, 0, 0);
        }
    };

    // Copies in issue order: codes 0, half stage 0 (int8: codes 1), half stage 1, codes 1 (int8: 2), half stage 2; then behind half stage i's barrier the
    // codes of the tile after the next (4-bit: i odd; int8: of half stage i + 3) and half stage i + 3.
    const int tiles = nst / kStep;
    auto codes = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < WC; ++k) issue_w(t, k);
    };
    auto rows = [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < XC; ++k) issue_x(i, k);
    };
    if (nst > 0) {
        codes(0);
        rows(0);
        if (W8 && tiles > 1) codes(1);
        if (nst > 1) rows(1);
        if (tiles <= 1)
            wait_copies<0>();
        else
            wait_copies<2 * XC + (W8 ? WC : 0)>();
        read_ws(0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the codes are in registers: their slot may be overwritten
        if (tiles > (W8 ? 2 : 1)) codes(W8 ? 2 : 1);
        if (nst > 2) rows(2);
        if (nst > 2)
            wait_vmcnt<2 * XC + (W8 ? 2 * WC : WC)>();
        else
            wait_vmcnt<0>();
        asm volatile("s_barrier" ::: "memory");
#pragma unroll
        for (int j = 0; j < NJ; ++j) read_x(0, 0, j);
#pragma unroll
        for (int k = 0; k < 4; ++k) convert(k >> 1, k & 1, 0, 0);
    }

    // Half stage i, h: its half of the 128-k tile (4-bit codes).  after: half stages that follow it, 3 standing for more of them.
    auto half = [&](int i, const int h, const int after) __attribute__((always_inline)) {
        constexpr int kFirst = NJ >= 8 ? 2 : 1;  // blocks multiplied ahead of the barrier
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            int slot = 0;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {  // row tiles 0 and 1; 2 and 3 are converted
                multiply(0, j);
#pragma unroll
                for (int k = j * 4 / NJ; k < (j + 1) * 4 / NJ; ++k) convert(2 + (k >> 1), k & 1, h, s);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (s == 1 && (W8 || h == 1) && after > 0) {
                // the next codes have landed once only what was issued after them is outstanding
                if (W8 && after >= 2)
                    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * XC + WC) : "memory");
                else
                    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(W8 ? XC : 2 * XC) : "memory");
                read_ws(W8 ? i + 1 : (i >> 1) + 1);
            }
#pragma unroll
            for (int j = 0; j < NJ; ++j) {  // row tiles 2 and 3; 0 and 1 of the next step are converted, its token rows read
                if (s == 1 && j == kFirst && after > 0) {
                    // Half stage i + 1 has landed once only what was issued for i + 2 is outstanding; this wavefront has read all of half stage i.
                    // The barrier says the same of the others: half stage i + 1 may be read, the slot of i overwritten.
                    if (after == 1)
                        wait_vmcnt<0>();
                    else if (W8 || h == 0)
                        wait_vmcnt<XC + WC>();
                    else
                        wait_vmcnt<XC>();
                    asm volatile("s_barrier" ::: "memory");
#pragma unroll
                    for (int jj = 0; jj < kFirst; ++jj) read_x(i + 1, 0, jj);
                }
                multiply(1, j);
                if (s == 0) {
#pragma unroll
                    for (int k = j * 4 / NJ; k < (j + 1) * 4 / NJ; ++k) convert(k >> 1, k & 1, h, 1);
                } else if (after > 0 && j >= kFirst) {
#pragma unroll
                    for (int k = (j - kFirst) * 4 / (NJ - kFirst); k < (j - kFirst + 1) * 4 / (NJ - kFirst); ++k) convert(k >> 1, k & 1, (h + 1) & 1, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (s == 0)
                    read_x(i, 1, j);
                else if (after > 0 && j >= kFirst)
                    read_x(i + 1, 0, j);
                if (s == 1 && j >= kFirst && after >= 3) {
                    constexpr int kPer = (WC + XC + NJ - kFirst - 1) / (NJ - kFirst);
#pragma unroll
                    for (int k = 0; k < kPer; ++k, ++slot) {
                        const int n = slot - (W8 || h == 1 ? WC : 0);
                        if (n < 0)
                            issue_w(W8 ? i + 3 : (i >> 1) + 2, slot);
                        else if (n < XC)
                            issue_x(i + 3, n);
                    }
                }
            }
        }
    };
    if constexpr (W8) {
        int i = 0;
        for (; i + 3 < nst; ++i) half(i, 0, 3);
        if (i + 2 < nst) half(i++, 0, 2);
        if (i + 1 < nst) half(i++, 0, 1);
        if (i < nst) half(i, 0, 0);
    } else {
        int i = 0;
        for (; i + 4 < nst; i += 2) {
            half(i, 0, 3);
            half(i + 1, 1, 3);
        }
        if (i + 2 < nst) {
            half(i, 0, 3);
            half(i + 1, 1, 2);
            i += 2;
        }
        if (i < nst) {
            half(i, 0, 1);
            half(i + 1, 1, 0);
        }
    }
    if (KS == 2) {
        for (int i = nst; i < first; ++i) asm volatile("s_barrier" ::: "memory");  // (as many barriers as the first group passes)
    }

    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // every wavefront is done with the rings
    const int n0 = nt * TN + wave * 64;
    char *region = lds_all + (threadIdx.x >> 6) * (32 * kStorePitch);
    if constexpr (KS == 1) {
        store_tile<!G32, NJ>(a, acc, n0, m0, region, lane);
    } else {
        // The two halves of K meet: the first group keeps the first H0 blocks of 16 token rows, the other the rest (an even number each), and each hands
        // the other's over through LDS ([group][wavefront][16-byte vector][lane]), over the dead rings.
        constexpr int H0 = (JP + 1) / 2 * 2, H1 = 2 * JP - H0;
        static_assert(16 * 2 * JP * 1024 <= 2 * L::kBytes, "the sums handed over fit over the rings");
        v4f *const to0 = reinterpret_cast<v4f *>(lds_all) + wave * (4 * H0 * 64) + lane;
        v4f *const to1 = reinterpret_cast<v4f *>(lds_all) + 16 * H0 * 64 + wave * (4 * H1 * 64) + lane;
        if (group) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < H0; ++j) to0[(i * H0 + j) * 64] = acc[i][j];
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < H1; ++j) to1[(i * H1 + j) * 64] = acc[i][H0 + j];
        }
        __syncthreads();
        if (group) {
            v4f out[4][H1];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < H1; ++j) out[i][j] = acc[i][H0 + j] + to1[(i * H1 + j) * 64];
            __syncthreads();
            store_tile<!G32, H1>(a, out, n0, m0 + H0 * 16, region, lane);
        } else {
            v4f out[4][H0];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < H0; ++j) out[i][j] = acc[i][j] + to0[(i * H0 + j) * 64];
            __syncthreads();
            store_tile<!G32, H0>(a, out, n0, m0, region, lane);
        }
    }
}

template <int FMT, int JP, int KS>
hipError_t launch_tile(GemmF16Args a, hipStream_t st) {
    constexpr size_t bytes = KS * TileLds<FMT, JP>::kBytes;
    if (const hipError_t e = allow_dynamic_lds<gemm_f16_tile_kernel<FMT, JP, KS>>(bytes); e != hipSuccess) return e;
    a.n_tiles = (a.N + TN - 1) / TN;
    a.m_tiles = (a.M + 32 * JP - 1) / (32 * JP);
    a.walk = tile_walk(a.n_tiles, a.m_tiles, a.K, false, (FMT == kW8C ? 1.0f : FMT == kW4C ? 0.5f : 0.5625f) * TN, 2.0f * 32 * JP);
    gemm_f16_tile_kernel<FMT, JP, KS><<<dim3((unsigned)(a.n_tiles * a.m_tiles)), 256 * KS, bytes, st>>>(a);
    return hipGetLastError();
}

template <bool PC, bool W8 = false>
hipError_t launch_fallback(GemmF16Args a, int M, hipStream_t st) {
    if (const hipError_t e = allow_dynamic_lds<gemm_f16_w4_kernel<PC, W8>>(kLdsBytes); e != hipSuccess) return e;
    a.n_tiles = (a.N + BN - 1) / BN;
    a.m_tiles = (M + BM - 1) / BM;
    a.walk = staged_tile_walk(a.n_tiles, a.m_tiles, a.K, false, (W8 ? 1.0f : PC ? 0.5f : 0.5625f) * BN, 2.0f * BM);
    gemm_f16_w4_kernel<PC, W8><<<dim3((unsigned)(a.n_tiles * a.m_tiles)), 256, kLdsBytes, st>>>(a);
    return hipGetLastError();
}

constexpr int kTileForms = 7;

template <int FMT>
hipError_t tile_form(const GemmF16Args &a, int form, hipStream_t st) {
    switch (form) {
        case 1: return launch_tile<FMT, 1, 1>(a, st);
        case 2: return launch_tile<FMT, 2, 1>(a, st);
        case 3: return launch_tile<FMT, 3, 1>(a, st);
        case 4: return launch_tile<FMT, 4, 1>(a, st);
        case 5: return launch_tile<FMT, 4, 2>(a, st);
        case 6: return launch_tile<FMT, 2, 2>(a, st);
        case 7: return launch_tile<FMT, 3, 2>(a, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace

bool tile_kernel_takes(const Geometry &g) { return g.K % (g.fmt == kW8C ? 64 : 128) == 0; }

// Estimated time of the main kernel and the form it is fastest in.  A tile takes `each` us and K / 1000 times `alone` on a
// compute unit of its own, `shared` where several are in flight.  The part that grows with K slows down with the number of compute units that are
// busy, since power is what they share: `cap` is about the share of the chip that runs at full clock.
// Fitted to 2157 shapes of 768 to 28672 channels, K of 256 to 14336 and 20 to 6500 rows (standard deviation 2 to 5 %); the choice is 0.2 % slower than the
// best of the first six forms on average, 4 % in one of a hundred shapes.  Form 7 lies between 5 and 6, and so do its numbers: within 3 % on 1562 more
// shapes of 150 to 4096 rows, the choice among all 0.05 % slower than the best (without form 7 1.1 %).
// us, forms 1 to 6, int4 in groups of 32: 2304 x 9216 1000 rows 99 / 84 / 96 / 113 / 96 / 67; 4096 x 2304 2048 rows 56 / 42 / 46 / 38 / 36 / 45.
// Forms 3 / 5 / 7: 2304 x 9216 2048 rows 97 / 96 / 89, x 2048 25.6 / 26.2 / 23.4; int4 4096 x 14336 1500 rows 139 / 141 / 130; int8 4096 x 4096 1400
// rows 48.4 / 48.4 / 45.6; 4096 x 2304 2048 rows, 256 tiles of 128 and 352 of 96, - / 35.8 / 50.4.
int tile_rows(int form) {
    static const int rows[kTileForms] = {32, 64, 96, 128, 128, 64, 96};
    return rows[form - 1];
}

float tile_us(const Geometry &g, int M, int num_cus, int *form) {
    struct Fit {
        float start, each, alone, shared, cap;
    };
    static const Fit fits[3][kTileForms] = {
        // int8
        {{2.23f, 0.76f, 6.38f, 4.23f, 1.11f}, {2.50f, 1.27f, 7.60f, 6.03f, 0.99f}, {3.02f, 1.56f, 9.26f, 7.83f, 1.00f},
         {3.30f, 2.07f, 11.20f, 9.61f, 0.95f}, {1.04f, 4.79f, 9.68f, 9.38f, 0.84f}, {0.83f, 3.39f, 6.16f, 5.75f, 0.87f}, {0.93f, 4.1f, 7.92f, 7.56f, 0.86f}},
        // int4, group scales
        {{2.38f, 0.47f, 6.97f, 4.86f, 1.16f}, {2.50f, 0.85f, 8.58f, 6.58f, 1.11f}, {2.54f, 1.38f, 9.87f, 8.36f, 1.03f},
         {2.81f, 1.79f, 11.54f, 10.02f, 0.98f}, {0.50f, 4.94f, 9.57f, 9.30f, 0.83f}, {0.49f, 3.52f, 6.77f, 6.34f, 0.95f}, {0.5f, 4.2f, 8.17f, 7.82f, 0.9f}},
        // int4
        {{2.49f, 0.51f, 5.36f, 3.67f, 1.14f}, {2.58f, 1.02f, 6.76f, 5.11f, 1.02f}, {2.61f, 1.73f, 8.14f, 6.77f, 0.98f},
         {2.91f, 2.09f, 10.01f, 8.79f, 1.00f}, {0.57f, 5.09f, 8.54f, 8.33f, 0.89f}, {0.71f, 3.42f, 5.26f, 4.91f, 0.89f}, {0.64f, 4.25f, 6.9f, 6.62f, 0.89f}}};
    const float k = 1e-3f * (float)g.K;
    float best = 0.0f;
    *form = 0;
    for (int i = 0; i < kTileForms; ++i) {
        if (i >= 4 && g.K < 256) break;  // (two halves of K: two steps of 128 at least)
        const Fit &f = fits[g.fmt][i];
        const int rows = tile_rows(i + 1), tiles = (g.N + TN - 1) / TN * ((M + rows - 1) / rows);
        const int full = tiles / num_cus, rest = tiles % num_cus;
        auto work = [&](int n) { return n == 0 ? 0.0f : n == 1 ? f.alone * k : (float)n * f.shared * k; };  // of a compute unit with n tiles
        auto slowed = [&](int busy) {
            const float u = (float)busy / (f.cap * (float)num_cus);
            return sqrtf(sqrtf(1.0f + u * u * u * u));
        };
        float us = f.start + (float)full * f.each + work(full) * slowed(num_cus);
        if (rest > 0) us += fmaxf(f.each + (work(full + 1) - work(full)) * slowed(rest), 0.0f);
        if (*form == 0 || us < best) best = us, *form = i + 1;
    }
    return best;
}

hipError_t launch_gemm_f16(const Geometry &g, const void *packed, const void *x, int M, void *y,
                           const void *residual, int gated_act, int num_cus, hipStream_t st) {
    // (a gated output is offered for int4 formats and K a multiple of 128)
    if (gated_act >= 0 && (!g.pair_half || (g.K % 128) != 0 || g.fmt == kW8C)) return hipErrorNotSupported;
    if (skinny_product(g, M, false, gated_act >= 0, num_cus)) return launch_skinny_f16(g, packed, x, M, y, residual, gated_act, num_cus, st);
    GemmF16Args a;
    a.w = static_cast<const uint4 *>(packed);
    a.x = static_cast<const uint4 *>(x);
    a.y = static_cast<_Float16 *>(y);
    a.res = static_cast<const _Float16 *>(residual);
    a.sw = reinterpret_cast<const float *>(static_cast<const char *>(packed) + g.scale_off);
    a.M = M;
    a.N = g.N;
    a.K = g.K;
    a.KT = g.KT;
    a.rt_stride = g.rt_stride;
    a.n_tiles = a.m_tiles = 0;
    a.walk = {};
    a.gated_act = gated_act;
    if (tile_kernel_takes(g) && (tuning().gemm_variant != 9 || gated_act >= 0)) {
        const int rest = skinny_tail_rows(g, M, gated_act >= 0, num_cus), most = M - rest;
        int form;
        tile_us(g, most, num_cus, &form);
        const int forced = tuning().gemm_variant - 30;  // (tests: a form by its number)
        if (forced >= 1 && forced <= (g.K < 256 ? 4 : kTileForms)) form = forced;
        a.M = most;
        const hipError_t e = g.fmt == kW8C ? tile_form<kW8C>(a, form, st) : g.fmt == kW4C ? tile_form<kW4C>(a, form, st) : tile_form<kW4G32>(a, form, st);
        if (e != hipSuccess || rest == 0) return e;
        const int n_out = gated_act >= 0 ? g.N / 2 : g.N;
        return launch_skinny_f16(g, packed, static_cast<const _Float16 *>(x) + (size_t)most * g.K, rest, a.y + (size_t)most * n_out,
                                 residual ? a.res + (size_t)most * g.N : nullptr, gated_act, num_cus, st);
    }
    if (g.fmt == kW8C) return launch_fallback<true, true>(a, M, st);
    const bool pc = g.fmt == kW4C;
    return pc ? launch_fallback<true>(a, M, st) : launch_fallback<false>(a, M, st);
}

}  // namespace qfc
