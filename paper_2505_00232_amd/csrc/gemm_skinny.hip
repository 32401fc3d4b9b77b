// Products of few token rows (from M = 9: batches beyond the decode kernel's eight rows, prompts of up to a
// few hundred tokens, see skinny_product): y[m,n] = sum_k x[m,k] * s * Wq[n,k], with binary16 activations (weights dequantized in
// registers) or int8 activations (exact int32 sums).
//
// What bounds them: the weight stream up to a few dozen rows, as in decode.  The tiles of the
// prefill kernels (256 channels x 64 or 128 tokens) give 16 workgroups for a layer of 4096
// channels, i.e. 16 of 256 compute units pull the weights.  Here, as in the decode kernel, a
// workgroup owns 16 R output channels (R packed row tiles) and all token rows (blocks of up to 64), and its
// wavefronts split K; their partial sums meet in LDS in fixed order (deterministic, no atomics, no
// traffic between workgroups, no workspace).
//
// Measured with the weights in HBM, 32 token rows, this kernel against the 256-channel tiles (us):
//   channels x k            4096 x 4096   4096 x 14336   6144 x 4096   28672 x 4096   128256 x 4096
//   int4 groups, binary16    7.8 / 32      18.3 / 107     9.0 / 32      22.0 / 34      79 / 68
//   int8 x int8 (with the quantization kernel)
//                           10.1 / 26      23.9 / 91     12.0 / 30      25.5 / 36      95 / 106
// The narrow layers are bound by the token rows: every compute unit pulls all of x (2 M K bytes) through
// its vector cache, seven times its share of the 4-bit weights at M = 32.  The wide ones are within 1.3
// (8-bit) to 1.7 (4-bit) of the time a 5.1 TB/s copy of the weights takes.
//
// MFMA shape 16 x 16: token rows are the row operand, in blocks of 16, weights the columns (a lane's 16
// bytes of a packed tile are one or more whole operands, loaded from memory straight into registers).
#include <type_traits>
#include <utility>

#include "qfc_internal.h"

namespace qfc {
namespace {

typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void *lptr_t;

struct SkinnyArgs {
    const u32x4 *w;       // packed row tiles
    const u32x4 *x;       // binary16 [M, K], or tiled int8 (see actquant.hip)
    const float *sw;      // per-channel scales [Np] (W8C, W4C)
    const float *sx;      // int8: per-token scales
    const _Float16 *res;  // [M, N] residual added before the rounding, or null
    void *out;
    int M, N, K, Kp, KT, RT;  // KT: packed k tiles per row tile, RT: row tiles
    int block_rows, blocks;   // token rows per workgroup, blocks of them
    int rt_stride;
    int steps_q, steps_rem;  // 128-k steps per wavefront: steps_q, one more for the first steps_rem
    float sw_mul;            // int8 x 4-bit: sums are 16 times the definition's (see gemm_i8.hip)
    int gated_act;
    int turned;  // int8: workgroups begin their k ranges at different steps
};

__device__ __forceinline__ h2 as_h2(uint32_t u) { return __builtin_bit_cast(h2, u); }

// eight biased int4 codes -> eight binary16 values (k ascending), exactly; with SC times a group scale
// (one binary16 rounding per weight, as in the large fp16 kernel)
template <bool SC>
__device__ __forceinline__ v8h dequant4(uint32_t w, h2 s) {
    const h2 c1032 = {(_Float16)1032.0f, (_Float16)1032.0f};
    const h2 c72 = {(_Float16)72.0f, (_Float16)72.0f};
    const h2 c16th = {(_Float16)0.0625f, (_Float16)0.0625f};
    const uint32_t lo = w & 0x0F0F0F0Fu, hi = w & 0xF0F0F0F0u;
    h2 p0 = as_h2(__builtin_amdgcn_perm(0x64646464u, lo, 0x04010400u)) - c1032;
    h2 p1 = as_h2(__builtin_amdgcn_perm(0x64646464u, lo, 0x04030402u)) - c1032;
    h2 p2 = as_h2(__builtin_amdgcn_perm(0x64646464u, hi, 0x04010400u)) * c16th - c72;
    h2 p3 = as_h2(__builtin_amdgcn_perm(0x64646464u, hi, 0x04030402u)) * c16th - c72;
    if (SC) p0 *= s, p1 *= s, p2 *= s, p3 *= s;
    return v8h{p0[0], p0[1], p1[0], p1[1], p2[0], p2[1], p3[0], p3[1]};
}
// eight int8 codes -> eight binary16 values, exactly
__device__ __forceinline__ v8h dequant8(uint32_t lo, uint32_t hi) {
    const h2 c1152 = {(_Float16)1152.0f, (_Float16)1152.0f};
    const uint32_t a = lo ^ 0x80808080u, b = hi ^ 0x80808080u;
    const h2 p0 = as_h2(__builtin_amdgcn_perm(0x64646464u, a, 0x04010400u)) - c1152;
    const h2 p1 = as_h2(__builtin_amdgcn_perm(0x64646464u, a, 0x04030402u)) - c1152;
    const h2 p2 = as_h2(__builtin_amdgcn_perm(0x64646464u, b, 0x04010400u)) - c1152;
    const h2 p3 = as_h2(__builtin_amdgcn_perm(0x64646464u, b, 0x04030402u)) - c1152;
    return v8h{p0[0], p0[1], p1[0], p1[1], p2[0], p2[1], p3[0], p3[1]};
}

// At most N vector-memory operations outstanding and no LDS operation; memory accesses do not move across.
template <int N>
__device__ __forceinline__ void wait_mem() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// The wavefronts' partial sums meet in LDS: red[wave][r][tb] = 16 tokens x 16 channels, the token rows
// permuted (bits 3:2 and 1:0 exchanged) so that the four tokens a store instruction writes lie in
// different banks.  (16 x 16 accumulator: lane = channel + 16 q holds tokens 4 q + e in register e.)
__device__ __forceinline__ int red_row(int tile, int token) { return (tile * 16 + ((token >> 2) | ((token & 3) << 2))) * 16; }

// The workgroup's first row tile and token block.  Workgroups are dealt to the 8 XCDs round robin: the token
// blocks of the same row tiles follow each other on one XCD, whose L2 then holds their weights.
__device__ __forceinline__ bool place(const SkinnyArgs &a, int R, int &rt0, int &m0, int &rows) {
    int group = blockIdx.x, block = 0;
    if (a.blocks > 1) {
        const int xcd = blockIdx.x % 8, j = blockIdx.x / 8;
        group = j / a.blocks * 8 + xcd;
        block = j % a.blocks;
    }
    rt0 = group * R;
    m0 = block * a.block_rows;
    rows = min(a.block_rows, a.M - m0);
    return rt0 < a.RT;
}

template <int R, int TB, typename T, typename ACC>
__device__ __forceinline__ void put_partials(T *red, const ACC (&acc)[R][TB], int wave, int lane) {
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb)
#pragma unroll
            for (int e = 0; e < 4; ++e) red[red_row((wave * R + r) * TB + tb, 4 * (lane >> 4) + e) + (lane & 15)] = acc[r][tb][e];
}

// Sum over the wavefronts (in order) and store phase.  T: float or int; CH: per-channel scales.
template <int R, int TB, typename T, bool CH>
__device__ __forceinline__ void finish(const SkinnyArgs &a, const T *red, int nwaves, int rt0, int m0, int rows) {
    constexpr bool kInt = std::is_same<T, int>::value;
    typedef T t4 __attribute__((ext_vector_type(4)));
    const bool gated = a.gated_act >= 0;
    const int half = a.N / 2;
    const int tiles = gated ? R / 2 : R;  // (gated: pairs of row tiles, R is even)
    auto total = [&](int r, int tb, int token, int n4) {
        t4 s = {0, 0, 0, 0};
        for (int w = 0; w < nwaves; ++w) s += *reinterpret_cast<const t4 *>(red + red_row((w * R + r) * TB + tb, token) + 4 * n4);
        return s;
    };
    auto scaled = [&](const t4 &s, int n, float sxm, float (&v)[4]) {
        float4 c = make_float4(1.0f, 1.0f, 1.0f, 1.0f);
        if (CH) c = *reinterpret_cast<const float4 *>(a.sw + n);
        const float cs[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = kInt ? (float)s[e] * sxm * (cs[e] * a.sw_mul) : CH ? (float)s[e] * cs[e] : (float)s[e];
    };
    for (int i = threadIdx.x; i < tiles * TB * 64; i += blockDim.x) {
        const int n4 = i & 3, m = (i >> 2) & 15, tb = (i >> 6) % TB, r = (i >> 6) / TB;
        if (tb * 16 + m >= rows) continue;
        const int token = m0 + tb * 16 + m;
        const float sxm = kInt ? a.sx[token] : 1.0f;
        if (gated) {
            // physical row tiles 2 t and 2 t + 1 of a layer packed in pairs hold the gate's and the other
            // branch's rows of the same 16 channels (operator fusion, section 3.6 of the paper)
            const int n = (rt0 + 2 * r) * 16 + 4 * n4, o = n / 2 + 2 * n4;  // o = (rt0 / 2 + r) * 16 + 4 n4
            if (o >= half) continue;
            float g[4], u[4];
            scaled(total(2 * r, tb, m, n4), n, sxm, g);
            scaled(total(2 * r + 1, tb, m, n4), n + 16, sxm, u);
            const GateCoeffs gc = gate_coeffs(a.gated_act);
            h4 hv;
#pragma unroll
            for (int e = 0; e < 4; ++e) hv[e] = (_Float16)(gate_activation(g[e], gc) * u[e]);
            *reinterpret_cast<h4 *>(static_cast<_Float16 *>(a.out) + (size_t)token * half + o) = hv;
            continue;
        }
        const int n = (rt0 + r) * 16 + 4 * n4;
        if (n >= a.N) continue;
        float v[4];
        scaled(total(r, tb, m, n4), n, sxm, v);
        _Float16 *y = static_cast<_Float16 *>(a.out) + (size_t)token * a.N + n;
        const _Float16 *res = a.res ? a.res + (size_t)token * a.N + n : nullptr;
        if ((a.N & 3) == 0) {
            if (res) {
                const h4 rv = *reinterpret_cast<const h4 *>(res);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] += (float)rv[e];
            }
            *reinterpret_cast<h4 *>(y) = h4{(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]};
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n + e < a.N) y[e] = (_Float16)(res ? v[e] + (float)res[e] : v[e]);
        }
    }
}

// ---------------------------------------------------------------- binary16 activations
// Per step of 128 k a wavefront holds its weights in registers (requested D steps ahead, see below) and reads the
// token rows from a private LDS ring of RING half steps (64 k: rows of 128 bytes, 16-byte octets
// XOR-swizzled as in the large fp16 kernel: conflict-free operand reads).  The ring is filled by
// direct memory -> LDS copies whose lanes cover whole 128-byte row pieces: fetching the operands from
// memory in their own order (16 rows x 64 bytes per instruction) reaches 9 TB/s out of L2 on this chip,
// row pieces 28 TB/s.  No workgroup barrier until the partial sums meet.
// Waiting: copies into LDS and loads into registers share the counter and complete in order within their
// own kind, so "at most the copies of RING - 1 stages outstanding" says that the oldest stage has
// landed whatever else is in flight; the weight loads are the compiler's own, which waits for
// them by their own count (the copies it does not see only make it wait earlier than needed).
// The price: the count includes the weight loads, so such a wait is also one for every weight load but the
// newest.  With a ring of two stages the loads issued at the end of a step have landed by the second half of the
// next step (where a step has more of them than a stage has copies, some by its first half), so that beyond the
// first D steps, which are requested together, the weights are about half a step ahead, whatever D is.
// Long K at few rows is bound by that: 4096 x 14336 int4 groups, 32 rows, takes 18 us, 2 us a step.
// Group scales multiply the weights (one binary16 rounding per weight), as in the large fp16 kernel.
// XB: blocks of 8 token rows.
template <int FMT, int XB, int R, int RING, int D, int MAXT>
__global__ __launch_bounds__(MAXT) void skinny_f16_kernel(SkinnyArgs a) {
    static_assert((RING == 2 || RING == 4 || RING == 8) && (2 * D) % RING == 0, "static ring slots");
    constexpr int TB = (XB + 1) / 2;
    constexpr int WV = FMT == kW8C ? 2 : 1;  // weight vectors per step and row tile
    constexpr int SLOT = TB * 2048;          // bytes of a half step in LDS
    static_assert((RING - 1) * XB <= 63, "6-bit wait counter");
    extern __shared__ u32x4 lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, q = lane >> 4;
    int rt0, m0, rows;
    if (!place(a, R, rt0, m0, rows)) return;  // (whole workgroups only)

    const int t0 = wave * a.steps_q + min(wave, a.steps_rem);
    const int nt = a.steps_q + (wave < a.steps_rem ? 1 : 0);
    const int nst = 2 * nt;
    const int nst_copy = min(nst, (a.K + 63) / 64 - 2 * t0);  // half steps that hold any k below K

    // (the last workgroup's row tiles may run past the layer's: they are clamped, results dropped)
    const u32x4 *wrow[R];
#pragma unroll
    for (int r = 0; r < R; ++r) wrow[r] = a.w + (size_t)min(rt0 + r, a.RT - 1) * a.rt_stride * 64;
    u32x4 wv[D][R][WV];
    u32x2 sv[D][R];
    auto load_w = [&](int slot, int t) __attribute__((always_inline)) {
        const int u = t >> 3;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (FMT == kW4G32) {
                const int spos = min(8 * u + 8, a.KT) + u;  // scale tile of the unit
                sv[slot][r] = reinterpret_cast<const u32x2 *>(wrow[r] + (size_t)spos * 64 + ((t & 7) >> 1) * 16 + c)[t & 1];
            }
#pragma unroll
            for (int v = 0; v < WV; ++v)
                wv[slot][r][v] = __builtin_nontemporal_load(wrow[r] + (size_t)(FMT == kW8C ? 2 * t + v : FMT == kW4G32 ? t + u : t) * 64 + lane);
        }
    };
    // copies of a half step: KiB i = token rows 8 i .. 8 i + 7, lane = (row, octet position).  Rows past the last (their
    // products are dropped) take the data of rows `back` before them, of the block before where the block is less than half
    // full: no line is copied by more than two instructions of a wavefront (many copies of the same lines in flight have been
    // seen to reach LDS after the counter said they were done, see gemm_i8.hip; this ring is reused for the partial sums).
    // (not copying them at all costs 3 to 20 %: lane masks, and a count of copies that is not a constant any more)
    const bool own = rows >= 4 * XB || m0 == 0;
    const int before = own ? 0 : a.block_rows, back = !own ? a.block_rows : m0 > 0 ? rows & ~7 : rows >= 16 ? 16 : 8;
    const char *xbase = reinterpret_cast<const char *>(a.x) + (size_t)(m0 - before) * a.K * 2;
    const int K8 = a.K / 8;
    const uint32_t ring0 = (uint32_t)(uintptr_t)(lptr_t)lds + wave * (RING * SLOT);
    auto copy_stage = [&](int s, int slot) __attribute__((always_inline)) {
        const int o0 = (2 * t0 + s) * 8;
        auto copy = [&](int i) __attribute__((always_inline)) {
            const int rl = 8 * i + (lane >> 3), o = o0 + ((lane & 7) ^ ((rl >> 1) & 7));
            const int row = before + (rl < rows ? rl : min(max(rl - back, -before), rows - 1));
            const uint32_t off = ((uint32_t)row * (uint32_t)K8 + (uint32_t)o) * 16u;
            copy16_to_lds(xbase, off, __builtin_amdgcn_readfirstlane(ring0 + slot * SLOT + i * 1024));
        };
        if (o0 + 8 <= K8) {
#pragma unroll
            for (int i = 0; i < XB; ++i) copy(i);
            return;
        }
        // octets beyond K: zeros (their weights are zero too, but zero times an infinity is not).  All eight, or
        // (K is a multiple of 32) the upper four: of an even KiB the lanes with bit 2 set hold those, of an odd KiB the others.
        auto clear = [&](int i) __attribute__((always_inline)) { lds[(wave * (RING * SLOT) + slot * SLOT + i * 1024) / 16 + lane] = u32x4{0, 0, 0, 0}; };
        if (o0 >= K8) {
#pragma unroll
            for (int i = 0; i < XB; ++i) clear(i);
        } else {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                if (((lane >> 2) & 1) == p) {
#pragma unroll
                    for (int i = p; i < XB; i += 2) copy(i);
                } else {
#pragma unroll
                    for (int i = p; i < XB; i += 2) clear(i);
                }
            }
        }
    };

    v4f acc[R][TB];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) acc[r][tb] = v4f{0.0f, 0.0f, 0.0f, 0.0f};

#pragma unroll
    for (int i = 0; i < D; ++i)
        if (i < nt) load_w(i, t0 + i);
#pragma unroll
    for (int s = 0; s < RING; ++s)
        if (s < nst) copy_stage(s, s);

    const char *xread = reinterpret_cast<const char *>(lds) + wave * (RING * SLOT) + c * 128;
    const int swz = (c >> 1) & 7;
    for (int b = 0; b < nt; b += D) {
#pragma unroll
        for (int i = 0; i < D; ++i) {
            if (b + i < nt) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int s = 2 * (b + i) + h;
                    const int slot = (2 * i + h) & (RING - 1);
                    if (s + RING <= nst_copy)
                        wait_mem<(RING - 1) * XB>();
                    else
                        wait_mem<0>();
                    v8h xv[2][TB];
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const int oct = FMT == kW8C ? 2 * q + j : 4 * j + q;
#pragma unroll
                        for (int tb = 0; tb < TB; ++tb)
                            xv[j][tb] = *reinterpret_cast<const v8h *>(xread + slot * SLOT + tb * 2048 + ((oct ^ swz) << 4));
                    }
                    wait_lds();  // the operands are in registers: their slot may be overwritten
                    if (s + RING < nst) copy_stage(s + RING, slot);
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            v8h fa;
                            h2 sc = {(_Float16)1.0f, (_Float16)1.0f};
                            if (FMT == kW4G32) sc = as_h2(__builtin_amdgcn_perm(0u, sv[i][r][h], j ? 0x03020302u : 0x01000100u));
                            if (FMT == kW8C)
                                fa = dequant8(wv[i][r][h][2 * j], wv[i][r][h][2 * j + 1]);
                            else
                                fa = dequant4<FMT == kW4G32>(wv[i][r][0][2 * h + j], sc);
#pragma unroll
                            for (int tb = 0; tb < TB; ++tb) acc[r][tb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(xv[j][tb], fa, acc[r][tb], 0, 0, 0);
                        }
                    }
                }
                if (b + i + D < nt) load_w(i, t0 + b + i + D);
            }
        }
    }
    __syncthreads();  // every wavefront is done with its ring
    float *red = reinterpret_cast<float *>(lds);
    put_partials<R, TB>(red, acc, wave, lane);
    __syncthreads();
    finish<R, TB, float, FMT != kW4G32>(a, red, blockDim.x >> 6, rt0, m0, rows);
}

// ---------------------------------------------------------------- int8 activations
// The quantized activations arrive in MFMA operand order (KiB tiles), so both operands go from memory
// straight into registers, D steps of 128 k ahead, every load instruction one contiguous KiB.  Codes of
// 4-bit weights are expanded as in gemm_i8.hip (sums times 16).
template <bool W4, int TB, int R, int D, int MAXT>
__global__ __launch_bounds__(MAXT) void skinny_i8_kernel(SkinnyArgs a) {
    constexpr int WV = W4 ? 1 : 2;
    extern __shared__ u32x4 lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int rt0, m0, rows;
    if (!place(a, R, rt0, m0, rows)) return;
    const int t0 = wave * a.steps_q + min(wave, a.steps_rem);
    const int nt = a.steps_q + (wave < a.steps_rem ? 1 : 0);
    const int XT = a.Kp / 64;
    const int first = a.turned ? rt0 / R / 8 % nt : 0;  // (whole row groups, so that token blocks still share weights in L2)
    auto step = [&](int i) __attribute__((always_inline)) { return t0 + (i + first < nt ? i + first : i + first - nt); };
    // (a block's last tiles of 16 rows may lie past the rows there are: clamped, results dropped)
    const u32x4 *xtile[TB];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) xtile[tb] = a.x + (size_t)min(m0 / 16 + tb, (a.M - 1) / 16) * XT * 64;

    const u32x4 *wrow[R];
#pragma unroll
    for (int r = 0; r < R; ++r) wrow[r] = a.w + (size_t)min(rt0 + r, a.RT - 1) * a.rt_stride * 64;
    u32x4 wv[D][R][WV], xv[D][TB][2];
    auto load = [&](int slot, int t) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int v = 0; v < WV; ++v) wv[slot][r][v] = __builtin_nontemporal_load(wrow[r] + (size_t)(W4 ? t : 2 * t + v) * 64 + lane);
#pragma unroll
        for (int tb = 0; tb < TB; ++tb)
#pragma unroll
            for (int v = 0; v < 2; ++v) xv[slot][tb][v] = xtile[tb][(size_t)(2 * t + v) * 64 + lane];
    };
    v4i acc[R][TB];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) acc[r][tb] = v4i{0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < D; ++i)
        if (i < nt) load(i, step(i));
    for (int b = 0; b < nt; b += D) {
#pragma unroll
        for (int i = 0; i < D; ++i) {
            if (b + i < nt) {
#pragma unroll
                for (int v = 0; v < 2; ++v) {  // k steps of 64
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        v4i fw;
                        if (W4) {
                            const uint32_t px = wv[i][r][0][2 * v], py = wv[i][r][0][2 * v + 1];
                            fw[0] = (int)(((px << 4) & 0xF0F0F0F0u) ^ 0x80808080u);
                            fw[1] = (int)((px & 0xF0F0F0F0u) ^ 0x80808080u);
                            fw[2] = (int)(((py << 4) & 0xF0F0F0F0u) ^ 0x80808080u);
                            fw[3] = (int)((py & 0xF0F0F0F0u) ^ 0x80808080u);
                        } else {
                            fw = __builtin_bit_cast(v4i, wv[i][r][W4 ? 0 : v]);
                        }
#pragma unroll
                        for (int tb = 0; tb < TB; ++tb)
                            acc[r][tb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(v4i, xv[i][tb][v]), fw, acc[r][tb], 0, 0, 0);
                    }
                }
                if (b + i + D < nt) load(i, step(b + i + D));
            }
        }
    }
    int *red = reinterpret_cast<int *>(lds);
    put_partials<R, TB>(red, acc, wave, lane);
    __syncthreads();
    finish<R, TB, int, true>(a, red, blockDim.x >> 6, rt0, m0, rows);
}

constexpr int kStreamSteps = 4, kStreamTiles = 2;

// The same products for up to 32 token rows and many channels: the workgroups stay (one grid of them fills the chip), a wavefront keeps
// its 512 k of the token rows in registers for good and walks over row tiles, two at a time.  A vector of weights is requested
// again, for the next tile, as soon as it has been multiplied, so that the weights' stream does not stop between tiles, and it is the
// only one: the token rows are read once per workgroup instead of once per four row tiles or so.
// What bounds it: the stream, which a barrier per group and the store phase still hold up (5.9 to 6.2 TB/s with K of 4096 and 8192). us, 24
// token rows, skinny_i8_kernel / this: 65536 x 4096 57.7 / 46.0; 128256 x 4096 103 / 90 (9 rows 98 / 84); 256000 x 4096 196 / 181; 65536 x
// 8192 105 / 88; 100000 x 1024 27.7 / 21.5.  Two row tiles at a time: with one the compiler has no registers left for requests in flight
// across the store phase.  4-bit weights, half the bytes in flight: 128256 x 4096 32 rows 49 / 53, not built.
template <int TB>
__global__ __launch_bounds__(1024) void skinny_i8_stream_kernel(SkinnyArgs a) {
    constexpr int R = kStreamTiles, KS = 2 * kStreamSteps;  // KS: k steps of 64 of a wavefront
    extern __shared__ u32x4 lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = blockDim.x >> 6, XT = a.Kp / 64, s0 = wave * KS;
    v4i xv[KS][TB];
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) {
            // (token rows past the last tile of 16: clamped, results dropped)
            xv[s][tb] = __builtin_bit_cast(v4i, a.x[((size_t)min(tb, (a.M - 1) / 16) * XT + s0 + s) * 64 + lane]);
        }
    u32x4 wv[KS];
    auto load = [&](int s, int tile) __attribute__((always_inline)) {
        wv[s] = __builtin_nontemporal_load(a.w + ((size_t)min(tile, a.RT - 1) * a.rt_stride + s0 + s) * 64 + lane);
    };
    int tile = blockIdx.x * R, buf = 0;
    const int stride = gridDim.x * R;
#pragma unroll
    for (int s = 0; s < KS; ++s) load(s, tile);
    auto group = [&](auto more) __attribute__((always_inline)) {
        v4i acc[R][TB];
#pragma unroll
        for (int r = 0; r < R; ++r) {
#pragma unroll
            for (int tb = 0; tb < TB; ++tb) acc[r][tb] = v4i{0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < KS; ++s) {
#pragma unroll
                for (int tb = 0; tb < TB; ++tb)
                    acc[r][tb] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xv[s][tb], __builtin_bit_cast(v4i, wv[s]), acc[r][tb], 0, 0, 0);
                if (r + 1 < R || decltype(more)::value) load(s, r + 1 < R ? tile + r + 1 : tile + stride);
            }
        }
        int *red = reinterpret_cast<int *>(lds) + buf * (waves * R * TB * 256);
        put_partials<R, TB>(red, acc, wave, lane);
        // (two buffers: whoever writes this one again has passed the barrier of the group in between, behind which nobody reads it.  The
        // requests of weights stay in flight.)
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        finish<R, TB, int, true>(a, red, waves, tile, 0, a.M);
        buf ^= 1;
    };
    for (; tile + stride < a.RT; tile += stride) group(std::true_type());
    group(std::false_type());
}

constexpr size_t kLdsLimit = 160 * 1024;

unsigned stream_grid(const SkinnyArgs &a, int waves, int num_cus) {  // (16 wavefronts of 128 registers fill a compute unit)
    return min((unsigned)((a.RT + kStreamTiles - 1) / kStreamTiles), (unsigned)(16 / waves * num_cus));
}

// Which int8 layers skinny_i8_stream_kernel takes (8-bit weights).  K of whole multiples of 4096: there the other kernel's workgroups are 64 KiB apart
// and meet in few memory channels, while here those of a compute unit spread over K.  us, that one / this, 24 rows: 32768 x 4096 26.9 / 25.3,
// 100000 x 4096 84.8 / 72.5, x 8192 161 / 136.  At other K both are level (65536 x 3072 36.6 / 36.1, x 5120 57.8 / 56.6, x 6144 66.2 / 67.5) or
// this loses (202048 x 2048 72 / 78; x 2560, five wavefronts on four SIMDs, 89 / 104).  From two rounds of the grid on, the last
// at least four fifths full: 28672 x 4096 20 rows 23.6 / 23.9; with K of 8192, where one workgroup fills a compute unit and nothing runs beside
// its last round, nine tenths from the fourth round on: 33000, 4.03 rounds, 16 rows 46.6 / 49.4, 26624, 3.25 rounds, 24 rows 40.4 / 41.7, 50304, 6.14
// rounds, 69.5 / 72.3, but 31104, 3.8 rounds, 51.4 / 47.8; up to 16 rows with K of 4096, whose stream leaves less to hide it in, from the fifth
// (99936, 6.1 rounds, 9 rows 66.8 / 69.4, 131758, 8.04 rounds, 10 rows 86.6 / 89.2; 57344, 3.5 rounds, 41.5 / 38.9).  K of 512 and 1024: the other kernel's
// wavefronts have one or
// two steps (152064 x 512 20.9 / 18.4; 65536 x 1024 19.8 / 15.1, 256000 x 1024 59.1 / 53.6).  There one or two wavefronts store a row tile, and that shows
// with many channels: up to 16 rows from about 160000 on (250000 x 512 9 rows 25.3 / 26.3, 164748 x 992 10 rows 31.5 / 32.5, 200000 x 1024 36.6 / 37.9;
// 140000 x 512 17.0 / 15.7), rows of single values earlier (131070 x 512 16 rows 16.6 / 18.0, 200001 x 1024 32 rows 50.4 / 55.4; 100002 24 rows 26.6 /
// 25.5).  Weights in HBM; both move by up to 10 % with where the weights lie, 152064 x 4096 12 rows 99.4 / 103.4 and 113 / 99 in two processes.
bool stream_takes(const SkinnyArgs &a, int num_cus) {
    if (a.M > 32 || tuning().skinny_waves > 0 || tuning().skinny_row_tiles > 0 || tuning().skinny_blocks > 0) return false;
    const int steps = a.Kp / 128, waves = steps / kStreamSteps;
    if (steps % kStreamSteps != 0 || waves > 16) return false;
    const int groups = (a.RT + kStreamTiles - 1) / kStreamTiles, grid = 16 / waves * num_cus;
    if (a.Kp <= 1024) return groups >= grid && (a.N % 4 != 0 ? a.N < 110000 : a.M > 16 || a.N < 155000);
    const int rounded = (groups + grid - 1) / grid * grid;
    const bool four_fifths = a.Kp == 4096 ? a.M > 16 || groups <= 4 * grid : groups <= 3 * grid;
    return a.Kp % 4096 == 0 && groups >= 2 * grid && (four_fifths ? 5 * groups >= 4 * rounded : 10 * groups >= 9 * rounded);
}

void split_steps(SkinnyArgs &a, int steps, int waves) {
    a.steps_q = steps / waves;
    a.steps_rem = steps % waves;
}

unsigned grid_for(const SkinnyArgs &a, int R) {
    const int groups = (a.RT + R - 1) / R;
    return (unsigned)(a.blocks > 1 ? round_up(groups, 8) * a.blocks : groups);
}

// Workgroups of the fullest XCD per compute unit of it (whose workgroups of one row group stay together).
float load_per_cu(const SkinnyArgs &a, int R, int num_cus) {
    const int groups = (a.RT + R - 1) / R;
    return a.blocks > 1 ? (float)((groups + 7) / 8 * a.blocks) * 8.0f / (float)num_cus : (float)groups / (float)num_cus;
}

// Wavefronts per workgroup: at most `most`, every one with the same number of steps if it divides; four where
// there are more workgroups than compute units, so that two share one and overlap (64 and 128 token rows, 18432 x
// 2304: 24.2 / 19.3 and 34.2 / 26.2 us with eight / four; 28672 x 4096 32.1 / 29.0 and 57.0 / 49.7; level for K of 9216 and 14336).
int waves_for(int steps, int most, unsigned workgroups, int num_cus) {
    const int forced = tuning().skinny_waves;
    if (forced > 0 && forced < most) most = forced;
    if (forced == 0 && workgroups > (unsigned)num_cus && most > 4) most = 4;
    const int w = steps < most ? steps : most;
    const int per = (steps + w - 1) / w;
    return (steps + per - 1) / per;
}

template <int FMT, int XB, int R>
hipError_t launch_f16(SkinnyArgs a, int num_cus, hipStream_t st) {
    constexpr int TB = (XB + 1) / 2;
    constexpr int RING = XB <= 2 ? 4 : 2;
    constexpr int D0 = R == 1 ? 8 : R <= 3 ? 4 : 2, D = FMT == kW8C && D0 > 2 ? D0 / 2 : D0;
    constexpr bool kWide = R == 1 && XB <= 4 && FMT != kW8C;  // few enough registers for 16 wavefronts
    constexpr int MAXT = kWide ? 1024 : 512;
    constexpr size_t ring = RING * TB * 2048, red = (size_t)R * TB * 1024, per_wave = ring > red ? ring : red;
    constexpr int most = (int)(kLdsLimit / per_wave) < MAXT / 64 ? (int)(kLdsLimit / per_wave) : MAXT / 64;
    const int steps = (a.K + 127) / 128, waves = waves_for(steps, most, grid_for(a, R), num_cus);
    split_steps(a, steps, waves);
    if (const hipError_t e = allow_dynamic_lds<skinny_f16_kernel<FMT, XB, R, RING, D, MAXT>>(kLdsLimit); e != hipSuccess) return e;
    skinny_f16_kernel<FMT, XB, R, RING, D, MAXT><<<dim3(grid_for(a, R)), dim3((unsigned)(waves * 64)), waves * per_wave, st>>>(a);
    return hipGetLastError();
}

template <bool W4, int TB, int R>
hipError_t launch_i8(SkinnyArgs a, int num_cus, hipStream_t st) {
    constexpr int VECS = R * (W4 ? 1 : 2) + 2 * TB;  // vectors per step
    constexpr int D = VECS <= 4 ? 4 : VECS <= 6 ? 3 : VECS <= 14 ? 2 : R * TB >= 12 ? 1 : 2;
    constexpr bool kWide = R == 1 && TB <= 2;
    constexpr int MAXT = kWide ? 1024 : 512;
    constexpr size_t per_wave = (size_t)R * TB * 1024;
    const int steps = a.Kp / 128, waves = waves_for(steps, MAXT / 64, grid_for(a, R), num_cus);
    split_steps(a, steps, waves);
    if (const hipError_t e = allow_dynamic_lds<skinny_i8_kernel<W4, TB, R, D, MAXT>>(kLdsLimit); e != hipSuccess) return e;
    skinny_i8_kernel<W4, TB, R, D, MAXT><<<dim3(grid_for(a, R)), dim3((unsigned)(waves * 64)), waves * per_wave, st>>>(a);
    return hipGetLastError();
}

template <int TB>
hipError_t launch_i8_stream(const SkinnyArgs &a, int num_cus, hipStream_t st) {
    const int waves = a.Kp / 128 / kStreamSteps;
    const size_t bytes = (size_t)2 * waves * kStreamTiles * TB * 1024;  // (at most 128 KiB)
    if (const hipError_t e = allow_dynamic_lds<skinny_i8_stream_kernel<TB>>(kLdsLimit); e != hipSuccess) return e;
    skinny_i8_stream_kernel<TB><<<dim3(stream_grid(a, waves, num_cus)), dim3((unsigned)(waves * 64)), bytes, st>>>(a);
    return hipGetLastError();
}

// Row tiles per workgroup, of the counts built: the busiest compute unit has `load` row tiles of weights
// to pull from memory and load / r times the token rows from L2, which deliver a byte about
// 2.5 times as fast (fitted to the sweep over r = 1 .. 8 of layers of 2304 to 28672 channels at 12 to 64 token rows).
template <int... RS>
int pick_row_tiles(const SkinnyArgs &a, float weight_bytes, float token_bytes, int num_cus, std::integer_sequence<int, RS...>) {
    const int forced = tuning().skinny_row_tiles;
    int best = 0;
    float best_cost = 0.0f;
    for (const int r : {RS...}) {
        if (a.gated_act >= 0 && r % 2) continue;
        if (forced == r) return r;
        // many rounds: balance does not matter, fewer registers and more workgroups per compute unit do
        // (128256 channels at 12 and 32 token rows, 4-bit weights: 54 and 61 us with 4, 61 and 69 us with 7 or 8)
        if (r > 4 && a.RT >= 16 * num_cus) continue;
        const float cost = ceilf(load_per_cu(a, r, num_cus)) * ((float)r * 16.0f * weight_bytes + 0.4f * (float)a.block_rows * token_bytes);
        if (best == 0 || cost < best_cost) best = r, best_cost = cost;
    }
    return best;
}

template <int FMT, int XB, int... RS>
hipError_t f16_rows(const SkinnyArgs &a, int num_cus, hipStream_t st, std::integer_sequence<int, RS...> rs) {
    const int pick = pick_row_tiles(a, FMT == kW8C ? 1.0f : FMT == kW4G32 ? 0.5625f : 0.5f, 2.0f, num_cus, rs);
    hipError_t e = hipErrorInvalidValue;
    ((pick == RS ? (void)(e = launch_f16<FMT, XB, RS>(a, num_cus, st)) : (void)0), ...);
    return e;
}

template <bool W4, int TB, int... RS>
hipError_t i8_rows(const SkinnyArgs &a, int num_cus, hipStream_t st, std::integer_sequence<int, RS...> rs) {
    const int pick = pick_row_tiles(a, W4 ? 0.5f : 1.0f, 1.0f, num_cus, rs);
    hipError_t e = hipErrorInvalidValue;
    ((pick == RS ? (void)(e = launch_i8<W4, TB, RS>(a, num_cus, st)) : (void)0), ...);
    return e;
}

// Row tiles per workgroup the kernels are built for (registers and LDS bound them: R * TB sums per lane)
typedef std::integer_sequence<int, 1, 2, 3, 4, 5, 6, 7, 8> Rows2;  // up to 32 token rows
typedef std::integer_sequence<int, 1, 2, 3, 4, 5, 6, 7> Rows2W8;
typedef std::integer_sequence<int, 1, 2, 3, 4, 5, 6> Rows3;
typedef std::integer_sequence<int, 1, 2, 3, 4> Rows4;

// (the same choice as f16_any and i8_any make)
int row_tiles_for(const SkinnyArgs &a, int fmt, bool int8_activations, int num_cus) {
    const float wb = fmt == kW8C ? 1.0f : fmt == kW4G32 ? 0.5625f : 0.5f, xb = int8_activations ? 1.0f : 2.0f;
    switch ((a.block_rows + 15) / 16) {
        case 1: return pick_row_tiles(a, wb, xb, num_cus, Rows2());
        case 2: return fmt == kW8C && !int8_activations ? pick_row_tiles(a, wb, xb, num_cus, Rows2W8()) : pick_row_tiles(a, wb, xb, num_cus, Rows2());
        case 3: return pick_row_tiles(a, wb, xb, num_cus, Rows3());
        case 4: return pick_row_tiles(a, wb, xb, num_cus, Rows4());
    }
    return 0;
}

template <int FMT>
hipError_t f16_any(const SkinnyArgs &a, int num_cus, hipStream_t st) {
    switch ((a.block_rows + 7) / 8) {
        case 1: case 2: return f16_rows<FMT, 2>(a, num_cus, st, Rows2());
        case 3: case 4: return f16_rows<FMT, 4>(a, num_cus, st, std::conditional_t<FMT == kW8C, Rows2W8, Rows2>());
        case 5: case 6: return f16_rows<FMT, 6>(a, num_cus, st, Rows3());
        case 7: case 8: return f16_rows<FMT, 8>(a, num_cus, st, Rows4());
    }
    return hipErrorInvalidValue;
}

template <bool W4>
hipError_t i8_any(const SkinnyArgs &a, int num_cus, hipStream_t st) {
    switch ((a.block_rows + 15) / 16) {
        case 1: return i8_rows<W4, 1>(a, num_cus, st, Rows2());
        case 2: return i8_rows<W4, 2>(a, num_cus, st, Rows2());
        case 3: return i8_rows<W4, 3>(a, num_cus, st, Rows3());
        case 4: return i8_rows<W4, 4>(a, num_cus, st, Rows4());
    }
    return hipErrorInvalidValue;
}

// Estimated time in us with R row tiles per workgroup, fitted to a sweep over formats, 2304 to 28672 channels, K of 2048 to
// 14336, 12 to 300 token rows in blocks of 16 to 64 and R of 1 to 8 (standard deviation 13 %).
float estimate_us(const SkinnyArgs &a, int fmt, bool int8_activations, int R, int num_cus) {
    const float l = load_per_cu(a, R, num_cus), k = 1e-3f * (float)a.K, r = (float)R, rows = (float)round_up(a.block_rows, 16);
    const float load = fmaxf(1.0f, 0.5f * (l + ceilf(l)));
    if (int8_activations) return load * (2.0f + 0.28f * r + k * (0.16f + 0.0118f * rows + (fmt == kW8C ? 0.23f : 0.08f) * r + 0.0023f * r * rows));
    const float w = fmt == kW8C ? 0.27f : fmt == kW4G32 ? 0.24f : 0.13f;
    return load * (1.9f + 0.45f * r + k * (0.21f + 0.0148f * rows + w * r + 0.0031f * r * rows));
}

// Equal blocks of whole tiles of 16 token rows (one block: all of them)
void cut_rows(SkinnyArgs &a, int blocks) {
    a.block_rows = round_up((a.M + blocks - 1) / blocks, blocks > 1 ? 16 : 1);
    a.blocks = (a.M + a.block_rows - 1) / a.block_rows;
}

// Blocks the token rows are cut into: as few as there can be, or more of 48, 32 or 16 rows where that is estimated to save a
// twentieth.  Every compute unit pulls its block of x through its vector cache; a layer of few row tiles leaves
// compute units idle, or gives each one row tile for up to 64 rows, and more blocks with more row tiles each pull fewer bytes:
// x falls with the blocks, weights (once per block, from the XCD's L2) rise.  us, fewest blocks / like this:
// int4 groups, binary16  4096 x 14336 64 rows 28.4 / 22.7; 2304 x 9216 77 rows 17.4 / 15.2, 128 20.6 / 17.7, 200 24.4 / 21.4
// int8, binary16         2304 x 9216 77 rows 19.1 / 16.3, 200 26.3 / 23.1
// int8 x int8            2304 x 9216 48 rows 13.0 / 10.8, 77 14.7 / 12.8; 6144 x 4096 64 rows 10.9 / 10.1
// int8 x int4            4096 x 14336 20 rows 13.6 / 12.1, 64 19.2 / 15.3; 6144 x 4096 64 rows 9.3 / 7.7; 2304 x 9216 77 rows 11.9 / 9.3
// (over 11 layers, 16 numbers of rows and each format 2 to 4 % faster on average; the worst where these kernels are taken at all: 2304 x 2048
// int4 groups, 400 rows 11.5 / 12.0; wide layers keep the fewest blocks: 28672 x 4096 int4 groups, 64 rows 30.9 / 34.9 with two.)
void choose_blocks(SkinnyArgs &a, int fmt, bool int8_activations, int num_cus) {
    if (tuning().skinny_blocks > 0) return;
    const SkinnyArgs fewest = a;
    float limit = 0.95f * estimate_us(a, fmt, int8_activations, row_tiles_for(a, fmt, int8_activations, num_cus), num_cus);
    for (const int rows : {48, 32, 16}) {
        SkinnyArgs b = fewest;
        cut_rows(b, (a.M + rows - 1) / rows);
        if (b.blocks <= fewest.blocks) continue;
        const float us = estimate_us(b, fmt, int8_activations, row_tiles_for(b, fmt, int8_activations, num_cus), num_cus);
        if (us < limit) a = b, limit = us;
    }
}

SkinnyArgs make_args(const Geometry &g, const void *packed, const void *x, const float *sx, int M, void *out,
                     const void *residual, int gated_act) {
    SkinnyArgs a;
    a.w = static_cast<const u32x4 *>(packed);
    a.x = static_cast<const u32x4 *>(x);
    a.sw = reinterpret_cast<const float *>(static_cast<const char *>(packed) + g.scale_off);
    a.sx = sx;
    a.res = static_cast<const _Float16 *>(residual);
    a.out = out;
    a.M = M;
    a.N = g.N;
    a.K = g.K;
    a.Kp = g.Kp;
    a.KT = g.KT;
    a.RT = g.RT;
    a.rt_stride = g.rt_stride;
    a.steps_q = a.steps_rem = 0;
    const int fewest = (M + kSkinnyRows - 1) / kSkinnyRows, forced = tuning().skinny_blocks;
    cut_rows(a, forced > fewest ? forced : fewest);
    a.sw_mul = 1.0f;
    a.turned = 0;
    a.gated_act = g.pair_half ? gated_act : -1;
    return a;
}

}  // namespace

// 33 to 64 token rows, layers of so many channels that their 256-channel tiles fill half the compute units and more:
// the largest K up to which those tiles are the faster ones (0: none), by the share of the compute units that
// they fill.  Measured at 33 to 64 rows, 32768 to 256000 channels, K of 512 to 14336 (us at 64 rows, these kernels / the
// tiles, int8 activations with the quantization kernel):
//   int8 x int4  34000 x 2048 18.4 / 17.5, x 4096 27.3 / 26.0; 40000 x 1024 17.3 / 13.3, x 4096 32.0 / 27.1; 57000 x 8192 68.8 / 64.8
//   int8 x int8  40000 x 1024 19.8 / 17.5, x 4096 42.8 / 42.6; 75000 x 512 22.7 / 21.3, x 1024 29.5 / 30.9; 100000 x 2048 53.0 / 50.5
// (Drawn for int8 tiles with 32 x 32 MFMAs: the present ones are a few percent faster, so that a line by them would lie a little higher.)
// Binary16 activations with whole steps of K: tile_us says.
static int tiles_up_to_k(const Geometry &g, int M, bool int8_activations, int num_cus) {
    constexpr int kAll = 1 << 30;
    const float fill = (float)((g.N + 255) / 256) / (float)num_cus;
    const bool w8 = g.fmt == kW8C;
    if (M <= 32 || fill < 0.5f) return 0;
    if (int8_activations) {
        if (M <= 48) return w8 ? 1024 : fill <= 1.0f ? 2048 : fill < 1.5f ? 0 : 512;
        if (fill <= 1.0f) return fill < 0.6f ? 2048 : kAll;
        return !w8 ? kAll : fill < 1.5f ? 512 : 3072;
    }
    if (fill < 0.6f || fill > 1.0f || !w8) return 0;  // (K that is not whole steps)
    const bool wide = fill >= 0.75f;
    return M <= 48 ? (wide ? 512 : 0) : wide ? 1024 : 512;
}

// Which products these kernels take.  Up to 64 token rows: all but those.  More rows: the tiles of 64 or 128
// tokens take the same time until they fill the chip, and long (they leave most of it idle); here the
// rows are cut into blocks, with the time growing with their number.  Both times are estimated: here see estimate_us, which where
// the two are near each other (65 to 1024 rows, 1500 to 65536 channels, K of 896 to 14336, 721 shapes) is 1 to 7 % high in the median (hence the
// 1.05) and from 16 % low to 27 % high in eight of ten; tiles
//   tile_us (binary16 activations), 10 + 10.3 K / 1000 (128 x 128, K that is not whole steps: staged_tiles_us); int8_tile_us, 3.5 + 9.3 K / 1000
//   (int8 x int4, K of an odd number of 128)
// Measured (us, weights in HBM, tiles / here): 4096 x 14336 int4, binary16 activations, 77 rows 83 / 24, 300 83 / 63, 512 83 / 76;
// 2304 x 9216 int4 groups 77 rows 65 / 15, 300 66 / 26, 1000 67 / 65; 18432 x 2304 77 rows 20.3 / 20.2, 200 29 / 40;
// 11000 x 3008 300 rows 50 / 37; int8, binary16 18432 x 2304 150 rows 24 / 35, 14336 x 4096 640 rows 78 / 118;
// int8 x int8  4096 x 14336 191 rows 39 / 29; 2048 x 14336 1002 rows 55 / 76; 4096 x 9216 214 rows 40 / 29, 516 rows 46 / 56; 6144 x 4096 300 rows 21.9 / 24.8
// int8 x int4  4096 x 14336 300 rows 39 / 47; 2304 x 9216 300 rows 28.5 / 20.7, 814 rows 30.5 / 41.7; 6144 x 4096 300 rows 17.5 / 20.0
static float skinny_us(const Geometry &g, int M, bool int8_activations, bool gated, int num_cus) {
    SkinnyArgs a = make_args(g, nullptr, nullptr, nullptr, M, nullptr, nullptr, gated ? 0 : -1);
    choose_blocks(a, g.fmt, int8_activations, num_cus);
    return estimate_us(a, g.fmt, int8_activations, row_tiles_for(a, g.fmt, int8_activations, num_cus), num_cus);
}

// Binary16 activations, 128 x 128 tiles: two workgroups share a compute unit, so that a second tile on it costs a third to
// three quarters of the first.  us, rounds of one tile per compute unit / this: 24000 x 8192 int8 65 rows, 0.73 rounds 93 / 94; 130 rows, 1.47
// 133 / 145; 277 rows, 2.2 224 / 255; 400 rows, 2.94 241 / 255; 640 rows, 3.67 306 / 299; 18432 x 3040 int4 800 rows, 3.94 115 / 135;
// 28672 x 4128 int4 800 rows, 6.13 264 / 305.
static float staged_tiles_us(const Geometry &g, int M, int num_cus) {
    const float fill = (float)((g.N + 127) / 128 * ((M + 127) / 128)) / (float)num_cus;
    const float pairs = floorf(0.5f * fill), rest = fill - 2.0f * pairs;
    const float last = rest == 0.0f ? 0.0f : rest > 1.0f ? 0.95f + 0.4f * rest : pairs == 0.0f ? 1.0f : 1.15f;
    return (10.0f + 10.3e-3f * (float)g.K) * (1.55f * pairs + last);
}

// Binary16 activations: what the plan of choose_blocks takes, for the choice between it and the large tiles.  estimate_us ranks the
// plans of one layer; across layers it is 23 % off (at K of 256 up to twice), this 9 %: fitted to 2870 shapes of 768 to 40000 channels, K of 128 to 14336
// and 9 to 1024 rows.  The choice is 0.3 % slower than the faster of both (estimate_us 1.1 %, with single shapes 1.5 times slower).
static float few_rows_us(const Geometry &g, int M, bool gated, int num_cus) {
    SkinnyArgs a = make_args(g, nullptr, nullptr, nullptr, M, nullptr, nullptr, gated ? 0 : -1);
    choose_blocks(a, g.fmt, false, num_cus);
    const int R = row_tiles_for(a, g.fmt, false, num_cus);
    const float l = load_per_cu(a, R, num_cus), k = 1e-3f * (float)g.K, r = (float)R, rows = (float)round_up(a.block_rows, 16);
    const float w = g.fmt == kW8C ? 0.337f : g.fmt == kW4G32 ? 0.288f : 0.191f;
    return 4.0f + fmaxf(1.0f, 0.5f * (l + ceilf(l))) * (0.0053f * r * rows + k * (0.0106f * rows + w * r + 0.0036f * r * rows));
}

// Binary16 activations: rows to leave to the kernels here where the tiles of the others then end with a full round, or without a tile of
// few rows, if that is estimated to save more than a second launch and a fiftieth; 0: none.  Returns the estimated time.
// us, tiles alone / like this: 2304 x 9216 int4 groups 3700 rows 164 / 137; 8192 x 4096 int8 1030 rows 69 / 67; 4096 x 4096 int4 2060 rows
// 63 / 55; 6144 x 4096 int4 3100 rows 131 / 119; 14336 x 14336 int4 groups 1271 rows 495 / 444.  Of 1500 random shapes the worst lost 6 %; a worse
// one is 22016 x 14336 int4 351 rows, 207 / 220.
static float tail_rows(const Geometry &g, int M, bool gated, int num_cus, int *rest) {
    int form;
    float best = tile_us(g, M, num_cus, &form);
    *rest = 0;
    if (tuning().gemm_variant != 0 || tuning().skinny_max_m >= 0) return best;
    const int n_tiles = (g.N + 255) / 256, form_rows = tile_rows(form);
    if (n_tiles * ((M + form_rows - 1) / form_rows) <= num_cus) return best;  // (one round: a tile of few rows keeps nothing waiting)
    for (const int rows : {form_rows, 128}) {  // (128: the best where no rows are left over)
        const int m_tiles = (M + rows - 1) / rows;
        const int full = (n_tiles * m_tiles - 1) / num_cus * num_cus / n_tiles * rows, whole = (M - 1) / rows * rows;
        for (const int most : {full, whole}) {
            const int r = M - most;
            if (most < 128 || r > kSkinnyMaxM) continue;
            const float us = tile_us(g, most, num_cus, &form) + few_rows_us(g, r, gated, num_cus) + 1.0f;
            if (us < 0.98f * best) best = us, *rest = r;
        }
        if (rows == 128) break;
    }
    return best;
}

int skinny_tail_rows(const Geometry &g, int M, bool gated, int num_cus) {
    int rest;
    tail_rows(g, M, gated, num_cus, &rest);
    return rest;
}

bool skinny_product(const Geometry &g, int M, bool int8_activations, bool gated, int num_cus) {
    if (tuning().gemm_variant != 0) return false;  // a large kernel is asked for by name
    if (tuning().skinny_max_m >= 0) return M <= tuning().skinny_max_m;
    if (M <= kSkinnyRows && (int8_activations || !tile_kernel_takes(g))) return g.K > tiles_up_to_k(g, M, int8_activations, num_cus);
    if (M > kSkinnyMaxM) return false;
    if (!int8_activations && tile_kernel_takes(g)) {
        if (M <= kSkinnyRows && g.N < 8192) return true;  // (where the tiles win there, K = 256, it is by 0.3 us, and the estimate costs the host that)
        int rest;
        const float here = few_rows_us(g, M, gated, num_cus), tiles = tail_rows(g, M, gated, num_cus, &rest);
        // (1.05: where both estimates are level the kernels here are the faster more often; up to 16 rows, whose blocks are half empty, 1.1.
        // Half a microsecond: at K of 512 and less, where the products are little more than launches, the estimate here is high by up to 1.1. us, tiles /
        // here, weights in HBM: int8 1404 x 192 73 rows 4.8 / 3.6, 345 x 256 146 rows 5.2 / 3.0, int4 311 x 256 442 rows 5.5 / 3.9, int4 groups 3527 x 256 69
        // rows 5.4 / 5.0, 80000 x 1024 9 rows 26 / 22; the other way round int4 4258 x 256 122 rows 5.0 / 7.4, 28000 x 512 20 rows 6.4 / 7.6 (in the
        // cache 5.7 / 6.0), int4 groups 128256 x 4096 32 rows 68 / 79.  612 shapes whose estimates are near each other, weights in HBM: 0.55 % behind the faster
        // of both, 0.73 % with 1.05 alone; the worst int8 2338 x 128 81 rows, tiles 4.3, here 6.0, int8 19937 x 11520 68 rows 76 / 90, and the other
        // way round 221 x 128 95 rows 4.7 / 3.9, 4404 x 2304 394 rows 20.6 / 18.9)
        return here < fmaxf((M <= 16 ? 1.1f : 1.05f) * tiles, tiles + 0.5f);
    }
    const float here = skinny_us(g, M, int8_activations, gated, num_cus);
    const long m128 = (M + 127) / 128;
    if (!int8_activations) {
        // Up to eight wavefronts share the steps here, and the time is that of the one with most (4096 x 14432, 113 steps: 7 % more than
        // 4096 x 14336).  The choice is 0.2 % slower than the faster of both over 319 shapes of 1500 to 65536 channels, K of 1024 to 14432
        // and 65 to 1000 rows; us, tiles / here: 18432 x 3040 int4 800 rows 115 / 146, 4096 x 14432 1000 rows 161 / 188; int8 28672 x 8192 96 rows
        // 94 / 85, 25698 x 10368 277 rows 311 / 270, 24000 x 8192 400 rows 241 / 270.
        const int steps = (g.K + 127) / 128, per_wave = (steps + 7) / 8;
        const float uneven = (float)(per_wave * ((steps + per_wave - 1) / per_wave)) / (float)steps;
        return uneven * here < 1.05f * staged_tiles_us(g, M, num_cus);
    }
    const float k = 1e-3f * (float)g.K;
    const bool w8 = g.fmt == kW8C;
    if (!w8 && g.Kp / 128 % 2 != 0) {
        // 128 x 128 tiles with both operands staged: two share a compute unit at an eighth more than one (us, weights in HBM, tiles / here: 28672 x 4224 65
        // rows 49 / 32, 240 rows, 1.75 per compute unit 53 / 57, 384 rows, 2.6 93 / 85, 1000 rows, 7 181 / 225; 11000 x 9600 240 rows 100 / 55, 384 rows
        // 101 / 76; 6144 x 2944 384 rows 31 / 20).  The choice was 0.3 % slower than the faster of both over 220 such shapes, weights in the cache.
        const float fill = (float)((g.N + 127) / 128 * m128) / (float)num_cus;
        return here < 1.04f * (3.5f + 9.3f * k) * (fill <= 1.0f ? 1.0f : 0.12f + ceilf(0.5f * fill));
    }
    // (skinny_us put to measured times over 1772 shapes of 65 to 1024 rows, standard deviation 9 to 14 %; the choice is 0.35 % slower than the faster of both (0.95 and
    // 1.1 % with a line drawn where rows are stored in 16 bytes): us, tiles / here, 6875 x 256 77 rows 15.7 / 9.5, 4635 x 1280 420 rows 20.1 / 15.8, int4 8482 x
    // 1024 230 rows 16.5 / 14.1)
    int form;
    return (w8 ? 3.0f + 0.84f * here : 4.75f + 0.88f * here) < int8_tile_us(g, M, g.N % 8 == 0, num_cus, &form);
}

hipError_t launch_skinny_f16(const Geometry &g, const void *packed, const void *x, int M, void *y, const void *residual,
                             int gated_act, int num_cus, hipStream_t st) {
    SkinnyArgs a = make_args(g, packed, x, nullptr, M, y, residual, gated_act);
    choose_blocks(a, g.fmt, false, num_cus);
    if (g.fmt == kW8C) return f16_any<kW8C>(a, num_cus, st);
    return g.fmt == kW4C ? f16_any<kW4C>(a, num_cus, st) : f16_any<kW4G32>(a, num_cus, st);
}

hipError_t launch_skinny_i8(const Geometry &g, const void *packed, const int8_t *xq_tiled, const float *sx, int M,
                            void *y, const void *residual, int gated_act, int num_cus, hipStream_t st) {
    SkinnyArgs a = make_args(g, packed, xq_tiled, sx, M, y, residual, gated_act);
    if (g.fmt == kW8C && stream_takes(a, num_cus)) return M <= 16 ? launch_i8_stream<1>(a, num_cus, st) : launch_i8_stream<2>(a, num_cus, st);
    choose_blocks(a, g.fmt, true, num_cus);
    if (g.fmt == kW4C) {
        a.sw_mul = 0.0625f;
        // Row tiles a multiple of 32 KiB apart: with every workgroup at the same k the weight stream comes from few memory
        // channels at a time.  us, same k / turned, 9 and 32 rows: 28672 x 4096 16.7 / 13.8 and 18.4 / 15.7, 20000 x 4096 11.4 / 10.2
        // and 13.2 / 12.2, 65536 x 4096 25.7 / 24.2 and 30.6 / 28.3, 6144 x 4096 6.1 / 5.7 and 6.8 / 6.7, 22016 x 8192 18.1 / 17.5
        // and 20.7 / 20.4; 8192 x 4096 32 and 65 rows 8.4 / 7.2 and 11.5 / 9.7.  From about 256 rows on the blocks of a row group no longer run
        // at the same time and share the weights in L2 less well when each begins elsewhere (4096 x 4096 400 rows 16.7 / 17.4, 1536 x 8192
        // 640 rows 16.3 / 18.0; over nine layers 1 % slower at 300, 3 at 400, 4 at 500).  Other K level (28672 x 3072 1 % slower);
        // 8-bit weights from 12 % faster (65536 x 4096) to 5 % slower (12288 x 4096): not turned.
        a.turned = a.rt_stride % 32 == 0 && M <= 256;
        return i8_any<true>(a, num_cus, st);
    }
    return i8_any<false>(a, num_cus, st);
}

}  // namespace qfc
