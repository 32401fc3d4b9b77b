// Prefill int8 product and its dequantizing epilogue (section 3.7 of the paper:
// int8 activations x pre-quantized int8 weights with integer instructions, then
// dequantization of the output):
//   acc[m,n] = sum_k xq[m,k] * Wq[n,k]        (int32, exact)
//   y[m,n]   = fp16(float(acc) * sx[m] * sw[n])
//
// Both operands arrive tiled the same way (KiB tiles of 16 rows x 64 k, lane
// (c, q) = 16 codes of row c at k = 16q).  A stage of the K loop (128 k) is a
// verbatim copy of KiB tiles into LDS, done by global_load_lds_dwordx4 (one
// wavefront instruction moves one tile from memory straight into LDS, no
// staging registers), in a ring of LDS stages that keeps several stages in
// flight, with one workgroup barrier per stage.
// An MFMA operand fragment (16 rows x 64 k) is a whole KiB tile, a lane's 16 bytes at
// lane * 16: conflict free without padding.
//
// Workgroup: 4 wavefronts in a 2 x 2 grid over a BN x BM tile (weight rows x
// token rows); each wavefront owns (BN/2) x (BM/2) outputs as 16x16 tiles of
// v_mfma_i32_16x16x64_i8 (register-only loops of probe.hip on codes of normal values, all compute units: 4.09 POP/s,
// v_mfma_i32_32x32x32_i8 3.35; one operand 16 x int4 4.54 / 3.54: power).  The weights are the row operand of the MFMA so that
// a lane ends up with 4 consecutive n of one token row (8-byte fp16 stores
// along the contiguous axis of y).  Tile ids are dealt so that every XCD works
// on a contiguous range of (weight tile, token tile) pairs and the token tiles
// that share a weight tile hit the same L2.
#include "qfc_internal.h"
#include "tile_waits.h"

namespace qfc {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const void *gptr_t;
typedef __attribute__((address_space(3))) void *lptr_t;

__host__ __device__ inline int stages_total(int Kp, int bk) { return Kp / bk; }

struct GemmI8Args {
    const uint4 *w;   // packed weights, tiles [row tile][Kp/64][64]
    const uint4 *x;   // tiled activations, tiles [row tile][Kp/64][64]
    const float *sw;  // [Np]
    const float *sx;  // [Mp] (null for raw accumulators)
    const _Float16 *res;  // [M, N] residual added before the rounding, or null
    void *out;
    int M, N, Kp, n_tiles, m_tiles;
    TileWalk walk;  // order of the tiles (see xcd_tile)
    int share;      // by_tokens: token tiles on an XCD, which divide the early touch of the weights among them
    // 4-bit weights enter the MFMA as 16 q (the code's nibble in the top half of a byte): the sums are
    // 16 times the definition's, exactly; channel scales are multiplied by 1/16, raw sums shifted by 4
    float sw_mul = 1.0f;
    int acc_shift = 0;
    int gated_act = -1;  // QFC_ACT_*: the layer is packed in pairs and y [M, N/2] = fp16(act(gate) * other)
};

// Store phase of a layer packed in pairs (operator fusion, section 3.6 of the paper: the element-wise
// operators of the two branches merged into the fully connected operator that produces them).
// Physical row tiles 2 t and 2 t + 1 are the gate's and the other branch's rows of the same 16 channels, so a lane holds both
// branches of a channel: scale both, multiply act(gate) with the other in fp32, round once.  8 TN output channels per
// wavefront, staged through LDS like the plain store phase and written as 16-byte pieces of rows of N / 2 values.
template <int TN, int TM>
__device__ __forceinline__ void epilogue_gated(const GemmI8Args &a, v4i (&acc)[TN][TM], uint4 *lds, int n_base,
                                               int m_base, int wave, int lane) {
    constexpr int WO = TN * 8;
    constexpr int PITCH = (WO + 8) * 2;  // bytes per staged row
    char *region = reinterpret_cast<char *>(lds) + wave * (32 * PITCH);
    const int half = a.N / 2;
    const int o0 = n_base / 2;  // first output channel of the wavefront
    const int c = lane & 15, q = lane >> 4;
    const GateCoeffs gc = gate_coeffs(a.gated_act);
    float4 sc[TN];
    float sxr[TM];
#pragma unroll
    for (int i = 0; i < TN; ++i) {
        float4 v = *reinterpret_cast<const float4 *>(a.sw + n_base + i * 16 + 4 * q);
        v.x *= a.sw_mul, v.y *= a.sw_mul, v.z *= a.sw_mul, v.w *= a.sw_mul;
        sc[i] = v;
    }
#pragma unroll
    for (int j = 0; j < TM; ++j) {
        const int m = m_base + j * 16 + c;
        sxr[j] = m < a.M ? a.sx[m] : 0.0f;
    }
    asm volatile("s_barrier" ::: "memory");  // all wavefronts are done with the stage buffers
#pragma unroll
    for (int j = 0; j < TM; j += 2) {
        const int mrow0 = m_base + j * 16;
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
            const float sxm = sxr[j + jj];
#pragma unroll
            for (int i = 0; i < TN; i += 2) {
                typedef _Float16 h4 __attribute__((ext_vector_type(4)));
                const float gs[4] = {sc[i].x, sc[i].y, sc[i].z, sc[i].w};
                const float us[4] = {sc[i + 1].x, sc[i + 1].y, sc[i + 1].z, sc[i + 1].w};
                h4 hv;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float g = (float)acc[i][j + jj][e] * sxm * gs[e];
                    const float u = (float)acc[i + 1][j + jj][e] * sxm * us[e];
                    hv[e] = (_Float16)(gate_activation(g, gc) * u);
                }
                *reinterpret_cast<h4 *>(region + (16 * jj + c) * PITCH + (i * 8 + 4 * q) * 2) = hv;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        constexpr int CH = WO / 8;  // 16-byte chunks per staged row
#pragma unroll
        for (int it = 0; it < 32 * CH / 64; ++it) {
            const int idx = it * 64 + lane;
            const int row = idx / CH, ch = idx % CH;
            const uint4 v = *reinterpret_cast<const uint4 *>(region + row * PITCH + ch * 16);
            const int mm = mrow0 + row, nn = o0 + ch * 8;
            if (mm < a.M && nn < half)
                *reinterpret_cast<uint4 *>(static_cast<_Float16 *>(a.out) + (size_t)mm * half + nn) = v;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

// Epilogue shared by the product kernels.
// A wavefront holds TN x TM tiles of 16 x 16 outputs whose first weight row is n_base and first
// token row is m_base.
template <int OUT_MODE, int TN, int TM>
__device__ __forceinline__ void epilogue(const GemmI8Args &a, v4i (&acc)[TN][TM], uint4 *lds, int n_base, int m_base,
                                         int wave, int lane) {
    constexpr int WN = TN * 16;
    const int c = lane & 15, q = lane >> 4;
    if (OUT_MODE == 0 && a.gated_act >= 0) {
        epilogue_gated<TN, TM>(a, acc, lds, n_base, m_base, wave, lane);
        return;
    }
    // Epilogue.  After the MFMAs a lane holds, per tile, four consecutive n (4 (lane / 16) ..) of one
    // token row (lane % 16): stored as they are,
    // every store instruction would touch 32 different rows of y with 8 bytes
    // each.  The scaled binary16 values therefore take a detour through LDS (one
    // block of 32 token rows x WN channels per wavefront at a time) and leave as
    // 16-byte stores that cover whole rows segments of 2 * WN contiguous bytes.
    if (OUT_MODE == 0 && (a.N % 8) == 0) {
        constexpr int PITCH = (WN + 8) * 2;  // bytes per staged row
        char *region = reinterpret_cast<char *>(lds) + wave * (32 * PITCH);
        const int n0 = n_base;
        // the scales of the lane's channels and token rows, requested once and before the barrier
        // (inside the loop over the row blocks they would be fetched again after every fence)
        float4 scw[TN];
        float sxr[TM];
#pragma unroll
        for (int i = 0; i < TN; ++i) {
            float4 v = *reinterpret_cast<const float4 *>(a.sw + n0 + i * 16 + 4 * q);
            v.x *= a.sw_mul, v.y *= a.sw_mul, v.z *= a.sw_mul, v.w *= a.sw_mul;  // (1 or 1/16: exact)
            scw[i] = v;
        }
#pragma unroll
        for (int j = 0; j < TM; ++j) {
            const int m = m_base + j * 16 + c;
            sxr[j] = m < a.M ? a.sx[m] : 0.0f;
        }
        asm volatile("s_barrier" ::: "memory");  // all wavefronts are done with the stage buffers
#pragma unroll
        for (int j = 0; j < TM; j += 2) {
            const int mrow0 = m_base + j * 16;
            const bool has_res = a.res != nullptr;
            if (has_res) stage_residual_block<WN / 8, PITCH>(region, a.res, mrow0, n0, a.M, a.N, lane);
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) {
                const float sxm = sxr[j + jj];
#pragma unroll
                for (int i = 0; i < TN; ++i) {
                    const int at = (16 * jj + c) * PITCH + (i * 16 + 4 * q) * 2;
                    const float4 sc = scw[i];
                    const v4i s = acc[i][j + jj];
                    typedef _Float16 h4 __attribute__((ext_vector_type(4)));
                    float v[4] = {(float)s[0] * sxm * sc.x, (float)s[1] * sxm * sc.y, (float)s[2] * sxm * sc.z, (float)s[3] * sxm * sc.w};
                    if (has_res) {
                        float rv[4];
                        staged_residual4(region, at, rv);
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] += rv[e];
                    }
                    const h4 hv = {(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]};
                    *reinterpret_cast<h4 *>(region + at) = hv;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            constexpr int CH = WN / 8;  // 16-byte chunks per staged row
#pragma unroll
            for (int it = 0; it < 32 * CH / 64; ++it) {
                const int idx = it * 64 + lane;
                const int row = idx / CH, ch = idx % CH;
                const uint4 v = *reinterpret_cast<const uint4 *>(region + row * PITCH + ch * 16);
                const int mm = mrow0 + row, nn = n0 + ch * 8;
                if (mm < a.M && nn < a.N)
                    *reinterpret_cast<uint4 *>(static_cast<_Float16 *>(a.out) + (size_t)mm * a.N + nn) = v;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        return;
    }
    asm volatile("s_barrier" ::: "memory");  // all wavefronts are done with the stage buffers
    // generic path (raw accumulators, or N not a multiple of 8): direct stores
    const bool vec_ok = (a.N % 4) == 0;
#pragma unroll
    for (int j = 0; j < TM; ++j) {
        const int m = m_base + j * 16 + c;
        if (m >= a.M) continue;
        float sxm = 1.0f;
        if (OUT_MODE == 0) sxm = a.sx[m];
#pragma unroll
        for (int i = 0; i < TN; ++i) {
            {
                const int n = n_base + i * 16 + 4 * q;
                if (n >= a.N) continue;
                if (OUT_MODE == 0) {
                    _Float16 *y = static_cast<_Float16 *>(a.out) + (size_t)m * a.N + n;
                    const float4 s = *reinterpret_cast<const float4 *>(a.sw + n);
                    const float sv[4] = {s.x * a.sw_mul, s.y * a.sw_mul, s.z * a.sw_mul, s.w * a.sw_mul};
                    _Float16 h[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float v = (float)acc[i][j][e] * sxm * sv[e];
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
                } else {
                    int32_t *o = static_cast<int32_t *>(a.out) + (size_t)m * a.N + n;
                    const int sh = a.acc_shift;  // (arithmetic shift of an exact multiple: exact)
                    if (vec_ok) {
                        *reinterpret_cast<int4 *>(o) = make_int4(acc[i][j][0] >> sh, acc[i][j][1] >> sh,
                                                                 acc[i][j][2] >> sh, acc[i][j][3] >> sh);
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (n + e < a.N) o[e] = acc[i][j][e] >> sh;
                    }
                }
            }
        }
    }
}

// Both operands staged.  No layer's automatic choice: 128 x 128 tiles are level with the direct-weights kernel below at best (us, this / that:
// 475 x 2112 2243 rows 28.7 / 28.7, 457 x 8960 1714 rows 65 / 50).  Kept, at one shape, as the second opinion that tests compare that
// kernel's large launches with.  Stages of two KiB k tiles (64 k each); NS = LDS stages (prefetch distance NS - 1)
template <int BN, int BM, int NS, int OUT_MODE>
__global__ __launch_bounds__(256, 2) void gemm_i8_kernel(GemmI8Args a) {
    constexpr int KTS = 2, BK = KTS * 64;
    constexpr int WN = BN / 2, WM = BM / 2;    // per-wavefront tile
    constexpr int TN = WN / 16, TM = WM / 16;  // 16x16 MFMA tiles per wavefront
    constexpr int W_TILES = BN / 16 * KTS, X_TILES = BM / 16 * KTS;  // KiB tiles per stage
    constexpr int STAGE_VECS = (W_TILES + X_TILES) * 64;
    extern __shared__ uint4 lds[];  // NS stages: [stage][W tiles | X tiles][64]

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave & 1, wm = wave >> 1;

    int nt, mt;
    xcd_tile(blockIdx.x, a.n_tiles, a.m_tiles, a.walk, nt, mt);
    const int KT = a.Kp / 64;

    // One wavefront instruction copies one KiB tile: tile t of the stage, t = wave,
    // wave + 4, ...  The tiles of one row tile are contiguous along K, so the source
    // of a tile advances by a constant per stage; the stage-0 pointers are
    // computed once.
    constexpr int NLOAD = (W_TILES + X_TILES) / 4;
    const uint4 *src0[NLOAD];
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
        const int t = wave + 4 * i;
        if (t < W_TILES)
            src0[i] = a.w + ((size_t)(nt * (BN / 16) + t / KTS) * KT + t % KTS) * 64 + lane;
        else
            src0[i] = a.x + ((size_t)(mt * (BM / 16) + (t - W_TILES) / KTS) * KT + (t - W_TILES) % KTS) * 64 + lane;
    }
    auto issue_stage = [&](int kt, int buf) {
        uint4 *dst = lds + buf * STAGE_VECS + wave * 64;
#pragma unroll
        for (int i = 0; i < NLOAD; ++i)
            __builtin_amdgcn_global_load_lds((gptr_t)(src0[i] + (size_t)kt * (KTS * 64)), (lptr_t)(dst + i * 256), 16, 0, 0);
    };

    v4i acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j) acc[i][j] = v4i{0, 0, 0, 0};

    // Software pipeline over k steps of 64.  While the MFMAs of step s run, the
    // fragments of step s + 1 are already being read from LDS (double-buffered in
    // registers; scheduling barriers keep the reads ahead of the MFMA block), and
    // NS - 1 stages of global -> LDS copies are in flight.  When step s + 1 is the
    // first of the next stage, the wait for that stage and the workgroup barrier
    // come before its reads, i.e. before the MFMAs of the last step of the current
    // stage.  The barrier is a bare s_barrier: __syncthreads() would drain every
    // outstanding copy and cancel the prefetch distance.  The copy issued after the
    // barrier overwrites the buffer of the stage that is ending: every wavefront
    // waited for its own last LDS reads of that stage before the barrier.
    constexpr int KS = BK / 64;
    auto load_frags = [&](v4i(&fa)[TN], v4i(&fb)[TM], int buf, int ks) {
        const uint4 *lw = lds + buf * STAGE_VECS;
        const uint4 *lx = lw + W_TILES * 64;
#pragma unroll
        for (int i = 0; i < TN; ++i) fa[i] = __builtin_bit_cast(v4i, lw[((wn * TN + i) * KTS + ks) * 64 + lane]);
#pragma unroll
        for (int j = 0; j < TM; ++j) fb[j] = __builtin_bit_cast(v4i, lx[((wm * TM + j) * KTS + ks) * 64 + lane]);
    };
    auto stage_ready = [&](int kt) {  // stage kt has landed for the whole workgroup
        if (kt + NS - 2 < stages_total(a.Kp, BK))
            wait_vmcnt<(NS - 2) * NLOAD>();
        else
            wait_vmcnt<0>();
        asm volatile("s_barrier" ::: "memory");
    };
    const int stages = stages_total(a.Kp, BK);
#pragma unroll
    for (int p = 0; p < NS - 1; ++p)
        if (p < stages) issue_stage(p, p);
    v4i fa[2][TN], fb[2][TM];
    stage_ready(0);
    if (NS - 1 < stages) issue_stage(NS - 1, NS - 1);
    load_frags(fa[0], fb[0], 0, 0);
    auto step = [&](int kt, const int ks, const int set) __attribute__((always_inline)) {  // set: registers of this step's operands
        if (ks < KS - 1) {
            load_frags(fa[set ^ 1], fb[set ^ 1], kt % NS, ks + 1);
        } else if (kt + 1 < stages) {
            stage_ready(kt + 1);
            if (kt + NS < stages) issue_stage(kt + NS, (kt + NS) % NS);
            load_frags(fa[set ^ 1], fb[set ^ 1], (kt + 1) % NS, 0);
        }
        __builtin_amdgcn_sched_barrier(0);  // keep the reads ahead of this step's MFMAs
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[set][i], fb[set][j], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    for (int kt = 0; kt < stages; ++kt) {
        step(kt, 0, 0);
        step(kt, 1, 1);
    }

    epilogue<OUT_MODE, TN, TM>(a, acc, lds, nt * BN + wn * WN, mt * BM + wm * WM, wave, lane);
}

// int8 activations x 4-bit per-channel weights (the "8/4/4" scheme of section 4.2 in the prefill
// stage of section 3.7): the same pipeline as gemm_i8_kernel with stages of 128 k.  A stage holds
// one packed KiB tile per 16 weight rows (16 rows x 128 k of 4-bit codes, copied verbatim) and
// two activation tiles per 16 token rows, the latter written by the quantizer in the k order of
// the packed codes.  A lane reads the two dwords of its packed vector that belong to a k step and
// expands them in registers: code u = q + 8 in a nibble becomes the byte (u ^ 8) << 4, which the
// MFMA reads as the signed value 16 q (5 vector instructions per 8 codes), so the int32 sums are
// exactly 16 times the definition's and the epilogue divides them out (scale * 1/16, or a shift).
template <int BN, int BM, int NS, int OUT_MODE>
__global__ __launch_bounds__(256, 2) void gemm_i8_w4_kernel(GemmI8Args a) {
    constexpr int WN = BN / 2, WM = BM / 2;
    constexpr int TN = WN / 16, TM = WM / 16;
    constexpr int W_TILES = BN / 16, X_TILES = BM / 16 * 2;  // KiB tiles per stage
    constexpr int STAGE_VECS = (W_TILES + X_TILES) * 64;
    static_assert((W_TILES + X_TILES) % 4 == 0, "tiles of a stage are dealt to four wavefronts");
    extern __shared__ uint4 lds[];  // NS stages: [stage][W tiles | X tiles][64]

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave & 1, wm = wave >> 1;
    int nt, mt;
    xcd_tile(blockIdx.x, a.n_tiles, a.m_tiles, a.walk, nt, mt);
    const int stages = a.Kp / 128;

    constexpr int NLOAD = (W_TILES + X_TILES) / 4;
    const uint4 *src0[NLOAD];
    int adv[NLOAD];  // vectors a tile's source advances per stage
#pragma unroll
    for (int i = 0; i < NLOAD; ++i) {
        const int t = wave + 4 * i;
        if (t < W_TILES) {
            src0[i] = a.w + ((size_t)(nt * (BN / 16) + t) * stages) * 64 + lane;
            adv[i] = 64;
        } else {
            const int tx = t - W_TILES;
            src0[i] = a.x + ((size_t)(mt * (BM / 16) + tx / 2) * (2 * stages) + tx % 2) * 64 + lane;
            adv[i] = 128;
        }
    }
    auto issue_stage = [&](int kt, int buf) {
        uint4 *dst = lds + buf * STAGE_VECS + wave * 64;
#pragma unroll
        for (int i = 0; i < NLOAD; ++i)
            __builtin_amdgcn_global_load_lds((gptr_t)(src0[i] + (size_t)kt * adv[i]), (lptr_t)(dst + i * 256), 16, 0, 0);
    };

    v4i acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j) acc[i][j] = v4i{0, 0, 0, 0};

    constexpr int KS = 2;  // k steps of 64 per stage
    auto load_frags = [&](v4i(&fa)[TN], v4i(&fb)[TM], int buf, int ks) {
        const char *lw = reinterpret_cast<const char *>(lds + buf * STAGE_VECS);
        const uint4 *lx = lds + buf * STAGE_VECS + W_TILES * 64;
#pragma unroll
        for (int i = 0; i < TN; ++i) {
            const uint2 p = *reinterpret_cast<const uint2 *>(lw + ((wn * TN + i) * 64 + lane) * 16 + ks * 8);
            fa[i][0] = (int)(((p.x << 4) & 0xF0F0F0F0u) ^ 0x80808080u);  // codes 0..3 of the first run's octet
            fa[i][1] = (int)((p.x & 0xF0F0F0F0u) ^ 0x80808080u);         // codes 4..7
            fa[i][2] = (int)(((p.y << 4) & 0xF0F0F0F0u) ^ 0x80808080u);  // the second run's octet
            fa[i][3] = (int)((p.y & 0xF0F0F0F0u) ^ 0x80808080u);
        }
#pragma unroll
        for (int j = 0; j < TM; ++j) fb[j] = __builtin_bit_cast(v4i, lx[((wm * TM + j) * 2 + ks) * 64 + lane]);
    };
    auto stage_ready = [&](int kt) {  // stage kt has landed for the whole workgroup
        if (kt + NS - 2 < stages)
            wait_vmcnt<(NS - 2) * NLOAD>();
        else
            wait_vmcnt<0>();
        asm volatile("s_barrier" ::: "memory");
    };
    static_assert((NS - 1) * NLOAD <= 63, "outstanding copies must fit the 6-bit counter");
#pragma unroll
    for (int p = 0; p < NS - 1; ++p)
        if (p < stages) issue_stage(p, p);
    v4i fa[2][TN], fb[2][TM];
    stage_ready(0);
    if (NS - 1 < stages) issue_stage(NS - 1, NS - 1);
    load_frags(fa[0], fb[0], 0, 0);
    for (int kt = 0; kt < stages; ++kt) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (ks < KS - 1) {
                load_frags(fa[(ks + 1) & 1], fb[(ks + 1) & 1], kt % NS, ks + 1);
            } else if (kt + 1 < stages) {
                stage_ready(kt + 1);
                if (kt + NS < stages) issue_stage(kt + NS, (kt + NS) % NS);
                load_frags(fa[(ks + 1) & 1], fb[(ks + 1) & 1], (kt + 1) % NS, 0);
            }
            __builtin_amdgcn_sched_barrier(0);  // keep the reads ahead of this step's MFMAs
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int j = 0; j < TM; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[ks & 1][i], fb[ks & 1][j], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    epilogue<OUT_MODE, TN, TM>(a, acc, lds, nt * BN + wn * WN, mt * BM + wm * WM, wave, lane);
}

// Variant with the weights going from memory straight into the MFMA operand registers, for int8 weights and for int4 per-channel
// ones (W4).  The packed layout already is operand order (a lane's 16 bytes of a KiB tile are 16 consecutive k of one row, or, 4-bit,
// its octets of four groups), so only the activations, which all four wavefronts share, pass through LDS.  Tile 256 (n) x 32 TM
// (m); wavefront w owns weight rows 64 w .. 64 w + 63 and all token rows (4 x 2 TM tiles of 16 x 16, 128 accumulator registers
// at TM = 4) and loads only its own weights, PW stages of 128 k ahead, into a ring of registers (slot = stage % PW,
// refilled right after the MFMAs that consumed it).  Activation stages: ring of NS LDS stages of two KiB tiles per 16 token rows (4-bit
// weights: in the k order of the packed dwords), CP tile copies per wavefront and stage.  A block of 16 token rows of a k step is replaced by the
// next step's as soon as it has been multiplied.  4-bit codes are expanded as in the kernel above, those of a stage's second k step during the MFMAs
// of the first.  Copies and loads past the end of K start
// over at stage 0, so that every iteration issues the same number of operations and the waits are
// constants.  Such copies go to a spare KiB behind the ring that is never read (and their sources
// are distinct stages, not one stage over and over: with about ten copies of the same lines in
// flight from one wavefront, data had been seen in ring slots after the counter had dropped to zero;
// the cause is not known, so no late copy may have a destination that anything reads or reuses).
// The number of stages must be even.
// CG wavefronts side by side: tiles of 64 CG channels x 32 TM tokens, 256 or 128 x 128 or 64.  KS groups of them share K (an even number of stages each) and
// hand their sums over through LDS at the end.  Which form: int8_tile_us.
// PF: a compute unit has only so many cache lines on their way to it (the product alone draws 58 GB/s per compute unit with weights in HBM, 69 with weights in the
// memory-side cache), so what bounds a
// layer of one round of tiles is how long a line is on its way, not the rate of HBM or of the matrix cores (4096 x 14336, 1024 rows, tiles of 256 x 64,
// weights in HBM: 88 us, and 88 without its MFMAs; in the cache 65).  The token tiles of the same weights therefore divide among them an early touch of every line, PW + NS - 1 stages
// ahead, one instruction per wavefront and stage, and the weights' own loads then find them in L2: 128 x 128 tiles in two parts of K 73.9 / 68.1 us, 2304 x 9216
// 1024 rows 48.8 / 44.6.  Tiles of 128 x 128 read 3.7 MB each where 256 x 64 read 4.6 (the same shapes 88 / 74 and 57 / 49 without the touch); for 4-bit weights,
// whose bytes are half as many, 256 x 64 stays the better one and the touch costs more than it saves (62.4 / 63.6).  A touch is a copy into the
// spare KiB like those past the end of K.
// PIPE: the first operands of a stage are read during the MFMAs of the stage before, so its copies must have landed a stage
// earlier.  For int8 weights in tiles of 64 tokens, which run where a compute unit has one of them: nothing else fills the time between the barrier
// and the first MFMA.  With 4-bit weights the wait, which then covers more, costs more than it saves (540 x 9984 1434 rows 50.0 / 51.5 us, 4096 x
// 4096 700 rows 25.5 / 26.1), and so it does in tiles of 64 tokens with K in two parts, whose ring of four stages would leave four operations
// outstanding instead of eight (without / with: 4096 x 14336 512 rows 51.8 / 56.6 us, 4096 x 4096 300 rows 20.1 / 21.2, 2304 x 9216 300 rows 37.3 / 40.5).
//
// What bounds it: power on real data (see the MFMA rates above), then the operand paths; where the tiles leave most of the chip idle, the latency of a
// stage.  us with the quantization kernel, 32 x 32 MFMAs (int8 weights: stages of
// 64 k) / this, weights in the cache, both in one session: 28672 x 4096 int8, 1024 rows 119.6 / 107.6, 4096 rows 461 / 442; int4 gated, 1024 rows 109.0 / 97.0,
// 300 rows 50.2 / 47.0; 6144 x 4096 int8, 1024 rows 35.0 / 32.1; 64-token tiles, 1024 rows: 4096 x 4096 int8 26.7 / 25.6, 4096 x 14336 int8
// 67.9 / 64.8, int4 66.0 / 60.5; 457 x 8960 int8, 1714 rows 49.1 / 49.7, 540 x 9984 int4, 1434 rows 48.2 / 48.2.  (240 shapes of 200 to 32768 channels and
// 300 to 4096 rows: 0.958 of the time, the worst narrow ones 767 x 4096 int8 1568 rows 33.4 / 34.2 and 1055 x 6144 1049 rows 39.8 / 40.6.  Without reading and
// expanding ahead, and with four stages of weights only where those divide K: 0.964, 457 x 8960 51.8, 540 x 9984 50.9.)
//
// The weight loads carry no streaming hint: the workgroups of the same weight tile (one per token tile)
// run side by side on one XCD, and with the lines marked evict-first the later ones miss in L2
// (measured: 4-19 % slower on every shape).
//
// The weight loads are assembly too: the compiler counts only the loads it knows when it places its
// waits, and with the copies in between those waits would drain most of the prefetch.  A load's
// destination registers are handed back to the compiler (an empty asm that "redefines" them) right
// after the explicit wait that covers the load, so that no MFMA can be scheduled ahead of that wait.
template <bool W4, int NS, int PW, int TM, int CG, int KS, bool PF, int OUT_MODE>
__global__ __launch_bounds__(CG * KS * 64, 2) void gemm_i8_dw_kernel(GemmI8Args a) {
    constexpr int BN = 64 * CG, BM = 32 * TM, TN = 4, WV = W4 ? 1 : 2;  // (WV: weight vectors per row tile and stage)
    constexpr int XT = BM / 16 * 2;  // activation tiles (KiB) per stage
    constexpr int CP = XT / CG;      // copies per wavefront and stage
    constexpr int XJ = 2 * TM;   // blocks of 16 token rows
    constexpr bool PIPE = !W4 && TM == 2 && !PF;
    static_assert(NS >= 3 && (TM == 2 || TM == 4), "tile shapes");
    extern __shared__ uint4 lds[];  // NS stages of XT tiles x 64 vectors
    const int lane = threadIdx.x & 63;
    const int group = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) / CG;  // which part of K
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) - group * CG;
    int nt, mt;
    xcd_tile(blockIdx.x, a.n_tiles, a.m_tiles, a.walk, nt, mt);
    // stages: of the layer, before the group's, of the group (an even number; the first groups may have two more)
    const int all = a.Kp / 128, pairs = all / 2, first = 2 * (group * (pairs / KS) + min(group, pairs % KS));
    const int KT = KS == 1 ? all : 2 * (pairs / KS + (group < pairs % KS ? 1 : 0));

    // weights: row tile i of the wavefront's four, whole packed KiB tiles, at offset woff[i] from the stage's base
    const uint4 *const wsrc = a.w + ((size_t)(nt * (BN / 16) + 4 * wave) * all + first) * (64 * WV);
    uint32_t woff[TN];
#pragma unroll
    for (int i = 0; i < TN; ++i) woff[i] = (uint32_t)(i * all * WV * 1024 + lane * 16);
    v4i wreg[PW][TN][WV];
    auto load_w = [&](int slot, int kt, int v, const bool bulk) __attribute__((always_inline)) {  // vector v of the row tiles; bulk: kt < KT is known
        const int kc = bulk || kt < KT ? kt : min(kt - KT, KT - 1);
#pragma unroll
        for (int i = 0; i < TN; ++i)
            asm volatile("global_load_dwordx4 %0, %1, %2 offset:%3" : "=&v"(wreg[slot][i][v]) : "v"(woff[i]), "s"(wsrc + (size_t)(WV * kc) * 64), "n"(v * 1024) : "memory");
    };
    // activations: tile t = 2 g + e of a stage is half e of the stage's 128 k for token rows 16 g ..
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)lds;
    const uint32_t ring0 = lds0 + group * (NS * XT * 1024);
    const uint4 *const ring = lds + group * (NS * XT * 64);
    const uint4 *xsrc = a.x + ((size_t)(mt * (BM / 16)) * 2 * all + 2 * first) * 64;
    constexpr uint32_t kSpare = KS * NS * XT * 1024;  // copies past the end of K land here; nothing reads it
    auto issue_x = [&](int kt, const bool bulk) __attribute__((always_inline)) {
        const bool real = bulk || kt < KT;
        const int kc = real ? kt : min(kt - KT, KT - 1);
#pragma unroll
        for (int h = 0; h < CP; ++h) {
            const int t = wave + CG * h;
            copy16_to_lds(xsrc + ((size_t)(t >> 1) * 2 * all + 2 * kc + (t & 1)) * 64, lane * 16,
                          real ? ring0 + ((kt % NS) * XT + t) * 1024 : lds0 + kSpare);
        }
    };

    // the touch of the weights of a stage far ahead (PF): of the 128-byte lines of the wavefront's row tiles, those that fall to this token tile
    constexpr int PFN = PF ? 1 : 0, kLines = 32 * WV;
    const int band = a.walk.by_tokens ? 0 : mt / a.walk.band * a.walk.band;  // token tiles that walk the same weights on this XCD, and which of them this is
    const int share = a.walk.by_tokens ? a.share : min(a.walk.band, a.m_tiles - band), mine = a.walk.by_tokens ? mt % share : mt - band;
    const int per = (kLines + share - 1) / share, pidx = min(mine * per + lane % per, kLines - 1);
    const uint32_t poff = (uint32_t)((pidx / (8 * WV)) * all * WV * 1024 + (pidx % (8 * WV)) * 128);
    constexpr int kPrefetch = NS - 1 + PW;
    auto prefetch = [&](int kt, const bool bulk) __attribute__((always_inline)) {
        if (!PF) return;
        const int kc = bulk || kt < KT ? kt : min(kt - KT, KT - 1);
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(poff), "s"(wsrc + (size_t)(WV * kc) * 64), "s"(lds0 + kSpare) : "memory", "m0");
    };

    v4i acc[TN][XJ];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < XJ; ++j) acc[i][j] = v4i{0, 0, 0, 0};

    constexpr bool kBulk = true, kEdge = false;
#pragma unroll
    for (int p = 0; p < PW; ++p)
#pragma unroll
        for (int v = 0; v < WV; ++v) load_w(p, p, v, kEdge);
#pragma unroll
    for (int p = 0; p < NS - 1; ++p) {
        issue_x(p, kEdge);
        prefetch(PW + p, kEdge);
    }

    // Waiting (see dw_waits).  At the top of iteration kt a wavefront has issued, after the copies of stage kt, the copies of NS - 2 later stages
    // (CP each), and after the loads of stage kt the loads of PW - 1 later stages - from iteration 0 on, thanks to the prologue.  With PIPE it is
    // stage kt + 1 whose copies must have landed, which has one stage fewer behind it.
    constexpr DwWaits kWaits = dw_waits(CP, 4 * WV, NS, PW, PIPE);
    // (the most operations a wavefront ever has outstanding: right after the refills of an iteration)
    static_assert((CP + PFN) * (NS - 1) + 4 * WV * PW <= 63, "wait counts must fit the 6-bit counter");

    v4i fb[XJ];  // (token rows of a k step of 64: a block is replaced by the next step's once it has been multiplied)
    auto read_x = [&](int kt, int ks, int j) __attribute__((always_inline)) {
        fb[j] = __builtin_bit_cast(v4i, ring[(kt % NS) * (XT * 64) + (2 * j + ks) * 64 + lane]);
    };
    if (PIPE) {
        wait_vmcnt<kWaits.first>();
        asm volatile("s_barrier" ::: "memory");
#pragma unroll
        for (int j = 0; j < XJ; ++j) read_x(0, 0, j);
    }
    auto stages_pw = [&](int kt0, const int count, const bool bulk) __attribute__((always_inline)) {  // count: PW, or 2
#pragma unroll
        for (int u = 0; u < count; ++u) {
            const int kt = kt0 + u;
            if (PIPE)
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kWaits.allowed) : "memory");  // (not the LDS counter: operand reads stay in flight)
            else
                wait_vmcnt<kWaits.allowed>();
            asm volatile("s_barrier" ::: "memory");
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int v = 0; v < WV; ++v) asm volatile("" : "+v"(wreg[u][i][v]));
            issue_x(kt + NS - 1, bulk);
            prefetch(kt + kPrefetch, bulk);
            if (!PIPE) {
#pragma unroll
                for (int j = 0; j < XJ; ++j) read_x(kt, 0, j);
            }
            v4i fa[2][TN];
            auto operand = [&](int ks, int i) __attribute__((always_inline)) {
                if (!W4) {
                    fa[ks][i] = wreg[u][i][W4 ? 0 : ks];
                    return;
                }
                const uint32_t px = (uint32_t)wreg[u][i][0][2 * ks], py = (uint32_t)wreg[u][i][0][2 * ks + 1];
                fa[ks][i][0] = (int)(((px << 4) & 0xF0F0F0F0u) ^ 0x80808080u);
                fa[ks][i][1] = (int)((px & 0xF0F0F0F0u) ^ 0x80808080u);
                fa[ks][i][2] = (int)(((py << 4) & 0xF0F0F0F0u) ^ 0x80808080u);
                fa[ks][i][3] = (int)((py & 0xF0F0F0F0u) ^ 0x80808080u);
            };
#pragma unroll
            for (int i = 0; i < TN; ++i) operand(0, i);
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
                for (int j = 0; j < XJ; ++j) {
#pragma unroll
                    for (int i = 0; i < TN; ++i)
                        acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[ks][i], fb[j], acc[i][j], 0, 0, 0);
                    if (ks == 0 && j < TN) operand(1, j);
                    if (ks == 0 || PIPE) {
                        __builtin_amdgcn_sched_barrier(0);
                        if (ks == 0)
                            read_x(kt, 1, j);
                        else
                            read_x(kt + 1, 0, j);
                    }
                }
                if (!W4 || ks == 1) load_w(u, kt + PW, W4 ? 0 : ks, bulk);  // (the vectors that this step was the last to use)
            }
        }
    };
    constexpr int kAhead = PF ? NS - 1 + PW : NS - 1 > PW ? NS - 1 : PW;  // how far past kt a pass issues
    int kt0 = 0;
    for (; kt0 + PW - 1 + kAhead < KT; kt0 += PW) stages_pw(kt0, PW, kBulk);
    for (; kt0 + PW <= KT; kt0 += PW) stages_pw(kt0, PW, kEdge);
    // The loads issued past the end of K are still writing their destination registers until the
    // wait returns, and the compiler does not know (it sees registers that nobody reads any more).
    // Naming them as inputs behind it keeps them allocated until after the wait, and the memory clobber
    // keeps the store phase's own loads from being moved above it.  (On either way to the end, so that none of them is
    // the same value on both, which the compiler might move to another register while its load is in flight.)
    auto drain = [&]() __attribute__((always_inline)) {
        wait_vmcnt<0>();
#pragma unroll
        for (int p = 0; p < PW; ++p)
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int v = 0; v < WV; ++v) asm volatile("" ::"v"(wreg[p][i][v]) : "memory");
    };
    if (PW > 2 && kt0 < KT) {
        stages_pw(kt0, 2, kEdge);
        drain();
    } else {
        drain();
    }
    if constexpr (KS == 1) {
        epilogue<OUT_MODE, TN, XJ>(a, acc, lds, nt * BN + wave * 64, mt * BM, wave, lane);
    } else {
        // The parts of K meet (whole numbers: in any order): group 0 keeps the first half of the token rows, group 1 the second, and everybody
        // hands over what it does not keep, [half][group][wavefront][16-byte vector][lane] over the dead rings, below the spare KiB.
        constexpr int H = XJ / 2;
        static_assert(2 * (KS - 1) * CG * TN * H <= KS * NS * XT, "the sums handed over fit over the rings");
        v4i *const given = reinterpret_cast<v4i *>(lds);
        auto slot = [&](int half, int from) { return given + (((half * (KS - 1) + from) * CG + wave) * (TN * H)) * 64 + lane; };
        for (int i = KT; i < 2 * ((pairs + KS - 1) / KS); ++i) asm volatile("s_barrier" ::: "memory");  // (as many as the first group's stages)
        asm volatile("s_barrier" ::: "memory");  // every wavefront has read its last stage and all its copies have landed (drain)
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            if (group == half) continue;
            v4i *to = slot(half, group > half ? group - 1 : group);
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int j = 0; j < H; ++j) to[(i * H + j) * 64] = acc[i][half * H + j];
        }
        __syncthreads();
        v4i out[TN][H];
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            if (group != half) continue;
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int j = 0; j < H; ++j) {
                    out[i][j] = acc[i][half * H + j];
#pragma unroll
                    for (int from = 0; from < KS - 1; ++from) out[i][j] += slot(half, from)[(i * H + j) * 64];
                }
        }
        __syncthreads();
        if (group >= 2) {  // nothing to store: the one barrier that the others pass in their store phase
            asm volatile("s_barrier" ::: "memory");
            return;
        }
        epilogue<OUT_MODE, TN, H>(a, out, lds, nt * BN + wave * 64, mt * BM + group * (H * 16), group * CG + wave, lane);
    }
}

template <bool W4, int NS, int PW, int TM, int CG, int KS, bool PF, int OUT_MODE>
hipError_t launch_dw(GemmI8Args a, hipStream_t st) {
    constexpr size_t ring_bytes = (size_t)KS * NS * (4 * TM) * 1024;  // + one spare KiB for the copies past the end of K
    constexpr size_t lds_bytes = ring_bytes + 1024;
    static_assert(ring_bytes >= (size_t)CG * (KS > 1 ? 2 : 1) * 32 * (64 + 8) * 2, "the store phase stages its blocks inside the ring, below the spare KiB");
    static_assert(lds_bytes <= (KS > 1 ? 160 : 80) * 1024, "two workgroups per compute unit, or one");
    static_assert(PW == 2 || PW == 4, "an even number of stages is passes of PW and two more");
    if ((a.Kp / 128) % 2 != 0 || a.Kp / 128 < 2 * KS) return hipErrorInvalidValue;
    if (const hipError_t e = allow_dynamic_lds<gemm_i8_dw_kernel<W4, NS, PW, TM, CG, KS, PF, OUT_MODE>>(lds_bytes); e != hipSuccess) return e;
    a.n_tiles = (a.N + 64 * CG - 1) / (64 * CG);
    a.m_tiles = (a.M + 32 * TM - 1) / (32 * TM);
    a.walk = tile_walk(a.n_tiles, a.m_tiles, a.Kp, true, (W4 ? 32.0f : 64.0f) * CG, 32.0f * TM);
    const int width = a.walk.band, per_xcd = (a.n_tiles * a.m_tiles + 7) / 8;
    a.share = min((per_xcd + width - 1) / width, min(a.m_tiles, 16));
    gemm_i8_dw_kernel<W4, NS, PW, TM, CG, KS, PF, OUT_MODE><<<dim3((unsigned)(a.n_tiles * a.m_tiles)), CG * KS * 64, lds_bytes, st>>>(a);
    return hipGetLastError();
}

template <int BN, int BM, int NS, int OUT_MODE>
hipError_t launch_staged(GemmI8Args a, hipStream_t st) {
    constexpr size_t lds_bytes = (size_t)NS * ((BN + BM) / 16 * 2) * 1024;
    static_assert(lds_bytes <= 160 * 1024, "LDS budget");
    if (const hipError_t e = allow_dynamic_lds<gemm_i8_kernel<BN, BM, NS, OUT_MODE>>(lds_bytes); e != hipSuccess) return e;
    a.n_tiles = (a.N + BN - 1) / BN;
    a.m_tiles = (a.M + BM - 1) / BM;
    a.walk = tile_walk(a.n_tiles, a.m_tiles, a.Kp, true, (float)BN, (float)BM);
    gemm_i8_kernel<BN, BM, NS, OUT_MODE><<<dim3((unsigned)(a.n_tiles * a.m_tiles)), 256, lds_bytes, st>>>(a);
    return hipGetLastError();
}

template <int BN, int BM, int NS, int OUT_MODE>
hipError_t launch_w4(GemmI8Args a, hipStream_t st) {
    constexpr size_t lds_bytes = (size_t)NS * (BN / 16 + BM / 8) * 1024;
    static_assert(lds_bytes <= 80 * 1024, "two workgroups per compute unit");
    static_assert(lds_bytes >= 4 * 32 * (BN / 2 + 8) * 2, "the store phase stages its blocks in the same LDS");
    if (const hipError_t e = allow_dynamic_lds<gemm_i8_w4_kernel<BN, BM, NS, OUT_MODE>>(lds_bytes); e != hipSuccess) return e;
    a.n_tiles = (a.N + BN - 1) / BN;
    a.m_tiles = (a.M + BM - 1) / BM;
    a.walk = staged_tile_walk(a.n_tiles, a.m_tiles, a.Kp, true, 0.5f * BN, (float)BM);
    gemm_i8_w4_kernel<BN, BM, NS, OUT_MODE><<<dim3((unsigned)(a.n_tiles * a.m_tiles)), 256, lds_bytes, st>>>(a);
    return hipGetLastError();
}

bool parts_fit(int Kp, int parts) { return Kp / 128 >= 2 * parts; }

// The kernel is chosen by size (int8_tile_us), or by number for tests: 4, 10, 12, 13, 14 (int8 weights), 20, 21, 23, 24, 25 (int4).  A number that
// names none of the call's kernels leaves the choice.
// Tiles of 256 x 64 hold the weights of four stages with int4 codes (an operation more in flight is one that the wait of a stage need not see done; us with the
// quantization kernel, two / four: 4096 x 4096 700 rows 25.3 / 24.4, 3101 x 8192 840 rows 48.9 / 46.6, the worst 2210 x 512 2197 rows 21.6 / 22.0), of two with
// int8 codes, where the longer start shows at small K and nothing is gained at large K (the 500 shapes that take these tiles: K up to 512 +4.9 % with
// four, up to 2048 +3.7 %, up to 4096 +1.6 %, 31 above 6144 level).
// Tiles of 256 x 128 touch their weights early where one round of them leaves latency to hide, K is long enough for it and a band of token tiles shares the work
// (us without / with: 2304 x 9216 2048 rows 68.9 / 66.5, 4352 x 9728 1096 rows 71.5 / 68.0, 48 shapes with K above 4096 -1.7 %; K of 4096 and less, 109 shapes
// +2 %, 3392 x 768 2135 rows 17.2 / 17.3, 2240 x 1024 3546 rows 19.6 / 20.8; a second round +3 %, 2304 x 9216 4096 rows 116 / 123; few token tiles +3 %,
// 9728 x 10240 423 rows 73.3 / 75.5; a walk by tokens, 1344 x 13056 3677 rows 104.6 / 108.5).
template <int OUT_MODE>
hipError_t launch_mode(const GemmI8Args &a, int chosen, int num_cus, hipStream_t st) {
    int variant = tuning().gemm_variant;
    if (variant != 4 && variant != 10 && variant != 12 && ((variant != 13 && variant != 14) || !parts_fit(a.Kp, 2))) variant = chosen;
    switch (variant) {
        case 4: return launch_staged<128, 128, 3, OUT_MODE>(a, st);
        case 10: {
            const long n_tiles = (a.N + 255) / 256, m_tiles = (a.M + 127) / 128;
            return a.Kp > 4096 && m_tiles >= kBand && m_tiles < 3 * n_tiles && n_tiles * m_tiles <= num_cus ? launch_dw<false, 4, 2, 4, 4, 1, true, OUT_MODE>(a, st)
                                                                                                            : launch_dw<false, 4, 2, 4, 4, 1, false, OUT_MODE>(a, st);
        }
        case 13: return launch_dw<false, 4, 2, 4, 2, 2, true, OUT_MODE>(a, st);
        case 14: return launch_dw<false, 4, 2, 2, 2, 2, true, OUT_MODE>(a, st);
    }
    return launch_dw<false, 8, 2, 2, 4, 1, false, OUT_MODE>(a, st);
}

template <int OUT_MODE>
hipError_t launch_mode_w4(const GemmI8Args &a, int chosen, hipStream_t st) {
    int variant = tuning().gemm_variant;
    if (variant != 20 && variant != 21 && variant != 23 && (variant != 24 || !parts_fit(a.Kp, 2)) && (variant != 25 || !parts_fit(a.Kp, 4))) variant = chosen;
    if ((a.Kp / 128) % 2 != 0) variant = 20;
    switch (variant) {
        case 20: return launch_w4<128, 128, 3, OUT_MODE>(a, st);
        case 21: return launch_dw<true, 4, 2, 4, 4, 1, false, OUT_MODE>(a, st);
        case 24: return launch_dw<true, 4, 4, 2, 2, 2, false, OUT_MODE>(a, st);
        case 25: return launch_dw<true, 4, 4, 2, 2, 4, false, OUT_MODE>(a, st);
    }
    return launch_dw<true, 8, 4, 2, 4, 1, false, OUT_MODE>(a, st);
}

}  // namespace

// Estimated time of the direct-weights kernel (with the quantization of the rows, but for what of it grows with the rows) and the form that it is fastest
// in, by its number.  A tile takes `each` us and K / 1000 times `alone` on a compute unit of its own, `shared` where several are in flight; of a last
// round that is not full, the part that grows with K takes at least the share `idle` of a full one's.  Fitted so that the choice costs least, over 2580 shapes of 256 to 40000
// channels, K of 256 to 14336 and 65 to 4096 rows, weights in HBM: int8 weights 0.22 % behind the fastest form (fitted to 350 aligned shapes before: 0.50 %), 6 of
// 1301 shapes more than 10 %, int4 weights 0.43 %.  us, 256 x 128 / 256 x 64 / in parts of K 128 x 128 / 128 x 64, int8 weights: 4096 x 14336 1024 rows 98 / 87 / 68 / 87,
// 512 rows 96 / 82 / 64 / 52, 2048 rows 110 / 156 / 133 / 171; 2112 x 6144 505 rows 44 / 34 / 31 / 24; 1600 x 2048 2026 rows 21.7 / 16.9 / 21.6 / 20.7; 30336 x 12544 96 rows
// 113 / 102 / 128 / 133; int4 (256 x 128 / 256 x 64 / 128 x 64 in two / in four parts): 2304 x 9216 814 rows 59 / 40 / 32.4 / 30.5, 4096 x 4096 512 rows
// 31 / 21.9 / 17.7 / 19.0.
// Outputs that are stored as they lie in the registers (accumulators; rows that are no multiple of 16 bytes) cost tiles of 256 x 128 more than the others: 4 us in
// the choice (int4 9001 x 1024 600 rows, 256 x 128 / 256 x 64, 31.1 / 24.9; int8 4100 x 1024 1211 rows 24.7 / 21.4).  What that store itself takes is in the time that
// is returned: 0.11 us per round and token row of a wavefront where single values are stored, 0.05 where four are (K of 256, 256 x 64, 8.3 us; odd channels 15.8).
float int8_tile_us(const Geometry &g, int M, bool staged_store, int num_cus, int *form) {
    struct Fit {
        int number, channels, tokens, parts;
        float start, each, alone, shared, idle;
    };
    static const Fit fits[2][4] = {{{10, 256, 128, 1, 7.07f, 2.27f, 7.40f, 5.71f, 0.77f}, {12, 256, 64, 1, 4.12f, 2.70f, 5.07f, 4.53f, 0.93f},
                                    {13, 128, 128, 2, 7.62f, 4.93f, 3.55f, 4.33f, 1.00f}, {14, 128, 64, 2, 3.43f, 2.74f, 2.96f, 3.14f, 0.98f}},
                                   {{21, 256, 128, 1, 6.06f, 2.51f, 6.66f, 5.52f, 0.75f}, {23, 256, 64, 1, 5.37f, 2.15f, 4.18f, 3.35f, 0.74f},
                                    {24, 128, 64, 2, 5.26f, 1.73f, 2.79f, 2.10f, 0.76f}, {25, 128, 64, 4, 3.45f, 5.06f, 2.46f, 2.18f, 0.78f}}};
    const float k = 1e-3f * (float)g.Kp, row_us = g.N % 8 == 0 ? 0.0f : g.N % 4 == 0 ? 0.05f : 0.11f;
    float best = 0.0f, store = 0.0f;
    *form = 0;
    for (const Fit &f : fits[g.fmt == kW4C]) {
        if (f.parts > 1 && !parts_fit(g.Kp, f.parts)) continue;
        // (one token tile: nobody to share the touch of the weights with; 28672 x 4096 66 rows 44.6, the others 36.4 and 40.3)
        if (f.number == 13 && M <= f.tokens) continue;
        const int tiles = (g.N + f.channels - 1) / f.channels * ((M + f.tokens - 1) / f.tokens), full = tiles / num_cus, rest = tiles % num_cus;
        auto work = [&](int n) { return n == 0 ? 0.0f : n == 1 ? f.alone * k : (float)n * f.shared * k; };  // of a compute unit with n tiles
        float us = f.start + (float)full * f.each + work(full);
        if (rest > 0) us += f.each + (work(full + 1) - work(full)) * (f.idle + (1.0f - f.idle) * (float)rest / (float)num_cus);
        if (!staged_store && f.channels * f.tokens == 256 * 128) us += 4.0f;
        if (*form == 0 || us < best) {
            best = us, *form = f.number;
            store = row_us * (float)(full + (rest > 0 ? 1 : 0)) * (float)(f.parts > 1 ? f.tokens / 2 : f.tokens);
        }
    }
    return best + store;
}

hipError_t launch_gemm_i8(const Geometry &g, const void *packed, const int8_t *xq_tiled,
                          const float *sx, int M, int Mp, void *out, int out_mode, const void *residual,
                          int gated_act, int num_cus, hipStream_t st) {
    (void)Mp;
    if (out_mode == 0 && skinny_product(g, M, true, gated_act >= 0 && g.pair_half, num_cus)) return launch_skinny_i8(g, packed, xq_tiled, sx, M, out, residual, gated_act, num_cus, st);
    GemmI8Args a;
    a.w = static_cast<const uint4 *>(packed);
    a.x = reinterpret_cast<const uint4 *>(xq_tiled);
    a.sw = reinterpret_cast<const float *>(static_cast<const char *>(packed) + g.scale_off);
    a.sx = sx;
    a.res = out_mode == 0 ? static_cast<const _Float16 *>(residual) : nullptr;
    a.out = out;
    a.M = M;
    a.N = g.N;
    a.Kp = g.Kp;
    a.n_tiles = a.m_tiles = a.share = 0;
    a.walk = {};
    a.gated_act = out_mode == 0 && g.pair_half ? gated_act : -1;
    int form;
    int8_tile_us(g, M, out_mode == 0 && g.N % 8 == 0, num_cus, &form);
    if (g.fmt == kW4C) {
        a.sw_mul = 0.0625f;
        a.acc_shift = 4;
        return out_mode == 0 ? launch_mode_w4<0>(a, form, st) : launch_mode_w4<1>(a, form, st);
    }
    return out_mode == 0 ? launch_mode<0>(a, form, num_cus, st) : launch_mode<1>(a, form, num_cus, st);
}

}  // namespace qfc
