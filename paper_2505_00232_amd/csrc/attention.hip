// Attention-side operators of the decode stage.
//
// 1. Rotary embedding fused with the layout transformation of the query, key and value
//    projections (section 3.6 of the paper): the QKV layer's output [B, S, (h_q + 2 h_kv) d] goes
//    to queries [B h_kv, S g, d] (g = h_q / h_kv query heads per KV head, row s g + j), the rotated
//    keys are appended to the K cache [B h_kv, C, d] as rows pos0 + s and the values to the V cache
//    (d, cache position) as columns pos0 + s.
// 2. The two matrix products of attention with the KV cache in the role of weights (section 3.8):
//    the K cache is stored (cache position, d), i.e. K^T of Q K^T, the V cache (d, cache position);
//    both are [N, K] operands exactly like a layer's logical weight matrix, and 16 bytes of a row
//    are one lane's MFMA operand.  Physically the V cache is cut into blocks of 64 positions,
//    [B h_kv, C / 64, d, 64]: a step of the kernel then reads 128 d contiguous bytes of V as it does
//    of K, instead of d pieces of 128 bytes that lie a whole cache row apart.  Here the two products and the softmax between them run
//    in one pass over the cache (the scores never leave registers): per step of 64 positions a
//    wavefront computes S^T = K Q^T with v_mfma_f32_16x16x32_f16 (keys as rows), updates the running
//    maximum and sum of every query row, and accumulates O^T += V P^T, where the positions are
//    taken in the order in which the score tiles leave them in the lanes (no cross-lane traffic:
//    the rows of the score tiles are assigned to positions so that lane (m, r) ends up with 2 x 8
//    contiguous positions for query row m, and reads the same positions of its V rows, 16 bytes each).  The context is split over workgroups and
//    wavefronts; partial (maximum, sum, O) triples meet in LDS and then in a second small kernel.
#include <type_traits>

#include "qfc_internal.h"
#include "attention_walk.h"

namespace qfc {
namespace {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr float kNegBig = -1.0e30f;
// Maximum of a query row that has seen no position yet (prefill): above every masked score times the scale, below every real one
constexpr float kFloorMax = -1.0e25f;
static_assert(kAttnMaxSplits <= 64, "the combine kernel takes one split per lane");

// ---------------------------------------------------------------- rotary embedding + layouts
// Few tokens (decode steps, short prompts): latency is all there is.
// One thread per (b, s, head, i), i < d / 2: the pair (i, i + d / 2) of one head of one token.
__global__ __launch_bounds__(256) void rope_qkv_few_kernel(const _Float16 *__restrict__ qkv, int B, int S, int h_q,
                                                           int h_kv, int d, int C, int pos0, double log_base,
                                                           _Float16 *__restrict__ q_out, _Float16 *__restrict__ kc,
                                                           _Float16 *__restrict__ vc) {
    const int half = d / 2;
    const int heads = h_q + 2 * h_kv;
    const long total = (long)B * S * heads * half;
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    const int i = (int)(idx % half);
    const int head = (int)((idx / half) % heads);
    const int s = (int)((idx / ((long)half * heads)) % S);
    const int b = (int)(idx / ((long)half * heads * S));
    const _Float16 *src = qkv + ((size_t)(b * S + s) * heads + head) * d;
    const double x0 = (double)(float)src[i], x1 = (double)(float)src[i + half];
    const int g = h_q / h_kv;
    if (head >= h_q + h_kv) {  // value head: no rotation, transposed into the cache
        const int kv = head - h_q - h_kv;
        const int p = pos0 + s;
        _Float16 *dst = vc + (((size_t)(b * h_kv + kv) * (C / 64) + p / 64) * d) * 64 + p % 64;
        dst[(size_t)i * 64] = src[i];
        dst[(size_t)(i + half) * 64] = src[i + half];
        return;
    }
    // angle = pos * base^(-2 i / d), in double so that long contexts keep the low bits of the angle
    const double ang = (double)(pos0 + s) * exp(-2.0 * (double)i / (double)d * log_base);
    double sn, cs;
    sincos(ang, &sn, &cs);
    const _Float16 y0 = (_Float16)(float)(x0 * cs - x1 * sn);
    const _Float16 y1 = (_Float16)(float)(x1 * cs + x0 * sn);
    _Float16 *dst;
    if (head < h_q) {
        const int kv = head / g, j = head % g;
        dst = q_out + ((size_t)(b * h_kv + kv) * (S * g) + (s * g + j)) * d;
    } else {
        const int kv = head - h_q;
        dst = kc + ((size_t)(b * h_kv + kv) * C + (pos0 + s)) * d;
    }
    dst[i] = y0;
    dst[i + half] = y1;
}

// Bound: HBM (read once, written once), once the angles and the fp64 products are out of the way: cos and sin in fp64 cost
// more than everything else together when every head of a token evaluates them (S = 1024, 40 heads to
// rotate: 34 us; 6000: 165 us, where reading and writing 147 MB takes 28).  So a workgroup takes T
// tokens, evaluates their d / 2 angles once into LDS, and rotates all heads with them, 16 bytes of each half
// of a head per thread.  The rotation itself is done in pairs of fp32 that carry all rounding errors (sum_of_products): with fp64 products, whose
// conversions and operations kept the vector unit busy for half of the time, the same kernel takes, us, fp64 / fp32 pairs: 1024 tokens of 48 heads of 128
// 11.8 / 9.2, 6000 42.3 / 34.4, 2048 tokens of 16 heads of 256 14.2 / 11.0.  The results are the same bits (35 million values of five shapes).
// Few tokens: the heads are split over several workgroups.
// Values: a workgroup takes the tokens of one block of 64 cache positions of one head, turns them in LDS and
// writes runs of up to 128 bytes of the transposed cache instead of single values 128 bytes apart.
typedef _Float16 rope_h2 __attribute__((ext_vector_type(2)));
// An fp64 value as the sum of two fp32 values, the second at most half a unit in the last place of the first (48 bits and the sign)
__device__ __forceinline__ float2 split_f64(double v) {
    const float hi = (float)v;
    return make_float2(hi, (float)(v - (double)hi));
}
// x0 c + x1 s, c = (c.x, c.y) and s likewise: both products with their rounding errors (fma), their sum with its own (Knuth's
// two-sum); what the last sum rounds off decides its lowest bit (rounding to odd), so that the conversion to binary16 rounds the real
// result once, ties included: the bits that fp64 gives.  Without a correction the plain sum stands: a zero keeps its sign, and an infinite x,
// which makes the corrections NaN, gives what it gives in fp64.
__device__ __forceinline__ float sum_of_products(float x0, float2 c, float x1, float2 s) {
#pragma clang fp contract(off)  // (the two-sum needs its own roundings)
    const float p = x0 * c.x, q = x1 * s.x, sum = p + q, of_q = sum - p;
    const float rest = ((p - (sum - of_q)) + (q - of_q)) + (fmaf(x0, c.x, -p) + fmaf(x1, s.x, -q));
    const float low = fmaf(x0, c.y, fmaf(x1, s.y, rest)), r = sum + low, off = low - (r - sum);
    const int bits = __float_as_int(r), odd = (bits - ((__float_as_int(off) ^ bits) < 0 ? 1 : 0)) | 1;
    return low < 0.0f || low > 0.0f ? (off != 0.0f ? __int_as_float(odd) : r) : sum;
}
// x0 cos - x1 sin and x1 cos + x0 sin, cos = (t.x, t.y), sin = (t.z, t.w)
__device__ __forceinline__ void rotate_pair(float x0, float x1, const float4 &t, float &y0, float &y1) {
    const float2 c = make_float2(t.x, t.y), s = make_float2(t.z, t.w);
    y0 = sum_of_products(x0, c, -x1, s);
    y1 = sum_of_products(x1, c, x0, s);
}
struct RopeArgs {
    const _Float16 *qkv;
    _Float16 *q_out, *kc, *vc;
    int B, S, h_q, h_kv, d, C, pos0;
    int T, rot_wgs, pblocks;  // tokens per workgroup, workgroups that rotate, cache blocks touched
    double log_base;
};
__global__ __launch_bounds__(256) void rope_qkv_kernel(RopeArgs a) {
    extern __shared__ float4 rope_lds[];  // (cos, its rest, sin, its rest)
    const int half = a.d / 2, heads = a.h_q + 2 * a.h_kv, g = a.h_q / a.h_kv;
    if ((int)blockIdx.x < a.rot_wgs) {
        const int tok0 = (int)blockIdx.x * a.T;
        const int nt = min(a.T, a.B * a.S - tok0);
        const int rot = a.h_q + a.h_kv, vecs = half / 8;
        // thread = octet v of the heads r, r + rows, ... of the workgroup's tokens (no divisions in the loop)
        const int rows = 256 / vecs, v = threadIdx.x % vecs;
        int head = threadIdx.x / vecs, t = 0;
        auto wrap = [&](int &h, int &tt) {
            while (h >= rot) h -= rot, ++tt;
        };
        wrap(head, t);
        const int b0 = tok0 / a.S, s0 = tok0 % a.S;
        auto source = [&](int h, int tt) { return a.qkv + ((size_t)(tok0 + tt) * heads + h) * a.d + 8 * v; };
        h8 x0, x1;  // of the thread's next item: requested before the angles are evaluated
        if (t < nt) {
            x0 = *reinterpret_cast<const h8 *>(source(head, t));
            x1 = *reinterpret_cast<const h8 *>(source(head, t) + half);
        }
        // angle = pos * base^(-2 i / d), in double so that long contexts keep the low bits of the angle
        for (int e = threadIdx.x; e < nt * half; e += 256) {
            const int i = e % half, slot = e - i + (i % 8) * vecs + i / 8;  // (threads read the octet i / 8 side by side)
            double sn, cs;
            sincos((double)(a.pos0 + (tok0 + e / half) % a.S) * exp(-2.0 * (double)i / (double)a.d * a.log_base), &sn, &cs);
            const float2 c = split_f64(cs), n = split_f64(sn);
            rope_lds[slot] = make_float4(c.x, c.y, n.x, n.y);
        }
        __syncthreads();
        while (t < nt) {
            const h8 u0 = x0, u1 = x1;
            int head1 = head + rows, t1 = t;
            wrap(head1, t1);
            if (t1 < nt) {
                x0 = *reinterpret_cast<const h8 *>(source(head1, t1));
                x1 = *reinterpret_cast<const h8 *>(source(head1, t1) + half);
            }
            int b = b0, s = s0 + t;
            while (s >= a.S) s -= a.S, ++b;
            const float4 *ang = rope_lds + t * half + v;
            h8 y0, y1;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                float r0, r1;
                rotate_pair((float)u0[i], (float)u1[i], ang[vecs * i], r0, r1);
                y0[i] = (_Float16)r0;
                y1[i] = (_Float16)r1;
            }
            _Float16 *dst;
            if (head < a.h_q)
                dst = a.q_out + ((size_t)(b * a.h_kv + head / g) * (a.S * g) + (s * g + head % g)) * a.d;
            else
                dst = a.kc + ((size_t)(b * a.h_kv + head - a.h_q) * a.C + (a.pos0 + s)) * a.d;
            *reinterpret_cast<h8 *>(dst + 8 * v) = y0;
            *reinterpret_cast<h8 *>(dst + half + 8 * v) = y1;
            head = head1, t = t1;
        }
        return;
    }
    // value heads: workgroup = (b, kv, block of 64 cache positions, 64 values)
    const int w = (int)blockIdx.x - a.rot_wgs, dc = a.d / 64;
    const int d0 = (w % dc) * 64, pb = w / dc % a.pblocks, kv = w / (dc * a.pblocks) % a.h_kv, b = w / (dc * a.pblocks * a.h_kv);
    const int p0 = (a.pos0 / 64 + pb) * 64;
    const int first = max(a.pos0 - p0, 0), last = min(a.pos0 + a.S - p0, 64);  // columns of the block to write
    // LDS rows of one token each, four bytes longer than 64 values: eight rows apart is eight banks apart
    constexpr int pitch = 64 + 2;
    _Float16 *tile = reinterpret_cast<_Float16 *>(rope_lds);
    const _Float16 *src0 = a.qkv + ((size_t)b * a.S * heads + a.h_q + a.h_kv + kv) * a.d + d0;
    for (int e = threadIdx.x; e < (last - first) * 8; e += 256) {
        const int c = first + e / 8, v = e % 8;
        const h8 x = *reinterpret_cast<const h8 *>(src0 + (size_t)(p0 + c - a.pos0) * heads * a.d + 8 * v);
#pragma unroll
        for (int i = 0; i < 4; ++i) *reinterpret_cast<rope_h2 *>(tile + c * pitch + 8 * v + 2 * i) = rope_h2{x[2 * i], x[2 * i + 1]};
    }
    __syncthreads();
    _Float16 *dst0 = a.vc + (((size_t)(b * a.h_kv + kv) * (a.C / 64) + p0 / 64) * a.d + d0) * 64;
    const int o0 = first / 8, no = (last + 7) / 8 - o0;  // octets of columns
    for (int e = threadIdx.x; e < 64 * no; e += 256) {
        const int o = o0 + e % no, dd = e / no;
        _Float16 *dst = dst0 + dd * 64 + 8 * o;
        if (8 * o >= first && 8 * o + 8 <= last) {
            h8 y;
#pragma unroll
            for (int i = 0; i < 8; ++i) y[i] = tile[(8 * o + i) * pitch + dd];
            *reinterpret_cast<h8 *>(dst) = y;
        } else {
            for (int i = 0; i < 8; ++i)
                if (8 * o + i >= first && 8 * o + i < last) dst[i] = tile[(8 * o + i) * pitch + dd];
        }
    }
}

// cos and sin of the rotary angles of `positions` positions: table[(pos * d / 2 + i) * 2] = cos, + 1 = sin
// of pos * base^(-2 i / d), the angle in fp64 as in the kernel above (long contexts keep its low bits).
__global__ __launch_bounds__(256) void rope_table_kernel(int d, int positions, double log_base, float *__restrict__ table) {
    const int half = d / 2;
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (long)positions * half) return;
    const int i = (int)(idx % half);
    const int pos = (int)(idx / half);
    const double ang = (double)pos * exp(-2.0 * (double)i / (double)d * log_base);
    double sn, cs;
    sincos(ang, &sn, &cs);
    table[2 * idx] = (float)cs;
    table[2 * idx + 1] = (float)sn;
}

// ---------------------------------------------------------------- attention over the cache
struct AttnArgs {
    const _Float16 *q;   // [G, M, D]
    const _Float16 *kc;  // [G, C, D]
    const _Float16 *vc;  // [G, C / 64, D, 64]
    float *ws_o;         // [G, splits, M, D] partial outputs (unnormalized)
    float *ws_ml;        // [G, splits, M, 2] partial (maximum, sum)
    _Float16 *out;       // [G, M, D]
    int M, g, S, C, n_ctx, splits;
    int groups;       // prefill: workgroup i works on KV head i % groups
    int block_rows;   // prefill: query rows per workgroup
    int chunk_steps;  // prefill: > 0 = walks are cut into chunks of this many steps (one workgroup each)
    int max_chunks;   // prefill: chunk slots per query row in the workspace
    float scale;
};
// prefill: steps of 32 positions that the walk of block j of `rows` query rows takes (the last row of the block sees most)
__host__ __device__ inline int prefill_steps(const AttnArgs &a, int j, int rows) {
    const int last = j * rows + rows - 1 < a.M - 1 ? j * rows + rows - 1 : a.M - 1;
    return (a.n_ctx - a.S + last / a.g + 1 + 31) / 32;
}

// Workgroup = 4 wavefronts and up to 16 query rows.  grid = (splits, G, blocks of 16 query rows).  A step covers TP pairs of score tiles = 32 TP positions:
// 64 for head sizes up to 128, 32 for 256 (whose operands of 64 positions would leave one wavefront per SIMD).
// Two workgroups per compute unit (up to head size 128) are said in the launch bounds so that the accumulators stay in
// ordinary registers (with the whole register file at its disposal the compiler parks them in
// accumulation registers and copies them back and forth for the rescaling).
template <int D>
__global__ __launch_bounds__(256, D <= 128 ? 2 : 1) void attn_partial_kernel(AttnArgs a) {
    constexpr int TP = D <= 128 ? 2 : 1;
    constexpr int SP = 32 * TP;  // positions per step
    constexpr int DJ = D / 32;  // MFMA steps along d of the score product
    constexpr int DT = D / 16;  // row tiles of O^T
    constexpr int PITCH = D + 4;  // floats per staged query row: O^T column, maximum, sum (16-byte aligned rows)
    extern __shared__ float lds[];  // [4][16][PITCH]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = lane & 15, r = lane >> 4;
    const int G = blockIdx.y;
    const int part = blockIdx.x, parts = a.splits;
    const int row0 = 16 * blockIdx.z, rows = min(16, a.M - row0);
    const int n_end = a.n_ctx - a.S + (row0 + rows - 1) / a.g + 1;  // positions the block's last row sees
    const int nb = (n_end + SP - 1) / SP;  // steps
    // the workgroup takes a contiguous range of steps; its wavefronts take every fourth step of it
    const int b0 = (int)((long)part * nb / parts) + wave, b1 = (int)((long)(part + 1) * nb / parts);

    // Q^T operand: lane (m, r) holds Q[row0 + m][32 j + 8 r .. + 7]; rows past the last are zero
    u32x4 qf[DJ];
#pragma unroll
    for (int j = 0; j < DJ; ++j) {
        const u32x4 zero = {0, 0, 0, 0};
        qf[j] = m < rows ? *reinterpret_cast<const u32x4 *>(a.q + ((size_t)G * a.M + row0 + m) * D + 32 * j + 8 * r) : zero;
    }
    // positions a query row may see: those before the end of its own token
    // (rows past the last are all-zero queries whose results are never stored: they see everything)
    const int lim = m < rows ? a.n_ctx - a.S + (row0 + m) / a.g + 1 : n_end;

    v4f acc[DT];
#pragma unroll
    for (int t = 0; t < DT; ++t) acc[t] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    float run_max = kNegBig, run_sum = 0.0f;  // run_sum: this lane's share (its 8 positions per block)

    const _Float16 *kbase = a.kc + (size_t)G * a.C * D;
    const _Float16 *vbase = a.vc + (size_t)G * D * a.C;
    // One step = 64 positions: four score tiles of 16 positions, two MFMA steps of 32 positions for
    // O^T.  All operands of a step are requested at once, so that each 128-byte line of a V row (64
    // positions) is fetched by one burst of one wavefront.  The loop is software pipelined without a
    // second set of registers: the next step's K operands are requested as soon as the score MFMAs
    // have consumed the current ones (they fly during the softmax and the O^T MFMAs), the next step's
    // V operands at the end of the step (they fly during the next score MFMAs and softmax).
    // Which position a row of a score tile stands for is free; row w of tile t is position
    //   k0 + 32 (t / 2) + 8 (w / 4) + 4 (t % 2) + w % 4,
    // so that the eight values lane (m, r) holds of tiles (2 u, 2 u + 1) are the contiguous positions
    // k0 + 32 u + 8 r .. + 7: its V operand of MFMA step u is one 16-byte load, and the four lanes r
    // of a V row read 64 contiguous bytes.  K: lane (w = lane & 15, r) reads d = 32 j + 8 r .. + 7 of
    // its position's row (a K row is contiguous whatever the order of the rows).
    u32x4 kf[2 * TP][DJ];
    u32x4 vf[DT][TP];
    auto load_k = [&](int blk) {
#pragma unroll
        for (int t = 0; t < 2 * TP; ++t) {
            const int pos = blk * SP + 32 * (t >> 1) + 8 * (m >> 2) + 4 * (t & 1) + (m & 3);
            const _Float16 *krow = kbase + (size_t)pos * D + 8 * r;
#pragma unroll
            for (int j = 0; j < DJ; ++j) kf[t][j] = *reinterpret_cast<const u32x4 *>(krow + 32 * j);
        }
    };
    auto load_v = [&](int blk) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            const int p0 = blk * SP;  // first position of the step: block p0 / 64 of the cache, column p0 % 64
            const _Float16 *vrow = vbase + ((size_t)(p0 / 64) * D + 16 * dt + m) * 64 + p0 % 64 + 8 * r;
#pragma unroll
            for (int u = 0; u < TP; ++u)
                vf[dt][u] = *reinterpret_cast<const u32x4 *>(vrow + 32 * u);
        }
    };
    if (b0 < b1) {
        load_k(b0);
        load_v(b0);
    }
    for (int blk = b0; blk < b1; blk += 4) {
        const int k0 = blk * SP;
        // ---- S^T = K Q^T; lane (m, r) holds positions k0 + 32 (t / 2) + 8 r + 4 (t % 2) + i
        v4f st[2 * TP];
#pragma unroll
        for (int t = 0; t < 2 * TP; ++t) {
            v4f acc_s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int j = 0; j < DJ; ++j)
                acc_s = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, kf[t][j]), __builtin_bit_cast(h8, qf[j]), acc_s, 0, 0, 0);
            st[t] = acc_s;
        }
        if (blk + 4 < b1) load_k(blk + 4);
        // ---- scaled (in units of log 2, so that exponentials are bare v_exp_f32) and, in the steps that
        // reach past the first query token's horizon, masked
        float sc[8 * TP];
        float bmax = kNegBig;
        const bool edge = k0 + SP > a.n_ctx - a.S + row0 / a.g + 1;  // same for the whole wavefront
        if (!edge) {
#pragma unroll
            for (int e = 0; e < 8 * TP; ++e) {
                sc[e] = st[e >> 2][e & 3] * a.scale;
                bmax = fmaxf(bmax, sc[e]);
            }
        } else {
#pragma unroll
            for (int t = 0; t < 2 * TP; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int pos = k0 + 32 * (t >> 1) + 8 * r + 4 * (t & 1) + i;
                    sc[4 * t + i] = pos < lim ? st[t][i] * a.scale : kNegBig;
                    bmax = fmaxf(bmax, sc[4 * t + i]);
                }
        }
        bmax = fmaxf(bmax, __shfl_xor(bmax, 16, 64));
        bmax = fmaxf(bmax, __shfl_xor(bmax, 32, 64));
        const float new_max = fmaxf(run_max, bmax);
        const float corr = __builtin_amdgcn_exp2f(run_max - new_max);
        run_max = new_max;
        float psum = 0.0f;
        h8 pv[TP];  // P^T operands of the MFMA steps: positions of tiles (0, 1), (2, 3)
#pragma unroll
        for (int e = 0; e < 8 * TP; ++e) {
            // a masked score is kNegBig: 2^(kNegBig - maximum) is 0 unless the row has seen no valid
            // position yet (maximum = kNegBig), which the test on the score itself excludes
            float p = __builtin_amdgcn_exp2f(sc[e] - new_max);
            if (edge) p = sc[e] > 0.5f * kNegBig ? p : 0.0f;
            psum += p;
            pv[e >> 3][e & 7] = (_Float16)p;
        }
        run_sum = run_sum * corr + psum;
        // positions at or past the end of the context may hold anything (0 * NaN would poison the sum)
        if (k0 + SP > n_end) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int u = 0; u < TP; ++u) {
                    const int p0 = k0 + 32 * u + 8 * r;
                    uint32_t w[4] = {vf[dt][u].x, vf[dt][u].y, vf[dt][u].z, vf[dt][u].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if (p0 + 2 * e >= n_end) w[e] &= 0xFFFF0000u;
                        if (p0 + 2 * e + 1 >= n_end) w[e] &= 0x0000FFFFu;
                    }
                    vf[dt][u] = u32x4{w[0], w[1], w[2], w[3]};
                }
        }
        // ---- O^T = O^T corr + V P^T (the running maxima settle early: most steps have corr = 1 in every lane)
        const bool rescale = __any(corr != 1.0f);
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            v4f o = acc[dt];
            if (rescale) {
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] *= corr;
            }
#pragma unroll
            for (int u = 0; u < TP; ++u) {
                o = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, vf[dt][u]), pv[u], o, 0, 0, 0);
            }
            acc[dt] = o;
        }
        if (blk + 4 < b1) load_v(blk + 4);
    }
    run_sum += __shfl_xor(run_sum, 16, 64);
    run_sum += __shfl_xor(run_sum, 32, 64);

    // ---- the four wavefronts meet in LDS: [wave][m][PITCH] = O^T column m, then (maximum, sum)
    float *mine = lds + (size_t)wave * 16 * PITCH + (size_t)m * PITCH;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) *reinterpret_cast<v4f *>(mine + 16 * dt + 4 * r) = acc[dt];  // rows d = 16 dt + 4 r + i
    if (r == 0) {
        mine[D] = run_max;
        mine[D + 1] = run_sum;
    }
    __syncthreads();
    // A thread takes four columns of a row: maxima, factors and sum once for the four.  Latency-bound where a workgroup has 16
    // rows (us, one column per thread / four: 77 tokens, 8 heads on 4 of 256 values 9.3 / 7.5, 32 on 8 of 128 7.0 / 5.9; one token,
    // 1280 positions 9.0 / 8.8 and 8.2 / 8.0 with the combination).
    for (int e = threadIdx.x; e < rows * (D / 4); e += 256) {
        const int mm = e / (D / 4), dd = 4 * (e % (D / 4));
        const float *row = lds + (size_t)mm * PITCH;
        float f[4], mx = kNegBig, l = 0.0f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            f[w] = row[(size_t)w * 16 * PITCH + D];
            mx = fmaxf(mx, f[w]);
        }
        v4f o = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const v4f part_o = *reinterpret_cast<const v4f *>(row + (size_t)w * 16 * PITCH + dd);
            f[w] = __builtin_amdgcn_exp2f(f[w] - mx);
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] += f[w] * part_o[i];
            l += f[w] * row[(size_t)w * 16 * PITCH + D + 1];
        }
        if (a.splits == 1) {
            h4 y;
#pragma unroll
            for (int i = 0; i < 4; ++i) y[i] = (_Float16)(o[i] / l);
            *reinterpret_cast<h4 *>(a.out + ((size_t)G * a.M + row0 + mm) * D + dd) = y;
        } else {
            const size_t p = ((size_t)G * a.splits + blockIdx.x) * a.M + row0 + mm;
            *reinterpret_cast<v4f *>(a.ws_o + p * D + dd) = o;
            if (dd == 0) {
                a.ws_ml[p * 2] = mx;
                a.ws_ml[p * 2 + 1] = l;
            }
        }
    }
}

// grid = (M, G, D / 64), one wavefront per query row and 64 columns: lane s first takes the (maximum,
// sum) pair of split s (splits <= 64) and the factors 2^(maximum_s - maximum) are shared by lane
// broadcast; lane l sums column 64 z + l of the partial outputs in split order.
template <int D>
__global__ __launch_bounds__(64) void attn_combine_kernel(AttnArgs a) {
    const int G = blockIdx.y, mm = blockIdx.x, lane = threadIdx.x;
    const int col = 64 * blockIdx.z + lane;
    const size_t row0 = ((size_t)G * a.splits) * a.M + mm;  // partial row of split s: row0 + s * M
    // The first 32 splits' columns are requested before the factors are known (splits past the last read the last one
    // again and count as 0: their factor is 0, but the last one may be infinite): one trip to memory instead of one for the
    // pairs and one for every eight splits.
    // us, walk and combination, before / after: 8 heads on 4 of 256 values, 1280 positions 8.7 / 8.0; 32 on 8 of 128, 1280 7.8 / 7.2,
    // 12001 17.1 / 16.0; head size 64, 4000 positions 8.4 / 7.6.
    float v[4][8];
    const float *src = a.ws_o + row0 * D + col;
    const size_t step = (size_t)a.M * D;
    auto fetch = [&](int k, int s) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 8; ++u) v[k][u] = src[(size_t)min(s + u, a.splits - 1) * step];
    };
    float mx = kNegBig, l = 0.0f;
    if (lane < a.splits) {
        mx = a.ws_ml[(row0 + (size_t)lane * a.M) * 2];
        l = a.ws_ml[(row0 + (size_t)lane * a.M) * 2 + 1];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (8 * k < a.splits) fetch(k, 8 * k);
    float top = mx;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) top = fmaxf(top, __shfl_xor(top, off, 64));
    const float f = lane < a.splits ? __builtin_amdgcn_exp2f(mx - top) : 0.0f;
    float lsum = f * l;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) lsum += __shfl_xor(lsum, off, 64);
    float o = 0.0f;
    for (int s = 0; s < a.splits; s += 32) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (s + 8 * k >= a.splits) break;
            if (s + 8 * k + 8 > a.splits) {  // (us, 1280 positions, the select in every group / in the last one only: 3.58 / 3.42)
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (s + 8 * k + u >= a.splits) v[k][u] = 0.0f;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) o = fmaf(__shfl(f, s + 8 * k + u, 64), v[k][u], o);
            if (s + 8 * k + 32 < a.splits) fetch(k, s + 8 * k + 32);
        }
    }
    a.out[((size_t)G * a.M + mm) * D + col] = (_Float16)(o / lsum);
}

// ---------------------------------------------------------------- attention, many query rows (prefill)
// More than 16 query rows per KV head.  A wavefront owns 32 query rows (the columns of
// v_mfma_f32_32x32x16_f16) and walks positions in steps of 32: S^T = K Q^T (32 positions x 32 queries),
// running maximum and sum per query (a query's 16 scores of a step sit in two lanes), O^T += V P^T.  As in the
// decode kernel the rows of the score tile are assigned to positions so that a lane's eight probabilities of
// an MFMA step are eight contiguous positions (row i = 16 c + 8 b + 4 h + r is position
// k0 + 16 c + 8 h + 4 b + r): P goes from the first product's result registers into the second product's
// operand registers as it is, and a lane's V operand is one 16-byte read.
// A workgroup is four wavefronts: PS of them share the same query rows and take every PS-th step of the walk
// (their results meet in LDS at the end), 4 / PS own different rows.  Causal walks are of very different length and a
// launch lasts as long as its longest: with PS = 2 that one is half as long, and there are twice as many workgroups to
// spread.  A stage of LDS holds the PS steps the workgroup works on together.
// LDS layouts (16-byte chunks, XOR-swizzled so that the operand reads are conflict free; the copy
// writes LDS linearly, so the swizzle is applied to the address it reads from memory):
//   K step: row = position (32), D / 8 chunks per row; chunk o of row p sits at o ^ swz(p)
//   V step: row = d (D), 4 chunks per row (32 positions); chunk c of row d sits at c ^ ((d >> 2) & 3)
// Causal: rows of token s see positions 0 .. n_ctx - S + s; the block stops at the last position
// its last row sees, rows that see less mask the rest.
// Registers: up to head size 128 two workgroups per compute unit, everything in ordinary registers; at 256 one, whose
// query operands and part of whose sums sit in accumulation registers (scores in ordinary ones: a flag of this file's build).
// What bounds it: at 8192 tokens (head size 128) power and both units: matrix cores busy 54 %, vector unit 59 % of the clocks, the
// clock at 1.6 to 1.8 GHz.  Short walks: latency (head size 128: 4 us before the first and behind the last step, a stage of a workgroup alone
// on its compute unit 0.5 to 0.6 us, of two together 1.2).
// Measured (us, 32 heads on 8 of 128; blocks of 128 rows with one walk each / this, both in one session, caches not in L2): 512 tokens
// 19.1 / 13.1, 1024 32.1 / 22.1, 2048 65 / 61.5, 6000 373 / 319, 8192 630 / 567 (0.97 PFLOP/s), 130 behind 2870 positions 31.6 / 24.8, 300 behind
// 6000 60 / 57; head size 64, 8 heads, 4096 tokens 53 / 38; head size 256, 8 heads on 4, 2048 tokens 58 / 49, 4096 175 / 128.
template <int D, int PS>
struct PrefillCfg {
    static constexpr int CPR = D / 8;           // 16-byte chunks per K row
    static constexpr int KB = 32 * D * 2;       // bytes of K (and of V) of a step
    static constexpr int RW = 4 / PS;           // wavefronts that own different rows
    static constexpr int ROWS = 32 * RW;        // query rows per workgroup
    static constexpr int NB = 6 * PS * KB <= (D <= 128 ? 48 : 96) * 1024 ? 3 : 2;  // LDS stages
    static constexpr int COPIES = KB / 4096;    // copies per wavefront and step, of K and of V
    static constexpr int MERGE = PS > 1 ? 4 * ((D / 32) * 4096 + 256) : 0;  // bytes of the wavefronts' results
    static constexpr int RING = 2 * NB * PS * KB;
    static constexpr int LDS = RING > MERGE ? RING : MERGE;
    static_assert(LDS <= (D <= 128 ? 80 : 160) * 1024 && 2 * PS * COPIES * NB <= 63, "LDS, and the 6-bit counter of outstanding copies");
    __device__ static int swz(int p) { return D >= 128 ? (p & 15) : ((p >> 1) & 7); }
};
// maximum over the lanes l and l ^ 32
__device__ __forceinline__ float both_halves_max(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

template <int D, int PS>
__global__ __launch_bounds__(256, D <= 128 ? 2 : 1) void attn_prefill_kernel(AttnArgs a) {
    typedef float v16f __attribute__((ext_vector_type(16)));
    typedef PrefillCfg<D, PS> Cfg;
    constexpr int DJ = D / 16;  // MFMA steps along d of the score product
    constexpr int DT = D / 32;  // row tiles of O^T
    constexpr int NB = Cfg::NB, KB = Cfg::KB, RW = Cfg::RW;
    constexpr int KP = DJ < 8 ? DJ : 8;  // K operands of a step requested during the step before
    extern __shared__ uint4 lds_raw[];
    char *const ldsb = reinterpret_cast<char *>(lds_raw);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rw = wave % RW, ps = wave / RW;
    const int q = lane & 31, h = lane >> 5;
    // (groups side by side: where 8 divides their number, the workgroups of one share the L2 of one XCD)
    const int G = (int)blockIdx.x % a.groups, item = (int)blockIdx.x / a.groups;
    const int nblocks = (a.M + Cfg::ROWS - 1) / Cfg::ROWS;
    // Longest walks first: the compute units that finish theirs take the shorter ones.  a.chunk_steps > 0 (a multiple of
    // PS; few blocks): the walk of a block is cut into chunks of that many steps, one workgroup
    // each; a block with more than one chunk leaves unnormalized partial results that a second kernel combines.
    int block = nblocks - 1 - item, chunk = 0, chunks = 1;
    if (a.chunk_steps > 0) {
        int w = item;
        for (block = nblocks - 1;; --block) {
            chunks = (prefill_steps(a, block, Cfg::ROWS) + a.chunk_steps - 1) / a.chunk_steps;
            if (w < chunks || block == 0) break;
            w -= chunks;
        }
        chunk = w;
        if (chunk >= chunks) return;  // (a grid larger than the chunk count: nothing to do)
    }
    const int r0 = block * Cfg::ROWS + rw * 32;  // first query row of the wavefront
    const int m = r0 + q;
    const bool real = m < a.M;
    // (the same in every lane: said explicitly, the divisions would otherwise be carried out per lane
    // and drag the loop control and the copy addresses into vector registers)
    const int lo_full = __builtin_amdgcn_readfirstlane(a.n_ctx - a.S + min(r0, a.M - 1) / a.g + 1);  // positions every row of the wavefront sees
    const int nb_all = __builtin_amdgcn_readfirstlane(prefill_steps(a, block, Cfg::ROWS));
    // the steps this workgroup takes: [sb, nb), in stages of PS
    const int sb = chunk * a.chunk_steps;
    const int nb = chunks > 1 ? min(nb_all, sb + a.chunk_steps) : nb_all;
    const int lim = min(real ? a.n_ctx - a.S + m / a.g + 1 : a.n_ctx, 32 * nb);  // end of the positions the lane's row sees in them

    // Q^T operand: lane (q, h) holds Q[m][16 j + 8 h .. + 7]
    h8 qf[DJ];
#pragma unroll
    for (int j = 0; j < DJ; ++j) {
        const h8 zero = {0};
        qf[j] = real ? *reinterpret_cast<const h8 *>(a.q + ((size_t)G * a.M + m) * D + 16 * j + 8 * h) : zero;
    }

    // ---- copies: the KiB pieces of a step are dealt to the wavefronts in turn
    const char *kbase = reinterpret_cast<const char *>(a.kc + (size_t)G * a.C * D);
    const char *vbase = reinterpret_cast<const char *>(a.vc + (size_t)G * D * a.C);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)lds_raw;
    constexpr int PP = KB / 1024;  // pieces per step
    static_assert(PP % 4 == 0, "the wavefronts' pieces of one round belong to the same step");
    constexpr int NO = Cfg::COPIES;
    uint32_t koffs[NO], voffs[NO];
#pragma unroll
    for (int i = 0; i < NO; ++i) {
        const int L = (4 * i + wave) * 64 + lane;  // 16-byte chunk of the step
        const int p = L / Cfg::CPR, o = (L % Cfg::CPR) ^ Cfg::swz(p);
        koffs[i] = (uint32_t)(p * (2 * D) + o * 16);
        const int d = L >> 2, c = (L & 3) ^ ((d >> 2) & 3);
        voffs[i] = (uint32_t)(d * 128 + c * 16);
    }
    auto uniform = [](const char *p) {  // (the same in every lane: keeps the address in scalar registers)
        const uint64_t x = reinterpret_cast<uint64_t>(p);
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x), hi = __builtin_amdgcn_readfirstlane((uint32_t)(x >> 32));
        return reinterpret_cast<const void *>(((uint64_t)hi << 32) | lo);
    };
    const uint32_t lds_wave = __builtin_amdgcn_readfirstlane(lds0 + wave * 1024);
    auto copy_k = [&](int t, int p, int slot) __attribute__((always_inline)) {
        const char *src = kbase + (size_t)(sb + t * PS + p) * KB;
#pragma unroll
        for (int i = 0; i < NO; ++i) copy16_to_lds_at(uniform(src), koffs[i], lds_wave + slot * (PS * KB), p * KB + 4096 * i);
    };
    auto copy_v = [&](int t, int p, int slot) __attribute__((always_inline)) {
        const int first = sb + t * PS;  // (even for PS = 2)
        const char *src = PS == 2 ? vbase + (size_t)(first / 2) * (D * 128) + p * 64 : vbase + (size_t)(first / 2) * (D * 128) + (first & 1) * 64;
#pragma unroll
        for (int i = 0; i < NO; ++i) copy16_to_lds_at(uniform(src), voffs[i], lds_wave + (NB + slot) * (PS * KB), p * KB + 4096 * i);
    };
    auto wait = [](auto n) __attribute__((always_inline)) {
        // (one asm: the operand reads before it are issued before it, and none may be in flight when the barrier opens)
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(decltype(n)::value) : "memory");
    };

    // operand read offsets of this lane inside the rings
    const int pp = 16 * (q >> 4) + 8 * ((q >> 2) & 1) + 4 * ((q >> 3) & 1) + (q & 3);  // position of score-tile row q
    int koff[DJ];
#pragma unroll
    for (int j = 0; j < DJ; ++j) koff[j] = ps * KB + pp * (2 * D) + (((2 * j + h) ^ Cfg::swz(pp)) * 16);
    int voff[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) voff[c] = NB * PS * KB + ps * KB + q * 64 + (((2 * c + h) ^ ((q >> 2) & 3)) * 16);
    auto read_k = [&](int j, int slot) __attribute__((always_inline)) { return *reinterpret_cast<const h8 *>(ldsb + koff[j] + slot * (PS * KB)); };

    v16f acc[DT], st;
    float run_max = kFloorMax, run_sum = 0.0f;
    float top;  // the lane's largest raw score of the step at hand
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[t][e] = 0.0f;
    h8 kf[KP];
    // register e = 8 c + 4 b + r of lane (q, h): position k0 + 8 h + (16 c + 4 b + r)
    auto mask = [&](v16f &s, int k0) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 16; ++e) s[e] = 16 * (e >> 3) + (e & 7) < lim - k0 - 8 * h ? s[e] : kNegBig;
    };
    auto largest = [&](const v16f &s) __attribute__((always_inline)) {
        float x = fmaxf(s[0], s[1]);
#pragma unroll
        for (int e = 2; e < 16; e += 2) x = fmaxf(fmaxf(x, s[e]), s[e + 1]);
        return x;
    };
    v16f sn;
    h8 vf[DT][2], pv[2];

    // ---- the walk (its order: attention_walk.h).  Before the loop: the scores of stage 0
    auto first = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < DJ; ++j) {
            const v16f zero = {0};
            st = __builtin_amdgcn_mfma_f32_32x32x16_f16(read_k(j, 0), qf[j], j == 0 ? zero : st, 0, 0, 0);
        }
        if (32 * (sb + ps) + 32 > lo_full || sb + ps >= nb) mask(st, 32 * (sb + ps));
        top = largest(st);
    };
    auto request_k = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < KP; ++j) kf[j] = read_k(j, slot);
    };
    // One step per stage.  Scores of the next step first (their MFMAs run beside the exponentials of this one), then, behind
    // the barrier that hands over the next stage, the second product (beside the rest of the exponentials and the next step's
    // maximum).  BULK: branch-free but for the rescaling, with an order of MFMAs and vector instructions asked of the scheduler.
    auto head = [&](int t, int slot, int slot1, auto bulk_c, bool next) __attribute__((always_inline)) {
        constexpr bool BULK = decltype(bulk_c)::value;
        const int k0 = 32 * (sb + t * PS + ps);
        if (__any(top * a.scale > run_max)) {
            const float nm = fmaxf(run_max, both_halves_max(top) * a.scale), corr = __builtin_amdgcn_exp2f(run_max - nm);
            run_max = nm;
            run_sum *= corr;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[dt][e] *= corr;
        }
        if (next) {
#pragma unroll
            for (int j = 0; j < DJ; ++j) {
                const v16f zero = {0};
                sn = __builtin_amdgcn_mfma_f32_32x32x16_f16(j < KP ? kf[j < KP ? j : 0] : read_k(j, slot1), qf[j], j == 0 ? zero : sn, 0, 0, 0);
            }
        }
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) vf[dt][c] = *reinterpret_cast<const h8 *>(ldsb + voff[c] + dt * 2048 + slot * (PS * KB));
        if (!BULK && k0 + 32 > a.n_ctx) {  // positions past the context may hold anything
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int c = 0; c < 2; ++c)
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        if (k0 + 16 * c + 8 * h + e >= a.n_ctx) vf[dt][c][e] = (_Float16)0.0f;
        }
        float sum4[4];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            // raw scores; the scale (in units of log 2) is applied inside the exponent: 2^(s scale - maximum); masked ones
            // give 0 (the maximum of a row that has seen nothing is far above them)
            const float p = __builtin_amdgcn_exp2f(fmaf(st[e], a.scale, -run_max));
            sum4[e & 3] = e < 4 ? p : sum4[e & 3] + p;
            pv[e >> 3][e & 7] = (_Float16)p;
        }
        run_sum += (sum4[0] + sum4[1]) + (sum4[2] + sum4[3]);
    };
    auto tail = [&](int t, auto bulk_c, bool next) __attribute__((always_inline)) {
        constexpr bool BULK = decltype(bulk_c)::value;
        const int k1 = 32 * (sb + (t + 1) * PS + ps);  // first position of the next step
        if (BULK || PS == 1 || k1 - 32 * PS < 32 * nb) {  // (a step that the last stage lacks: its V operands are anything)
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vf[dt][c], pv[c], acc[dt], 0, 0, 0);
        }
        if (next) {
            if (!BULK && (k1 + 32 > lo_full || k1 >= 32 * nb)) mask(sn, k1);
            top = largest(sn);
            st = sn;
        }
        if (BULK) {  // every MFMA followed by its share of the vector instructions (56 of the exponentials, 8 of the maximum)
#pragma unroll
            for (int j = 0; j < DJ; ++j) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
            }
#pragma unroll
            for (int j = 0; j < DT; ++j) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
            }
#pragma unroll
            for (int j = 0; j < DT; ++j) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
            }
        }
    };
    const int full = lo_full / 32 - 1 - sb - ps;  // (steps up to lo_full / 32 - 1 are unmasked)
    prefill_walk<NB, PS, Cfg::COPIES>(nb - sb, full < 0 ? 0 : full / PS, copy_k, copy_v, wait, first, request_k, head, tail);
    run_sum += __shfl_xor(run_sum, 32, 64);

    // ---- the PS wavefronts of the same rows meet in LDS; each then finishes the d tiles dt = ps, ps + PS, ...
    if constexpr (PS > 1) {
        constexpr int PER_WAVE = DT * 4096;
        float *ml = reinterpret_cast<float *>(ldsb + 4 * PER_WAVE);  // [wave][q]: maximum, sum
        asm volatile("s_barrier" ::: "memory");  // everyone is done with the rings
        if (h == 0) {
            ml[(wave * 32 + q) * 2] = run_max;
            ml[(wave * 32 + q) * 2 + 1] = run_sum;
        }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
            if (dt % PS != ps)
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    *reinterpret_cast<v4f *>(ldsb + wave * PER_WAVE + (dt * 4 + b) * 1024 + lane * 16) =
                        v4f{acc[dt][4 * b], acc[dt][4 * b + 1], acc[dt][4 * b + 2], acc[dt][4 * b + 3]};
        __syncthreads();
        float f[PS], own = 0.0f;
        run_max = kFloorMax;
#pragma unroll
        for (int w = 0; w < PS; ++w) run_max = fmaxf(run_max, ml[((w * RW + rw) * 32 + q) * 2]);
        run_sum = 0.0f;
#pragma unroll
        for (int w = 0; w < PS; ++w) {
            const float *src = ml + ((w * RW + rw) * 32 + q) * 2;
            f[w] = __builtin_amdgcn_exp2f(src[0] - run_max);
            run_sum += f[w] * src[1];
            own = w == ps ? f[w] : own;
        }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            if (dt % PS != ps) continue;
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[dt][e] *= own;
#pragma unroll
            for (int w = 0; w < PS; ++w) {
                if (w == ps) continue;
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const v4f o = *reinterpret_cast<const v4f *>(ldsb + (w * RW + rw) * PER_WAVE + (dt * 4 + b) * 1024 + lane * 16);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[dt][4 * b + e] = fmaf(f[w], o[e], acc[dt][4 * b + e]);
                }
            }
        }
    }
    if (!real) return;
    // lane (q, h) holds O^T rows d = 32 dt + 8 b + 4 h + r of column q: four consecutive d per b
    const size_t slot = ((size_t)G * a.max_chunks + chunk) * a.M + m;  // (rows side by side: 4 KiB apart they meet in one memory channel)
    const float inv = 1.0f / run_sum;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
        if (PS > 1 && dt % PS != ps) continue;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int d = 32 * dt + 8 * b + 4 * h;
            const v4f o = {acc[dt][4 * b], acc[dt][4 * b + 1], acc[dt][4 * b + 2], acc[dt][4 * b + 3]};
            if (chunks > 1)  // partial result: unnormalized O^T column, maximum (in units of log 2) and sum
                *reinterpret_cast<v4f *>(a.ws_o + slot * D + d) = o;
            else
                *reinterpret_cast<h4 *>(a.out + ((size_t)G * a.M + m) * D + d) =
                    h4{(_Float16)(o[0] * inv), (_Float16)(o[1] * inv), (_Float16)(o[2] * inv), (_Float16)(o[3] * inv)};
        }
    }
    if (chunks > 1 && h == 0 && ps == 0) {
        a.ws_ml[slot * 2] = run_max;
        a.ws_ml[slot * 2 + 1] = run_sum;
    }
}

// Chunked walks: the rows of blocks with more than one chunk.  One wavefront per query row; lane l
// takes the D / 64 consecutive values from d = l D / 64.
template <int D>
__global__ __launch_bounds__(256) void attn_prefill_combine_kernel(AttnArgs a) {
    constexpr int PER = D / 64;
    const int lane = threadIdx.x & 63;
    const int m = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    const int G = blockIdx.y;
    if (m >= a.M) return;
    const int chunks = (prefill_steps(a, m / a.block_rows, a.block_rows) + a.chunk_steps - 1) / a.chunk_steps;
    if (chunks <= 1) return;  // written by the first kernel
    const size_t slot0 = (size_t)G * a.max_chunks * a.M + m;  // chunk c's: slot0 + c * M
    // lane c < chunks holds chunk c's (maximum, sum); all loads of the row are requested at once
    static_assert(kPrefillMaxChunks == 8, "the reductions below cover eight lanes");
    float mx = kNegBig, l = 0.0f;
    if (lane < chunks) {
        mx = a.ws_ml[(slot0 + (size_t)lane * a.M) * 2];
        l = a.ws_ml[(slot0 + (size_t)lane * a.M) * 2 + 1];
    }
    float part[kPrefillMaxChunks][PER];
#pragma unroll
    for (int c = 0; c < kPrefillMaxChunks; ++c) {
#pragma unroll
        for (int e = 0; e < PER; ++e) part[c][e] = 0.0f;
        if (c >= chunks) continue;  // (the same for the whole wavefront)
        const float *src = a.ws_o + (slot0 + (size_t)c * a.M) * D + lane * PER;
#pragma unroll
        for (int e = 0; e < PER; ++e) part[c][e] = src[e];
    }
    float top = mx;
#pragma unroll
    for (int off = 1; off < 8; off <<= 1) top = fmaxf(top, __shfl_xor(top, off, 64));
    top = __shfl(top, 0, 64);
    const float f = lane < chunks ? __builtin_amdgcn_exp2f(mx - top) : 0.0f;
    float den = f * l;
#pragma unroll
    for (int off = 1; off < 8; off <<= 1) den += __shfl_xor(den, off, 64);
    den = __shfl(den, 0, 64);
    float o[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) o[e] = 0.0f;
#pragma unroll
    for (int c = 0; c < kPrefillMaxChunks; ++c) {
        const float fc = __shfl(f, c, 64);  // 0 for c >= chunks
#pragma unroll
        for (int e = 0; e < PER; ++e) o[e] = fmaf(fc, part[c][e], o[e]);
    }
    const float inv = 1.0f / den;
    _Float16 *dst = a.out + ((size_t)G * a.M + m) * D + lane * PER;
#pragma unroll
    for (int e = 0; e < PER; ++e) dst[e] = (_Float16)(o[e] * inv);
}

template <int D, int PS>
hipError_t launch_attn_prefill(const AttnArgs &a, hipStream_t st) {
    constexpr int rows = PrefillCfg<D, PS>::ROWS, lds = PrefillCfg<D, PS>::LDS;
    if (a.block_rows != rows) return hipErrorInvalidValue;
    if (const hipError_t e = allow_dynamic_lds<attn_prefill_kernel<D, PS>>(lds); e != hipSuccess) return e;
    const int nblocks = (a.M + rows - 1) / rows;
    int items = nblocks;
    if (a.chunk_steps > 0) {
        items = 0;
        for (int j = 0; j < nblocks; ++j) items += (prefill_steps(a, j, rows) + a.chunk_steps - 1) / a.chunk_steps;
    }
    attn_prefill_kernel<D, PS><<<dim3((unsigned)(items * a.groups)), 256, lds, st>>>(a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.chunk_steps == 0) return e;
    attn_prefill_combine_kernel<D><<<dim3((unsigned)((a.M + 3) / 4), (unsigned)a.groups), 256, 0, st>>>(a);
    return hipGetLastError();
}

template <int D>
hipError_t launch_attn(const AttnArgs &a, int G, hipStream_t st) {
    const size_t lds = (size_t)4 * 16 * (D + 4) * sizeof(float);
    if (const hipError_t e = allow_dynamic_lds<attn_partial_kernel<D>>(lds); e != hipSuccess) return e;
    attn_partial_kernel<D><<<dim3((unsigned)a.splits, (unsigned)G, (unsigned)((a.M + 15) / 16)), 256, lds, st>>>(a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || a.splits == 1) return e;
    attn_combine_kernel<D><<<dim3((unsigned)a.M, (unsigned)G, D / 64), 64, 0, st>>>(a);
    return hipGetLastError();
}

}  // namespace

// Decode: workgroups per (batch, KV head) group.  One workgroup per compute unit, as far as there are steps: a
// compute unit pulls about 35 GB/s with the operands of four wavefronts in flight, so the cache is
// spread over all of them even if only one wavefront of a workgroup has a step, and a second batch of workgroups
// on some compute units is what the launch would wait for.  Not for up to four steps (one per wavefront of a single
// workgroup, and no second launch), and beyond 24 only with two steps each (the combination gets
// slower).  Where one workgroup per compute unit leaves more than 40 % of them idle: two per compute unit.
// Measured (us, G = groups; 1 to 64 workgroups each, the best of them / this rule / 4 steps per workgroup as
// long as there are 2 workgroups per compute unit): head size 128, G = 8: 1280 positions 8.0 / 8.0 / 9.5, 12001
// 15.9 / 16.1 / 18.1; G = 56: 3000 21.5 / 21.5 / 25.8, 9000 51.3 / 51.3 / 61.0; G = 256: 300 11.6 / 11.6 /
// 14.5; head size 256, G = 4: 1280 8.7 / 8.7 / 12.9; G = 20: 9000 40.1 / 40.1 / 51.8; G = 44: 1500 20.0 / 20.0 / 27.6.
int attn_splits(int G, int M, int d, int n_ctx, int num_cus) {
    const int step = d <= 128 ? 64 : 32, steps = (n_ctx + step - 1) / step;
    if (steps <= 4 || num_cus < 1) return 1;
    int s = num_cus / G;
    if (5L * G * s < 3L * num_cus) s = 2 * num_cus / G;
    // More KV heads than compute units and a last round that is a third full or less: four walks each.  What that saves, the idle part of one round, grows with the
    // positions; the partial results, written and read, grow with the heads and the query rows: taken from positions x idle share = heads x (1.8 + 0.15
    // rows) on, where it was nowhere slower over 780 combinations of 257 to 4112 heads of 64, 128 and 256, 1 to 16 rows, 448 to 6000 positions (without that
    // line up to 1.56 times, 4112 heads of 256, 448 positions, 16 rows 389 / 607).  us, one / four: 288 heads of 128, 1 row, 900 positions 38.1 / 33.2, 1500 59.8 /
    // 47.0; of 256, 3000 226 / 174; 528 of 128, 1500 91.6 / 81.1; 264 of 256, 16 rows, 1500 120.0 / 109.1, and before the line 900 78.4 / 78.0.
    // From half a round on level or slower (384 of 64 3000 60.5 / 56.9, 448 of 128 1500 66.2 / 68.9), and so are short walks (288 of 256 400 37.8 / 41.8).
    const int last = G % num_cus;
    if (G > num_cus && last > 0 && 20 * last <= 7 * num_cus && steps >= 14 && 20L * n_ctx * (num_cus - last) >= (36L + 3L * M) * G * num_cus) s = 4;
    if (s > 24 && s > steps / 2) s = steps / 2 > 24 ? steps / 2 : 24;
    if (s > steps) s = steps;
    if (s > kAttnMaxSplits) s = kAttnMaxSplits;
    return s < 1 ? 1 : s;
}

// More than 16 query rows (prompts): blocks of 16 rows in the decode kernel, or the kernel for blocks of 64 and 128.  That one
// reads each position once per block, but takes 4 to 7 us before its first and behind its last step.
// Here the positions are read once per 16 rows and the walks are split over wavefronts and
// workgroups, which wins as long as there is little to walk (blocks x 64 positions) and the compute units hold the
// blocks at once; long walks have to be split over more workgroups, whose results are combined.  Measured (us, blocks of 64 or 128 / of 16):
// head size 64, 8 groups of 2 heads, 400 tokens 9.1 / 7.5, 4 of 8, 301 tokens behind 572 12.0 / 9.8, 8 of 1, 155 behind 1802 11.8 / 13.7;
// head size 128, 1 group of 8, 17 tokens 6.4 / 4.9 (of 1 head, two blocks of one step 4.5 / 4.8), 2 of 4, 77 behind 500 12.7 / 10.3, 1 of 1, 20
// behind 4234 22.6 / 23.9; head size 256, 1 group, 400 tokens 17.6 / 11.4, 4 of 2, 77 behind 500 18.6 / 13.3, 300 16.3 / 14.1, 2 of 4, 135 behind
// 732 18.2 / 24.1.  Over 816 shapes of 17 to 512 tokens behind 0 to 5000 positions, 1 to 32 groups, the choice is 0.2 % slower than the faster of both.
static bool few_row_blocks(int G, int M, int d, int n_ctx, int num_cus) {
    const long blocks = (long)G * ((M + 15) / 16), steps = (n_ctx + 63) / 64;
    if ((n_ctx <= 32 && M <= 32) || blocks > (d <= 64 ? 2 : 1) * num_cus) return false;
    if (d <= 64) return blocks * steps <= (steps <= 24 ? 3000 : 2000);
    return blocks * steps <= (steps <= 8 ? 2500 : d > 128 ? 800 : steps <= 32 ? 1000 : 0);
}

// Workgroups per block of 16 query rows and KV head: the estimated time (us) of the walk and the combination.
static int row_block_splits(int G, int M, int d, int n_ctx, int num_cus) {
    const int step = d <= 128 ? 64 : 32, steps = (n_ctx + step - 1) / step, blocks = (M + 15) / 16;
    const float step_us = d <= 64 ? 2.0f : 3.7f, slots = (float)num_cus * (d <= 128 ? 2.0f : 1.0f);
    int best = 1;
    float best_us = 0.0f;
    for (int s = 1; s <= kPrefillMaxChunks; ++s) {
        const float load = (float)G * (float)blocks * (float)s / slots;
        float us = (load > 1.0f ? load : 1.0f) * (float)((steps + 4 * s - 1) / (4 * s)) * step_us;
        if (s > 1) us += 2.2f + (float)G * (float)M * (float)s * (float)d * 8.0f / 0.7e6f;
        if (s == 1 || us < best_us) best = s, best_us = us;
    }
    return best;
}

// The many-query-rows path needs partial results only where it may cut walks into chunks: launches
// with no more blocks of 128 query rows than compute units.
static bool prefill_may_chunk(int G, int M, int num_cus) {
    const long wgs = (long)((M + 127) / 128) * G;
    const int forced = tuning().attn_chunks;
    return forced >= 0 ? forced != 0 : wgs <= num_cus;
}

// Prefill: wavefronts that share a walk (returned) and chunks of the walks (a.chunk_steps, a.block_rows), the combination with
// the shortest estimated time (us).  Stages a workgroup takes one after the other: `longest` for the last one to finish,
// `total` per compute unit.  Per stage: alone on its compute unit / as one of two (times two: head size 256 has the unit for itself); fixed: before the first and
// behind the last stage.  Chunks cost a second launch and the partial results, written and read.  Over 290
// shapes (17 to 6000 tokens behind 0 to 6000 positions, 1 to 64 groups of 1 to 8 heads of 64, 128 and 256) the choice is 0.9 % slower than the
// best combination where this kernel runs (head size 64 1.2, 128 1.0, 256 0.3), 6 shapes more than 6 %, the worst 16.
static int plan_prefill(AttnArgs &a, int d, int num_cus) {
    const int forced_shares = tuning().attn_shares, forced_chunks = tuning().attn_chunks;
    const bool may_chunk = prefill_may_chunk(a.groups, a.M, num_cus);
    const float alone[2] = {d <= 64 ? 0.43f : d <= 128 ? 0.58f : 1.13f, d <= 64 ? 0.45f : d <= 128 ? 0.65f : 1.55f};
    const float busy[2] = {d <= 64 ? 0.50f : d <= 128 ? 0.79f : 1.13f, d <= 64 ? 0.52f : d <= 128 ? 0.95f : 1.55f};
    const float shared[2] = {d <= 64 ? 0.40f : d <= 128 ? 0.57f : 1.13f, d <= 64 ? 0.44f : d <= 128 ? 0.63f : 1.85f};
    const float fixed[2] = {d <= 128 ? 4.0f : 6.0f, d <= 128 ? 4.5f : 6.0f};
    const long slots = (long)num_cus * (d <= 128 ? 2 : 1);
    const int exactly = forced_chunks > kPrefillMaxChunks ? kPrefillMaxChunks : forced_chunks;  // (from 2 on)
    const float second = fminf(7.0f, 2.5f + (float)((long)a.groups * a.M) / 520.0f);  // the second launch
    int best = 0;
    float best_us = 0.0f;
    for (int ps = 1; ps <= 2; ++ps) {
        if (forced_shares > 0 && ps != forced_shares) continue;
        const int rows = 128 / ps, nblocks = (a.M + rows - 1) / rows, longest = prefill_steps(a, nblocks - 1, rows);
        if (best == 0) best = ps, best_us = 1e30f, a.block_rows = rows, a.chunk_steps = 0;
        int last_len = 0;
        for (const int k : {1, 2, 3, 4, 6, 8}) {
            if (exactly > 1 ? k != exactly : exactly == 1 ? k == 1 : k > 1 && (!may_chunk || best_us < fixed[ps - 1] + second + 4.0f * alone[ps - 1])) continue;
            const int len = ((longest + k - 1) / k + ps - 1) / ps * ps;
            if (len == last_len || (k > 1 && (len < 4 || len >= longest))) continue;
            last_len = len;
            long items = 0, total = 0;
            double partial_bytes = 0.0;
            for (int j = 0; j < nblocks; ++j) {
                const int steps = prefill_steps(a, j, rows), c = (steps + len - 1) / len;
                items += c;
                total += (steps + ps - 1) / ps;
                if (c > 1) partial_bytes += (double)rows * c * d * 8.0 * a.groups;
            }
            if (k > 1 && items * a.groups > slots && forced_chunks <= 0) break;  // (a second round of chunks)
            const float per_cu = (float)items * (float)a.groups / (float)num_cus, stages = (float)(len / ps);
            float us = fixed[ps - 1];
            if (k > 1)
                us += (per_cu > 1.0f ? 2.0f * shared[ps - 1] : alone[ps - 1]) * stages + second + (float)(partial_bytes / 7.0e6);
            else
                us += fmaxf((per_cu > 1.0f ? busy : alone)[ps - 1] * stages, shared[ps - 1] * (float)total * (float)a.groups / (float)num_cus);
            if (us < best_us) best = ps, best_us = us, a.block_rows = rows, a.chunk_steps = k > 1 ? len : 0;
        }
    }
    return best;
}

size_t attn_prefill_workspace(int G, int M, int d, int num_cus) {
    if (!prefill_may_chunk(G, M, num_cus)) return 256;
    return (size_t)G * M * kPrefillMaxChunks * (d + 2) * sizeof(float);
}

// Tokens per workgroup of rope_qkv_kernel: at most as many as one evaluation of an angle per thread covers; fewer, so that there are about four
// workgroups per compute unit (1024 tokens x 48 x 128, 1 / 2 / 4 tokens: 9.2 / 10.3 / 12.7 us), unless their heads leave a quarter of the threads idle and more
// and there are two per compute unit all the same (1216 x 3 x 128, 1 / 2 tokens: 5.7 / 5.1 us; 4793 x 2 x 64, 4 / 8: 7.1 / 6.8; for the last quarter it does not pay, 816 x
// 12 x 128, 1 / 3: 5.9 / 7.0, nor with one per compute unit, 1939 x 10 x 64, 3 / 7: 6.1 / 7.2).  Over 2298 shapes 1.5 % behind the best number.
int rope_tokens(long total, int heads, int d) {
    const int items = heads * (d / 16);  // (a thread rotates 16 values of a token at a time)
    const long most = 512 / d, busy = (192 + items - 1) / items;
    long T = busy < total / 512 ? busy : total / 512;
    if (T < total / 1024) T = total / 1024;
    return T < 1 ? 1 : T > most ? (int)most : (int)T;
}

hipError_t launch_rope_qkv(const void *qkv, int B, int S, int h_q, int h_kv, int d, int C, int pos0, float base,
                           void *q_out, void *kc, void *vc, hipStream_t st) {
    const long total = (long)B * S;
    // Few tokens, and more of them where their heads are few: a workgroup that shares the angles of a token has little else
    // to do (us, this kernel / the other, tokens x heads x values: 77 x 16 x 256 3.9 / 4.25, 2000 x 3 x 64 4.4 / 5.7; 300 x 48 x 128 11.4 / 6.5; drawn
    // with the rotation in fp64: 328 x 6 x 128 4.5 / 5.0, 200 x 16 x 128 5.1 / 4.9, 200 x 48 x 64 5.7 / 5.0)
    if (total < 128 || total * (h_q + 2 * h_kv) * d < (400L << 10)) {
        const long pairs = total * (h_q + 2 * h_kv) * (d / 2);
        rope_qkv_few_kernel<<<(unsigned)((pairs + 255) / 256), 256, 0, st>>>(
            static_cast<const _Float16 *>(qkv), B, S, h_q, h_kv, d, C, pos0, log((double)base),
            static_cast<_Float16 *>(q_out), static_cast<_Float16 *>(kc), static_cast<_Float16 *>(vc));
        return hipGetLastError();
    }
    RopeArgs a;
    a.qkv = static_cast<const _Float16 *>(qkv);
    a.q_out = static_cast<_Float16 *>(q_out);
    a.kc = static_cast<_Float16 *>(kc);
    a.vc = static_cast<_Float16 *>(vc);
    a.B = B, a.S = S, a.h_q = h_q, a.h_kv = h_kv, a.d = d, a.C = C, a.pos0 = pos0;
    a.log_base = log((double)base);
    a.T = rope_tokens(total, h_q + h_kv, d);
    a.rot_wgs = (int)((total + a.T - 1) / a.T);
    a.pblocks = (pos0 + S - 1) / 64 - pos0 / 64 + 1;
    const size_t angles = (size_t)a.T * (d / 2) * sizeof(float4), tile = (size_t)64 * 66 * 2;
    rope_qkv_kernel<<<(unsigned)(a.rot_wgs + B * h_kv * a.pblocks * (d / 64)), 256, angles > tile ? angles : tile, st>>>(a);
    return hipGetLastError();
}

hipError_t launch_rope_table(int d, float base, int positions, float *table, hipStream_t st) {
    const long total = (long)positions * (d / 2);
    rope_table_kernel<<<(unsigned)((total + 255) / 256), 256, 0, st>>>(d, positions, log((double)base), table);
    return hipGetLastError();
}

hipError_t launch_attention(const void *q, const void *kc, const void *vc, int G, int S, int g, int d, int C,
                            int n_ctx, void *workspace, void *out, int num_cus, hipStream_t st) {
    AttnArgs a;
    a.q = static_cast<const _Float16 *>(q);
    a.kc = static_cast<const _Float16 *>(kc);
    a.vc = static_cast<const _Float16 *>(vc);
    a.M = S * g;
    a.g = g;
    a.S = S;
    a.C = C;
    a.n_ctx = n_ctx;
    a.splits = tuning().attn_splits > 0 ? (int)tuning().attn_splits : attn_splits(G, a.M, d, n_ctx, num_cus);
    if (num_cus < 1) num_cus = 1;
    a.groups = G;
    a.max_chunks = kPrefillMaxChunks;
    const int shares = a.M > 16 ? plan_prefill(a, d, num_cus) : 1;
    a.scale = 1.4426950408889634f / sqrtf((float)d);  // scores in units of log 2
    a.ws_o = static_cast<float *>(workspace);
    a.ws_ml = a.ws_o + (size_t)G * (a.M > 16 ? kPrefillMaxChunks : kAttnMaxSplits) * a.M * d;
    a.out = static_cast<_Float16 *>(out);
    bool few = a.M <= 16;
    if (!few) {
        const int forced = tuning().attn_few;
        few = forced >= 0 ? forced != 0 : few_row_blocks(G, a.M, d, n_ctx, num_cus);
        if (few) {  // partial results fit the workspace of the chunks
            const int most = prefill_may_chunk(G, a.M, num_cus) ? kPrefillMaxChunks : 1;
            if (tuning().attn_splits == 0) a.splits = row_block_splits(G, a.M, d, n_ctx, num_cus);
            if (a.splits > most) a.splits = most;
        }
    }
    if (!few) {
        switch (d) {
            case 64: return shares == 1 ? launch_attn_prefill<64, 1>(a, st) : launch_attn_prefill<64, 2>(a, st);
            case 128: return shares == 1 ? launch_attn_prefill<128, 1>(a, st) : launch_attn_prefill<128, 2>(a, st);
            case 256: return shares == 1 ? launch_attn_prefill<256, 1>(a, st) : launch_attn_prefill<256, 2>(a, st);
            default: return hipErrorInvalidValue;
        }
    }
    switch (d) {
        case 64: return launch_attn<64>(a, G, st);
        case 128: return launch_attn<128>(a, G, st);
        case 256: return launch_attn<256>(a, G, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace qfc
