// Measurement probe, not part of the product path: a register-only loop of back-to-back MFMAs with
// no memory traffic at all, to find out what rate and what shader clock the matrix cores hold with
// constant and with random operands.  The prefill kernels' fractions of the published peak are
// read against these figures.
#include <type_traits>

#include "qfc_internal.h"
#include "../../include/qfc_experimental.h"

namespace qfc {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint32_t mix(uint32_t x) {
    x ^= x >> 16; x *= 0x7feb352du; x ^= x >> 15; x *= 0x846ca68bu; x ^= x >> 16;
    return x;
}

// About normal, variance one: the sum of four uniform values
__device__ __forceinline__ float bell(uint32_t id) {
    const uint32_t u = mix(id), v = mix(id ^ 0x9e3779b9u);
    const float s = (float)(u & 65535u) + (float)(u >> 16) + (float)(v & 65535u) + (float)(v >> 16);
    return (s * (1.0f / 65536.0f) - 2.0f) * 1.7320508f;
}

// Values as the products meet them: codes of normal values (int8; int4 the integers -8 .. 7), normal activations
__device__ __forceinline__ float code(uint32_t id, bool int4) { return fminf(fmaxf(rintf(bell(id) * (int4 ? 2.5f : 28.0f)), int4 ? -8.0f : -127.0f), int4 ? 7.0f : 127.0f); }

enum Operands { kConstant = 0, kRandomBits = 1, kNormal = 2, kInt4 = 3 };  // kInt4: the first operand's codes

__device__ __forceinline__ v4i int8_operand(uint32_t id, int operands, bool first) {
    v4i r;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        uint32_t w = operands == kConstant ? 0x01010101u : mix(id + e);
        if (operands >= kNormal) {
            const bool int4 = operands == kInt4 && first;  // (as the kernels multiply them: 16 times the code)
            w = 0;
            for (int b = 0; b < 4; ++b) w |= ((uint32_t)(int)(code((id + e) * 4 + b, int4) * (int4 ? 16.0f : 1.0f)) & 255u) << (8 * b);
        }
        r[e] = (int)w;
    }
    return r;
}
__device__ __forceinline__ v8h half_operand(uint32_t id, int operands, bool first) {
    v8h r;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const _Float16 bits = (_Float16)((int)(mix(id + e) & 2047) - 1024) * (_Float16)(1.0f / 1024);  // finite, in [-1, 1)
        r[e] = operands == kConstant ? (_Float16)1.0f : operands == kRandomBits ? bits : operands == kInt4 && first ? (_Float16)code(id + e, true) : (_Float16)bell(id + e);
    }
    return r;
}

// KIND 0: v_mfma_i32_32x32x32_i8, 1: v_mfma_f32_32x32x16_f16, eight accumulators, eight operand pairs used in rotation (with random operands
// consecutive MFMAs see unrelated bits; with constant ones every operand register holds the same value).  4: v_mfma_i32_16x16x64_i8,
// 5: v_mfma_f32_16x16x32_f16, the 4 x 8 tiles of a wavefront of the product kernels in their order, 4 and 8 operands.  32 MFMAs per iteration.
// ticks[2 b] = shader clock ticks, ticks[2 b + 1] = ticks of the constant 100 MHz counter, both over the loop of workgroup b's first wavefront.
template <int KIND>
__global__ __launch_bounds__(256, 2) void probe_mfma_kernel(int iters, int operands, uint64_t *ticks) {
    constexpr bool kHalf = KIND & 1, kSmall = KIND & 4;
    constexpr int NA = kSmall ? 4 : 8, NACC = kSmall ? 32 : 8, E = kSmall ? 4 : 16;
    typedef std::conditional_t<kHalf, v8h, v4i> In;
    typedef std::conditional_t<kSmall, std::conditional_t<kHalf, v4f, v4i>, std::conditional_t<kHalf, v16f, v16i>> Acc;
    Acc acc[NACC];
    In a[NA], b[8];
    const uint32_t id = blockIdx.x * 256 + threadIdx.x;
#pragma unroll
    for (int i = 0; i < NACC; ++i)
#pragma unroll
        for (int e = 0; e < E; ++e) acc[i][e] = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if constexpr (kHalf) {
            if (i < NA) a[i] = half_operand(id * 128 + i * 16, operands, true);
            b[i] = half_operand(id * 128 + i * 16 + 8, operands, false);
        } else {
            if (i < NA) a[i] = int8_operand(id * 64 + i * 8, operands, true);
            b[i] = int8_operand(id * 64 + i * 8 + 4, operands, false);
        }
    }
    const uint64_t c0 = clock64(), w0 = wall_clock64();
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int r = 0; r < 32; ++r) {
            if constexpr (KIND == 0)
                acc[r & 7] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[(r + (r >> 3)) & 7], b[r & 7], acc[r & 7], 0, 0, 0);
            else if constexpr (KIND == 1)
                acc[r & 7] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[(r + (r >> 3)) & 7], b[r & 7], acc[r & 7], 0, 0, 0);
            else if constexpr (KIND == 4)
                acc[r] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[r & 3], b[r >> 2], acc[r], 0, 0, 0);
            else
                acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[r & 3], b[r >> 2], acc[r], 0, 0, 0);
        }
        if (kHalf && (it & 63) == 63) {  // keep the fp32 sums finite
#pragma unroll
            for (int i = 0; i < NACC; ++i)
#pragma unroll
                for (int e = 0; e < E; ++e) acc[i][e] *= 0.5f;
        }
    }
    const uint64_t c1 = clock64(), w1 = wall_clock64();
    int s = 0;
    float fs = 0.0f;
#pragma unroll
    for (int i = 0; i < NACC; ++i)
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if constexpr (kHalf)
                fs += acc[i][e];
            else
                s += acc[i][e];
        }
    s += __float_as_int(fs);
    if (threadIdx.x == 0) {
        ticks[2 * blockIdx.x] = c1 - c0 + (s == 0x7fffffff ? 1 : 0);  // (the sums are used, so the loop stays)
        ticks[2 * blockIdx.x + 1] = w1 - w0;
    }
}

}  // namespace
}  // namespace qfc

extern "C" qfc_status_t qfc_probe_mfma(int32_t kind, int32_t random_operands, int32_t iters, int32_t workgroups,
                                       uint64_t *ticks, void *stream) {
    if ((kind != 0 && kind != 1 && kind != 4 && kind != 5) || iters < 1 || iters > (1 << 22) || workgroups < 1 || workgroups > 4096 || !ticks)
        return QFC_ERR_INVALID_ARG;
    if (reinterpret_cast<uintptr_t>(ticks) & 7u) return QFC_ERR_ALIGNMENT;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int operands = random_operands == qfc::kConstant || random_operands == qfc::kNormal || random_operands == qfc::kInt4 ? random_operands : (int)qfc::kRandomBits;
    const dim3 grid((unsigned)workgroups);
    switch (kind) {
        case 0: qfc::probe_mfma_kernel<0><<<grid, 256, 0, st>>>(iters, operands, ticks); break;
        case 1: qfc::probe_mfma_kernel<1><<<grid, 256, 0, st>>>(iters, operands, ticks); break;
        case 4: qfc::probe_mfma_kernel<4><<<grid, 256, 0, st>>>(iters, operands, ticks); break;
        default: qfc::probe_mfma_kernel<5><<<grid, 256, 0, st>>>(iters, operands, ticks); break;
    }
    return hipGetLastError() == hipSuccess ? QFC_OK : QFC_ERR_HIP;
}
