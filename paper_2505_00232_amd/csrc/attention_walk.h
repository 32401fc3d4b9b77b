// Order of a prefill walk (attention.hip, attn_prefill_kernel): which copies into LDS are issued when, what is waited
// for and which stage is read from which slot.  It is the kernel's control flow, apart from the kernel so that a host program can run
// it too, with operations that only record what they are asked for (tests/attention_walk.cpp).
#pragma once
#include <type_traits>

namespace qfc {

// A walk of `steps` steps is taken in T stages of PS steps (the last stage may lack one), with rings of NB stages for K and
// for V.  Batch b = K of stage b + 1 and V of stage b; per wavefront a step is COPIES copies of K and as many of V.
// `unmasked`: leading stages whose successor no row of this wavefront masks.  The operations:
//   copy_k(t, p, slot), copy_v(..)       request step p of stage t into its place of slot `slot`
//   wait(n)              this wavefront's copies up to the n newest have landed, its reads of LDS are done; then the barrier
//   first()              scores of stage 0, K from slot 0
//   request_k(slot)      K operands of the stage in `slot`, for the next head
//   head(t, slot, next_slot, bulk, next)  scores of stage t + 1 if there is one (`next`), V operands of stage t, exponentials
//   tail(t, bulk, next)  second product of stage t, maximum of stage t + 1
// Nothing is copied but the walk's steps, each once: nothing can land behind the walk in LDS that is in use again, and no line
// is on its way twice.  What a place holds whose step the last stage lacks is not known: the operations discard its
// scores and leave out its second product (a zero probability times an infinite value is no zero).  (Direct-to-LDS copies of the same lines, ten and more in flight from one wavefront,
// have been seen in LDS after the counter said they were done.)  Counts of outstanding copies are relied on only where every batch
// they cover is whole; elsewhere the counter is waited empty.
template <int NB, int PS, int COPIES, class CopyK, class CopyV, class Wait, class First, class RequestK, class Head, class Tail>
__host__ __device__ __forceinline__ void prefill_walk(int steps, int unmasked, const CopyK &copy_k, const CopyV &copy_v, const Wait &wait,
                                                      const First &first, const RequestK &request_k, const Head &head, const Tail &tail) {
    constexpr int CB = 2 * PS * COPIES;  // copies of a batch
    constexpr std::true_type kBulk;
    constexpr std::false_type kEdge;
    const int T = (steps + PS - 1) / PS;
    auto stage = [&](const auto &copy, int t, int slot, auto bulk) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < PS; ++p) {
            if (decltype(bulk)::value || t * PS + p < steps) copy(t, p, slot);
        }
    };
    auto next_slot = [](int slot) __attribute__((always_inline)) { return slot + 1 == NB ? 0 : slot + 1; };

    stage(copy_k, 0, 0, kEdge);
#pragma unroll
    for (int b = 0; b < NB - 1; ++b) {
        stage(copy_k, b + 1, b + 1, kEdge);
        stage(copy_v, b, b, kEdge);
    }
    if (steps >= NB * PS)
        wait(std::integral_constant<int, (NB - 1) * CB>{});
    else
        wait(std::integral_constant<int, 0>{});
    first();
    // batch 0 is there (fewer steps: everything is), and K of stage 0 has been read by all
    wait(std::integral_constant<int, (NB - 2) * CB>{});
    stage(copy_k, NB, 0, kEdge);
    stage(copy_v, NB - 1, NB - 1, kEdge);
    if (1 < T) request_k(1 % NB);

    // bulk: the next stage exists and is not masked, and the batch to issue is whole
    auto step = [&](int t, int slot, auto bulk) __attribute__((always_inline)) {
        constexpr bool BULK = decltype(bulk)::value;
        const int slot1 = next_slot(slot);
        head(t, slot, slot1, bulk, BULK || t + 1 < T);
        // the next batch has landed for everyone, and everyone has read this stage's V and the next one's K
        wait(std::integral_constant<int, BULK ? (NB - 2) * CB : 0>{});
        stage(copy_k, t + NB + 1, slot1, bulk);
        stage(copy_v, t + NB, slot, bulk);
        if (BULK || t + 2 < T) request_k(next_slot(slot1));
        tail(t, bulk, BULK || t + 1 < T);
    };
    const int whole = T - NB - 1 - (steps % PS != 0), bulk_end = unmasked < whole ? unmasked : whole;
    int t = 0;
    for (; t + NB <= bulk_end; t += NB)
#pragma unroll
        for (int s = 0; s < NB; ++s) step(t + s, s, kBulk);
    for (int slot = 0; t < T; ++t) {  // (t is a multiple of NB here)
        step(t, slot, kEdge);
        slot = next_slot(slot);
    }
}

}  // namespace qfc
