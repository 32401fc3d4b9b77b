// How many operations of a wavefront of gemm_i8_dw_kernel may be outstanding where it goes on to read (also compiled for the host, by a test).
#pragma once

namespace qfc {

// Loads into registers, copies into LDS and early touches of the weights share one counter (vmcnt) and are taken to complete in order only within
// their own kind.  (Measured for loads and copies: with waits that assumed one common order, stages were read before their copies had
// landed.  Touches are copies of another width that mostly come from HBM, and nothing shows that they stay behind copies that L2 has.)
// Where at most `allowed` operations are outstanding, what a stage needs is not among them: an unfinished copy would have all later copies
// behind it, an unfinished load all later loads.  Touches count on neither side.
struct DwWaits {
    int first;    // before the first stage's copies are read (PIPE)
    int allowed;  // at the top of a stage: its loads, and its copies (PIPE: the next stage's), have landed
};
// copies, loads: of a stage, per wavefront; NS: stages of the copies' ring, NS - 1 of them issued ahead; PW: stages of loads, all issued ahead
constexpr DwWaits dw_waits(int copies, int loads, int NS, int PW, bool pipe) {
    const int after_copies = copies * (NS - (pipe ? 3 : 2)), after_loads = loads * (PW - 1);
    return {copies * (NS - 2), after_copies < after_loads ? after_copies : after_loads};
}

}  // namespace qfc
