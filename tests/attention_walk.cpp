// Runs the order of a prefill walk (csrc/attention_walk.h) for the four wavefronts of a workgroup with operations that take
// notes, and checks the notes against a model of LDS: copies land at the latest where a wait says so and are seen by
// the others behind the barrier of that wait; until then their destination holds nothing that may be read.
// Usage: attention_walk (prints one line per fault; 0 = none).
#include <algorithm>
#include <cstdio>
#include <deque>
#include <vector>

#include "attention_walk.h"

namespace {

int faults = 0;

struct Copy { char kind; int step, place, issued, landed; };  // place: slot * PS + p; epochs (barriers passed) of both
struct Read { char kind; int step, place, epoch; };

struct Notes {
    std::vector<Copy> copies;
    std::vector<Read> reads;
    std::vector<int> scored, added;
    int epochs = 0, most_of_a_line = 0;
    size_t outstanding = 0;
};

template <int NB, int PS, int COPIES>
Notes run(int steps, int unmasked, int ps) {
    Notes n;
    const int T = (steps + PS - 1) / PS;
    std::deque<size_t> flying;  // (one entry per step copied: COPIES instructions)
    auto copy = [&](char kind, int t, int p, int slot) {
        const int step = t * PS + p, same = 1 + (int)std::count_if(flying.begin(), flying.end(), [&](size_t i) {
            return n.copies[i].kind == kind && n.copies[i].step == step; });
        n.most_of_a_line = std::max(n.most_of_a_line, same);
        if (t >= T || step >= steps) printf("steps %d: a copy of step %d\n", steps, step), ++faults;
        if (slot < 0 || slot >= NB || p < 0 || p >= PS) printf("steps %d: a copy into slot %d.%d\n", steps, slot, p), ++faults;
        flying.push_back(n.copies.size());
        n.copies.push_back({kind, step, slot * PS + p, n.epochs, -1});
    };
    auto read = [&](char kind, int t, int slot) {
        const int step = t * PS + ps;
        if (step < steps) n.reads.push_back({kind, step, slot * PS + ps, n.epochs});
    };
    int requested = 0;  // stage whose K operands were requested last
    n.scored.assign(steps, 0), n.added.assign(steps, 0);
    auto count = [&](std::vector<int> &of, int t) { if (t * PS + ps < steps) ++of[t * PS + ps]; };
    qfc::prefill_walk<NB, PS, COPIES>(
        steps, unmasked, [&](int t, int p, int slot) { copy('K', t, p, slot); },
        [&](int t, int p, int slot) { copy('V', t, p, slot); },
        [&](auto left) {
            while (flying.size() * COPIES > (size_t)decltype(left)::value) n.copies[flying.front()].landed = n.epochs, flying.pop_front();
            ++n.epochs;
        },
        [&]() { read('K', 0, 0), count(n.scored, 0); },
        [&](int slot) { read('K', ++requested, slot); },
        [&](int t, int slot, int next_slot, auto bulk, bool next) {
            if (decltype(bulk)::value && (!next || t + 1 > unmasked)) printf("steps %d: stage %d as bulk\n", steps, t), ++faults;
            if (next) {
                if (requested != t + 1) printf("steps %d: stage %d scored, operands of %d\n", steps, t + 1, requested), ++faults;
                read('K', t + 1, next_slot), count(n.scored, t + 1);
            }
            read('V', t, slot);
        },
        [&](int t, auto, bool) { count(n.added, t); });
    n.outstanding = flying.size();
    return n;
}

template <int NB, int PS, int COPIES>
void check(int steps, const std::vector<int> &unmasked) {
    std::vector<Notes> w;
    for (int i = 0; i < 4; ++i) w.push_back(run<NB, PS, COPIES>(steps, unmasked[i], i / (4 / PS)));
    auto fault = [&](const char *what, int wave) { printf("NB %d PS %d steps %d wavefront %d: %s\n", NB, PS, steps, wave, what), ++faults; };
    for (int i = 0; i < 4; ++i) {
        const int ps = i / (4 / PS);
        if (w[i].epochs != w[0].epochs) fault("another number of barriers", i);
        if (w[i].outstanding) fault("copies in flight behind the walk", i);
        if (w[i].most_of_a_line > 1 || w[i].copies.size() != 2 * (size_t)steps) fault("a step not copied exactly once", i);
        for (int s = 0; s < steps; ++s)
            if (w[i].scored[s] != (s % PS == ps) || w[i].added[s] != (s % PS == ps)) fault("a step not taken exactly once", i);
        for (const Read &r : w[i].reads)
            for (int o = 0; o < 4; ++o) {  // every wavefront copies a share of every step
                const Copy *last = nullptr;
                for (const Copy &c : w[o].copies) {
                    if (c.kind != r.kind || c.place != r.place) continue;
                    // a copy issued in the epoch of the read may land before it
                    if (c.issued <= r.epoch) last = &c;
                }
                if (!last || last->step != r.step) fault("a read of another step's place", i);
                else if (last->landed < 0 || last->landed >= r.epoch) fault("a read before the data has landed", i);
            }
    }
}

template <int NB, int PS, int COPIES>
void check_all() {
    for (int steps = 1; steps <= 12 * PS + 1; ++steps) {
        const int T = (steps + PS - 1) / PS;
        for (int u = 0; u <= T; ++u) check<NB, PS, COPIES>(steps, {u, u, u, u}), check<NB, PS, COPIES>(steps, {0, u / 2, u, std::max(0, u - 1)});
    }
}

}  // namespace

int main() {
    check_all<3, 1, 1>(), check_all<3, 2, 1>();  // head size 64
    check_all<3, 1, 2>(), check_all<2, 2, 2>();  // 128
    check_all<3, 1, 4>(), check_all<2, 2, 4>();  // 256
    printf("%d faults\n", faults);
    return faults != 0;
}
