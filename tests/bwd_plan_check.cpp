// The split backward core's schedule (csrc/snn_bwd_core.hip) over every small
// case, on the CPU: what its waves read and write in the adjoint ring between
// two barriers, by the rules that the kernel uses (csrc/snn_bwd_plan.h).
// Argument "no-tail": without the meeting before the steps past the last spikes
// (a planted mistake that has to be found).
#include <cstdio>
#include <cstring>
#include <vector>

#include "snn_bwd_plan.h"

namespace {

// Between two barriers (an epoch), every wave's accesses come in any order.
struct Access {
    int epoch, step;     // the step whose row is read or written
    bool write, helper;
};

// The steps of `act` (last first) have spikes.  A neuron wave's epochs: the
// helpers count theirs by the same barriers.
std::vector<Access> run(int T, int S, const std::vector<int>& act, bool tail) {
    std::vector<Access> log;
    const int run_max = S - 1;
    int epoch = 0, last = T;
    for (int n : act) {
        const int gap = last - n;
        if (ring_lapped(gap - 1, run_max)) ++epoch;
        for (int m = last - 1; m > n; --m) log.push_back({epoch, m, true, false});
        if (gap > 1) ++epoch;
        // the helpers' sums of slots 1 .. S - 1, beside the step itself
        for (int m = n + 1; m < n + S && m < T; ++m) log.push_back({epoch, m, false, true});
        log.push_back({epoch, n, true, false});
        ++epoch;
        log.push_back({epoch, n, false, false});             // the jumps' terms of slot 0
        last = n;
    }
    if (tail && !act.empty() && ring_lapped(last, run_max)) ++epoch;
    for (int m = last - 1; m >= 0; --m) log.push_back({epoch, m, true, false});
    return log;
}

// Reads that another wave's write of the same epoch may overtake, or that find
// another step's row.
int faults(int T, int S, const std::vector<int>& act, bool tail) {
    const std::vector<Access> log = run(T, S, act, tail);
    int bad = 0;
    for (const Access& r : log) {
        if (r.write) continue;
        int held = -1;                                       // the row's step before the epoch
        for (const Access& w : log) {
            if (!w.write || w.step % S != r.step % S) continue;
            if (w.epoch < r.epoch) held = w.step;
            if (w.epoch == r.epoch) ++bad;
        }
        bad += held != r.step;
    }
    return bad;
}

}  // namespace

int main(int argc, char** argv) {
    const bool tail = !(argc > 1 && !strcmp(argv[1], "no-tail"));
    long long cases = 0, bad = 0;
    // all sets of active steps of trials of up to 11 steps, and sparse ones of longer
    for (int S = 2; S <= 9; ++S) {
        for (int T = 1; T <= 11; ++T)
            for (unsigned set = 0; set < 1u << T; ++set) {
                std::vector<int> act;
                for (int n = T - 1; n >= 0; --n)
                    if (set >> n & 1) act.push_back(n);
                ++cases;
                bad += faults(T, S, act, tail) != 0;
            }
        for (int T = 12; T <= 40; ++T)
            for (int n1 = 0; n1 < T; ++n1)
                for (int n0 = 0; n0 <= n1; ++n0) {
                    ++cases;
                    bad += faults(T, S, n0 < n1 ? std::vector<int>{n1, n0} : std::vector<int>{n1}, tail) != 0;
                }
    }
    printf("%lld cases, %lld with a race\n", cases, bad);
    return bad ? 1 : 0;
}
