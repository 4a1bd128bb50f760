// The split backward core's plan (csrc/snn_bwd_core.hip) over every small case,
// on the CPU, by the rules that the kernel uses (csrc/snn_bwd_plan.h): what its
// waves read and write in the adjoint ring between two barriers, and which cells
// the terms of slots >= 1 read.
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

// Every entry of a far table: the cell of its arrival, or, where nothing arrives
// (slot 0, posts past the layer), one of the row after the spike's step.
int wrong_cells(int S, int nq, int slots) {
    const unsigned bytes = (unsigned)(S * nq * 8);
    int bad = 0;
    for (int n = 0; n < 2 * S; ++n)
        for (int slot = -1; slot < slots; ++slot)            // -1: past the layer, loaded as 0
            for (int j = 0; j < nq; ++j) {
                const unsigned e = slot < 0 ? 0u : far_entry((unsigned)slot, (unsigned)nq);
                const unsigned at = far_cell((unsigned)((n % S + 1) * nq * 8), (unsigned)j, e, bytes);
                const bool arrives = slot > 0;
                const unsigned want = (unsigned)(((n + (arrives ? slot : 1)) % S * nq + j) * 8);
                bad += far_arrives(e) != arrives || at != want || at >= bytes;
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
    // (slots of a projection: up to the rows of its post layer's ring)
    int cells = 0;
    for (int S = 2; S <= 9; ++S)
        for (int nq : {1, 3, 64, 70})
            for (int slots = 1; slots <= S; ++slots) cells += wrong_cells(S, nq, slots);
    cells += wrong_cells(256, 79, 256);
    printf("%d wrong cells\n", cells);
    printf("%lld cases, %lld with a race\n", cases, bad);
    return bad || cells ? 1 : 0;
}
