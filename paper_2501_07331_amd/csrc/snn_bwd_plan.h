// When the waves of the split backward core have to meet, as functions of sizes
// alone: used by the kernel, and by a check of every case on the CPU.
//
// An adjoint ring of S >= 2 rows holds lambda_I - lambda_V of the post layer's
// nq neurons, step m in row m % S.
#pragma once

// Whether a wave that runs this many steps from the step after (in reverse time)
// one with spikes, without a barrier, writes that step's row again, which
// another wave may still be reading: run_max is S - 1 of the shortest ring.
constexpr bool ring_lapped(int steps, int run_max) { return steps > run_max; }
