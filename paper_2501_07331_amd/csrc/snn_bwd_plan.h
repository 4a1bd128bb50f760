// Which ring cells the split backward core reads and when its waves have to
// meet, as functions of sizes alone: used by the kernels that build its tables
// and run it, and by a check of every case on the CPU.
//
// An adjoint ring of S >= 2 rows holds lambda_I - lambda_V of the post layer's
// nq neurons, step m in row m % S.
#pragma once

// Entry of a far table for a synapse of the given slot: 0 for slot 0 (the
// spiking neuron's own lane takes those terms), else a mark in the top bit and
// the cells from the row of the step after the spike's to the arrival's.  Posts
// past the layer load 0 likewise.
constexpr unsigned far_entry(unsigned slot, unsigned nq) {
    return slot == 0 ? 0u : 0x80000000u | (slot - 1) * nq;
}
constexpr bool far_arrives(unsigned entry) { return (int)entry < 0; }

// Byte offset in the ring of the cell that an entry's term reads: next is the
// byte offset of the row of the spike's step plus one row, bytes the ring's.
// The mark is shifted out; entries 0 read the row of the step after the spike's,
// which, unlike that of the step itself, no wave writes meanwhile.  (The sum is
// below two rings: at most S rows in next and S - 2 in the entry.)
constexpr unsigned far_cell(unsigned next, unsigned col, unsigned entry, unsigned bytes) {
    const unsigned x = next + col * 8u + entry * 8u;
    return x < bytes ? x : x - bytes;
}

// Whether a wave that runs this many steps from the step after (in reverse time)
// one with spikes, without a barrier, writes that step's row again, which
// another wave may still be reading: run_max is S - 1 of the shortest ring.
constexpr bool ring_lapped(int steps, int run_max) { return steps > run_max; }
