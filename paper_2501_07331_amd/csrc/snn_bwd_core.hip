// The LIF adjoint core of libsnn with its adjoint rings in LDS (gfx950,
// wave64): one workgroup per sample runs lambda of the LIF layers in reverse
// time (Table 1, backward dynamics; Methods, the lambda_V jump with delayed
// postsynaptic adjoints).  All fp64.
//
// A step's critical path is lambda of every neuron: free dynamics, the
// trajectory and ring row, the delayed postsynaptic sum of every spike of the
// step, the jumps, then the next step.  With one set of waves doing all of it
// the step took about 3000 cycles, most of them spent on finding the spikes'
// data and on the sums.  So the waves are split:
//
//  neuron waves  (ceil(widest layer / 64)): lane j owns neuron j of every LIF
//                layer: jumps, dynamics, trajectory, ring row; nothing else.
//  helper waves  (H of them): wave h takes the step's spikes h, h + H, ...
//                (layers in order): A = A2 + sum_j w (lambda_V - lambda_I)_j
//                at the arrivals, over the post neurons of its projections,
//                lanes over posts; A and the jump's two factors go to the
//                spiking neuron's slot in LDS.
//
// Spikes and their records are known from the forward, so a helper loads its
// spikes' ids two steps ahead and their weight rows one step ahead.  The sum
// is split at delay 0: terms with slots >= 1 read ring rows that are complete
// a step earlier, so the helpers take them while the neuron waves run the
// step's dynamics.  The few terms with slot 0 are left to the spiking neuron's
// own lane, which holds the first of them (post neuron, weight) in registers
// (split_tables_kernel) and reads the step's own row after the step's barrier.
// Where some neuron has more than kNearCap synapses of slot 0 (delays near
// zero throughout), the helpers take those terms too, between the step's
// barrier and a second one.
//
// Terms that do not arrive are loaded with the others and have weight 0; the
// cell that is loaded in their place (snn_bwd_plan.h: always one of the post
// layer's ring, in a row that no wave writes meanwhile) may hold an infinity or
// a NaN, so the high word of what it holds is cleared: 0 times a finite value.
//
// Both loops run over the steps that have spikes (backward_prep_kernel lists
// them): instructions and above all branches that merely pass over an empty
// step cost as much as its arithmetic.  Between two of them the neuron waves
// run the free dynamics in a loop of its own, without barriers.
//
// Measured, 700-256-20 recurrent, T = 1000: the core 1232 -> 539 us at batch 256
// (a workgroup per CU), 1170 -> 440 us at 32; the recurrent layer of 128, T =
// 300, batch 128: 460 -> 190 us.  Two barriers a step with the slot 0 terms in
// the helpers: 781; a loop over all steps: 796; four helpers instead of twelve:
// 1043; the jump's factors by fp64 division in the helpers: 648; with a jump's
// factor of lambda_V, 24 bytes a record and slot, made beforehand: 577; its two
// terms loaded apart: 582 (first-spike core of two layers 261).  Leaving out
// the trajectory stores changes nothing: it is bound by the chain of LDS round
// trips of a step with spikes, about 1400 cycles.
#include "snn_bwd_plan.h"
#include "snn_device.h"

namespace {

// Barrier over LDS only: this wave's LDS accesses complete, its device-memory
// ones (trajectory stores, prefetched loads) stay in flight.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);       // lgkmcnt(0); vmcnt, expcnt at their maximum
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Sum of x over the 64 lanes, in lane 63 (a fixed order): within rows of 16,
// then row 0 into 1 and 2 into 3, then rows 0-1 into 2-3.
__device__ __forceinline__ double wave_sum_f64(double x) {
    x += dpp_f64<0xB1>(x);                    // quad_perm [1,0,3,2]
    x += dpp_f64<0x4E>(x);                    // quad_perm [2,3,0,1]
    x += dpp_f64<0x141>(x);                   // row_half_mirror
    x += dpp_f64<0x140>(x);                   // row_mirror
    x += dpp_f64<0x142, 0xA>(x);              // row_bcast:15 into rows 1, 3
    x += dpp_f64<0x143, 0xC>(x);              // row_bcast:31 into rows 2, 3
    return x;
}

// What the core needs of a call beside the records, per sample: the steps that
// have spikes of any LIF layer, last first (act), and their number; for every
// record the numerator's terms from elsewhere (A2) and r = 1 / (I- - theta) of its
// jump lambda_V <- lambda_V + r (theta lambda_V + A); r < 0 marks a skipped one, I-
// <= theta (r is 0 for a current that has overflowed to infinity: a jump that
// changes nothing).
__global__ void __launch_bounds__(256) backward_prep_kernel(CoreBwdArgs a, int nl) {
    const int tid = threadIdx.x, lane = tid & 63, b = blockIdx.x;
    for (int l = 0; l < nl; ++l) {
        const BwdLayer& y = a.ly[l];
        const size_t r0 = (size_t)b * a.cap;
        const int cnt = y.rec_idx[(size_t)b * (a.T + 1) + a.T];
        for (int q = tid; q < cnt; q += 256) {
            // tau_m dV/dt just before the crossing is I- - theta (V- = theta)
            const double den = __dsub_rn((double)y.recI[r0 + q], a.theta), r = 1.0 / den;
            y.jump[r0 + q] = make_double2(y.A2 ? y.A2[r0 + q] : 0.0, den > 0.0 ? r : -1.0);
        }
    }
    if (tid >= 64) return;
    int* act = a.act + (size_t)b * a.T;
    int cnt = 0;
    for (int n0 = a.T - 1; n0 >= 0; n0 -= 64) {
        const int n = n0 - lane;
        bool any = false;
        for (int l = 0; l < nl; ++l) {
            const int* idx = a.ly[l].rec_idx + (size_t)b * (a.T + 1) + max(n, 0);
            any |= idx[1] > idx[0];
        }
        any = any && n >= 0;
        const unsigned long long m = __ballot(any);
        if (any) act[cnt + lanes_below(m)] = n;
        cnt += __popcll(m);
    }
    if (lane == 0) a.nact[b] = cnt;
}

// The spike masks, from the records, where the forward core does not write them:
// a workgroup takes 256 words of a sample's [T][NW] in layer blockIdx.y.
__global__ void __launch_bounds__(256) backward_masks_kernel(CoreBwdArgs a) {
    const int chunks = (a.T * a.NW + 255) / 256, b = (int)blockIdx.x / chunks;
    const int k = ((int)blockIdx.x - b * chunks) * 256 + (int)threadIdx.x;
    if (k >= a.T * a.NW) return;
    const BwdLayer& y = a.ly[blockIdx.y];
    const int n = k / a.NW, w = k - n * a.NW;
    const int* idx = y.rec_idx + (size_t)b * (a.T + 1) + n;
    const int* id = y.recn + (size_t)b * a.cap;
    unsigned long long m = 0;
    for (int r = idx[0]; r < idx[1]; ++r) m |= id[r] >> 6 == w ? 1ull << (id[r] & 63) : 0ull;
    y.masks[(size_t)b * a.T * a.NW + k] = m;
}

// MC: 64-post chunks of the widest LIF-post layer, at most.
template <int NL, int NP, int MC>
struct BwdSplit {
    static_assert(NP > 0, "layers without LIF-post projections have a core of their own");
    // a step's weight rows loaded a step ahead, in a second register set (wide
    // layers have no registers for one: loaded at the step itself), for the
    // first RW spikes of every helper
    static constexpr bool PF = NP * MC <= 8;
    static constexpr int RW = NP * MC <= 4 ? 2 : 1;
    static constexpr int CH = MC < 4 ? MC : 4;               // chunks whose ring reads go out together

    // far-table rows of one spike (all its LIF-post projections, this lane's
    // posts lane + 64 c) and its jump's A2 and r
    struct Row {
        uint2 w[NP][MC];
        double2 J;
    };

    // Position of spike q of a step (layers in order): layer l, record index
    // r of the sample; false: the step has fewer spikes.
    struct Step;
    static __device__ __forceinline__ bool locate(int q, const Step& s, int& l, int& r) {
        bool found = false;
        l = 0;
        r = 0;
#pragma unroll
        for (int m = 0; m < NL; ++m) {
            const int c = s.en[m] - s.st[m];
            if (!found && q < c) {
                found = true;
                l = m;
                r = s.st[m] + q;
            }
            if (!found) q -= c;
        }
        return found;
    }

    // (Loads of uniform addresses through a per-lane zero that the compiler
    // cannot see: scalar loads would count on the LDS counter.  The layers'
    // records lie one after the other: one base for all, as scalar registers are
    // short, 4-200-3 with a spiking output 252 us with one each, now 232.)
    static __device__ __forceinline__ int lane_zero() {
        int zero;
        asm volatile("v_mov_b32 %0, 0" : "=v"(zero));
        return zero;
    }

    static __device__ __forceinline__ int load_id(const CoreBwdArgs& a, int b, int l, int r) {
        return (a.ly[0].recn + ((size_t)l * a.B + b) * a.cap + r)[lane_zero()];
    }

    // Byte offsets of this lane's posts in a row of projection pp of layer l;
    // posts past the layer: past any matrix (the loads read 0).
    static __device__ __forceinline__ unsigned col(const BwdLayer& y, int pp, int c, int lane) {
        const int j = c * 64 + lane;
        return j < y.nq[pp] ? (unsigned)(j * 8) : 0x80000000u;
    }

    static __device__ __forceinline__ void load_row(const CoreBwdArgs& a, int b, int l, int r, int id, int lane,
                                                    Row& R) {
        R.J = (a.ly[0].jump + ((size_t)l * a.B + b) * a.cap + r)[lane_zero()];
#pragma unroll
        for (int m = 0; m < NL; ++m) {
            if (m != l) continue;
            const BwdLayer& y = a.ly[m];
#pragma unroll
            for (int pp = 0; pp < NP; ++pp) {
                if (pp >= y.npost) continue;
                const int rb = y.nq[pp] * 8;
                const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                    (void*)y.far[pp], (short)0, y.npre[pp] * rb, 0x00020000);
#pragma unroll
                for (int c = 0; c < MC; ++c) {
                    const auto v = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)col(y, pp, c, lane), id * rb, 0);
                    R.w[pp][c] = make_uint2((unsigned)v[0], (unsigned)v[1]);
                }
            }
        }
    }

    // x where `in`, else a finite value (the high word cleared).
    static __device__ __forceinline__ double finite_unless(bool in, double x) {
        const unsigned long long u = (unsigned long long)__double_as_longlong(x);
        const unsigned hi = in ? (unsigned)(u >> 32) : 0u;
        return __longlong_as_double((long long)(((unsigned long long)hi << 32) | (unsigned)u));
    }

    // This lane's terms of slots >= 1 of one spike of layer l, subtracted from
    // v: the far table's weights times the ring cells of the arrivals (rows of
    // steps past T - 1 were never written: zero).  nm: byte offset of the
    // step's own row in each post ring.
    static __device__ __forceinline__ void far_terms(const CoreBwdArgs& a, const int (&nm)[NL][NP], int l, int lane,
                                                     const Row& R, double& v) {
#pragma unroll
        for (int m = 0; m < NL; ++m) {
            if (m != l) continue;
            const BwdLayer& y = a.ly[m];
#pragma unroll
            for (int pp = 0; pp < NP; ++pp) {
                if (pp >= y.npost) continue;
                const int nq = y.nq[pp];
                const unsigned bytes = (unsigned)(y.qS[pp] * nq * 8), next = (unsigned)((nm[m][pp] + nq * 8));
                const unsigned char* ring = smem + y.qring_lds[pp];
#pragma unroll
                for (int c0 = 0; c0 < MC; c0 += CH) {
                    double d[CH];
#pragma unroll
                    for (int u = 0; u < CH; ++u) {
                        const unsigned e = R.w[pp][c0 + u].y;
                        const unsigned at = far_cell(next, (unsigned)min((c0 + u) * 64 + lane, nq - 1), e, bytes);
                        d[u] = finite_unless(far_arrives(e), *(const lds_f64*)(ring + at));
                    }
#pragma unroll
                    for (int u = 0; u < CH; ++u)
                        v = __fma_rn(-(double)__uint_as_float(R.w[pp][c0 + u].x), d[u], v);
                }
            }
        }
    }

    // The terms of slot 0 of one spike, from the weights themselves.
    static __device__ __forceinline__ void near_terms(const CoreBwdArgs& a, const int (&nm)[NL][NP], int l, int id,
                                                      int lane, double& v) {
#pragma unroll
        for (int m = 0; m < NL; ++m) {
            if (m != l) continue;
            const BwdLayer& y = a.ly[m];
#pragma unroll
            for (int pp = 0; pp < NP; ++pp) {
                if (pp >= y.npost) continue;
                const int nq = y.nq[pp];
                for (int j0 = 0; j0 < nq; j0 += 64) {
                    const int j = min(j0 + lane, nq - 1);
                    const uint2 e = y.ws[pp][(size_t)id * nq + j];
                    const double d = *(const lds_f64*)(smem + y.qring_lds[pp] + nm[m][pp] + j * 8);
                    const double t = __fma_rn(-(double)__uint_as_float(e.x), d, v);
                    v = j0 + lane < nq && e.y == 0 ? t : v;
                }
            }
        }
    }

    // The slots of the spiking neurons, by neuron: the jump's data with the
    // sum so far.  [2 (parity of the active step's index)][lif_total].
    static __device__ __forceinline__ double2* slots(const CoreBwdArgs& a, int k) {
        return reinterpret_cast<double2*>(smem + a.slot_off) + (k & 1) * a.lif_total;
    }

    static __device__ __forceinline__ void put(const CoreBwdArgs& a, int k, int l, int id, int lane, const Row& R,
                                               double v) {
        int off = 0;
#pragma unroll
        for (int m = 0; m < NL; ++m)
            if (m == l) off = a.ly[m].lif_off;
        double2* s = slots(a, k) + off + id;
        const double x = wave_sum_f64(v);
        if (lane == 63) *s = make_double2(R.J.x + x, R.J.y);
    }

    // Active steps of the sample in blocks of 64, one per lane: the step, the
    // records of every layer at it, and the byte offset of its row in each
    // post ring.
    struct Block {
        int n, st[NL], en[NL], nm[NL][NP];
    };
    static __device__ __forceinline__ void load_block(const CoreBwdArgs& a, int b, int k, int K, int lane, Block& B) {
        B.n = (a.act + (size_t)b * a.T)[min((k & ~63) + lane, K - 1)];
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const int* idx = a.ly[l].rec_idx + (size_t)b * (a.T + 1) + B.n;
            B.st[l] = idx[0];
            B.en[l] = idx[1];
#pragma unroll
            for (int pp = 0; pp < NP; ++pp) B.nm[l][pp] = B.n % a.ly[l].qS[pp] * (a.ly[l].nq[pp] * 8);
        }
        __builtin_amdgcn_s_waitcnt(kWaitVm0);
    }

    // Active step k (uniform); past the last: step -1, no records.
    struct Step {
        int n, st[NL], en[NL], nm[NL][NP];
    };
    static __device__ __forceinline__ void get_step(const CoreBwdArgs& a, int b, int k, int K, int lane, Block& B,
                                                    Step& s) {
        if (k >= K) {
            s.n = -1;
#pragma unroll
            for (int l = 0; l < NL; ++l) s.en[l] = s.st[l];
            return;
        }
        if ((k & 63) == 0) load_block(a, b, k, K, lane, B);
        s.n = __builtin_amdgcn_readlane(B.n, k & 63);
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            s.st[l] = __builtin_amdgcn_readlane(B.st[l], k & 63);
            s.en[l] = __builtin_amdgcn_readlane(B.en[l], k & 63);
#pragma unroll
            for (int pp = 0; pp < NP; ++pp) s.nm[l][pp] = __builtin_amdgcn_readlane(B.nm[l][pp], k & 63);
        }
    }

    static __device__ __forceinline__ int total(const Step& s) {
        int t = 0;
#pragma unroll
        for (int l = 0; l < NL; ++l) t += s.en[l] - s.st[l];
        return t;
    }

    // The barriers of active step n (gap: steps from the last active step, or
    // from step T, to it), the same for every wave:
    //  - ring_lapped(gap - 1): the jumps of the last active step have read its
    //    ring row, which the free steps would overwrite;
    //  - gap > 1: row n + 1 is in, and the delayed sums of step n may read it
    //    (for gap 1 the last step's own barrier says so);
    //  - row n is in, and with LISTS the slots of step n.
    // After the last active step, ring_lapped(n): its jumps have read its row,
    // which the free steps down to step 0 would overwrite.
    static __device__ __forceinline__ void before_sums(const CoreBwdArgs& a, int gap) {
        if (gap > 1) lds_barrier();
    }

    // ---- helper waves

    // Active step k with its rows cur (landed), the rows of step k + 1 into
    // nxt, the ids of step k + 2 into id.
    template <bool LISTS>
    static __device__ __forceinline__ void help_step(const CoreBwdArgs& a, int b, int h, int lane, int k, int K,
                                                     int& last, Block& B, Step& s0, Step& s1, Step& s2,
                                                     int (&id0)[RW], int (&id)[RW], Row (&cur)[RW], Row (&nxt)[RW]) {
        // loads issued a step ago have landed: this step's rows, the next ids
        __builtin_amdgcn_s_waitcnt(kWaitVm0);
        const int n = s0.n, gap = last - n, tot = total(s0);
        int id1[RW];
        get_step(a, b, k + 2, K, lane, B, s2);
#pragma unroll
        for (int u = 0; u < RW; ++u) {
            int l, r;
            id1[u] = __builtin_amdgcn_readfirstlane(id[u]);
            if constexpr (PF) {
                if (locate(h + u * a.H, s1, l, r)) load_row(a, b, l, r, id1[u], lane, nxt[u]);
            } else {
                if (locate(h + u * a.H, s0, l, r)) load_row(a, b, l, r, id0[u], lane, cur[u]);
            }
            if (locate(h + u * a.H, s2, l, r)) id[u] = load_id(a, b, l, r);
        }
        if (ring_lapped(gap - 1, a.run_max)) lds_barrier();
        before_sums(a, gap);
        // phase 1: terms of slots >= 1 (all terms in phase 2 where the slot-0
        // ones are the helpers')
#pragma unroll
        for (int u = 0; u < RW; ++u) {
            int l, r;
            if (!LISTS || !locate(h + u * a.H, s0, l, r)) break;
            double v = 0.0;
            far_terms(a, s0.nm, l, lane, cur[u], v);
            put(a, k, l, id0[u], lane, cur[u], v);
        }
        // spikes past the first RW of every helper: loaded now
        if (LISTS && tot > RW * a.H) more<false>(a, b, h + RW * a.H, lane, k, s0, tot);
        lds_barrier();                                       // row n is in
        if (!LISTS) {
            more<true>(a, b, h, lane, k, s0, tot);
            lds_barrier();                                   // the slots are in
        }
        last = n;
        s0 = s1;
        s1 = s2;
#pragma unroll
        for (int u = 0; u < RW; ++u) id0[u] = id1[u];
    }

    // Spikes q0, q0 + H, ... of the step, nothing of them loaded yet; NEAR:
    // with the terms of slot 0.
    template <bool NEAR>
    static __device__ __forceinline__ void more(const CoreBwdArgs& a, int b, int q0, int lane, int k, const Step& s,
                                                int tot) {
        for (int q = q0; q < tot; q += a.H) {
            int l, r;
            if (!locate(q, s, l, r)) break;
            const int id = __builtin_amdgcn_readfirstlane(load_id(a, b, l, r));
            Row R;
            load_row(a, b, l, r, id, lane, R);
            double v = 0.0;
            if (NEAR) near_terms(a, s.nm, l, id, lane, v);
            far_terms(a, s.nm, l, lane, R, v);
            put(a, k, l, id, lane, R, v);
        }
    }

    template <bool LISTS>
    static __device__ void help(const CoreBwdArgs& a, int b, int h, int lane) {
        const int K = a.nact[b];
        Block B{};
        Step s0{}, s1{}, s2{};
        get_step(a, b, 0, K, lane, B, s0);
        get_step(a, b, 1, K, lane, B, s1);
        Row X[RW], Y[RW];
        int id0[RW], id[RW], last = a.T;
#pragma unroll
        for (int u = 0; u < RW; ++u) {
            int l, r;
            id0[u] = id[u] = 0;
            if (locate(h + u * a.H, s0, l, r)) {
                id0[u] = __builtin_amdgcn_readfirstlane(load_id(a, b, l, r));
                if constexpr (PF) load_row(a, b, l, r, id0[u], lane, X[u]);
            }
            if (locate(h + u * a.H, s1, l, r)) id[u] = load_id(a, b, l, r);
        }
        int k = 0;
        for (; k + 1 < K; k += 2) {
            help_step<LISTS>(a, b, h, lane, k, K, last, B, s0, s1, s2, id0, id, X, Y);
            if constexpr (PF)
                help_step<LISTS>(a, b, h, lane, k + 1, K, last, B, s0, s1, s2, id0, id, Y, X);
            else
                help_step<LISTS>(a, b, h, lane, k + 1, K, last, B, s0, s1, s2, id0, id, X, Y);
        }
        if (k < K) help_step<LISTS>(a, b, h, lane, k, K, last, B, s0, s1, s2, id0, id, X, Y);
        if (K > 0 && ring_lapped(last, a.run_max)) lds_barrier();
    }

    // ---- neuron waves

    // The first near synapses of this lane's neurons: minus the weights, and
    // the LDS addresses of their posts in ring row 0.
    struct Near {
        double w[NL][kNearRegs];
        int at[NL][kNearRegs];
        int cnt[NL];                                         // of this lane's neuron
        int most[NL];                                        // over the wave's (uniform)
    };

    // LDS address of a near entry's post in ring row 0, and its projection in
    // bit 0.
    static __device__ __forceinline__ int near_at(const BwdLayer& y, unsigned e) {
        return (int)(e & 0xFFFFu) + (NP > 1 && (e >> 16) ? y.qring_lds[NP - 1] + 1 : y.qring_lds[0]);
    }

    static __device__ __forceinline__ void near_load(const CoreBwdArgs& a, int j, Near& N) {
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const BwdLayer& y = a.ly[l];
            const int i = y.lif_off + min(j, y.n - 1);
            N.cnt[l] = j < y.n && y.npost > 0 ? a.ncnt[i] : 0;
            int most = N.cnt[l];
#pragma unroll
            for (int d = 32; d; d >>= 1) most = max(most, __shfl_xor(most, d, 64));
            N.most[l] = __builtin_amdgcn_readfirstlane(most);
#pragma unroll
            for (int u = 0; u < kNearRegs; ++u) {
                // an entry past the list: weight 0 of the first post's cell (a layer
                // without LIF posts has no entries, and near_sum reads no cell)
                const uint2 e = a.near[(size_t)i * kNearCap + u];
                const bool in = u < N.cnt[l];
                N.w[l][u] = in ? -(double)__uint_as_float(e.x) : 0.0;
                N.at[l][u] = in ? near_at(y, e.y) : (y.npost > 0 ? y.qring_lds[0] : 0);
            }
        }
    }

    // x minus the sum of this lane's near terms of layer l, the step's row at
    // byte offset ro0 (ro1) of its projections' post rings.
    static __device__ __forceinline__ double near_sum(const CoreBwdArgs& a, const Near& N, int l, int j, int ro0,
                                                      int ro1, double x) {
        const BwdLayer& y = a.ly[l];
        auto cell = [&](int at) {
            return *(const lds_f64*)(smem + (NP > 1 ? (at & ~1) + ((at & 1) ? ro1 : ro0) : at + ro0));
        };
#pragma unroll
        for (int u0 = 0; u0 < kNearRegs; u0 += 4) {
            if (N.most[l] <= u0) break;
            double d[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) d[u] = finite_unless(u0 + u < N.cnt[l], cell(N.at[l][u0 + u]));
#pragma unroll
            for (int u = 0; u < 4; ++u) x = __fma_rn(N.w[l][u0 + u], d[u], x);
        }
        if (N.most[l] > kNearRegs) {
            for (int u = kNearRegs; u < N.cnt[l]; ++u) {
                const uint2 e = a.near[(size_t)(y.lif_off + j) * kNearCap + u];
                x = __fma_rn(-(double)__uint_as_float(e.x), cell(near_at(y, e.y)), x);
            }
        }
        return x;
    }

    struct Lane {
        double lv[NL], lI[NL];
        double2* tr[NL];                     // this lane's trajectory cell of the next step
        int own[NL], ownS[NL];               // LDS address of its cell in the own ring, and of row S
    };

    // One step of free dynamics: the trajectory and the ring row.  (At step
    // T - 1 the adjoints are zero and stay zero.)
    static __device__ __forceinline__ void free_step(const CoreBwdArgs& a, int j, Lane& L) {
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const BwdLayer& y = a.ly[l];
            const double v = L.lv[l];
            L.lI[l] = __dadd_rn(__dmul_rn(a.beta, L.lI[l]), __dmul_rn(a.cc, v));
            L.lv[l] = __dmul_rn(a.alpha, v);
            const double d = __dsub_rn(L.lI[l], L.lv[l]);
            if (j < y.n) {
                if (NL == 1 || y.ring_lds >= 0) *(lds_f64*)(smem + L.own[l]) = d;
                *L.tr[l] = make_double2(L.lI[l], d);
            }
            L.tr[l] -= a.lif_total;
            L.own[l] -= y.n * 8;
            L.own[l] = L.own[l] < y.ring_lds ? L.own[l] + y.S * y.n * 8 : L.own[l];
        }
    }

    template <bool LISTS>
    static __device__ void neurons(const CoreBwdArgs& a, int b, int wave, int lane) {
        const int T = a.T, j = wave * 64 + lane, K = a.nact[b];
        Lane L;
        Near N;
        if (LISTS) near_load(a, j, N);
        unsigned long long mk[NL];
        const unsigned long long* mp[NL];
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const BwdLayer& y = a.ly[l];
            L.lv[l] = L.lI[l] = 0.0;
            L.own[l] = y.ring_lds + ((T - 1) % y.S * y.n + min(j, y.n - 1)) * 8;
            L.tr[l] = a.traj + ((size_t)b * T + (T - 1)) * a.lif_total + y.lif_off + min(j, y.n - 1);
            mp[l] = y.masks + (size_t)b * T * a.NW + wave;
            mk[l] = 0;
        }
        int deg = 0;
        Block B{};
        Step s{};
        int last = T;
        for (int k = 0; k < K; ++k) {
            get_step(a, b, k, K, lane, B, s);
            if ((k & 63) == 0) {
#pragma unroll
                for (int l = 0; l < NL; ++l) mk[l] = mp[l][(size_t)B.n * a.NW];
                __builtin_amdgcn_s_waitcnt(kWaitVm0);
            }
            const int gap = last - s.n;
            if (ring_lapped(gap - 1, a.run_max)) lds_barrier();
            for (int g = gap; g > 1; --g) free_step(a, j, L);
            before_sums(a, gap);
            free_step(a, j, L);
            lds_barrier();                                   // row n is in, and (LISTS) the slots
            if (!LISTS) lds_barrier();                       // the slots are in
            last = s.n;
#pragma unroll
            for (int l = 0; l < NL; ++l) {
                const unsigned lo = __builtin_amdgcn_readlane((unsigned)mk[l], k & 63);
                const unsigned hi = __builtin_amdgcn_readlane((unsigned)(mk[l] >> 32), k & 63);
                const unsigned long long m = ((unsigned long long)hi << 32) | lo;
                if (m == 0) continue;
                if ((m >> lane) & 1ull) {
                    const double2 q = slots(a, k)[a.ly[l].lif_off + j];
                    const double A = LISTS ? near_sum(a, N, l, j, s.nm[l][0], s.nm[l][NP - 1], q.x) : q.x;
                    const double v = __fma_rn(q.y, __fma_rn(a.theta, L.lv[l], A), L.lv[l]);
                    L.lv[l] = q.y >= 0.0 ? v : L.lv[l];
                    deg += q.y >= 0.0 ? 0 : 1;
                }
            }
        }
        if (K > 0 && ring_lapped(last, a.run_max)) lds_barrier();
        for (int g = last; g > 0; --g) free_step(a, j, L);
        if (deg) atomicAdd(&a.st->degenerate, (unsigned long long)deg);
    }

    static __device__ void run(const CoreBwdArgs& a) {
        const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const bool lists = a.st->near_pre <= kNearCap;
        // the rings start at zero: rows not written yet are read, and masked
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const BwdLayer& y = a.ly[l];
            if (y.ring_lds < 0) continue;
            for (int k = tid; k < y.S * y.n; k += blockDim.x) ((lds_f64*)(smem + y.ring_lds))[k] = 0.0;
        }
        __syncthreads();
        if (wave < a.NW) {
            __builtin_amdgcn_s_setprio(3);                   // the chain of steps runs through these
            if (lists) neurons<true>(a, b, wave, lane); else neurons<false>(a, b, wave, lane);
        } else {
            if (lists) help<true>(a, b, wave - a.NW, lane); else help<false>(a, b, wave - a.NW, lane);
        }
    }
};

template <int NL, int NP, int MC>
__global__ void __launch_bounds__(1024) backward_split_kernel(CoreBwdArgs a) {
    BwdSplit<NL, NP, MC>::run(a);
}

// The instantiation for n_lif LIF layers with at most np LIF-post projections
// each, posts of at most mc chunks of 64; NULL: none (more layers need more
// scalar registers for their arguments than a wave has).
const void* split_kernel(int n_lif, int np, int mc) {
    if (n_lif == 1 && np == 1)
        return mc <= 2 ? (const void*)backward_split_kernel<1, 1, 2>
               : mc <= 4 ? (const void*)backward_split_kernel<1, 1, 4>
               : mc <= 8 ? (const void*)backward_split_kernel<1, 1, 8> : nullptr;
    if (n_lif == 2 && np == 1)
        return mc <= 2 ? (const void*)backward_split_kernel<2, 1, 2>
               : mc <= 4 ? (const void*)backward_split_kernel<2, 1, 4> : nullptr;
    if (n_lif == 2 && np == 2)
        return mc <= 2 ? (const void*)backward_split_kernel<2, 2, 2>
               : mc <= 4 ? (const void*)backward_split_kernel<2, 2, 4> : nullptr;
    return nullptr;
}

}  // namespace

hipError_t launch_backward_masks(const CoreBwdArgs& a, int n_lif, hipStream_t s) {
    const int chunks = (a.T * a.NW + 255) / 256;
    hipLaunchKernelGGL(backward_masks_kernel, dim3((unsigned)(a.B * chunks), n_lif), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_backward_prep(const CoreBwdArgs& a, int n_lif, hipStream_t s) {
    hipLaunchKernelGGL(backward_prep_kernel, dim3(a.B), dim3(256), 0, s, a, n_lif);
    return hipGetLastError();
}

hipError_t launch_backward_split(const CoreBwdArgs& a, int n_lif, int np, size_t lds, hipStream_t s) {
    const int waves = a.NW + a.H;
    if (n_lif < 1 || n_lif > SNN_MAX_LIF || a.NW < 1 || a.H < 1 || waves > 16) return hipErrorInvalidValue;
    int mc = 0;
    for (int l = 0; l < n_lif; ++l) {
        if (a.ly[l].n > 64 * a.NW || a.ly[l].npost > np || a.ly[l].ring_lds == -1) return hipErrorInvalidValue;
        for (int pp = 0; pp < a.ly[l].npost; ++pp) {
            if (a.ly[l].qring_lds[pp] < 0) return hipErrorInvalidValue;
            mc = max(mc, (a.ly[l].nq[pp] + 63) / 64);
        }
    }
    const void* f = split_kernel(n_lif, np, mc);
    if (!f) return hipErrorInvalidValue;
    CoreBwdArgs arg = a;
    void* args[] = {&arg};
    return hipLaunchKernel(f, dim3(a.B), dim3(64 * waves), args, lds, s);
}

bool backward_split_serves(int n_lif, int np, int maxn) {
    return split_kernel(n_lif, np, (maxn + 63) / 64) != nullptr;
}

hipError_t set_split_lds_limits(size_t bytes, int* bad) {
    static const int cases[7][3] = {{1, 1, 2}, {1, 1, 4}, {1, 1, 8}, {2, 1, 2}, {2, 1, 4}, {2, 2, 2}, {2, 2, 4}};
    for (int k = 0; k < 7; ++k) {
        const hipError_t e = hipFuncSetAttribute(split_kernel(cases[k][0], cases[k][1], cases[k][2]),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e != hipSuccess) {
            if (bad) *bad = k;
            return e;
        }
    }
    return hipSuccess;
}
