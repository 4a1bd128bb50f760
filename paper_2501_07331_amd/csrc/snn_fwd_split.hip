// The LIF forward core of libsnn with its delay rings in LDS (gfx950,
// wave64): one workgroup per sample runs the LIF layers over T steps (Table 1,
// forward dynamics with delayed current jumps).  All fp32, in the order of the
// definition: a ring cell sums its weights in emission order (step, then
// presynaptic neuron), bit for bit.
//
// A step's critical path is short: a neuron's arrivals, its dynamics, its
// spike, and the spikes of the others that reach it without delay.  With one
// set of waves doing everything a step took about 2500 cycles, nearly all of
// it the scatter of the step's spikes (weight rows from L2, ordered
// read-modify-writes of ring cells) and the spike records.  So the waves are
// split, with one barrier a step, at which the step's spikes are in LDS (mask
// words, counts and per-wave lists, kept for four steps):
//
//  neuron waves   lane j owns neuron j of every LIF layer: dynamics, ballot;
//                 after the barrier its arrivals: the ring cell, then the
//                 synapses of slot 1 from the last step's spikes and those of
//                 slot 0 from the step's own, in presynaptic order.  A cell sums
//                 in emission order, so the latest two emissions can stay out
//                 of the ring: each lane holds its synapses of slots 1 and 0
//                 (presynaptic neuron, weight) in registers and tests the
//                 neurons' bits in the mask words.
//  scatter waves  one per 64 columns of every LIF -> LIF ring: spikes with
//                 slots >= 2 into the ring, one step late: a step's weight rows
//                 are loaded while the last step's are added.
//  record wave    spike records, mask words and record indices, off the path.
//  readout wave   the leaky-integrator readout fed by a LIF layer, if it fits
//                 (an LDS ring of its own), one step late likewise.
//
// Where some neuron has more synapses of slots 0 and 1 than near_limit (delays
// near zero throughout), the neuron waves take them from the weight rows of the
// spikes instead, which they hold from one step to the next (dense_add: a step's
// rows give its slot 0 at once and its slot 1 a step later).  T = 500, batch 128,
// delays up to 5: 256 neurons 504 us, 128 362, 64 312 (both steps' rows loaded
// in the step: 683, 481, 374; the general core 512, 405, 355; T = 1000, batch
// 256: 1122 and 1057, left to the general core by the host).
//
// Measured, 700-256-20 recurrent, T = 1000: the core with the readout 1063 -> 792
// us at batch 256, 1042 -> 772 us at 32; T = 4000 at a quarter of the time step,
// batch 64: 3248 -> 2010 us; the recurrent layer of 128, T = 300, batch 128: 432
// -> 286 us.  Bound
// by the ordered adds into the rings (without them 475 of 772 us; without the
// readout wave 111 less).  Slot 0 alone kept near: 885; ring cells read four
// together instead of two: 804 against 780; lists of 16 instead of 24 or 32
// registers 2549 against 2010 (fine grid).
#include "snn_bwd_plan.h"
#include "snn_device.h"

namespace {

__device__ __forceinline__ void lds_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);       // lgkmcnt(0); vmcnt, expcnt at their maximum
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Tables of the LIF -> LIF projections, from their (weight, slot) pairs.
//  workgroups [0, rowblocks): one wave per neuron i of the LIF layers: its
//      rows of the far tables: of the backward core (far: weight bits, far_entry),
//      of the forward core (ffar [n + 1][nq]: weight bits, slot times the bytes of
//      a ring row) with slots 0 and 1 as weight +0 at the largest slot (a cell
//      that no pending step reads; a readout's table has all slots); row n of
//      ffar, which stands in for spikes past a chunk's end, likewise; and its
//      synapses of slot 0 for the backward core, projections then posts in order:
//      the first kNearCap (weight bits; LDS byte offset of the post's fp64 ring
//      column, projection << 16) and their number.
//  the others: 64 posts of a projection each: the posts' synapses of slot 1
//      (where post_slots is 2), then slot 0, each in presynaptic order: the first
//      kPostCap (weight bits; neuron, slot << 16) and their number.
// The largest numbers go to the status block.  (One launch for both directions in
// every forward: whether a backward follows is not known there, and weights and
// delays may have changed when it comes.)
__global__ void __launch_bounds__(512) split_tables_kernel(SplitTables a) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (a.st->bad_input) return;
    if ((int)blockIdx.x < a.rowblocks) {
        int i = (int)blockIdx.x * 8 + wave, l = 0;
        if (i >= a.lif_total) return;
        const int g = i;
        while (i >= a.n[l]) i -= a.n[l++];
        int cnt = 0;
        for (int pp = 0; pp < a.npost[l]; ++pp) {
            const SplitProj& p = a.pr[a.out[l][pp]];
            const int nq = p.nq;
            for (int j0 = 0; j0 < nq; j0 += 64) {
                const int j = j0 + lane;
                const size_t k = (size_t)i * nq + min(j, nq - 1);
                const uint2 e = p.ws[k];
                const bool zero = j < nq && e.y == 0;
                const unsigned long long m = __ballot(zero);
                const int pos = cnt + lanes_below(m);
                const unsigned top = (unsigned)((p.S - 1) * nq);
                if (j < nq) {
                    if (p.far) p.far[k] = make_uint2(zero ? 0u : e.x, far_entry(e.y, (unsigned)nq));
                    if (p.ffar) p.ffar[k] = e.y < 2 ? make_uint2(0u, top * 4u) : make_uint2(e.x, e.y * (unsigned)(nq * 4));
                    if (p.ffar && i == p.npre - 1) p.ffar[(size_t)p.npre * nq + j] = make_uint2(0u, top * 4u);
                }
                if (zero && pos < kNearCap)
                    a.near[(size_t)g * kNearCap + pos] = make_uint2(e.x, (unsigned)(j * 8) | ((unsigned)pp << 16));
                cnt += __popcll(m);
            }
        }
        if (a.ro.ffar && l == a.ro_l) {
            const int C = a.ro.nq;
            for (int k = lane; k < C; k += 64) {
                const uint2 e = a.ro.ws[(size_t)i * C + k];
                a.ro.ffar[(size_t)i * C + k] = make_uint2(e.x, e.y * (unsigned)(C * 4));
                if (i == a.ro.npre - 1)
                    a.ro.ffar[(size_t)a.ro.npre * C + k] = make_uint2(0u, (unsigned)((a.ro.S - 1) * C * 4));
            }
        }
        if (lane == 0) {
            a.ncnt[g] = cnt;
            if (cnt > kNearRegs) atomicMax(&a.st->near_pre, cnt);
        }
        return;
    }
    __shared__ int part[2][8][64];
    int blk = (int)blockIdx.x - a.rowblocks, q = 0;
    while (blk >= (a.pr[q].nq + 63) / 64) blk -= (a.pr[q++].nq + 63) / 64;
    const SplitProj& p = a.pr[q];
    const int nq = p.nq, j = blk * 64 + lane, jc = min(j, nq - 1);
    const int per = (p.npre + 7) / 8, i0 = min(wave * per, p.npre), i1 = min(i0 + per, p.npre);
    int cnt[2] = {0, 0};
#pragma unroll 8
    for (int i = i0; i < i1; ++i) {
        const unsigned sl = p.ws[(size_t)i * nq + jc].y;
        cnt[0] += sl == 1 && a.post_slots > 1;
        cnt[1] += sl == 0;
    }
    part[0][wave][lane] = cnt[0];
    part[1][wave][lane] = cnt[1];
    __syncthreads();
    int pos[2] = {0, 0}, all = 0;
    for (int h = 0; h < 2; ++h) {
        pos[h] = all;
        for (int w = 0; w < 8; ++w) {
            const int c = part[h][w][lane];
            pos[h] += w < wave ? c : 0;
            all += c;
        }
    }
    if (j < nq) {
        uint2* out = p.post + (size_t)j * kPostCap;
        if (cnt[0] + cnt[1] > 0) {
#pragma unroll 8
            for (int i = i0; i < i1; ++i) {
                const uint2 e = p.ws[(size_t)i * nq + jc];
                if (e.y < a.post_slots) {
                    const int at = e.y ? pos[0]++ : pos[1]++;
                    if (at < kPostCap) out[at] = make_uint2(e.x, (unsigned)i | (e.y << 16));
                }
            }
        }
        if (wave == 0) {
            p.pcnt[j] = all;
            if (all > 4) atomicMax(&a.st->near_post, all);
        }
    }
}

// NWM: the most neuron waves (64-neuron groups of the widest LIF layer).
template <int NL, int NP, int NWM>
struct FwdSplit {
    typedef __attribute__((address_space(3))) unsigned short lds_u16;
    typedef __attribute__((address_space(3))) unsigned lds_u32;
    typedef __attribute__((address_space(3))) unsigned long long lds_u64;
    // head of the LDS, four steps deep (slot n & 3 for step n): spike counts of
    // the neuron waves (16 bits each), mask words (with one more slot before
    // the first, a copy of the last, so that the slot before a step's is at a
    // fixed distance), spike lists (neuron of wave w's r-th spike), I- of the
    // listed spikes
    static constexpr int D = 4;
    static constexpr int MASKS = NL * NWM * 8, CNTS = NL * NWM * 2, LIST = NL * NWM * 64;
    static constexpr int CNT0 = 0, MASK0 = (CNT0 + D * CNTS + 15) / 16 * 16, LIST0 = MASK0 + (D + 1) * MASKS,
                         CUR0 = LIST0 + D * LIST * 2, HEAD = CUR0 + D * LIST * 4;
    // near synapses a lane holds in registers (the rest is read from memory in
    // every step with spikes: delays drawn from 0 .. 50 give a neuron 7.7 of them
    // among 256, and the most of 256 neurons about 17)
    static constexpr int EN = NL == 1 && NWM == 4 ? kPostCap : 16;
    // The longest lists taken synapse by synapse, with nw neuron waves; longer
    // ones in the dense form.  T = 500, batch 128, list and dense form: one layer
    // of 64, lists of 31, 212 and 312 us, of 128 (30) 244 and 362, of 256 (31) 379
    // and 508 (with 24 registers 374, 381, 464: a memory access an entry and step);
    // of 300 (16 registers), 20: 548 and 665, 26: 808 and 670, T = 2000 2320 and
    // 1647; two layers of 100 and 60, 21 to 24: 428 and 444; of 256 each, 25 to
    // 30: 773 and 860.
    static __device__ __forceinline__ int near_limit(int nw) {
        return NL == 1 ? (nw <= 4 ? kPostCap : EN + 8) : nw <= 2 ? EN + 8 : kPostCap;
    }
    static constexpr int U = 2 * D;                  // steps that input arrivals are loaded ahead
    static constexpr int kRound = 2;                 // ring cells read together (see cells_add)
    static constexpr int KG = 4;                     // spikes whose rows are loaded and added together
    // spikes of a step whose rows are loaded a step ahead (as the registers allow)
    static constexpr int PK = NL == 1 && NWM == 4 ? 16 : 8;

    // The spikes of a layer at a step (uniform): how many, and how many before
    // each wave's.
    struct Spikes {
        int pre[NWM], total;
    };
    static __device__ __forceinline__ void spikes_of(int n, int l, Spikes& s) {
        const lds_u64* c = (const lds_u64*)(smem + CNT0 + (n & (D - 1)) * CNTS + l * NWM * 2);
        unsigned long long v[NWM / 4];
#pragma unroll
        for (int k = 0; k < NWM / 4; ++k) v[k] = c[k];
        s.total = 0;
#pragma unroll
        for (int k = 0; k < NWM / 4; ++k) {
            const unsigned long long u = uniform64(v[k]);
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                s.pre[4 * k + h] = s.total;
                s.total += (int)(u >> (16 * h)) & 0xFFFF;
            }
        }
    }

    // Position in the lists of spike r of a layer (r < total).
    static __device__ __forceinline__ int list_at(const Spikes& s, int n, int l, int r) {
        int at = r;
#pragma unroll
        for (int k = 1; k < NWM; ++k) at = r >= s.pre[k] ? k * 64 + r - s.pre[k] : at;
        return ((n & (D - 1)) * NL + l) * NWM * 64 + at;
    }
    // Neuron of spike r0 + k in lane k, `pad` past the last (total > 0).
    static __device__ __forceinline__ int list_ids(const Spikes& s, int n, int l, int r0, int pad) {
        const int r = r0 + (int)(threadIdx.x & 63);
        const int id = ((const lds_u16*)(smem + LIST0))[list_at(s, n, l, min(r, s.total - 1))];
        return r < s.total ? id : pad;
    }

    // ---- neuron waves

    struct Lane {
        float V[NL], I[NL];
        int own[NL];
        // per LIF-sourced projection into the layer: the ring cell of the next
        // arrival (LDS address) and its wrap, the synapses of slots 1 and 0
        int cell[NL][NP], row[NL][NP], last[NL][NP];
        unsigned nw[NL][NP][EN];             // weight bits (0 past the list)
        int nat[NL][NP][EN], nbit[NL][NP][EN];   // LDS address of the neuron's mask word (step slot 0), bit
        int most[NL][NP];                    // longest list of the wave (uniform)
        int on[NL];                          // the last step had spikes of the layer (uniform)
    };

    // Mask word of a post-list entry's neuron (layer sl): of the step itself
    // (slot 0) or the one before (slot 1), for a step of slot 0 in the ring of
    // steps.
    static __device__ __forceinline__ int near_at(int sl, unsigned e) {
        return MASK0 + MASKS + sl * NWM * 8 + (int)((e & 0xFFFFu) >> 5) * 4 - (e >> 16 ? MASKS : 0);
    }

    static __device__ __forceinline__ void near_regs(const CoreFwdArgs& a, int j, int l, int e, int x, Lane& L) {
        const FwdLayer& y = a.ly[l];
        const bool live = j < y.n;
        const int jc = min(j, y.n - 1), cnt = live ? a.role[l].in_pcnt[e][jc] : 0;
        int most = cnt;
#pragma unroll
        for (int d = 32; d; d >>= 1) most = max(most, __shfl_xor(most, d, 64));
        L.most[l][x] = __builtin_amdgcn_readfirstlane(most);
#pragma unroll
        for (int u = 0; u < EN; ++u) {
            const uint2 v = a.role[l].in_post[e][(size_t)jc * kPostCap + u];
            const bool in = u < cnt;
            const int i = in ? (int)(v.y & 0xFFFFu) : 0;
            L.nw[l][x][u] = in ? v.x : 0u;
            L.nat[l][x][u] = near_at(y.in_l[e], in ? v.y : 0u);
            L.nbit[l][x][u] = i & 31;
        }
    }

    // x plus the synapses of slot 1 of the last step's spikes, then of slot 0 of
    // the step's, in presynaptic order (a neuron that did not spike adds +0,
    // which changes no x: a ring cell is never -0).  par: the step's slot.
    static __device__ __forceinline__ float near_add(const CoreFwdArgs& a, int j, int par, int l, int e, int x,
                                                     const Lane& L, float v) {
#pragma unroll
        for (int u0 = 0; u0 < EN; u0 += 8) {
            if (L.most[l][x] <= u0) break;
            constexpr int G = EN < 8 ? EN : 8;
            unsigned w[G];
#pragma unroll
            for (int u = 0; u < G; ++u) w[u] = *(const lds_u32*)(smem + par * MASKS + L.nat[l][x][u0 + u]);
#pragma unroll
            for (int u = 0; u < G; ++u) {
                const unsigned s = (unsigned)__builtin_amdgcn_sbfe((int)w[u], L.nbit[l][x][u0 + u], 1);
                v = __fadd_rn(v, __uint_as_float(s & L.nw[l][x][u0 + u]));
            }
        }
        // the rest of the list: four entries' loads together, with two layers (no
        // registers left: 275 us against 266, 4-200-3 with a spiking output) one
        if constexpr (NL > 1) {
            if (L.most[l][x] > EN) {
                const FwdLayer& y = a.ly[l];
                const int jc = min(j, y.n - 1), cnt = j < y.n ? a.role[l].in_pcnt[e][jc] : 0;
#pragma unroll 1
                for (int u = EN; u < cnt; ++u) {
                    const uint2 q = a.role[l].in_post[e][(size_t)jc * kPostCap + u];
                    const unsigned w = *(const lds_u32*)(smem + par * MASKS + near_at(y.in_l[e], q.y));
                    v = __fadd_rn(v, (w >> (q.y & 31)) & 1u ? __uint_as_float(q.x) : 0.0f);
                }
            }
        } else if constexpr (EN < kPostCap) {
            constexpr int TG = 4;
            const FwdLayer& y = a.ly[l];
            const int jc = min(j, y.n - 1), cnt = j < y.n ? a.role[l].in_pcnt[e][jc] : 0;
#pragma unroll 1
            for (int u0 = EN; u0 < L.most[l][x]; u0 += TG) {
                uint2 q[TG];
                unsigned w[TG];
#pragma unroll
                for (int u = 0; u < TG; ++u) {
                    q[u] = a.role[l].in_post[e][(size_t)jc * kPostCap + u0 + u];
                    if (u0 + u >= cnt) q[u] = make_uint2(0u, 0u);
                }
#pragma unroll
                for (int u = 0; u < TG; ++u) w[u] = *(const lds_u32*)(smem + par * MASKS + near_at(y.in_l[e], q[u].y));
#pragma unroll
                for (int u = 0; u < TG; ++u) {
                    const unsigned k = (unsigned)__builtin_amdgcn_sbfe((int)w[u], (int)(q[u].y & 31u), 1);
                    v = __fadd_rn(v, __uint_as_float(k & q[u].x));
                }
            }
        }
        return v;
    }

    // The rows of a step's first HR spikes that a lane holds of one projection:
    // the step's slot 0 is added from them, a step later its slot 1.
    static constexpr int HR = NL == 1 ? 16 : 8, DG = NL == 1 ? KG : KB;   // (DG: loaded together)
    struct Held {
        Spikes s;
        uint2 w[HR];
    };

    // Rows r0 .. r0 + DG (of the lane's ids; past the spikes: loaded, not used).
    static __device__ __forceinline__ void dense_load(__amdgpu_buffer_rsrc_t rs, int col8, int row8, int ids, int r0,
                                                      uint2* w) {
#pragma unroll
        for (int k = 0; k < DG; ++k) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b64(rs, col8, __builtin_amdgcn_readlane(ids, r0 + k) * row8, 0);
            w[k] = make_uint2((unsigned)v[0], (unsigned)v[1]);
        }
    }
    static __device__ __forceinline__ float dense_sum(const uint2* w, int left, unsigned slot, float v) {
#pragma unroll
        for (int k = 0; k < DG; ++k)
            v = __fadd_rn(v, k < left && w[k].y == slot ? __uint_as_float(w[k].x) : 0.0f);
        return v;
    }

    // The spikes of step n past the held ones, their rows loaded now.
    static __device__ __forceinline__ float dense_rest(__amdgpu_buffer_rsrc_t rs, int col8, int row8, const Spikes& s,
                                                       int n, int sl, unsigned slot, float v) {
#pragma unroll 1
        for (int r0 = HR; r0 < s.total; r0 += DG) {
            uint2 x[DG];
            dense_load(rs, col8, row8, list_ids(s, n, sl, r0, 0), 0, x);
            v = dense_sum(x, s.total - r0, slot, v);
        }
        return v;
    }

    // x plus the same synapses, from the weight rows of the two steps' spikes (n:
    // the step).
    static __device__ __forceinline__ float dense_add(const CoreFwdArgs& a, int j, int n, int l, int e, Held& H,
                                                      float v) {
        const FwdLayer& y = a.ly[l];
        const int nq = y.n, sl = y.in_l[e], col8 = min(j, nq - 1) * 8;
        // (an argument indexed by a value that the compiler does not know makes it
        // reload arguments within the loops instead of keeping them in scalar
        // registers: one layer 303 us against 296, 12-128-27 recurrent, T = 300,
        // batch 128; with two layers, which have none left, 264 against 285,
        // 4-200-3 with a spiking output, T = 600, batch 256)
        const int npre = NL == 1 ? nq : a.ly[sl].n;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)a.role[l].in_ws[e], (short)0, npre * nq * 8,
                                                                            0x00020000);
        const Spikes last = H.s;
        uint2 w[HR];
#pragma unroll
        for (int k = 0; k < HR; ++k) w[k] = H.w[k];
        spikes_of(n, sl, H.s);
        if (H.s.total > 0) {
            const int ids = list_ids(H.s, n, sl, 0, 0);
#pragma unroll
            for (int g = 0; g < HR; g += DG)
                if (g == 0 || H.s.total > g) dense_load(rs, col8, nq * 8, ids, g, H.w + g);
        }
#pragma unroll
        for (int g = 0; g < HR; g += DG)
            if (last.total > g) v = dense_sum(w + g, last.total - g, 1u, v);
        if (last.total > HR) v = dense_rest(rs, col8, nq * 8, last, n - 1, sl, 1u, v);
#pragma unroll
        for (int g = 0; g < HR; g += DG)
            if (H.s.total > g) v = dense_sum(H.w + g, H.s.total - g, 0u, v);
        if (H.s.total > HR) v = dense_rest(rs, col8, nq * 8, H.s, n, sl, 0u, v);
        return v;
    }

    template <bool DENSE>
    static __device__ __forceinline__ void step(const CoreFwdArgs& a, int j, int wave, int lane, int n, int par,
                                                float ain, Lane& L, Held (&H)[NL][NP]) {
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const float gi = __fmul_rn(a.gamma, L.I[l]);
            const float Vm = __fmaf_rn(a.alpha, L.V[l], gi);
            L.I[l] = __fmul_rn(a.beta, L.I[l]);
            const bool spk = j < a.ly[l].n && Vm >= a.theta;
            L.V[l] = spk ? 0.0f : Vm;
            const unsigned long long m = __ballot(spk);
            if (lane == 0) {
                lds_u64* w = (lds_u64*)(smem + MASK0 + MASKS + l * NWM * 8) + wave;
                w[par * (MASKS / 8)] = m;
                if (par == D - 1) w[-(MASKS / 8)] = m;
                ((lds_u16*)(smem + CNT0 + par * CNTS + l * NWM * 2))[wave] = (unsigned short)__popcll(m);
            }
            if (spk) {
                const int at = ((par * NL + l) * NWM + wave) * 64 + lanes_below(m);
                ((lds_u16*)(smem + LIST0))[at] = (unsigned short)j;
                ((lds_f32*)(smem + CUR0))[at] = L.I[l];
                ++L.own[l];
            }
        }
        lds_barrier();                                       // the step's spikes are in; in the rings, the
                                                             // emissions of all steps but the last two
        // arrivals, projection by projection in projection order; the cell is
        // then free for a later step
        float x[NL][NP];
        unsigned long long any[NL];
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            any[l] = 0;
#pragma unroll
            for (int k = 0; k < NWM / 4; ++k)
                any[l] |= ((const lds_u64*)(smem + CNT0 + par * CNTS + l * NWM * 2))[k];
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                if (q >= a.role[l].nrec) continue;
                lds_f32* c = (lds_f32*)(smem + L.cell[l][q]);
                x[l][q] = *c;
                *c = 0.0f;
                L.cell[l][q] += L.row[l][q];
                L.cell[l][q] = L.cell[l][q] > L.last[l][q] ? L.cell[l][q] - (a.ly[l].in_S[q + (l == 0)]) * L.row[l][q]
                                                           : L.cell[l][q];
            }
        }
        int on[NL];
#pragma unroll
        for (int l = 0; l < NL; ++l) on[l] = uniform64(any[l]) != 0;
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const FwdLayer& y = a.ly[l];
            if (l == 0) L.I[0] = __fadd_rn(L.I[0], ain);     // layer 1's first projection is the inputs'
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                if (q >= a.role[l].nrec) continue;
                const int e = q + (l == 0);
                // the source layer: l itself, or l - 1 (a feed-forward projection)
                const bool prev = l > 0 && y.in_l[e] != l;
                if (prev ? on[l > 0 ? l - 1 : 0] | L.on[l > 0 ? l - 1 : 0] : on[l] | L.on[l])
                    x[l][q] = DENSE ? dense_add(a, j, n, l, e, H[l][q], x[l][q]) : near_add(a, j, par, l, e, q, L, x[l][q]);
                L.I[l] = __fadd_rn(L.I[l], x[l][q]);
            }
        }
#pragma unroll
        for (int l = 0; l < NL; ++l) L.on[l] = on[l];
    }

    template <bool DENSE>
    static __device__ void neurons(const CoreFwdArgs& a, int b, int wave, int lane) {
        const int j = wave * 64 + lane, T = a.T;
        Lane L;
        Held H[NL][NP];                                      // (used with DENSE only)
#pragma unroll
        for (int l = 0; l < NL; ++l)
#pragma unroll
            for (int q = 0; q < NP; ++q) H[l][q].s.total = 0;
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const FwdLayer& y = a.ly[l];
            L.V[l] = L.I[l] = 0.0f;
            L.own[l] = 0;
            L.on[l] = 0;
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                L.most[l][q] = 0;
                if (q >= a.role[l].nrec) continue;
                const int e = q + (l == 0), row = y.n * 4;
                // (lanes past the layer: the dummy row's first cell, never read)
                L.row[l][q] = j < y.n ? row : 0;
                L.cell[l][q] = y.in_ring_lds[e] * 4 + (j < y.n ? j * 4 : y.in_S[e] * row);
                L.last[l][q] = j < y.n ? y.in_ring_lds[e] * 4 + y.in_S[e] * row - 4 : 0x7FFFFFFF;
                if (!DENSE) near_regs(a, j, l, e, q, L);
            }
        }
        gptr<const float> ain = (gptr<const float>)(a.A_in + (size_t)b * T * a.n1 + min(j, a.n1 - 1));
        if constexpr (DENSE) {
#pragma unroll 1
            for (int n = 0; n < T; ++n) step<true>(a, j, wave, lane, n, n & (D - 1), ain[(size_t)n * a.n1], L, H);
        } else {
            // each step's arrival in a register of its own, reloaded for step n
            // + U as soon as it is used: no register moves while its load is in
            // flight (a move would wait for it), and U - 1 loads stay in flight
            float x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = ain[(size_t)min(u, T - 1) * a.n1];
            int n0 = 0;
#pragma unroll 1
            for (; n0 + U <= T; n0 += U) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const float v = x[u];
                    step<false>(a, j, wave, lane, n0 + u, u & (D - 1), v, L, H);
                    x[u] = ain[(size_t)min(n0 + U + u, T - 1) * a.n1];
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (n0 + u < T) step<false>(a, j, wave, lane, n0 + u, u & (D - 1), x[u], L, H);
        }
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const FwdLayer& y = a.ly[l];
            if (j < y.n) {
                a.Vf[(size_t)b * a.nstate + a.soff[l] + j] = L.V[l];
                a.If[(size_t)b * a.nstate + a.soff[l] + j] = L.I[l];
                // integer sums over the samples: exact in any order
                if (y.ncount && L.own[l]) atomicAdd(&y.ncount[j], L.own[l]);
            }
        }
    }

    // ---- scatter waves

    // Adds w[k] to the cells at LDS address at[k] in order, in rounds of P
    // (see column_add_rounds).
    template <int P, int K>
    static __device__ __forceinline__ void cells_add(const int (&at)[K], const float (&w)[K]) {
#pragma unroll
        for (int h = 0; h < K; h += P) {
            float v[P];
#pragma unroll
            for (int k = 0; k < P; ++k) v[k] = *(lds_f32*)(smem + at[h + k]);
#pragma unroll
            for (int k = 0; k < P; ++k) {
                float base = v[k];
#pragma unroll
                for (int i = 0; i < k; ++i) base = at[h + i] == at[h + k] ? v[i] : base;
                v[k] = __fadd_rn(base, w[h + k]);
            }
#pragma unroll
            for (int k = 0; k < P; ++k) *(lds_f32*)(smem + at[h + k]) = v[k];
        }
    }

    // A ring's columns of one wave, and the rows of its table that the wave
    // adds to them.  A step's rows are loaded as its spikes come in and added
    // one step later, while the next step's are loaded.
    struct Adder {
        __amdgpu_buffer_rsrc_t rs;
        int col8, row8;                      // byte offset of this lane's entry in a row, bytes of a row
        int pad;                             // the table's row of zeros
        int ring;                            // LDS address of the ring
        unsigned nm, row, bytes;             // this lane's cell of the step added last, from the ring's
                                             // start; bytes of a ring row, of the ring
        bool live;
        Spikes s;                            // the step loaded last, its first PK rows
        uint2 w[PK / KG][KG];

        __device__ __forceinline__ void init(const uint2* tab, int npre, int nq, int S, int ring_at, int j) {
            rs = __builtin_amdgcn_make_buffer_rsrc((void*)tab, (short)0, (npre + 1) * nq * 8, 0x00020000);
            const int jc = min(j, nq - 1);
            col8 = jc * 8;
            row8 = nq * 8;
            pad = npre;
            ring = ring_at;
            row = (unsigned)(nq * 4);
            bytes = (unsigned)S * row;
            nm = (unsigned)(jc * 4) + bytes - row;
            live = j < nq;
            s.total = 0;
#pragma unroll
            for (int k = 0; k < NWM; ++k) s.pre[k] = 0;
#pragma unroll
            for (int g = 0; g < PK / KG; ++g)
#pragma unroll
                for (int k = 0; k < KG; ++k) w[g][k] = make_uint2(0u, 0u);
        }
        // rows of spikes k0 .. k0 + KG of the ids' byte offsets in a vector
        __device__ __forceinline__ void load(int offs, int k0, uint2 (&x)[KG]) const {
#pragma unroll
            for (int k = 0; k < KG; ++k) {
                const auto v = __builtin_amdgcn_raw_buffer_load_b64(rs, col8, __builtin_amdgcn_readlane(offs, k0 + k), 0);
                x[k] = make_uint2((unsigned)v[0], (unsigned)v[1]);
            }
        }
        __device__ __forceinline__ void add(const uint2 (&x)[KG]) const {
            int at[KG];
            float v[KG];
#pragma unroll
            for (int k = 0; k < KG; ++k) {
                const unsigned c = nm + x[k].y;              // c < 2 rings
                at[k] = ring + (int)min(c, c - bytes);
                v[k] = __uint_as_float(x[k].x);
            }
            if (live) cells_add<kRound>(at, v);
        }
        // Loads step n of layer l (n < T), adds step n - 1.
        __device__ __forceinline__ void step(int n, int T, int l) {
            const Spikes last = s;
            // the last step's rows, once they have landed: in registers that are
            // ordinary values to the compiler, with no load to wait for
            uint2 v[PK / KG][KG];
            if (last.total > 0) {
                __builtin_amdgcn_s_waitcnt(kWaitVm0);
#pragma unroll
                for (int g = 0; g < PK / KG; ++g)
#pragma unroll
                    for (int k = 0; k < KG; ++k) {
                        v[g][k] = w[g][k];
                        asm volatile("" : "+v"(v[g][k].x), "+v"(v[g][k].y));
                    }
            }
            s.total = 0;
            if (n < T) spikes_of(n, l, s);
            if (s.total > 0) {
                const int offs = list_ids(s, n, l, 0, pad) * row8;
#pragma unroll
                for (int g = 0; g < PK / KG; ++g)
                    if (g == 0 || s.total > g * KG) load(offs, g * KG, w[g]);
            }
            nm = min(nm + row, nm + row - bytes);            // the cell of step n - 1
            if (last.total > 0) {
#pragma unroll
                for (int g = 0; g < PK / KG; ++g)
                    if (g == 0 || last.total > g * KG) add(v[g]);
                if (last.total > PK) {
#pragma unroll 1
                    for (int r0 = PK; r0 < last.total; r0 += KG) {   // rare: loaded now
                        load(list_ids(last, n - 1, l, r0, pad) * row8, 0, v[0]);
                        add(v[0]);
                    }
                }
            }
        }
    };

    // Scatter wave t: 64 columns of the ring of a LIF -> LIF projection
    // (layers, then projections, then column blocks in order).
    static __device__ void scatter(const CoreFwdArgs& a, int t, int lane) {
        const uint2* far = nullptr;
        int l = 0, npre = 0, nq = 0, S = 1, ring = 0, c0 = 0;
#pragma unroll
        for (int m = 0; m < NL; ++m)
#pragma unroll
            for (int pp = 0; pp < NP; ++pp) {
                if (pp >= a.ly[m].npost) continue;
                const int nb = (a.ly[m].nq[pp] + 63) / 64;
                if (t >= 0 && t < nb) {
                    far = a.role[m].ffar[pp];
                    l = m;
                    npre = a.ly[m].npre[pp];
                    nq = a.ly[m].nq[pp];
                    S = a.ly[m].S[pp];
                    ring = a.ly[m].ring_lds[pp] * 4;
                    c0 = t * 64;
                }
                t -= nb;
            }
        Adder A;
        A.init(far, npre, nq, S, ring, c0 + lane);
        A.nm = min(A.nm - A.row, A.nm - A.row + A.bytes);    // (step -1 is added at step 0)
#pragma unroll 1
        for (int n = 0; n < a.T; ++n) {
            lds_barrier();                                   // the step's spikes are in
            if (S > 2) A.step(n, a.T, l);                    // (else every synapse is near)
        }
    }

    // ---- record wave

    static __device__ void records(const CoreFwdArgs& a, int b, int lane) {
        const int T = a.T, cap = a.cap;
        int cnt[NL], idx[NL];
        unsigned long long mk[NL][NWM];
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            cnt[l] = idx[l] = 0;
#pragma unroll
            for (int k = 0; k < NWM; ++k) mk[l][k] = 0;
        }
#pragma unroll 1
        for (int n = 0; n < T; ++n) {
            lds_barrier();                                   // the step's spikes are in
            const bool mine = (n & 63) == lane;
#pragma unroll
            for (int l = 0; l < NL; ++l) {
                const FwdLayer& y = a.ly[l];
                Spikes s;
                spikes_of(n, l, s);
                // (record indices never pass the capacity; the caller's count
                // stays exact)
                idx[l] = mine ? min(cnt[l], cap) : idx[l];
                if (y.steptab && lane < 2)
                    y.steptab[((size_t)b * T + n) * SNN_STEP_ROW + lane] = lane ? min(cnt[l], cap) : s.total;
                if (s.total == 0) continue;
                const lds_u64* w = (const lds_u64*)(smem + MASK0 + (1 + (n & (D - 1))) * MASKS + l * NWM * 8);
#pragma unroll
                for (int k = 0; k < NWM; ++k) mk[l][k] = mine ? w[k] : mk[l][k];
#pragma unroll 1
                for (int r0 = 0; r0 < s.total; r0 += 64) {
                    const int r = r0 + lane;
                    if (r < s.total) {
                        const int at = list_at(s, n, l, r);
                        const int id = ((const lds_u16*)(smem + LIST0))[at];
                        const float I = ((const lds_f32*)(smem + CUR0))[at];
                        const int pos = cnt[l] + r;
                        if (y.steptab && r < SNN_STEP_IDS) y.steptab[((size_t)b * T + n) * SNN_STEP_ROW + 2 + r] = id;
                        if (pos < cap) {
                            const size_t o = (size_t)b * cap + pos;
                            y.rec_n[o] = id;
                            y.rec_s[o] = n;
                            y.rec_I[o] = I;
                            y.out_step[o] = n;
                            y.out_neuron[o] = id;
                        }
                    }
                }
                cnt[l] += s.total;
            }
            if ((n & 63) == 63 || n == T - 1) {
                const int n0 = n & ~63;
                if (n0 + lane <= n) {
#pragma unroll
                    for (int l = 0; l < NL; ++l) {
                        const FwdLayer& y = a.ly[l];
                        y.rec_idx[(size_t)b * (T + 1) + n0 + lane] = idx[l];
#pragma unroll
                        for (int k = 0; k < NWM; ++k)
                            if (k < a.NW && a.role[l].masks) a.role[l].masks[((size_t)b * T + n0 + lane) * a.NW + k] = mk[l][k];
                    }
                }
#pragma unroll
                for (int l = 0; l < NL; ++l)
#pragma unroll
                    for (int k = 0; k < NWM; ++k) mk[l][k] = 0;
            }
        }
        if (lane == 0) {
#pragma unroll
            for (int l = 0; l < NL; ++l) {
                const FwdLayer& y = a.ly[l];
                y.rec_idx[(size_t)b * (T + 1) + T] = min(cnt[l], cap);
                y.rec_cnt[b] = min(cnt[l], cap);
                y.out_count[b] = cnt[l];
                if (cnt[l] > cap) a.st->overflow = 1;
                atomicAdd(&a.st->layer_spikes[l], (unsigned long long)cnt[l]);
            }
        }
    }

    // ---- readout wave: lane k owns output k

    static __device__ void readout(const CoreFwdArgs& a, int b, int lane) {
        const int T = a.T, C = a.ro_C;
        const bool live = lane < C, sum = a.ro_loss == SNN_LOSS_CE_SUM;
        Adder A;
        A.init(a.ro_far, a.ro_nfeed, C, a.ro_S, a.ro_off, lane);
        A.nm = min(A.nm - A.row, A.nm - A.row + A.bytes);    // (step -1 is added at step 0)
        LiState q{};
        // step n's rows go out, then step n - 1 is finished: its spikes into the
        // ring, the LI step with the arrivals of its cell
#pragma unroll 1
        for (int n = 0; n <= T; ++n) {
            if (n < T) lds_barrier();                        // the step's spikes are in
            A.step(n, T, a.ro_feed);
            if (n == 0) continue;
            float x = 0.0f;
            if (live) {
                lds_f32* c = (lds_f32*)(smem + A.ring + (int)A.nm);
                x = *c;
                *c = 0.0f;
            }
            if (sum)
                li_update<true>(a.alpha, a.beta, a.gamma, n - 1, x, q);
            else
                li_update<false>(a.alpha, a.beta, a.gamma, n - 1, x, q);
        }
        if (!live) return;
        a.z[(size_t)b * C + lane] = sum ? __fmul_rn(a.ro_scale, q.acc) : q.best;
        a.nstar[(size_t)b * C + lane] = sum ? -1 : q.nst;
        a.Vf[(size_t)b * a.nstate + (a.nstate - C) + lane] = q.V;
        a.If[(size_t)b * a.nstate + (a.nstate - C) + lane] = q.I;
    }

    static __device__ void run(const CoreFwdArgs& a) {
        if (a.st->bad_input) return;
        const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const bool dense = a.st->near_post > near_limit(a.NW);
        // head and rings start at zero
        for (int k = tid * 4; k < a.ro_end; k += blockDim.x * 4) *(lds_u32*)(smem + k) = 0u;
        __syncthreads();
        if (wave < a.NW) {
            __builtin_amdgcn_s_setprio(3);                   // the chain of steps runs through these
            if (dense) neurons<true>(a, b, wave, lane); else neurons<false>(a, b, wave, lane);
        } else if (wave < a.NW + a.NS) {
            __builtin_amdgcn_s_setprio(2);
            scatter(a, wave - a.NW, lane);
        } else if (wave == a.NW + a.NS) {
            records(a, b, lane);
        } else {
            __builtin_amdgcn_s_setprio(2);
            readout(a, b, lane);
        }
    }
};

// Most waves of a workgroup: fewer than 16 leave a wave more registers.
constexpr int split_waves(int nl, int nwm) { return nl == 1 ? (nwm == 4 ? 10 : 16) : 12; }

template <int NL, int NP, int NWM>
__global__ void __launch_bounds__(64 * split_waves(NL, NWM)) forward_split_kernel(CoreFwdArgs a) {
    FwdSplit<NL, NP, NWM>::run(a);
}

struct SplitFn {
    const void* f;
    int head, waves;
};

// The instantiation for n_lif LIF layers with at most np LIF-post projections
// each and nw neuron waves; {NULL}: none.
SplitFn split_kernel(int n_lif, int np, int nw) {
#define SNN_FS(NL, NP, M) SplitFn{(const void*)forward_split_kernel<NL, NP, M>, FwdSplit<NL, NP, M>::HEAD, split_waves(NL, M)}
    if (n_lif == 1 && np == 1) return nw <= 4 ? SNN_FS(1, 1, 4) : nw <= 8 ? SNN_FS(1, 1, 8) : SplitFn{nullptr, 0, 0};
    if (n_lif == 2 && np == 1 && nw <= 4) return SNN_FS(2, 1, 4);
#undef SNN_FS
    return SplitFn{nullptr, 0, 0};
}

}  // namespace

// LDS bytes of the split core before its rings, and its most waves; -1: it does
// not serve the network.
int forward_split_head(int n_lif, int np, int nw, int* waves) {
    const SplitFn f = split_kernel(n_lif, np, nw);
    *waves = f.waves;
    return f.f ? f.head : -1;
}

const void* forward_split_fn(int n_lif, int np, int nw) { return split_kernel(n_lif, np, nw).f; }

hipError_t launch_split_tables(const SplitTables& a, hipStream_t s) {
    int blocks = a.rowblocks;
    for (int p = 0; p < a.np; ++p) blocks += (a.pr[p].nq + 63) / 64;
    hipLaunchKernelGGL(split_tables_kernel, dim3(blocks), dim3(512), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_forward_split(const CoreFwdArgs& a, int n_lif, int np, size_t lds, hipStream_t s) {
    const SplitFn f = split_kernel(n_lif, np, a.NW);
    const int waves = a.NW + a.NS + 1 + (a.ro_C > 0 ? 1 : 0);
    int ns = 0;
    for (int l = 0; l < n_lif; ++l) {
        if (a.ly[l].npost > np || a.role[l].nrec > np || a.ly[l].n > 64 * a.NW) return hipErrorInvalidValue;
        for (int pp = 0; pp < a.ly[l].npost; ++pp) {
            if (a.ly[l].ring_lds[pp] * 4 < f.head) return hipErrorInvalidValue;
            ns += (a.ly[l].nq[pp] + 63) / 64;
        }
    }
    if (!f.f || ns != a.NS || waves > f.waves || a.ro_C > 64 || (size_t)a.ro_end > lds) return hipErrorInvalidValue;
    CoreFwdArgs arg = a;
    void* args[] = {&arg};
    return hipLaunchKernel(f.f, dim3(a.B), dim3(64 * waves), args, lds, s);
}

hipError_t set_forward_split_lds_limits(size_t bytes, int* bad) {
    static const int cases[3][3] = {{1, 1, 4}, {1, 1, 8}, {2, 1, 4}};
    for (int k = 0; k < 3; ++k) {
        const hipError_t e = hipFuncSetAttribute(split_kernel(cases[k][0], cases[k][1], cases[k][2]).f,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e != hipSuccess) {
            if (bad) *bad = k;
            return e;
        }
    }
    return hipSuccess;
}
