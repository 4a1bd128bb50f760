// The cores of libsnn for a LIF layer that feeds no LIF layer (gfx950, wave64):
// one layer, not recurrent, between the inputs and the readout (or the output
// layer itself).  Its neurons do not reach each other within a trial, so the
// steps of a wave's 64 neurons are a serial loop of a few instructions with no
// exchange between waves: the forward meets at a barrier every kFfBlock steps
// to place the spike records, the backward at none.  (With the recurrent
// networks' core, two barriers a step, 4-200-3 at 600 steps and batch 64 took
// 303 us forward and 218 us backward; now 88 and 56, with 54 for the readout,
// then a kernel of its own.)
#include "snn_device.h"

namespace {

constexpr int kFfBlock = 16;

// ------------------------------------------------------------------ forward

// One workgroup per sample, lane j of wave w owns neuron 64 w + j.  A block of
// steps: dynamics, every step's ballot and I- held in registers, the input
// arrival of a step reloaded for the next block as soon as it is used; the
// block's masks go to LDS; after a barrier every wave knows the records before
// each of its spikes (lane u: step u) and writes its own.  All fp32, in the
// order of the definition.
__global__ void __launch_bounds__(1024) forward_ff_kernel(CoreFwdArgs a) {
    if (a.st->bad_input) return;
    typedef __attribute__((address_space(3))) unsigned long long lds_u64;
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, T = a.T, NW = a.NW, cap = a.cap;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const FwdLayer& y = a.ly[0];
    const bool live = tid < y.n;
    const size_t r0 = (size_t)b * cap;
    gptr<const float> ain = (gptr<const float>)(a.A_in + (size_t)b * T * a.n1 + min(tid, a.n1 - 1));
    // this lane's mask word of the block at step 0 (in vector registers: as an
    // argument it was loaded in every block, 90 us against 85)
    gptr<unsigned long long> mrow = (gptr<unsigned long long>)(a.role[0].masks + ((size_t)b * T + lane) * NW + wave);
    asm volatile("" : "+v"(mrow));
    float V = 0.0f, I = 0.0f;
    int own = 0, cnt = 0;
    float x[kFfBlock];
#pragma unroll
    for (int u = 0; u < kFfBlock; ++u) x[u] = ain[(size_t)min(u, T - 1) * a.n1];
#pragma unroll 1
    for (int n0 = 0; n0 < T; n0 += kFfBlock) {
        float Im[kFfBlock];
        unsigned long long m[kFfBlock], mine = 0;
#pragma unroll
        for (int u = 0; u < kFfBlock; ++u) {
            const bool in = n0 + u < T;                      // (past the trial nothing changes)
            const float gi = __fmul_rn(a.gamma, I);
            const float Vm = __fmaf_rn(a.alpha, V, gi);
            const float Id = __fmul_rn(a.beta, I);
            const bool spk = in && live && Vm >= a.theta;
            m[u] = __ballot(spk);
            mine = lane == u ? m[u] : mine;
            Im[u] = Id;
            const float V2 = spk ? 0.0f : Vm, I2 = __fadd_rn(Id, x[u]);
            V = in ? V2 : V;
            I = in ? I2 : I;
            x[u] = ain[(size_t)min(n0 + kFfBlock + u, T - 1) * a.n1];
        }
        // masks of the block, two blocks deep (the next block's are written while
        // a slower wave still reads these)
        lds_u64* mk = (lds_u64*)smem + ((n0 / kFfBlock) & 1) * NW * kFfBlock;
        if (lane < kFfBlock) {
            mk[wave * kFfBlock + lane] = mine;
            if (n0 + lane < T) mrow[(size_t)n0 * NW] = mine;
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);                  // lgkmcnt(0): LDS only
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        int before = 0, tot = 0;                             // lane u: spikes at step u of lower waves, of all
        for (int w = 0; w < NW; ++w) {
            const int c = __popcll(mk[w * kFfBlock + (lane & (kFfBlock - 1))]);
            before += w < wave ? c : 0;
            tot += c;
        }
        int incl = tot;
#pragma unroll
        for (int d = 1; d < kFfBlock; d <<= 1) {
            const int v = __shfl_up(incl, d, kFfBlock);
            incl += (lane & (kFfBlock - 1)) >= d ? v : 0;
        }
        const int start = cnt + incl - tot;                  // first record of step u
        // (record indices never pass the capacity; the caller's count stays
        // exact)
        if (wave == 0 && lane < kFfBlock && n0 + lane < T)
            y.rec_idx[(size_t)b * (T + 1) + n0 + lane] = min(start, cap);
        cnt += __builtin_amdgcn_readlane(incl, kFfBlock - 1);
        const int base = start + before;
#pragma unroll
        for (int u = 0; u < kFfBlock; ++u) {
            if (m[u] == 0) continue;
            if ((m[u] >> lane) & 1ull) {
                ++own;
                const int pos = __builtin_amdgcn_readlane(base, u) + lanes_below(m[u]);
                if (pos < cap) {
                    y.rec_n[r0 + pos] = tid;
                    y.rec_s[r0 + pos] = n0 + u;
                    y.rec_I[r0 + pos] = Im[u];
                    y.out_step[r0 + pos] = n0 + u;
                    y.out_neuron[r0 + pos] = tid;
                }
            }
        }
    }
    if (live) {
        a.Vf[(size_t)b * a.nstate + a.soff[0] + tid] = V;
        a.If[(size_t)b * a.nstate + a.soff[0] + tid] = I;
        // integer sums over the samples: exact in any order
        if (y.ncount && own) atomicAdd(&y.ncount[tid], own);
    }
    if (tid == 0) {
        y.rec_idx[(size_t)b * (T + 1) + T] = min(cnt, cap);
        y.rec_cnt[b] = min(cnt, cap);
        y.out_count[b] = cnt;
        if (cnt > cap) a.st->overflow = 1;
        atomicAdd(&a.st->layer_spikes[0], (unsigned long long)cnt);
    }
}

// ------------------------------------------------------------------ backward

// lambda of the layer over reverse time (fp64): the jump numerators are known
// before (the readout's and the losses' terms: no LIF posts), so a wave runs
// alone: in blocks of 64 steps, lane k holds step k's mask word and the index of
// its first record of this wave; the data of the next spiking step's jumps is
// loaded while the steps before it run.
__global__ void __launch_bounds__(64) backward_ff_kernel(CoreBwdArgs a) {
    const int NW = a.NW, b = blockIdx.x / NW, wave = blockIdx.x - b * NW, lane = threadIdx.x, T = a.T;
    const BwdLayer& y = a.ly[0];
    const int j = wave * 64 + lane, jc = min(j, y.n - 1);
    const bool live = j < y.n;
    const unsigned long long* masks = y.masks + (size_t)b * T * NW;
    const int* idx = y.rec_idx + (size_t)b * (T + 1);
    const size_t r0 = (size_t)b * a.cap;
    double lv = 0.0, lI = 0.0;
    int deg = 0;
    double2* tr = a.traj + ((size_t)b * T + (T - 1)) * a.lif_total + jc;
    auto free_steps = [&](int g) {
        // (at step T - 1 the adjoints are zero and stay zero)
#pragma unroll 1
        for (; g > 0; --g) {
            const double v = lv;
            lI = __dadd_rn(__dmul_rn(a.beta, lI), __dmul_rn(a.cc, v));
            lv = __dmul_rn(a.alpha, v);
            if (live) *tr = make_double2(lI, __dsub_rn(lI, lv));
            tr -= a.lif_total;
        }
    };
    int n = T;                                               // steps below n are to be run
#pragma unroll 1
    for (int n0 = (T - 1) & ~63; n0 >= 0; n0 -= 64) {
        const int k = min(n0 + lane, T - 1);
        unsigned long long own = 0;
        int base = idx[k];
        for (int w = 0; w <= wave; ++w) {
            const unsigned long long m = masks[(size_t)k * NW + w];
            base += w < wave ? __popcll(m) : 0;
            own = m;
        }
        own = n0 + lane < T ? own : 0;
        unsigned long long act = __ballot(own != 0);
        float I = 0.0f;
        double A = 0.0;
        unsigned long long m = 0;
        int s = -1;
        // the step's I- and numerators of the top active step of act
        auto fetch = [&]() {
            s = act ? 63 - __builtin_clzll(act) : -1;
            if (s < 0) return;
            const unsigned lo = __builtin_amdgcn_readlane((unsigned)own, s);
            const unsigned hi = __builtin_amdgcn_readlane((unsigned)(own >> 32), s);
            m = ((unsigned long long)hi << 32) | lo;
            const size_t r = r0 + __builtin_amdgcn_readlane(base, s) + lanes_below(m);
            if ((m >> lane) & 1ull) {
                I = y.recI[r];
                A = y.A2 ? y.A2[r] : 0.0;
            }
            act &= ~(1ull << s);
        };
        fetch();
#pragma unroll 1
        while (s >= 0) {
            const unsigned long long ms = m;
            const int sn = n0 + s;
            free_steps(n - sn);
            n = sn;
            const float Is = I;
            const double As = A;
            if ((ms >> lane) & 1ull) {
                // tau_m dV/dt just before the crossing is I- - theta (V- = theta)
                const double den = __dsub_rn((double)Is, a.theta);
                if (den > 0.0)
                    lv = __dadd_rn(lv, __dadd_rn(__dmul_rn(a.theta, lv), As) / den);
                else
                    ++deg;
            }
            fetch();
        }
        free_steps(n - n0);
        n = n0;
    }
    if (deg) atomicAdd(&a.st->degenerate, (unsigned long long)deg);
}

}  // namespace

hipError_t launch_forward_ff(const CoreFwdArgs& a, hipStream_t s) {
    if (a.NW < 1 || a.NW > 16 || a.ly[0].n > 64 * a.NW || a.ly[0].npost != 0) return hipErrorInvalidValue;
    const size_t lds = (size_t)2 * a.NW * kFfBlock * sizeof(unsigned long long);
    hipLaunchKernelGGL(forward_ff_kernel, dim3(a.B), dim3(64 * a.NW), lds, s, a);
    return hipGetLastError();
}

hipError_t launch_backward_ff(const CoreBwdArgs& a, hipStream_t s) {
    if (a.NW < 1 || a.NW > 16 || a.ly[0].n > 64 * a.NW || a.ly[0].npost != 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(backward_ff_kernel, dim3(a.B * a.NW), dim3(64), 0, s, a);
    return hipGetLastError();
}
