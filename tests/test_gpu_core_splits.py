"""The forms the LIF cores take, at the sizes where their splits can go wrong,
against the oracle: the forward bit for bit, every dW and dD element within
1e-6 + 1e-4 |ref| of its fp64 definition.

* Recurrent layers: synapses of the smallest delays are kept out of the delay
  rings in lists of fixed length.  Delays all zero or of 0 and 1 (every list
  over its length: the general form), of a few steps (lists between the
  registers and the length), of 20 and 50 (short lists); widths of one, two,
  four and five wavefronts with remainders, two layers, and cluster mode.
* Feed-forward layers: blocks of 16 steps forward and 64 backward (trials of one
  step, one short, full and one over) and 1 to 1024 neurons, with a
  leaky-integrator readout or first-spike loss on the layer itself.
* Few samples with long trials: the input scan in segments, with an empty sample
  and delays longer than a segment.
"""
import dataclasses

import numpy as np
import pytest

from workloads import LOSS_DMSE, Workload
from workloads.configs import CONFIGS, projections
from workloads.generators import labels

from .gpu_util import assert_backward_close, assert_forward_bitexact, run_gpu, run_oracle

N_IN = 40


def _net(layers, T, B, high, d_in=12, drive=None, loss=None, rate=0.04, seed=7, empty=None):
    """A workload of its own weights: high is the upper end of the LIF -> LIF delays."""
    pr = projections(layers)
    lif = lambda l: layers[l][1] == 1
    rng = np.random.default_rng(seed)
    rec = max(1, int(round(high)))
    kw = dict(name="core-splits", T=T, B=B, layers=layers, dmse_delta=1.0,
              delay_range=tuple(rec if a > 0 and lif(q) else d_in for a, q in pr))
    if loss is not None:
        kw["loss"] = loss
    cfg = dataclasses.replace(CONFIGS[4], **kw)
    steps, neurons, off = [], [], [0]
    for b in range(B):
        s, i = np.nonzero(rng.random((T, N_IN)) < (0.0 if b == empty else rate))
        steps.append(s)
        neurons.append(i)
        off.append(off[-1] + s.size)
    W, D = [], []
    for p, (a, q) in enumerate(pr):
        shape = (layers[a][0], layers[q][0])
        mean, sd = {True: (drive or 0.55, 0.2), False: (0.0, 0.3)}[a == 0]
        if a > 0 and lif(q):
            mean, sd = (0.0, 0.3 / np.sqrt(shape[0])) if a == q else (6.0 / shape[0], 3.0 / shape[0])
        W.append(rng.normal(mean, sd, shape).astype(np.float32))
        hi = high if a > 0 and lif(q) else d_in
        D.append(rng.uniform(0.0, hi, shape).astype(np.float32))
    return Workload(cfg, B, T, np.array(off, np.int32), np.concatenate(steps).astype(np.int32),
                    np.concatenate(neurons).astype(np.int32), W, D, labels(cfg, B))


def _check(wl, least=1.0, flags=0):
    orc = run_oracle(wl, modes=("f64",))
    per = orc["fwd"].count.sum(axis=1) / (wl.B * np.array([n for n, k, _ in wl.cfg.layers if k == 1]))
    print(f"[splits] {wl.cfg.layers} T={wl.T} B={wl.B} spikes per neuron {per}", flush=True)
    assert per.min() >= least                    # every layer carries spikes
    gpu = run_gpu(wl, flags=flags)
    assert gpu["rc"] == 0
    assert_forward_bitexact(gpu, orc, wl)
    assert np.allclose(gpu["loss"], orc["loss"], rtol=1e-6, atol=1e-7)
    assert_backward_close(gpu, orc)


def _lif(*n, out=5, rec=1):
    return ((N_IN, 0, 0),) + tuple((k, 1, rec) for k in n) + ((out, 2, 0),)


REC = [(w, h, f) for w in ((70,), (256,)) for h in (0.0, 1.4, 6.0, 20.0, 50.0) for f in (0, 1)] + \
      [((33,), 1.4, 0), ((300,), 20.0, 0), ((300,), 1.4, 0), ((64, 130), 20.0, 0), ((64, 130), 1.4, 0),
       ((64, 130), 6.0, 1), ((64, 130), 1.4, 1)]


@pytest.mark.gpu
@pytest.mark.parametrize("widths,high,cluster", REC)
def test_recurrent_cores_over_delay_ranges(widths, high, cluster):
    import paper_2501_07331_amd as snn
    _check(_net(_lif(*widths), 90, 3, high), flags=snn.SNN_FLAG_CLUSTER if cluster else 0)


@pytest.mark.gpu
@pytest.mark.parametrize("widths", [(64, 130), (256, 100)])
def test_two_feed_forward_layers(widths):
    """One LIF -> LIF projection, none recurrent."""
    _check(_net(_lif(*widths, rec=0), 90, 3, 20.0))


@pytest.mark.gpu
@pytest.mark.parametrize("n,T", [(1, 64), (63, 65), (64, 63), (65, 17), (65, 16), (65, 15), (130, 130), (1024, 80)])
def test_feed_forward_core_block_edges(n, T):
    _check(_net(_lif(n, rec=0), T, 3, 1.0, d_in=min(12, T - 1), drive=1.2), least=0.1)


@pytest.mark.gpu
@pytest.mark.parametrize("n,T", [(1, 1), (5, 2), (3, 16)])
def test_feed_forward_core_shortest_trials(n, T):
    _check(_net(_lif(n, rec=0), T, 2, 1.0, d_in=1, drive=4.0, rate=0.3), least=0.0)


@pytest.mark.gpu
@pytest.mark.parametrize("n,T", [(5, 33), (70, 129)])
def test_first_spike_loss_on_the_first_layer(n, T):
    _check(_net(((N_IN, 0, 0), (n, 1, 0)), T, 4, 1.0, drive=1.2, loss=LOSS_DMSE), least=0.5)


@pytest.mark.gpu
@pytest.mark.parametrize("T,B,d_in", [(400, 2, 12), (400, 1, 150), (160, 3, 149), (33, 2, 5)])
def test_input_scan_in_segments(T, B, d_in):
    _check(_net(_lif(70), T, B, 20.0, d_in=d_in, rate=0.02, empty=1 if B > 1 else None), least=0.3)
