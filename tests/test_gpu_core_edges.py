"""The split LIF cores where their waves run apart the farthest, against the
oracle: the forward bit for bit, every dW and dD element within 1e-6 + 1e-4
|ref| of its fp64 definition, finite, and the same bits in a second call."""
import dataclasses

import numpy as np
import pytest

from workloads import LOSS_DMSE
from workloads.configs import projections

from .gpu_util import assert_backward_close, assert_forward_bitexact, run_gpu, run_oracle
from .test_gpu_core_splits import N_IN, _lif, _net


def _later(wl, steps):
    """The same trials after `steps` silent steps."""
    return dataclasses.replace(wl, cfg=dataclasses.replace(wl.cfg, T=wl.T + steps), T=wl.T + steps,
                               in_step=(wl.in_step + steps).astype(np.int32))


def _check(wl, silent=0, least=1.0, **kw):
    orc = run_oracle(wl, modes=("f64",))
    per = orc["fwd"].count.sum(axis=1) / (wl.B * np.array([n for n, k, _ in wl.cfg.layers if k == 1]))
    first = min(int(orc["fwd"].step[l, b, 0]) for l in range(len(per)) for b in range(wl.B)
                if orc["fwd"].count[l, b])
    print(f"[edges] {wl.cfg.layers} T={wl.T} B={wl.B} spikes per neuron {per}, first at {first}", flush=True)
    assert per.min() >= least and first >= silent
    gpu = run_gpu(wl, **kw)
    assert gpu["rc"] == 0
    assert_forward_bitexact(gpu, orc, wl)
    assert np.allclose(gpu["loss"], orc["loss"], rtol=1e-6, atol=1e-7)
    assert all(np.isfinite(x).all() for x in gpu["dW"] + gpu["dD"])
    assert_backward_close(gpu, orc)
    again = run_gpu(wl, **kw)
    for x, y in zip(gpu["dW"] + gpu["dD"], again["dW"] + again["dD"]):
        assert np.array_equal(x.view(np.uint32), y.view(np.uint32)), "a second call differs"


@pytest.mark.gpu
@pytest.mark.parametrize("widths,high", [((100,), 4.0), ((100,), 6.0), ((130,), 8.0), ((256,), 1.0), ((70, 100), 6.0)])
def test_steps_past_the_first_spikes(widths, high):
    """More silent steps at the start of every trial than an adjoint ring has
    rows, so that in reverse time the waves run past the last spikes' row while
    another one may still read it; neurons with more synapses of slot 0 than
    registers, and (1.0) with more than a list holds."""
    rows = int(round(high)) + 1
    _check(_later(_net(_lif(*widths), 90, 3, high), 5 * rows), silent=5 * rows)


@pytest.mark.gpu
@pytest.mark.parametrize("n,out,rec", [(200, 3, 0), (200, 3, 1), (70, 5, 0), (70, 5, 1), (64, 130, 0), (33, 1, 0)])
def test_hidden_layer_and_first_spike_output(n, out, rec):
    """A spiking output layer, which feeds no LIF layer: its jumps have no terms
    of slot 0, whatever the LDS holds."""
    _check(_net(((N_IN, 0, 0), (n, 1, rec), (out, 1, 0)), 120, 4, 20.0, loss=LOSS_DMSE))


@pytest.mark.gpu
def test_upper_layer_that_is_not_recurrent():
    """Two hidden layers, the lower one recurrent."""
    _check(_net(((N_IN, 0, 0), (100, 1, 1), (40, 1, 0), (5, 2, 0)), 90, 3, 6.0))


@pytest.mark.gpu
def test_overflowed_currents_are_not_degenerate_jumps():
    """Weights whose sums overflow: the neuron's current is infinite and it spikes
    at every step, with jumps that change nothing and are not counted as skipped;
    the gradients of the other neurons' synapses are as ever."""
    wl = _net(_lif(70), 90, 3, 20.0)
    wl.W[0][:, 0] = 3e38
    orc = run_oracle(wl, modes=("f64",))
    assert np.isinf(orc["fwd"].I_final).any()
    gpu = run_gpu(wl)
    assert_forward_bitexact(gpu, orc, wl)
    dW64, dD64, deg = orc["f64"]
    print(f"[edges] skipped jumps: {gpu['stats']['degenerate_jumps']}, oracle {deg}", flush=True)
    assert gpu["stats"]["degenerate_jumps"] == deg
    for g, r in zip(gpu["dW"] + gpu["dD"], dW64 + dD64):
        g, r = np.asarray(g, np.float64)[:, 1:], r[:, 1:]
        assert np.isfinite(r).all() and (np.abs(g - r) <= 1e-6 + 1e-4 * np.abs(r)).all()


@pytest.mark.gpu
@pytest.mark.parametrize("widths,high", [((64, 130), 1.0), ((256, 100), 1.0), ((256, 100), 6.0), ((33, 33), 0.0)])
def test_near_synapses_between_feed_forward_layers(widths, high):
    """Two layers, one projection between them, its smallest delays in lists over
    their length (taken from the weight rows) and within it."""
    _check(_net(_lif(*widths, rec=0), 90, 3, high))


@pytest.mark.gpu
@pytest.mark.parametrize("widths", [(64,), (200,), (300,)])
@pytest.mark.parametrize("near", [15, 16, 17, 24, 25, 28, 29, 32, 33])
def test_one_neuron_with_a_list_at_its_limits(widths, near):
    """One neuron with this many recurrent synapses of slots 0 and 1 among longer
    ones: lists that fill the registers, pass them, and pass what is taken from
    lists at all."""
    wl = _net(_lif(*widths), 90, 2, 6.0)
    p = projections(wl.cfg.layers).index((1, 1))
    wl.D[p][:] = np.float32(4.0)
    wl.D[p][:near, 3] = np.arange(near, dtype=np.float32) % 2
    _check(wl)


@pytest.mark.gpu
@pytest.mark.parametrize("layers,B,high", [
    (_lif(33), 1300, 6.0), (_lif(130), 520, 6.0), (_lif(256), 520, 1.0), (_lif(70), 1030, 6.0),
    (_lif(33, 40), 1030, 6.0), (((N_IN, 0, 0), (70, 1, 0), (3, 1, 0)), 1030, 6.0), (_lif(300), 520, 1.0),
    (_lif(512), 3, 1.0), (_lif(512), 3, 20.0), (_lif(200), 140, 1.0), (_lif(200), 140, 15.0)])
def test_batches_of_several_samples_a_cu(layers, B, high):
    """More samples than compute units, where the general cores take over from the
    split ones one after the other, and the widest layer that the split backward
    core serves with its slot-0 synapses in the lists and past them; a layer with
    short delays, on more than half the units, to either side of its rule."""
    loss = LOSS_DMSE if layers[-1][1] == 1 else None
    _check(_net(layers, 24, B, high, d_in=3, drive=1.0, rate=0.1, loss=loss), least=0.2)


@pytest.mark.gpu
@pytest.mark.parametrize("T,B", [(1023, 1), (1024, 1), (5000, 1), (3000, 3)])
def test_long_trials_are_validated_to_their_last_event(T, B):
    """Few samples with long trials, whose events and steps several workgroups
    share; an event out of order or range anywhere is refused."""
    import paper_2501_07331_amd as snn
    wl = _net(_lif(5, rec=0), T, B, 1.0, drive=0.35, rate=0.01)
    _check(wl)
    n = len(wl.in_step)
    for at in (0, n // 3, n - 1):
        for what in ("in_step", "in_neuron"):
            bad = dataclasses.replace(wl, **{what: getattr(wl, what).copy()})
            getattr(bad, what)[at] = T if what == "in_step" else N_IN
            with pytest.raises(snn.SNNError):
                run_gpu(bad, backward=False)


@pytest.mark.gpu
def test_device_memory_of_a_handle():
    """A record slot costs a handle its record (12 bytes), its grouped step (2) and
    its readout jump term (8); a step the arrivals, the trajectories, the spike
    masks and two indices: nothing beside them that only one core uses."""
    import torch
    import paper_2501_07331_amd as snn
    B, n, C = 256, 256, 20

    def used(T, cap):
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        net = snn.Network([(100, 0, 0), (n, 1, 1), (C, 2, 0)], 20.0, 5.0, 1.0, 1.0, 50, B, T, snn.SNN_LOSS_CE_SUM,
                          1.0 / T, cap, proj_max_delay=[50, 50, 50])
        x = free - torch.cuda.mem_get_info()[0]
        net.close()
        return x

    used(100, 64)
    slack = 24 << 20                                     # allocations in steps of 2 MiB
    base = used(500, 64)
    a, b = used(500, 64 * n) - base, used(1000, 64) - base
    per_record, per_step = 12 + 2 + 8, 4 * n + 16 * (n + C) + 8 * n // 64 + 8
    print(f"[edges] bytes a record {a / (B * 64 * (n - 1))}, a step {b / (B * 500)}", flush=True)
    assert a <= per_record * B * 64 * (n - 1) + slack
    assert b <= per_step * B * 500 + slack
