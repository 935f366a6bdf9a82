"""The synapse part of a source block in one launch, where it can go wrong:
many chunks and one, chunks without rows, more rows than are staged at once,
more entries than a window, segments longer than the direct map's, rows forced
and delivered in the same block, rows that are only delivered (exc -> exc
plasticity), the widest slices, blocks of one step and blocks cut short. Equal
to the step-by-step path bit for bit."""

import pytest

import workloads as wl
from workloads.presets import PLASTIC_EXC_EXC
from paper_2107_04092_amd import snn

from gpu_common import gpu_net, log, same_state

pytestmark = pytest.mark.gpu
LDS = snn.SNN_DELIVER_LDS_SLICE

CASES = [
    # preset overrides, slice width, chunks, extra config
    (dict(n=64, p_or_fanout=50, p_fire=0.05), 64, 1, dict()),
    (dict(n=513, p_or_fanout=300, p_fire=0.02), 512, 2, dict(history_bits=128)),
    (dict(n=2000, p_or_fanout=900, p_fire=0.01), 4096, 3, dict()),
    (dict(n=30000, p_or_fanout=40, p_fire=0.3), 2048, 1, dict()),
    (dict(n=6000, p_or_fanout=3000, p_fire=0.05), 2048, 2, dict(compressed_targets=0)),
    (dict(n=9001, n_exc=4001, p_or_fanout=200, p_fire=0.02, plastic=PLASTIC_EXC_EXC), 1024, 1,
     dict(history_bits=128)),
    # one in seven rows of a block both forced and delivered in it
    (dict(n=20011, p_or_fanout=100, p_fire=0.008), 1024, 4, dict()),
    (dict(n=20011, p_or_fanout=100, p_fire=0.008), 640, 1, dict(plastic_blocks=1)),
    (dict(n=20011, p_or_fanout=64, p_fire=0.004), 2048, 2,
     dict(plastic_blocks=2, history_bits=128)),
    (dict(n=100003, p_or_fanout=20, p_fire=0.005), 2048, 2, dict(stdp_filter=3)),
    (dict(n=5000, p_or_fanout=100, p_fire=0.02), 512, 1, dict(plasticity_algorithm=1)),
    # hardly any row is forced: seven eighths of the slots deliver
    (dict(n=6251, p_or_fanout=200, p_fire=0.1), 64, 4, dict()),
    (dict(n=6251, p_or_fanout=200, p_fire=0.1), 64, 1, dict(history_bits=128)),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%d-w%d-c%d" % (c[0]["n"], c[1], c[2]))
def test_run_equals_step_by_step(case):
    kw, width, chunks, cfg = case
    p = wl.preset("stress", **kw)
    log("source run: %s width %d %s" % (kw, width, cfg))
    a = gpu_net(p, slice_width=width, spike_chunks=chunks, **cfg)
    b = gpu_net(p, slice_width=width, spike_chunks=chunks, **dict(cfg, plastic_blocks=-1))
    assert a.graph()["block_steps"] > 0
    for k in (1, 2, 70, 17, 131):
        a.step(k, LDS)
        b.step(k, LDS)
        same_state(a, b, "%d steps" % k)
    a.flush_plasticity()
    b.flush_plasticity()
    same_state(a, b, "flush")


WIDE = [
    # beyond the ranges of the common form: slices of more than 4096 targets,
    # more neurons than the recency bitmap holds, no bitmap asked for, no edges
    (dict(n=20011, p_or_fanout=150, p_fire=0.008), 4160, 1, dict(history_bits=128)),
    (dict(n=20011, p_or_fanout=150, p_fire=0.008), 6528, 2, dict(compressed_targets=0)),
    (dict(n=50000, p_or_fanout=64, p_fire=0.01), 4608, 1, dict()),
    (dict(n=784001, p_or_fanout=6, p_fire=0.005), 2048, 1, dict()),
    (dict(n=420001, p_or_fanout=10, p_fire=0.005), 2048, 1, dict(stdp_filter=3)),
    (dict(n=3001, p_or_fanout=0, p_fire=0.01), 512, 2, dict()),
]


@pytest.mark.parametrize("case", WIDE, ids=lambda c: "%d-w%d" % (c[0]["n"], c[1]))
def test_wide_form_equals_step_by_step(case):
    kw, width, chunks, cfg = case
    p = wl.preset("stress", **kw)
    log("source run, wide: %s width %d %s" % (kw, width, cfg))
    a = gpu_net(p, slice_width=width, spike_chunks=chunks, **cfg)
    b = gpu_net(p, slice_width=width, spike_chunks=chunks, **dict(cfg, plastic_blocks=-1))
    assert a.graph()["block_steps"] > 0
    for k in (1, 70, 17):
        a.step(k, LDS)
        for _ in range(k):
            b.update_neurons()
            b.update_plasticity()
            b.deliver_spikes(LDS)
            b.advance()
        same_state(a, b, "%d steps" % k)
    # the launches are those of blocks: two for 16 steps are recorded as one
    # neuron part, far below 16 neuron updates of the step-by-step path
    for net in (a, b):
        net.record_kernel_times(64)
        net.step(64, LDS)
    (ta, _), (tb, _) = a.kernel_times(), b.kernel_times()
    log("neuron part per step: %.2f us in blocks, %.2f us step by step" % (
        ta["neuron"] * 1e3, tb["neuron"] * 1e3))
    assert ta["neuron"] < tb["neuron"]


def test_more_edges_than_32_bits_count():
    """4.32 billion synapses (35 GB): the first edges of the last rows take more
    than 32 bits."""
    import torch
    p = wl.preset("stress", n=360001, p_or_fanout=12000, p_fire=0.0005)
    log("source run: %d rows of 12,000" % p.n)
    nets = [gpu_net(p, slice_width=2048, spike_chunks=1, plastic_blocks=b) for b in (0, -1)]
    assert nets[0].n_edges > 1 << 32 and nets[0].graph()["block_steps"] > 0
    for k in (17, 50):
        for net in nets:
            net.step(k, LDS)
        same_state(*nets, "%d steps" % k, weights=False)
        wa, wb = (net.graph()["w"].view(torch.int32) for net in nets)
        step = 1 << 28
        for at in range(0, wa.numel(), step):
            assert torch.equal(wa[at:at + step], wb[at:at + step]), at
        log("  %d steps: weights equal" % k)


def test_a_call_of_one_step_is_a_step():
    """Single-step calls between longer ones: the same states, in the launches
    of the step-by-step path (a block of one step takes twice the time)."""
    import torch
    p = wl.preset("stress", n=20011, p_or_fanout=100)
    a = gpu_net(p, slice_width=1024, spike_chunks=2)
    b = gpu_net(p, slice_width=1024, spike_chunks=2, plastic_blocks=-1)
    assert a.graph()["block_steps"] == 16
    for k in (1, 5, 1, 1, 33, 1, 64, 1):
        a.step(k, LDS)
        b.step(k, LDS)
        same_state(a, b, "%d steps" % k)

    def us(net):
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        torch.cuda.synchronize()
        ev[0].record(net.stream)
        for _ in range(100):
            net.step(1, LDS)
        ev[1].record(net.stream)
        torch.cuda.synchronize()
        return ev[0].elapsed_time(ev[1]) * 10

    ta, tb = (min(us(net) for _ in range(5)) for net in (a, b))
    log("one step per call: %.1f us, step by step %.1f us" % (ta, tb))
    assert ta < 1.25 * tb  # (a block of one step: 1.56 times)
