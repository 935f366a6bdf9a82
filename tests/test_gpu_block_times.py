"""Recorded kernel times: of the launches that an unrecorded call makes (fused
passes with fewer workgroups per slice than configured among them); and of
source blocks: a launch of up to 16 steps counts for as many, so the means are
per step whatever the block lengths, and a recording that ends inside a call
ends with a block."""

import pytest

import workloads as wl
from paper_2107_04092_amd import snn

from gpu_common import gpu_net, log, same_state, torch_mod

pytestmark = pytest.mark.gpu
LDS = snn.SNN_DELIVER_LDS_SLICE


@pytest.mark.parametrize("steps", [1, 16, 20, 37])
def test_source_block_times_are_per_step(steps):
    torch = torch_mod()
    p = wl.preset("stress", n=60001, p_or_fanout=333)
    net = gpu_net(p)
    assert net.graph()["block_steps"] == 16
    net.step(64, LDS)
    net.record_kernel_times(steps)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    a.record(net.stream)
    net.step(steps, LDS)
    b.record(net.stream)
    torch.cuda.synchronize()
    t, recorded = net.kernel_times()
    log("%d steps: %s, %.3f ms in all" % (steps, t, a.elapsed_time(b)))
    assert recorded == steps
    # the kernels run one after another inside the interval, so their times
    # add up to no more than it (0.5 us per event for the clocks' resolution)
    kernels = (t["neuron"] + t["delivery"]) * steps
    assert 0 < kernels <= a.elapsed_time(b) + 0.002


def test_recording_that_ends_inside_a_call():
    p = wl.preset("stress", n=9001, p_or_fanout=100, p_fire=0.02)
    a, b = gpu_net(p), gpu_net(p)
    a.record_kernel_times(21)
    for k in (13, 30):
        a.step(k, LDS)
        b.step(k, LDS)
    t, recorded = a.kernel_times()
    assert recorded == 21 and t["neuron"] > 0 and t["delivery"] > 0
    same_state(a, b, "recorded and not")


@pytest.mark.parametrize("name,chunks,fused", [("brunel_plus", 4, True), ("brunel_plus", 16, True),
                                               ("brunel_plus", 17, False), ("stress", 16, True),
                                               ("stress", 17, False)])
def test_the_recorded_launches_are_those_of_unrecorded_calls(name, chunks, fused):
    """110 slices of the configured workgroups do not fit the pass's slots: up
    to 16 per slice it takes fewer, beyond that the parts run by themselves,
    recorded or not."""
    n = 64 * 110 - 13
    kw = dict(n=n, delay=1, p_or_fanout=0.01, n_exc=n * 4 // 5) if name == "brunel_plus" else dict(
        n=n, p_or_fanout=60, p_fire=0.02, delay=1)
    p = wl.preset(name, **kw)
    a = gpu_net(p, slice_width=64, spike_chunks=chunks)
    assert (a.graph()["block_steps"] > 0) == (fused and name == "stress")
    a.record_kernel_times(20)
    a.step(20, LDS)
    t, recorded = a.kernel_times()
    assert recorded == 20 and t["neuron"] > 0 and t["delivery"] > 0
    assert (t["plasticity"] == 0) == fused
