"""The fused synapse pass with fewer workgroups per slice than configured
(more slices than its slots hold) or more (few slices): the same states, inputs and weights as the
separate part calls with the configured number, bit for bit."""

import pytest

import workloads as wl
from paper_2107_04092_amd import snn

from gpu_common import gpu_net, log, same_state

pytestmark = pytest.mark.gpu
LDS = snn.SNN_DELIVER_LDS_SLICE


@pytest.mark.parametrize("case", [
    # slices, configured workgroups per slice
    (110, 4), (98, 5), (130, 3), (300, 64), (500, 2),
], ids=lambda c: "%d-slices-%d" % c)
@pytest.mark.parametrize("name", ["brunel_plus", "stress"])
def test_fewer_workgroups_per_slice(name, case):
    slices, chunks = case
    n = 64 * slices - 13
    log("fused pass: %s, %d slices, %d workgroups each" % (name, slices, chunks))
    kw = dict(n=n, delay=1, p_or_fanout=0.01) if name == "brunel_plus" else dict(
        n=n, p_or_fanout=60, p_fire=0.02, delay=1)
    if name == "brunel_plus":
        kw["n_exc"] = n * 4 // 5
    p = wl.preset(name, **kw)
    a = gpu_net(p, slice_width=64, spike_chunks=chunks)
    b = gpu_net(p, slice_width=64, spike_chunks=chunks, plastic_blocks=-1)
    for k in (1, 40, 69):
        a.step(k, LDS)
        for _ in range(k):
            b.update_neurons()
            b.update_plasticity()
            b.deliver_spikes(LDS)
            b.advance()
        same_state(a, b, "%d steps" % k)


@pytest.mark.parametrize("case", [
    # slices, configured workgroups per slice
    (1, 1), (7, 1), (13, 3), (50, 1), (51, 1),
], ids=lambda c: "%d-slices-%d" % c)
@pytest.mark.parametrize("name", ["brunel_plus", "stress"])
def test_more_workgroups_per_slice(name, case):
    slices, chunks = case
    n = 64 * slices - 13
    log("fused pass: %s, %d slices, %d workgroups each" % (name, slices, chunks))
    kw = dict(n=n, delay=1, p_or_fanout=0.1, n_exc=n * 4 // 5) if name == "brunel_plus" else dict(
        n=n, p_or_fanout=20, p_fire=0.02, delay=1)
    p = wl.preset(name, **kw)
    a = gpu_net(p, slice_width=64, spike_chunks=chunks, plastic_blocks=-1)
    b = gpu_net(p, slice_width=64, spike_chunks=chunks, plastic_blocks=-1)
    for k in (1, 40, 69):
        a.step(k, LDS)
        for _ in range(k):
            b.update_neurons()
            b.update_plasticity()
            b.deliver_spikes(LDS)
            b.advance()
        same_state(a, b, "%d steps" % k)


@pytest.mark.parametrize("cfg", [
    dict(), dict(history_bits=128, compressed_targets=0), dict(stdp_xcd=2),
], ids=str)
@pytest.mark.parametrize("chunks", [3, 4])
def test_busy_steps_take_more_workgroups_per_slice(chunks, cfg):
    """Steps on both sides of the number of spikes (1,470 with 9.1 entries per row
    and slice) from which the configured workgroups per slice deliver."""
    n = 64 * 110 - 13
    log("fused pass: busy steps, %d workgroups per slice, %s" % (chunks, cfg))
    p = wl.preset("stress", n=n, p_or_fanout=1000, p_fire=0.21, delay=1)
    a = gpu_net(p, slice_width=64, spike_chunks=chunks, plastic_blocks=-1, **cfg)
    b = gpu_net(p, slice_width=64, spike_chunks=chunks, plastic_blocks=-1, **cfg)
    for k in (1, 20, 9):
        a.step(k, LDS)
        for _ in range(k):
            b.update_neurons()
            b.update_plasticity()
            b.deliver_spikes(LDS)
            b.advance()
        same_state(a, b, "%d steps" % k)
