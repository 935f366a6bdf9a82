"""Delivery of a delay block (networks without plasticity, D >= 2): states,
lists, masks, input and statistics equal the separate part calls bit for bit,
with segments shorter than a team of lanes, at and beyond the entries a lane
keeps in flight, more spikes than are looked up at once, one and two
accumulators, both kinds of targets, ragged last slices and cut blocks."""

import pytest

import workloads as wl
from workloads.presets import PLASTIC_NONE
from paper_2107_04092_amd import snn

from gpu_common import gpu_net, log, same_state

pytestmark = pytest.mark.gpu
LDS = snn.SNN_DELIVER_LDS_SLICE

CASES = [
    # name, preset overrides, slice width, extra config
    ("brunel", dict(n=6007, n_exc=4800, delay=4), 1024, dict()),              # 102 per segment
    ("brunel", dict(n=5003, n_exc=4000, delay=9, p_or_fanout=0.15), 1280, dict()),  # 192
    ("brunel", dict(n=9001, n_exc=7200, delay=3, p_or_fanout=0.3), 2304,
     dict(compressed_targets=0)),                                             # 691
    ("brunel", dict(n=6007, n_exc=4800, delay=20), 1024, dict(compressed_targets=0)),
    ("vogels", dict(n=12345, n_exc=9000, delay=5, p_or_fanout=0.0065), 2048, dict()),
    ("vogels", dict(n=5003, n_exc=4000, delay=12, p_or_fanout=0.016), 256, dict(history_bits=128)),
    ("tiny", dict(n=7777, n_exc=6000, delay=2, p_or_fanout=0.003), 64, dict()),
    ("stress", dict(n=30001, p_or_fanout=30, p_fire=0.3, delay=17, plastic=PLASTIC_NONE), 2048,
     dict()),                                                                 # 9,000 spikes a step
    ("stress", dict(n=4100, p_or_fanout=3000, p_fire=0.01, delay=6, plastic=PLASTIC_NONE), 4096,
     dict()),
]


def parts(net, k):
    for _ in range(k):
        net.update_neurons()
        net.update_plasticity()
        net.deliver_spikes(LDS)
        net.advance()


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s-%d-w%d-d%d" % (
    c[0], c[1]["n"], c[2], c[1]["delay"]))
def test_block_delivery_equals_the_parts(case):
    name, kw, width, cfg = case
    p = wl.preset(name, **kw)
    log("block delivery: %s %s width %d" % (name, kw, width))
    a = gpu_net(p, slice_width=width, spike_chunks=1, **cfg)
    b = gpu_net(p, slice_width=width, spike_chunks=1, **cfg)
    for k in (1, 2, 37, 50):
        a.step(k, LDS)
        parts(b, k)
        same_state(a, b, "%d steps" % k, weights=False)
