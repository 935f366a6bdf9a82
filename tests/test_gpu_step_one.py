"""One launch per step (networks without plasticity, D = 1, beyond one
workgroup): states, lists, masks, input and statistics equal the separate part
calls bit for bit, at ragged sizes, one and several slices or rounds per
workgroup, rows shared by 4 to 64 lanes, more spikes than are listed at once,
calls of one step and of many, mixed with part calls, and captured."""

import pytest

import workloads as wl
from workloads.presets import PLASTIC_NONE
from paper_2107_04092_amd import snn

from gpu_common import gpu_net, log, same_state

pytestmark = pytest.mark.gpu
LDS = snn.SNN_DELIVER_LDS_SLICE

CASES = [
    # name, preset overrides, slice width, chunks, extra config
    ("vogels", dict(n=4097, n_exc=3277), 1024, 1, dict()),
    ("vogels", dict(n=5003, n_exc=4000, p_or_fanout=0.016), 256, 3, dict(history_bits=128)),
    ("vogels", dict(n=12345, n_exc=9000, p_or_fanout=0.0065), 2048, 2, dict()),
    ("vogels", dict(n=65536, n_exc=52000, p_or_fanout=0.0012), 640, 1, dict()),
    ("brunel", dict(n=6007, n_exc=4800, delay=1), 1024, 4, dict()),
    ("brunel", dict(n=9001, n_exc=7200, delay=1, p_or_fanout=0.3), 2304, 1,
     dict(compressed_targets=0)),
    ("tiny", dict(n=7777, n_exc=6000, p_or_fanout=0.003), 64, 2, dict()),
    ("stress", dict(n=30001, p_or_fanout=30, p_fire=0.3, plastic=PLASTIC_NONE), 2048, 2, dict()),
    ("stress", dict(n=4100, p_or_fanout=3000, p_fire=0.01, plastic=PLASTIC_NONE), 4096, 1,
     dict(history_bits=128)),
]


def parts(net, k):
    for _ in range(k):
        net.update_neurons()
        net.update_plasticity()
        net.deliver_spikes(LDS)
        net.advance()


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s-%d-w%d" % (c[0], c[1]["n"], c[2]))
def test_one_launch_per_step_equals_the_parts(case):
    name, kw, width, chunks, cfg = case
    p = wl.preset(name, **kw)
    log("one launch per step: %s %s width %d" % (name, kw, width))
    a = gpu_net(p, slice_width=width, spike_chunks=chunks, **cfg)
    b = gpu_net(p, slice_width=width, spike_chunks=chunks, **cfg)
    for k in (1, 1, 2, 40, 65):
        a.step(k, LDS)
        parts(b, k)
        same_state(a, b, "%d steps" % k, weights=False)
    parts(a, 3)
    a.step_static(5, LDS)
    parts(b, 8)
    same_state(a, b, "mixed", weights=False)


BUSY = [
    # the same, with bursts: steps of no spikes, of a few and of a third of the
    # neurons, so that groups run whole and in two to all of their parts
    ("vogels", dict(n=4097, n_exc=3277, p_or_fanout=0.1), 1024, 4, dict()),
    ("vogels", dict(n=20011, n_exc=16000, p_or_fanout=0.02), 64, 1, dict(history_bits=128)),
    ("vogels", dict(n=9001, n_exc=7200, p_or_fanout=0.1), 4096, 16, dict(history_bits=128)),
    ("brunel", dict(n=12345, n_exc=9876, delay=1), 4096, 3, dict()),
    ("brunel", dict(n=16385, n_exc=13000, delay=1, p_or_fanout=0.03), 2048, 9,
     dict(compressed_targets=0)),
    ("tiny", dict(n=65536, n_exc=52000, p_or_fanout=0.002), 512, 2, dict()),
]


@pytest.mark.parametrize("case", BUSY, ids=lambda c: "%s-%d-w%d" % (c[0], c[1]["n"], c[2]))
def test_busy_steps_in_parts(case):
    name, kw, width, chunks, cfg = case
    p = wl.preset(name, v_inf=400.0, tau_ref=0.3, w_exc=1e-3, w_inh=-1e-3, **kw)
    log("busy steps in parts: %s %s width %d" % (name, kw, width))
    a = gpu_net(p, slice_width=width, spike_chunks=chunks, **cfg)
    b = gpu_net(p, slice_width=width, spike_chunks=chunks, **cfg)
    for k in (1, 2, 30, 7):
        a.step(k, LDS)
        parts(b, k)
        same_state(a, b, "%d steps" % k, weights=False)
    assert a.stats()["spikes"] > 40 * p.n // 20


def test_captured():
    import torch
    p = wl.preset("vogels", n=6001, n_exc=4800, p_or_fanout=0.013)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        a = gpu_net(p, stream=s)
        b = gpu_net(p, stream=s)
        for steps in (1, 6):
            g = a.capture(steps, LDS)
            for r in range(5):
                a.replay(g)
                parts(b, steps)
                same_state(a, b, "replay %d of %d steps" % (r, steps), weights=False)
            snn.snn_graph_destroy(g)
