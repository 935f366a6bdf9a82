"""Deliveries by teams of lanes where rows are very uneven: segments of more
entries than a team adds by itself (left to all waves in pieces) at the limits
of teams and pieces, hubs beside empty rows, every target in one slice, equal
targets, more rows than are looked up at once; both kinds of targets, one and
two accumulators. Equal to the separate part calls bit for bit."""

import numpy as np
import pytest

import workloads as wl
from workloads.presets import PLASTIC_NONE
from paper_2107_04092_amd import snn

from gpu_common import gpu_net, log, same_state, torch_mod

pytestmark = pytest.mark.gpu
LDS = snn.SNN_DELIVER_LDS_SLICE


def uneven(kind, n, rs):
    """(src, dst) of an edge list."""
    if kind == "hubs":          # one row in fifty of 9,000 entries, the others of 20
        deg = np.full(n, 20)
        deg[::50] = 9000
    elif kind == "lognormal":
        deg = np.minimum(rs.lognormal(3.5, 1.8, n), 8000).astype(np.int64)
        deg[rs.random_sample(n) < 0.1] = 0
    elif kind == "limits":      # lengths at the teams' and the pieces' limits
        deg = rs.choice([0, 1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257,
                         511, 512, 513, 1023, 1025, 2049, 4096, 4097], n)
    else:
        deg = np.full(n, 150)
    src = np.repeat(np.arange(n), deg)
    dst = rs.randint(0, n, len(src))
    if kind == "near":          # targets near the source: whole rows in a slice
        dst = (src + rs.randint(-200, 200, len(src))) % n
    elif kind == "limits":      # ... and rows of one slice, equal targets among them
        dst = (src // 64 * 64 + rs.randint(0, 64, len(src))) % n
    return src.astype(np.int32), dst.astype(np.int32)


def nets(kind, model, n, width, count=2, **kw):
    name, over = model
    p = wl.preset(name, n=n, n_exc=n * 3 // 4, **over)
    rs = np.random.RandomState(n)
    src, dst = uneven(kind, n, rs)
    w = np.where(src < p.n_exc, p.w_exc, p.w_inh).astype(np.float32)
    st = wl.initial_state(p)
    out = []
    for _ in range(count):
        net = gpu_net(p, slice_width=width, spike_chunks=2, build=False, **kw)
        net.build_edges(src, dst, w)
        net.set_state(0, v=torch_mod().from_numpy(st["v"]))
        out.append(net)
    return out


def parts(net, k):
    for _ in range(k):
        net.update_neurons()
        net.update_plasticity()
        net.deliver_spikes(LDS)
        net.advance()


def source(fire, delay):
    return "stress", dict(p_or_fanout=0, p_fire=fire, delay=delay, plastic=PLASTIC_NONE)


@pytest.mark.parametrize("narrow", [0, 1])
@pytest.mark.parametrize("kind", ["hubs", "lognormal", "limits", "near"])
@pytest.mark.parametrize("fire,n,width", [(0.002, 6011, 1024), (0.03, 6011, 256),
                                          (0.4, 5003, 4096)])
def test_block_delivery(kind, fire, n, width, narrow):
    log("delay blocks: %s, n=%d, width %d, %g per step" % (kind, n, width, fire))
    a, b = nets(kind, source(fire, 5), n, width, compressed_targets=narrow)
    for k in (1, 3, 21):
        a.step(k, LDS)
        parts(b, k)
        same_state(a, b, "%d steps" % k, weights=False)
    assert a.stats()["delivered_events"] > 0


@pytest.mark.parametrize("kind", ["hubs", "limits"])
def test_block_delivery_two_inputs(kind):
    log("delay blocks, CUBA: %s" % kind)
    a, b = nets(kind, ("vogels", dict(p_or_fanout=0, delay=4, v_inf=-45.0)), 5003, 512)
    for k in (3, 60):
        a.step(k, LDS)
        parts(b, k)
        same_state(a, b, "%d steps" % k, weights=False)
    assert a.stats()["delivered_events"] > 0


def us_per_step(net, steps):
    torch = torch_mod()
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    best = 1e9
    for _ in range(7):
        torch.cuda.synchronize()
        ev[0].record(net.stream)
        net.step(steps, LDS)
        ev[1].record(net.stream)
        torch.cuda.synchronize()
        best = min(best, ev[0].elapsed_time(ev[1]) * 1e3 / steps)
    return best


def uneven_over_even(n, fire, delay):
    """Time of a network with uneven rows over that of one with the same number
    of edges in rows of one length."""
    torch = torch_mod()
    p = wl.preset("stress", n=n, p_or_fanout=0, p_fire=fire, delay=delay, plastic=PLASTIC_NONE)
    us = []
    for kind in ("hubs", "even"):
        rs = np.random.RandomState(1)
        if kind == "hubs":
            deg = np.full(n, 200)
            deg[::100] = 14000
        else:
            deg = np.full(n, (200 * 99 + 14000) // 100)
        src = np.repeat(np.arange(n), deg).astype(np.int32)
        dst = rs.randint(0, n, len(src)).astype(np.int32)
        net = gpu_net(p, slice_width=1024, spike_chunks=4, build=False)
        net.build_edges(src, dst, np.full(len(src), 0.1, np.float32))
        net.step(96, LDS)
        us.append(us_per_step(net, 96))
    log("n=%d, D=%d, %g per step: %.2f us with hubs, %.2f us even" % (n, delay, fire, *us))
    return us[0] / us[1]


def test_hubs_cost_no_more_than_their_entries_in_delay_blocks():
    """(left to single teams: 2.3 times)"""
    assert uneven_over_even(20011, 0.05, 6) < 1.4
