"""Small networks in one workgroup, at the edges of its rounds, of its history
folding (every 32 steps) and of its input conversion; and the external drive's
table walk.

The steps of one launch are compared bit for bit with the separate part calls
of the same library (another kernel for each part), the drive with the oracle.
"""

import numpy as np
import pytest

import workloads as wl
from workloads.presets import PLASTIC_NONE
from paper_2107_04092_amd import snn

from gpu_common import gpu_net, to_np, log, same_state

pytestmark = pytest.mark.gpu
LDS = snn.SNN_DELIVER_LDS_SLICE

CASES = [
    # name, preset overrides, extra config
    ("tiny", dict(n=1, n_exc=1), dict()),
    ("tiny", dict(n=64, n_exc=50, p_or_fanout=0.3), dict()),
    ("tiny", dict(n=1023, n_exc=800), dict(history_bits=128)),
    ("tiny", dict(n=1025, n_exc=800, delay=2), dict()),
    ("tiny", dict(n=2049, n_exc=1600, v_inf=-45.0), dict(history_bits=128)),
    ("vogels", dict(n=2047, n_exc=1600), dict()),
    ("vogels", dict(n=4096, n_exc=3000, delay=5), dict(history_bits=128)),
    # inputs of some 10^6 mV: the sums leave the range of the short conversion
    ("vogels", dict(n=1500, n_exc=1200, w_exc=3.0e5, w_inh=-3.1e5), dict()),
    # heavy activity: many more spikes per step than waves, rows of one to
    # several rounds of targets
    ("stress", dict(n=4090, p_or_fanout=700, p_fire=0.2, plastic=PLASTIC_NONE), dict()),
    ("stress", dict(n=1024, p_or_fanout=40, p_fire=0.01, plastic=PLASTIC_NONE, delay=3), dict()),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s-%d" % (c[0], c[1]["n"]))
def test_one_workgroup_equals_the_parts(case):
    name, kw, cfg = case
    p = wl.preset(name, **kw)
    log("one workgroup: %s %s %s" % (name, kw, cfg))
    a = gpu_net(p, slice_width=256, spike_chunks=3, **cfg)
    b = gpu_net(p, slice_width=256, spike_chunks=3, **cfg)
    for k in (1, 2, 31, 32, 33, 64, 3):
        a.step(k, LDS)
        for _ in range(k):
            b.update_neurons()
            b.update_plasticity()
            b.deliver_spikes(LDS)
            b.advance()
        same_state(a, b, "%d steps" % k, weights=False)


@pytest.mark.parametrize("table", [
    [2 ** 31], [0], [2 ** 32 - 1], [1 << 29, 2 << 29, 3 << 29, 4 << 29],
    [1 << 28, 1 << 29, 1 << 30, 3 << 30, 2 ** 32 - 5],
    [(q + 1) * (2 ** 32 // 33) for q in range(32)],
], ids=lambda t: "%d-entries-%x" % (len(t), t[0]))
def test_drive_table_matches_oracle(table):
    """Tables of every fill (none, one group, the whole capacity; saturated or
    not): spikes and potentials of a driven network equal the oracle's."""
    from oracle import oracle
    log("drive table of %d entries" % len(table))
    p = wl.preset("brunel", n=700, n_exc=560, p_or_fanout=0.05, delay=1, j_ext=0.7,
                  poisson_mu=0.0)
    net = snn.Network(snn.config_from_preset(p, table))
    net.build_random(p.graph_kind, p.p_or_fanout, p.w_exc, p.w_inh)
    o = oracle.Oracle(p, np.asarray(table, np.uint32))
    o.build_random()
    net.step(40, LDS)
    o.step(40)
    s, n = net.state(), o.neurons()
    assert np.array_equal(to_np(s["hist"]).view(np.uint64), n["hist"])
    assert np.array_equal(to_np(s["v"]).view(np.uint32), n["v"].view(np.uint32))
