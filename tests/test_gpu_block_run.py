"""The run of a plastic block at the edges of its stretches: steps cut by the
entries the map holds and by the records LDS holds, a step that does not fit
by itself, a row with as many entries in one group as a row can have, rows
with events in consecutive steps (loaded again after the step before), and
the external drive drawn for several steps at once. Equal to the step-by-step
path bit for bit."""

import pytest

import workloads as wl
from paper_2107_04092_amd import snn

from gpu_common import gpu_net, log, same_state

pytestmark = pytest.mark.gpu
LDS = snn.SNN_DELIVER_LDS_SLICE

CASES = [
    # one group, rows of 16384 entries: every step in portions of one record
    ("stress", dict(n=64, p_or_fanout=16384, p_fire=0.15, delay=4), 64, dict()),
    # about 24,000 entries per group and step: no step fits the map
    ("stress", dict(n=300, p_or_fanout=2000, p_fire=0.2, delay=12), 64, dict()),
    # about 3,000 per group and step: blocks of a few stretches
    ("stress", dict(n=300, p_or_fanout=1000, p_fire=0.05, delay=12), 64,
     dict(history_bits=128)),
    # more than 4,096 records in a block, and in a step
    ("stress", dict(n=20000, p_or_fanout=8, p_fire=0.04, delay=16), 64, dict()),
    ("stress", dict(n=20000, p_or_fanout=8, p_fire=0.4, delay=3), 256, dict()),
    # consecutive events of a row at every distance, 32-bit targets
    ("stress", dict(n=700, p_or_fanout=60, p_fire=0.5, delay=9), 128,
     dict(compressed_targets=0)),
    # the drive: 8, 4 and 2 steps per draw, blocks that end inside one
    ("brunel_plus", dict(n=1501, n_exc=1200, delay=16), 64, dict()),
    ("brunel_plus", dict(n=1501, n_exc=1200, delay=8), 128, dict()),
    ("brunel_plus", dict(n=1501, n_exc=1200, delay=6), 256, dict(plasticity_algorithm=1)),
]


@pytest.mark.parametrize("case", CASES,
                         ids=lambda c: "%s-%d-%d-w%d" % (c[0], c[1]["n"], c[1]["delay"], c[2]))
def test_run_equals_step_by_step(case):
    name, kw, width, cfg = case
    p = wl.preset(name, **kw)
    log("block run: %s %s width %d" % (name, kw, width))
    cfg = dict(cfg, plastic_block_width=width)
    a = gpu_net(p, slice_width=256, spike_chunks=1, **cfg)
    b = gpu_net(p, slice_width=256, spike_chunks=1, **dict(cfg, plastic_blocks=-1))
    assert a.graph()["block_steps"] > 0 and a.graph()["block_width"] == width
    for k in (1, 37, 70):
        a.step(k, LDS)
        b.step(k, LDS)
        same_state(a, b, "%d steps" % k)
