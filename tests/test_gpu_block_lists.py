"""The per-step lists after plastic blocks (rebuilt from the masks that the
block's run and plan leave, beside the last block's deferred updates), at the
sizes where a mask word, a mask row or the ring is partly filled, and over
calls of one block, of two and of odd counts (the list counts alternate
between two halves): equal to the step-by-step path bit for bit."""

import pytest

import workloads as wl
from paper_2107_04092_amd import snn

from gpu_common import gpu_net, log, same_state

pytestmark = pytest.mark.gpu
LDS = snn.SNN_DELIVER_LDS_SLICE

CASES = [
    ("stress", dict(n=65536, p_or_fanout=20, p_fire=0.01, delay=64), dict()),
    ("stress", dict(n=65473, p_or_fanout=20, p_fire=0.3, delay=2), dict()),
    ("stress", dict(n=1, p_or_fanout=1, p_fire=0.5, delay=3), dict()),
    ("stress", dict(n=129, p_or_fanout=9, p_fire=0.1, delay=33), dict(history_bits=128)),
    ("brunel_plus", dict(n=2111, n_exc=1700, delay=5), dict(plastic_block_width=64)),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s-%d" % (c[0], c[1]["n"]))
def test_lists_after_blocks(case):
    name, kw, cfg = case
    p = wl.preset(name, **kw)
    a = gpu_net(p, slice_width=1024, spike_chunks=1, **cfg)
    b = gpu_net(p, slice_width=1024, spike_chunks=1, **dict(cfg, plastic_blocks=-1))
    for k in (1, 1, 2, 3, p.delay, 2 * p.delay + 1, 90):
        log("lists after blocks: %s n=%d, %d steps" % (name, p.n, k))
        a.step(k, LDS)
        b.step(k, LDS)
        same_state(a, b, "%d steps" % k)
