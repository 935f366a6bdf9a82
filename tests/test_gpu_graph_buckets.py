"""Building rows by buckets, at the edges of its plan: one row, one bucket,
empty rows and buckets, the most rows per bucket, buckets up to the sort's
capacity and beyond it (the general path), targets so unevenly spread that a
bucket is sorted row by row, equal targets told apart by weight, and indices
out of range. Row pointers, targets, weights (their bits), compressed targets
and pivots equal a numpy sort's."""

import numpy as np
import pytest

from paper_2107_04092_amd import snn
import workloads as wl

from gpu_common import to_np, log

pytestmark = pytest.mark.gpu


def build(n, src, dst, w, width=64):
    p = wl.preset("brunel", n=n, n_exc=n, slice_width=width, spike_chunks=1, delay=1)
    net = snn.Network(snn.config_from_preset(p))
    net.build_edges(src, dst, w)
    return net


def check(net, n, src, dst, w, width=64):
    order = np.lexsort((w, dst, src))
    src, dst, w = src[order], dst[order], w[order]
    rp = np.searchsorted(src, np.arange(n + 1))
    g = net.graph()
    assert np.array_equal(to_np(g["row_ptr"]), rp)
    assert np.array_equal(to_np(g["col"]), dst)
    assert np.array_equal(to_np(g["w"]).view(np.uint32), w.view(np.uint32))
    assert np.array_equal(to_np(g["col16"]).view(np.uint16), (dst % width).astype(np.uint16))
    s = np.arange(g["n_slices"] + 1) * width
    piv = to_np(g["pivots"])
    for k in (0, n // 2, n - 1):
        assert np.array_equal(piv[k], np.searchsorted(dst[rp[k]:rp[k + 1]], s)), k


def edges(kind, n, e, rs):
    src = rs.randint(0, n, e)
    dst = rs.randint(0, n, e)
    if kind == "hub targets":       # a quarter of the edges end at three neurons
        dst[rs.random_sample(e) < 0.25] = rs.randint(0, 3)
        dst[: e // 8] = n - 1
    elif kind == "few sources":     # rows of thousands beside empty ones
        src = (src % 7) * (n // 7)
    elif kind == "one bucket full":  # more than the sort holds, in rows that fit
        src[: min(e, 15000)] = rs.randint(0, min(n, 2), min(e, 15000))
    w = rs.choice(np.float32([-1.5, -0.0, 0.0, 0.25, 3.0, 1e-30]), e).astype(np.float32)
    if kind == "signs":
        w = rs.standard_normal(e).astype(np.float32)
    else:
        w = w + np.float32(0)  # (-0.0 and 0.0 compare equal in numpy: one of them)
    return src.astype(np.int32), dst.astype(np.int32), w


@pytest.mark.parametrize("case", [
    ("plain", 1, 5000), ("plain", 2, 1), ("plain", 700, 0), ("plain", 1023, 50000),
    ("signs", 3000, 400000), ("plain", 140001, 300000), ("plain", 70000, 70000),
    ("hub targets", 2000, 100000), ("hub targets", 20011, 500000), ("few sources", 300, 60000),
    ("few sources", 5000, 70000), ("one bucket full", 600, 80000), ("plain", 8, 90000),
    ("plain", 12, 150000), ("one bucket full", 5000, 16000), ("few sources", 40000, 60000),
    ("signs", 255, 30000), ("signs", 256, 30000), ("plain", 513, 700),
], ids=lambda c: "%s-%d-%d" % c)
def test_edge_lists(case):
    kind, n, e = case
    log("edge list: %s, n=%d, %d edges" % case)
    src, dst, w = edges(kind, n, e, np.random.RandomState(n + e))
    check(build(n, src, dst, w), n, src, dst, w)


@pytest.mark.parametrize("bad", [(-1, 0), (0, 5000), (5000, 3)], ids=str)
def test_index_out_of_range_is_refused(bad):
    rs = np.random.RandomState(3)
    src, dst, w = edges("plain", 5000, 60000, rs)
    src[777], dst[777] = bad
    with pytest.raises(snn.SnnError):
        build(5000, src, dst, w)


@pytest.mark.parametrize("n,fanout", [(1, 2), (600, 12288), (1000, 12289), (5000, 300),
                                      (70001, 9), (33, 16384)])
def test_fixed_fanout_rows_are_sorted(n, fanout):
    log("fixed fan-out: n=%d, %d targets per row" % (n, fanout))
    p = wl.preset("stress", n=n, p_or_fanout=fanout, slice_width=64, spike_chunks=1)
    net = snn.Network(snn.config_from_preset(p))
    net.build_random(p.graph_kind, p.p_or_fanout, p.w_exc, p.w_inh)
    g = net.graph()
    col = to_np(g["col"]).reshape(n, fanout)
    draws = wl.rng_u32(p.seed, 1, np.arange(n, dtype=np.uint64)[:, None],
                       np.arange(fanout, dtype=np.uint64)[None, :]).astype(np.uint64)
    want = np.sort(((draws * np.uint64(n)) >> np.uint64(32)).astype(np.int32), axis=1)
    assert np.array_equal(col, want)
    assert np.array_equal(to_np(g["row_ptr"]), np.arange(n + 1) * fanout)
    assert np.array_equal(to_np(g["col16"]).view(np.uint16).reshape(n, fanout), want % 64)
