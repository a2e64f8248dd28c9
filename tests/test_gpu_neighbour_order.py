"""Graphs whose edge ids are scattered over their rows (an edge list in
arrival order) keep a second listing of their hub rows' CSRs by neighbour id,
which the passes that gather node rows walk.  Every such pass against the
oracle, and the exported formats, which stay in edge-id order; on graphs whose
hub rows lie on one side only; and on a graph whose rows' ids lie together,
which keeps no second listing."""
import numpy as np
import pytest
import torch

import oracle as orc
from paper_1909_01315_amd import gnnk, synth
from _gpu import Pair, assert_close, assert_exact, check_formats, dev
from test_gpu_gat import oracle_gat, oracle_gat_backward
from test_gpu_random_cases import gat_grad_bounds

pytestmark = pytest.mark.gpu
E = (1 << 20) + 77
S = synth.SEED_BASE + 700


def skewed(rng, n, hot_ids=None):
    """ids of which a tenth (or the first hot_ids) take nine tenths of the draws"""
    a = rng.integers(0, n, E)
    hot = rng.random(E) < 0.9
    a[hot] = rng.integers(0, hot_ids or max(n // 10, 1), int(hot.sum()))
    return a.astype(np.int32)


# sources, destinations, their hot ones (0: none, no hub rows), the directions
# listed; row ids of one, two and three radix digits.  (A row of E / 33 edges
# or more would have its ids next to each other by chance alone.)
GRAPHS = {"both": (3000, 2500, 300, 250, 3), "in": (300000, 2500, 0, 250, 1), "out": (3000, 300000, 300, 0, 2),
          "one pass": (300, 400, 100, 120, 3), "three passes": (300001, 270000, 1000, 900, 3)}


@pytest.fixture(scope="module", params=list(GRAPHS))
def pair(request):
    rng = np.random.default_rng(11)
    n_src, n_dst, hot_src, hot_dst, listed = GRAPHS[request.param]
    src = skewed(rng, n_src, hot_src) if hot_src else rng.integers(0, n_src, E).astype(np.int32)
    dst = skewed(rng, n_dst, hot_dst) if hot_dst else rng.integers(0, n_dst, E).astype(np.int32)
    p = Pair(src, dst, n_src, n_dst, ptr64=request.param == "in")
    info = p.g.info()
    assert info["identity_eids"] == 0 and info["neighbour_lists"] == listed
    return p


def test_formats_stay_in_edge_id_order(pair):
    check_formats(pair)


@pytest.fixture
def reset_schedule():
    yield
    gnnk.set_option("schedule", 0)


@pytest.mark.parametrize("schedule", [0, 2, 3])
def test_sums_and_their_gradients(pair, schedule, reset_schedule):
    gnnk.set_option("schedule", schedule)  # 2, 3: the edge-parallel walks
    p = pair
    X = synth.normal(S, "x", (p.o.n_src, 2, 8))
    w = synth.uniform(S, "w", (E, 2, 1), 0.5, 1.5)
    dZ = synth.normal(S, "dz", (p.o.n_dst, 2, 8))
    for op, red, rhs in (("copy_lhs", "sum", None), ("copy_lhs", "mean", None), ("mul", "sum", w)):
        assert_close(gnnk.gspmm(p.g, op, red, dev(X), None if rhs is None else dev(rhs)),
                     orc.gspmm(p.o, op, red, X, rhs), name=f"{op}/{red}")
        dl, dr = gnnk.gspmm_backward(p.g, op, red, dev(X), None if rhs is None else dev(rhs), dev(dZ))
        rl, rr = orc.gspmm_backward(p.o, op, red, X, rhs, dZ)
        assert_close(dl, rl, name=f"{op}/{red} dX")
        if rhs is not None:
            assert_close(dr, rr, name=f"{op}/{red} dW")


def test_max_ties_and_its_gradient(pair):
    # small integers: almost every maximum is tied, and the smallest edge id
    # wins whatever the order of the walk
    p = pair
    X = np.random.default_rng(3).integers(-3, 4, (p.o.n_src, 1, 40)).astype(np.float32)
    z, au, ae = gnnk.gspmm(p.g, "copy_lhs", "max", dev(X), want_args=True)
    rz, ru, re_ = orc.gspmm(p.o, "copy_lhs", "max", X)
    assert_exact(z, rz)
    assert_exact(au, ru)
    assert_exact(ae, re_)
    dZ = synth.normal(S, "dzm", (p.o.n_dst, 1, 40))
    dl, _ = gnnk.gspmm_backward(p.g, "copy_lhs", "max", dev(X), None, dev(dZ), arg_rhs=ae)
    rl, _ = orc.gspmm_backward(p.o, "copy_lhs", "max", X, None, dZ, arg_e=re_)
    assert_close(dl, rl)


def test_sddmm_and_its_gradients(pair):
    p = pair
    X, Y = synth.normal(S, "sx", (p.o.n_src, 2, 8)), synth.normal(S, "sy", (p.o.n_dst, 2, 8))
    for op, shape in (("dot", (E, 2, 1)), ("add", (E, 2, 8))):
        out = gnnk.gsddmm(p.g, op, dev(X), "u", dev(Y), "v")
        ref = orc.gsddmm(p.o, op, X, "u", Y, "v")
        (assert_close if op == "dot" else assert_exact)(out, ref)
        g = synth.normal(S, "sg" + op, shape)
        dl, dr = gnnk.gsddmm_backward(p.g, op, dev(X), "u", dev(Y), "v", dev(g))
        rl, rr = orc.gsddmm_backward(p.o, op, X, "u", Y, "v", g)
        assert_close(dl, rl)
        assert_close(dr, rr)


def test_fused_attention_and_its_gradients(pair):
    p = pair
    f = synth.normal(S, "gf", (p.o.n_src, 2, 8))
    l, r = synth.normal(S, "gl", (p.o.n_src, 2, 1)), synth.normal(S, "gr", (p.o.n_dst, 2, 1))
    dz = synth.normal(S, "gz", (p.o.n_dst, 2, 8))
    ref, ref_a = oracle_gat(p.o, f, l, r, 0.2)
    out, a, st = gnnk.gat_aggregate(p.g, dev(f), dev(l), dev(r), 0.2, want_attn=True, want_stats=True)
    assert_close(out, ref)
    assert_close(a, ref_a)
    assert_close(gnnk.gat_aggregate(p.g, dev(f), dev(l), dev(r), 0.2), ref)
    got = gnnk.gat_aggregate_backward(p.g, dev(f), dev(l), dev(r), 0.2, st, dev(dz))
    refs = oracle_gat_backward(p.o, f, l, r, 0.2, dz)
    bounds = gat_grad_bounds(p.o, f, l, r, dz, 0.2)
    for x, y, b in zip(got, refs, bounds):
        d = np.abs(x.cpu().numpy().astype(np.float64).reshape(y.shape) - y)
        assert np.all(d <= np.maximum(1e-6 + 1e-5 * np.abs(y), b.reshape(y.shape)))


def test_rows_whose_ids_lie_together_keep_their_order():
    """An edge list grouped by destination, the groups in another order: a
    row's ids lie together, and results and formats are those of the oracle."""
    rng = np.random.default_rng(5)
    n = 2000
    dst = np.sort(skewed(rng, n))[::-1].copy()
    src = skewed(rng, n)
    p = Pair(src, dst, n, n)
    info = p.g.info()
    assert info["identity_eids"] == 0 and info["neighbour_lists"] == 0
    check_formats(p)
    X, w = synth.normal(S, "tx", (n, 2, 8)), synth.uniform(S, "tw", (E, 2, 1), 0.5, 1.5)
    assert_close(gnnk.gspmm(p.g, "mul", "sum", dev(X), dev(w)), orc.gspmm(p.o, "mul", "sum", X, w))
    dZ = synth.normal(S, "tz", (n, 2, 8))
    for x, y in zip(gnnk.gspmm_backward(p.g, "mul", "sum", dev(X), dev(w), dev(dZ)),
                    orc.gspmm_backward(p.o, "mul", "sum", X, w, dZ)):
        assert_close(x, y)


@pytest.mark.parametrize("order", ["by source", "by source and destination", "by source, destinations descending"])
def test_edge_lists_sorted_by_source_keep_their_order(order):
    """The in-rows list their neighbours in order as they are, and the edge
    ids of a reverse row lie together."""
    rng = np.random.default_rng(6)
    n = 20000
    src, dst = skewed(rng, n), skewed(rng, n)
    second = rng.random(E) if order == "by source" else (-dst if "descending" in order else dst)
    at = np.lexsort((second, src))
    src, dst = src[at], dst[at]
    p = Pair(src, dst, n, n)
    info = p.g.info()
    assert info["identity_eids"] == 0 and info["neighbour_lists"] == 0
    check_formats(p)
    X, w, dZ = (synth.normal(S, k, sh) for k, sh in (("sx", (n, 2, 8)), ("sw", (E, 2, 1)), ("sz", (n, 2, 8))))
    assert_close(gnnk.gspmm(p.g, "mul", "sum", dev(X), dev(w)), orc.gspmm(p.o, "mul", "sum", X, w))
    for x, y in zip(gnnk.gspmm_backward(p.g, "mul", "sum", dev(X), dev(w), dev(dZ)),
                    orc.gspmm_backward(p.o, "mul", "sum", X, w, dZ)):
        assert_close(x, y)


def test_validate_reads_the_listings():
    rng = np.random.default_rng(9)
    n = 2000
    p = Pair(skewed(rng, n), skewed(rng, n), n, n)
    info = p.g.info()
    assert info["neighbour_lists"] == 3
    p.g.validate()
    lists = p.g._keep[1]
    assert lists.numel() == info["lists_bytes"]
    words = lists[: lists.numel() // 4 * 4].view(torch.int32)
    # four arrays of E words each, 256 bytes aligned, the segment orders of a
    # direction after its two
    for at in (E - 1, -(-E // 64) * 64 + E - 1):
        kept = int(words[at])
        words[at] = 1 << 30
        with pytest.raises(gnnk.GnnkError) as err:
            p.g.validate()
        assert err.value.status == gnnk.ERANGE
        words[at] = kept
    p.g.validate()


def test_from_csr_with_scattered_ids():
    rng = np.random.default_rng(8)
    n = 2000
    o = orc.OGraph(skewed(rng, n), skewed(rng, n), n, n)
    ip, ii, ie = orc.csr(o)
    g = gnnk.Graph.from_csr(dev(ip.astype(np.int32)), dev(ii), dev(ie), n)
    assert g.info()["neighbour_lists"] == 3
    X = synth.normal(S, "cx", (n, 1, 16))
    assert_close(gnnk.gspmm(g, "copy_lhs", "sum", dev(X)), orc.gspmm(o, "copy_lhs", "sum", X))
    dx, _ = gnnk.gspmm_backward(g, "copy_lhs", "sum", dev(X), None, dev(X))
    assert_close(dx, orc.gspmm_backward(o, "copy_lhs", "sum", X, None, X)[0])
    for rev in (False, True):
        for a, b in zip(g.csr_export(reverse=rev)[1:], orc.csr(o, reverse=rev)[1:]):
            assert_exact(a, b)
    g.destroy()
