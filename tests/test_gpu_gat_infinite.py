"""Infinities in the fused attention.  A row's answer depends on its own
edges alone, whatever its length leaves in the last batch of a walk or in the
last group of segments of a hub row: an infinite feature gives an infinite
value in its column and nothing elsewhere, and an edge whose score alone is
+inf takes the whole weight of its row.  Rows of one lane group, of one
wavefront and hub rows, at lengths around the batches (4 edges per lane group)
and around groups of four 64-edge segments; every edge has a source of its
own."""
import numpy as np
import pytest
import torch

from paper_1909_01315_amd import gnnk, synth
from _gpu import Pair, as_f64, dev, host

pytestmark = pytest.mark.gpu
S = synth.SEED_BASE + 900
DEGREES = [1, 2, 3, 4, 5, 6, 7, 8, 9, 31, 32, 33, 63, 64, 65, 128, 129, 256, 257, 300, 320, 321, 512, 513, 641]
FIRST = np.concatenate([[0], np.cumsum(DEGREES)[:-1]])  # first edge (and source) of each row
E = int(sum(DEGREES))
ROW = np.repeat(np.arange(len(DEGREES)), DEGREES)


@pytest.fixture(scope="module")
def pair():
    gnnk.set_option("seg_edges", 64)
    p = Pair(np.arange(E, dtype=np.int32), ROW.astype(np.int32), E, len(DEGREES))
    gnnk.set_option("seg_edges", 0)
    assert p.g.info()["hub_dst_rows"] == sum(d > 64 for d in DEGREES)
    return p


@pytest.fixture(autouse=True)
def reset_options():
    yield
    gnnk.set_option("no_fast", 0)


def inputs(H, F, dtype):
    """float32 values that the type holds"""
    made = (lambda a: a) if dtype == "f32" else (lambda a: as_f64(synth.to_bf16_bits(a)).astype(np.float32))
    return (made(synth.normal(S, f"f{H}.{F}", (E, H, F))), made(synth.normal(S, f"l{H}", (E, H, 1))),
            made(synth.normal(S, f"r{H}", (len(DEGREES), H, 1))),
            made(np.abs(synth.normal(S, f"z{H}.{F}", (len(DEGREES), H, F))) + 0.5))


def to_gpu(a, dtype):
    t = dev(a)
    return t if dtype == "f32" else t.to(torch.bfloat16)


def attention(el, er):
    """(E, H) softmax over each row of leaky(el + er), in 64 bits"""
    s = el[:, :, 0].astype(np.float64) + er[ROW, :, 0]
    s = np.where(s > 0, s, 0.2 * s)
    a = np.exp(s - np.maximum.reduceat(s, FIRST)[ROW])
    return a / np.add.reduceat(a, FIRST)[ROW]


CASES = [(8, 16, "f32"), (1, 8, "f32"), (2, 33, "f32"), (8, 64, "f32"), (4, 16, "bf16"), (2, 33, "bf16")]


@pytest.mark.parametrize("no_fast", [0, 1])
@pytest.mark.parametrize("H,F,dtype", CASES)
def test_infinite_features_stay_in_their_column(pair, H, F, dtype, no_fast):
    gnnk.set_option("no_fast", no_fast)
    feat, el, er, _ = inputs(H, F, dtype)
    a = attention(el, er)
    ref = np.add.reduceat(a[:, :, None] * feat, FIRST)
    feat[FIRST, :, 0] = np.inf                      # the first edge of every row
    ref[:, :, 0] = np.inf
    for r, d in enumerate(DEGREES):                 # and the first of a group of four segments
        if d > 256:
            feat[FIRST[r] + 256, :, 1] = -np.inf
            ref[r, :, 1] = -np.inf
    out = gnnk.gat_aggregate(pair.g, to_gpu(feat, dtype), to_gpu(el, dtype), to_gpu(er, dtype), 0.2)
    out = as_f64(host(out))
    assert np.array_equal(np.isinf(ref), np.isinf(out)), "infinite where the reference is, and nowhere else"
    assert np.all(out[np.isinf(ref)] == ref[np.isinf(ref)])
    fin = np.isfinite(ref)
    tol = 1e-6 + (1e-5 if dtype == "f32" else 1e-2) * np.abs(ref[fin])
    assert np.all(np.abs(out[fin] - ref[fin]) <= tol)


@pytest.mark.parametrize("no_fast", [0, 1])
@pytest.mark.parametrize("H,F,dtype", CASES)
def test_one_infinite_score_takes_the_whole_weight(pair, H, F, dtype, no_fast):
    gnnk.set_option("no_fast", no_fast)
    feat, el, er, _ = inputs(H, F, dtype)
    for at in (lambda d: 0, lambda d: d // 2, lambda d: d - 1):
        top = FIRST + np.array([at(d) for d in DEGREES])
        l = el.copy()
        l[top] = np.inf
        out = gnnk.gat_aggregate(pair.g, to_gpu(feat, dtype), to_gpu(l, dtype), to_gpu(er, dtype), 0.2)
        assert np.array_equal(as_f64(host(out)), feat[top].astype(np.float64))


@pytest.mark.parametrize("no_fast", [0, 1])
@pytest.mark.parametrize("H,F,dtype", CASES)
def test_infinite_features_in_the_backward(pair, H, F, dtype, no_fast):
    """dZ > 0 and +inf in the first edge of every row: S = sum of a da is +inf
    there, so d_el = sum of a (da - S) lk is -inf for the other edges of the
    row and NaN for that one; d_feat, which neither enters, stays.  An infinite
    dZ gives an infinite d_feat in its column."""
    gnnk.set_option("no_fast", no_fast)
    feat, el, er, dz = inputs(H, F, dtype)
    args = [to_gpu(x, dtype) for x in (el, er)]
    _, st = gnnk.gat_aggregate(pair.g, to_gpu(feat, dtype), *args, 0.2, want_stats=True)
    ref, _, _ = gnnk.gat_aggregate_backward(pair.g, to_gpu(feat, dtype), *args, 0.2, st, to_gpu(dz, dtype))
    first = np.zeros(E, bool)
    first[FIRST] = True
    up = feat.copy()
    up[FIRST, :, 0] = np.inf
    df, dl, _ = gnnk.gat_aggregate_backward(pair.g, to_gpu(up, dtype), *args, 0.2, st, to_gpu(dz, dtype))
    assert torch.equal(df, ref)
    dl = as_f64(host(dl))[:, :, 0]
    assert np.all(np.isneginf(dl[~first])) and np.all(np.isnan(dl[first]))
    dz[:, :, 0] = np.inf
    df, _, _ = gnnk.gat_aggregate_backward(pair.g, to_gpu(feat, dtype), *args, 0.2, st, to_gpu(dz, dtype))
    df, ref = as_f64(host(df)), as_f64(host(ref))
    assert np.all(df[:, :, 0] == np.inf) and np.array_equal(df[:, :, 1:], ref[:, :, 1:])
