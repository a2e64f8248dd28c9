"""Rows that no wide vector divides, or that are not aligned to one: a head's
last vector overlaps the one before it.  Every pass that takes such rows
against the oracle, at widths around the vectors' sizes, around the 32-column
words of the winner masks and past one pass of the wavefront, fp32 and bf16,
with tables whose base and row stride are aligned to single elements, hub rows,
and the compile-time and the runtime layouts."""
import numpy as np
import pytest
import torch

import oracle as orc
from paper_1909_01315_amd import gnnk, synth
from _gpu import Pair, assert_close, assert_exact, dev
from test_gpu_gat import oracle_gat

pytestmark = pytest.mark.gpu
S = synth.SEED_BASE + 800
N, M, E = 160, 120, 4000


@pytest.fixture(scope="module")
def pair():
    gnnk.set_option("seg_edges", 64)
    rng = np.random.default_rng(2)
    src = (rng.integers(0, N, E) ** 2 // N).astype(np.int32)  # hub sources and destinations
    dst = (rng.integers(0, M, E) ** 2 // M).astype(np.int32)
    p = Pair(src, dst, N, M)
    gnnk.set_option("seg_edges", 0)
    assert p.g.info()["hub_dst_rows"] > 0 and p.g.info()["hub_src_rows"] > 0
    return p


@pytest.fixture(autouse=True)
def reset_options():
    yield
    gnnk.set_option("no_fast", 0)


def shifted(a, pad):
    """a on the GPU inside a larger buffer: base and row stride off by `pad` elements"""
    t = dev(a)
    if not pad:
        return t
    rows, h, f = t.shape
    buf = torch.zeros(rows * (h * f + pad) + pad, dtype=t.dtype, device=t.device)
    v = buf[pad:].view(-1)[: rows * (h * f + pad)].view(rows, h * f + pad)[:, : h * f].view(rows, h, f) \
        if h == 1 else buf[pad:].as_strided((rows, h, f), (h * f + pad, f, 1))
    v.copy_(t)
    return v


WIDTHS = [(1, 5, 0), (1, 7, 0), (1, 9, 0), (1, 15, 1), (1, 33, 0), (1, 35, 0), (1, 39, 3), (1, 47, 0), (1, 64, 1),
          (1, 261, 0), (1, 515, 0), (3, 5, 0), (3, 9, 1), (2, 45, 0), (7, 13, 0),
          # the narrowest rows that overlap, and the widest that do not
          (1, 13, 0), (1, 14, 0), (1, 17, 0), (1, 18, 1), (2, 5, 0), (2, 9, 0), (4, 5, 0), (3, 6, 0)]


@pytest.mark.parametrize("no_fast", [0, 1])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("H,F,pad", WIDTHS)
def test_rows_of_any_width(pair, H, F, pad, dtype, no_fast):
    gnnk.set_option("no_fast", no_fast)
    p, kind = pair, dtype
    made = (lambda a: a) if dtype == "f32" else synth.to_bf16_bits
    X = made(synth.normal(S, f"x{H}.{F}", (N, H, F)))
    Y = made(synth.normal(S, f"y{H}.{F}", (M, H, F)))
    w = made(synth.uniform(S, f"w{H}", (E, H, 1), 0.5, 1.5))
    Xd, Yd, wd = shifted(X, pad), shifted(Y, pad), dev(w)
    assert_close(gnnk.gspmm(p.g, "copy_lhs", "mean", Xd), orc.gspmm(p.o, "copy_lhs", "mean", X), kind, "mean")
    assert_close(gnnk.gspmm(p.g, "mul", "sum", Xd, wd), orc.gspmm(p.o, "mul", "sum", X, w), kind, "u_mul_e")
    for op, red, rhs, rd in (("copy_lhs", "mean", None, None), ("mul", "sum", w, wd)):
        for a, b, n in zip(gnnk.gspmm_backward(p.g, op, red, Xd, rd, Yd), orc.gspmm_backward(p.o, op, red, X, rhs, Y),
                           ("dX", "dW")):
            if b is not None:
                assert_close(a, b, kind, f"{op} {n}")
    z, _, ae = gnnk.gspmm(p.g, "copy_lhs", "max", Xd, want_args=True)
    rz, _, re_ = orc.gspmm(p.o, "copy_lhs", "max", X)
    assert_exact(z, rz, "max")
    assert_exact(ae, re_, "arg edge")
    dl, _ = gnnk.gspmm_backward(p.g, "copy_lhs", "max", Xd, None, Yd, arg_rhs=ae)
    assert_close(dl, orc.gspmm_backward(p.o, "copy_lhs", "max", X, None, Y, arg_e=re_)[0], kind, "max dX")
    z, _, ae = gnnk.gspmm(p.g, "mul", "max", Xd, wd, want_args=True)
    rz, _, re_ = orc.gspmm(p.o, "mul", "max", X, w)
    assert_exact(z, rz, "u_mul_e max")
    for a, b, n in zip(gnnk.gspmm_backward(p.g, "mul", "max", Xd, wd, Yd, arg_rhs=ae),
                       orc.gspmm_backward(p.o, "mul", "max", X, w, Y, arg_e=re_), ("dX", "dW")):
        assert_close(a, b, kind, f"u_mul_e max {n}")
    assert_close(gnnk.gsddmm(p.g, "dot", Xd, "u", Yd, "v"), orc.gsddmm(p.o, "dot", X, "u", Y, "v"), kind, "dot")
    assert_exact(gnnk.gsddmm(p.g, "add", Xd, "u", Yd, "v"), orc.gsddmm(p.o, "add", X, "u", Y, "v"), "add")
    g = made(synth.normal(S, f"g{H}", (E, H, 1)))
    for a, b, n in zip(gnnk.gsddmm_backward(p.g, "dot", Xd, "u", Yd, "v", dev(g)),
                       orc.gsddmm_backward(p.o, "dot", X, "u", Y, "v", g), ("dX", "dY")):
        assert_close(a, b, kind, f"dot {n}")


@pytest.mark.parametrize("no_fast", [0, 1])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("H,F,pad", [(1, 5, 0), (3, 45, 0), (2, 33, 1), (1, 261, 0), (5, 7, 2), (2, 9, 0), (1, 129, 0),
                                     (1, 515, 1), (4, 47, 3)])
def test_fused_attention_of_any_width(pair, H, F, pad, dtype, no_fast):
    from test_gpu_gat import oracle_gat_backward
    from test_gpu_random_cases import check, check_bound, gat_grad_bounds

    # nothing is rounded between its steps: for bf16 the reference is the
    # oracle chain on the exactly widened inputs, at the bf16 tolerance
    gnnk.set_option("no_fast", no_fast)
    p = pair
    made = (lambda a: a) if dtype == "f32" else synth.to_bf16_bits
    wide = (lambda a: a) if dtype == "f32" else orc.bf16_to_f32
    f, dz = made(synth.normal(S, f"f{H}.{F}", (N, H, F))), made(synth.normal(S, f"z{H}.{F}", (M, H, F)))
    l, r = made(synth.normal(S, f"l{H}", (N, H, 1))), made(synth.normal(S, f"r{H}", (M, H, 1)))
    fd, zd, ld, rd = shifted(f, pad), shifted(dz, pad), dev(l), dev(r)
    f, dz, l, r = wide(f), wide(dz), wide(l), wide(r)
    out, a, st = gnnk.gat_aggregate(p.g, fd, ld, rd, 0.2, want_attn=True, want_stats=True)
    ref, ref_a = oracle_gat(p.o, f, l, r, 0.2)
    check(dtype, out, ref, "out")
    check(dtype, a, ref_a, "attention")
    got = gnnk.gat_aggregate_backward(p.g, fd, ld, rd, 0.2, st, zd)
    bounds = gat_grad_bounds(p.o, f, l, r, dz, 0.2)
    for n, x, y, b in zip(("d feat", "d el", "d er"), got, oracle_gat_backward(p.o, f, l, r, 0.2, dz), bounds):
        check_bound(x, y, b, n, 1e-2 if dtype == "bf16" else 1e-5)
