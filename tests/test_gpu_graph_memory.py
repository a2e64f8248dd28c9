"""The memory of a graph build: what a handle keeps (28 bytes per edge and its
tables), temporaries that go back to the caller, and the optional rows listed
by neighbour, which only graphs that gain from them ask for and any caller can
decline; and the one-buffer constructors, which keep no listing."""
import ctypes

import numpy as np
import pytest
import torch

import oracle as orc
from paper_1909_01315_amd import gnnk
from _gpu import Pair, assert_close, check_formats, dev

pytestmark = pytest.mark.gpu
N, E = 3000, (1 << 20) + 77


def edges(order):
    rng = np.random.default_rng(4)
    src, dst = ((rng.random(E) ** 3 * N).astype(np.int32) for _ in range(2))
    if order == "sorted":
        at = np.lexsort((src, dst))
        src, dst = src[at], dst[at]
    return src, dst


def kept(g):
    return sum(t.numel() for t in g._keep if t is not None)


@pytest.mark.parametrize("order", ["sorted", "arrival"])
@pytest.mark.parametrize("neighbour_lists", [True, False])
def test_a_handle_keeps_its_arrays_alone(order, neighbour_lists):
    src, dst = edges(order)
    o = orc.OGraph(src, dst, N, N)
    g = gnnk.Graph.from_coo(dev(src), dev(dst), N, N, neighbour_lists=neighbour_lists)
    info = g.info()
    lists = order == "arrival" and neighbour_lists
    assert info["neighbour_lists"] == (3 if lists else 0)
    assert (info["lists_bytes"] >= 16 * E) == lists and (info["lists_bytes"] == 0) != lists
    # 28 bytes per edge, and tables of hub rows and segments: at most 2 E / 64
    # segments of 36 bytes in each of four tables
    assert info["kept_bytes"] <= kept(g) - info["lists_bytes"] <= 28 * E + 4 * 36 * 2 * E // 64 + 100 * N + (1 << 16)
    p = Pair.__new__(Pair)
    p.o, p.g = o, g
    check_formats(p)
    X = np.random.default_rng(1).standard_normal((N, 2, 8)).astype(np.float32)
    assert_close(gnnk.gspmm(g, "copy_lhs", "sum", dev(X)), orc.gspmm(o, "copy_lhs", "sum", X))
    dx, _ = gnnk.gspmm_backward(g, "copy_lhs", "sum", dev(X), None, dev(X))
    assert_close(dx, orc.gspmm_backward(o, "copy_lhs", "sum", X, None, X)[0])
    g.destroy()


def test_temporaries_go_back_to_the_allocator():
    src, dst = (dev(x) for x in edges("arrival"))
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    g = gnnk.Graph.from_coo(src, dst, N, N)
    # (the allocator leaves up to 1 MiB of a large block with its tensor)
    assert torch.cuda.memory_allocated() - before <= kept(g) + (2 << 20) < kept(g) + 20 * E
    g.destroy()


def test_the_build_runs_on_another_stream():
    """temporaries are taken from the build stream's pool: work of the current
    stream that takes the same memory next cannot overwrite them"""
    src, dst = edges("arrival")
    s, d = dev(src), dev(dst)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    g = gnnk.Graph.from_coo(s, d, N, N, stream=side)
    noise = [torch.full((20 * E,), 255, dtype=torch.uint8, device="cuda") for _ in range(3)]
    torch.cuda.synchronize()
    p = Pair.__new__(Pair)
    p.o, p.g = orc.OGraph(src, dst, N, N), g
    check_formats(p)
    del noise
    g.destroy()


def test_one_buffer():
    lib = gnnk.load()
    src, dst = edges("arrival")
    s, d = dev(src), dev(dst)
    n = ctypes.c_size_t(0)
    assert lib.graph_workspace_bytes(N, N, E, gnnk.I32, ctypes.byref(n)) == gnnk.OK
    ws = torch.empty(n.value, dtype=torch.uint8, device="cuda")

    def create(size):
        h = ctypes.c_void_p()
        st = lib.graph_create_coo(N, N, E, s.data_ptr(), d.data_ptr(), gnnk.I32, ws.data_ptr(), size,
                                  torch.cuda.current_stream().cuda_stream, ctypes.byref(h))
        return st, h

    assert create(20 * E)[0] == gnnk.ENOMEM
    st, h = create(n.value)
    assert st == gnnk.OK
    g = gnnk.Graph(h, [ws], N, N, E)
    info = g.info()
    assert info["neighbour_lists"] == 0 and info["kept_bytes"] < info["workspace_bytes"] <= n.value
    torch.cuda.synchronize()
    ws[info["kept_bytes"]:] = 255  # free once the build is done
    X = np.random.default_rng(1).standard_normal((N, 2, 8)).astype(np.float32)
    ref = orc.gspmm(orc.OGraph(src, dst, N, N), "copy_lhs", "sum", X)
    assert_close(gnnk.gspmm(g, "copy_lhs", "sum", dev(X)), ref)
    # the size that graph_info names is enough for the same graph, and one byte
    # less is not
    g.destroy()
    need = info["workspace_bytes"]
    assert create(need - 1)[0] == gnnk.ENOMEM
    st, h = create(need)
    assert st == gnnk.OK
    g = gnnk.Graph(h, [ws], N, N, E)
    assert_close(gnnk.gspmm(g, "copy_lhs", "sum", dev(X)), ref)
    g.destroy()


def test_memory_that_a_build_refuses():
    lib = gnnk.load()
    src, dst = (dev(x) for x in edges("arrival"))
    w, t = ctypes.c_size_t(0), ctypes.c_size_t(0)
    assert lib.graph_build_bytes(N, N, E, gnnk.I32, ctypes.byref(w), ctypes.byref(t)) == gnnk.OK
    ws = torch.empty(w.value + 256, dtype=torch.uint8, device="cuda")
    tmp = torch.empty(t.value + 256, dtype=torch.uint8, device="cuda")
    odd = torch.empty(20 * E, dtype=torch.uint8, device="cuda")
    asked = []

    @ctypes.CFUNCTYPE(ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t)
    def none(_, n):
        asked.append(n)
        return None

    @ctypes.CFUNCTYPE(ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t)
    def misaligned(_, n):
        return odd.data_ptr() + 4

    def build(ws_ptr, ws_n, tmp_ptr, tmp_n, lists):
        mem = gnnk._MEMORY.pack(ws_ptr, ws_n, tmp_ptr, tmp_n,
                                ctypes.cast(lists, ctypes.c_void_p).value if lists else 0, 0)
        h = ctypes.c_void_p()
        st = lib.graph_build_coo(N, N, E, src.data_ptr(), dst.data_ptr(), gnnk.I32, mem,
                                 torch.cuda.current_stream().cuda_stream, ctypes.byref(h))
        if h.value:
            assert st == gnnk.OK
            g = gnnk.Graph(h, [ws], N, N, E)
            listed = g.info()["neighbour_lists"]
            g.destroy()
            return listed
        return ("refused", st)

    W, T = ws.data_ptr(), tmp.data_ptr()
    assert build(W, w.value, T, t.value - 1, None) == ("refused", gnnk.ENOMEM)
    assert build(W, 28 * E, T, t.value, None) == ("refused", gnnk.ENOMEM)
    assert build(W + 16, w.value, T, t.value, None) == ("refused", gnnk.EINVAL)
    assert build(W, w.value, T + 16, t.value, None) == ("refused", gnnk.EINVAL)
    assert build(W, w.value, 0, t.value, None) == ("refused", gnnk.ENOMEM)
    assert build(W, w.value, T, t.value, misaligned) == ("refused", gnnk.EINVAL)
    assert build(W, w.value, T, t.value, None) == 0
    assert build(W, w.value, T, t.value, none) == 0 and len(asked) == 1 and asked[0] >= 16 * E
    torch.cuda.synchronize()
