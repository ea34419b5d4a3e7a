"""The exchange of row maxima between the chunks of a composite rotation (GPU): calls on
several streams at once, and captured calls that are replayed, give what a call alone
gives; every form that exchanges (online permutation and folded, each chunk width, a
partial last tile); and a chunk that gives up a wait always shows in the token scales."""
import ctypes as C

import pytest
import torch

import paper_2605_28803_amd as oq
from paper_2605_28803_amd import _lib

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")

# K, folded: chunks of 4096, 2048, 1024 and 512 channels, and 4096 channels folded with more than 1024 rows.
FORMS = [(16384, False), (8192, False), (6144, False), (5120, False), (4608, False), (16384, True), (4608, True),
         (4096, True)]


def _inputs(M, K, folded, scale):
    g = torch.Generator(device=DEV).manual_seed(M + K)
    X = (torch.randn((M, K), generator=g, device=DEV) * scale).half()
    perm = None if folded else torch.randperm(K, generator=g, device=DEV).int()
    Rt = (torch.randn((K // 64, 64, 64), generator=g, device=DEV) / 8).half().view(torch.int16)
    return X, perm, Rt


@pytest.mark.parametrize("K,folded", FORMS)
def test_calls_overlap_on_streams(K, folded):
    """Four streams, each with its own rows (of different magnitudes, so that a maximum of another call would show)."""
    print(f"exchange streams K={K} folded={folded}", flush=True)
    ins = [_inputs(1100 + 17 * i, K, folded, 4.0 ** i) for i in range(4)]
    ref = [oq.rotate_quantize_act_composite(*x) for x in ins]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in ins]
    out = [[], [], [], []]
    for _ in range(6):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                out[i].append(oq.rotate_quantize_act_composite(*ins[i]))
    torch.cuda.synchronize()
    for i, (q, s) in enumerate(ref):
        assert torch.isfinite(s).all()
        for q2, s2 in out[i]:
            assert torch.equal(q2, q) and torch.equal(s2, s)


@pytest.mark.parametrize("K,folded", [(8192, False), (4096, True)])
def test_captured_calls(K, folded):
    """A call captured without any before it (nothing is allocated), replayed over other inputs and outputs that hold
    other values, with calls of its own between."""
    print(f"exchange graph K={K} folded={folded}", flush=True)
    M = 1039
    X, perm, Rt = _inputs(M, K, folded, 1.0)
    other = _inputs(M, K, folded, 8.0)[0].flip(0).contiguous()
    Xq = torch.empty((M, K // 2), dtype=torch.uint8, device=DEV)
    xs = torch.empty((M,), device=DEV)
    src = X.clone()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        oq.rotate_quantize_act_composite(src, perm, Rt, Xq=Xq, x_scale=xs)
    for i in range(4):
        src.copy_(X if i % 2 == 0 else other)
        Xq.fill_(i)
        xs.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        q, s = oq.rotate_quantize_act_composite(src, perm, Rt)
        torch.cuda.synchronize()
        assert torch.equal(Xq, q) and torch.equal(xs, s)


@pytest.mark.parametrize("K,folded,chunks", [(16384, False, 4), (5120, False, 5), (4608, True, 9), (4096, True, 4)])
def test_a_chunk_that_gives_up_shows_in_the_scales(K, folded, chunks):
    """Each chunk in turn gives up its wait for the maxima, then its wait for the acknowledgements: no token scale is a
    number, and nothing past the outputs is written.  A call with no such chunk gives the ordinary result."""
    M = 1031
    X, perm, Rt = _inputs(M, K, folded, 1.0)
    f = _lib.load().oq_test_composite_give_up
    f.argtypes = [C.c_void_p, C.c_int64, C.c_int64, C.c_int64, C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p, C.c_int32,
                  C.c_void_p]
    f.restype = C.c_int
    ref, rs = oq.rotate_quantize_act_composite(X, perm, Rt)
    for chunk in [-1] + list(range(2 * chunks)):
        print(f"give up K={K} folded={folded} chunk={chunk}", flush=True)
        Xq = torch.zeros((M + 1, K // 2), dtype=torch.uint8, device=DEV)
        xs = torch.full((M + 1,), 5.0, device=DEV)
        st = f(X.data_ptr(), M, K, K, None if perm is None else perm.data_ptr(), Rt.data_ptr(), Xq.data_ptr(),
               xs.data_ptr(), chunk, torch.cuda.current_stream().cuda_stream)
        assert st == 0
        torch.cuda.synchronize()
        if chunk < 0:
            assert torch.equal(Xq[:M], ref) and torch.equal(xs[:M], rs)
        else:
            assert torch.isnan(xs[:M]).all()
        assert not Xq[M].any() and xs[M].item() == 5.0
