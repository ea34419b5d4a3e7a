"""The composite rotation's chunk widths at their edges (GPU).

Every width built that holds a whole row (512, 1024, 1536, 2048, 3072 and 4096,
with 16- and, folded and with more than 1024 rows, 32-row tiles), other widths,
which take the other kernels, and every chunk width above 4096 with its raw-row sizes, at one
row, one row short of and past a tile, and past the 1024-row rule: codes by the
boundary rule of the oracle fed the same block matrices, token scales within the
same bound."""
import numpy as np
import pytest
import torch

import paper_2605_28803_amd as oq
from oracle import composite
from tests import parity
from tests.test_gpu_composite import DEV, U32, _device, _operands, _tau

pytestmark = pytest.mark.gpu

CASES = [(1, 512), (17, 512), (1040, 512), (15, 1024), (33, 1024), (1025, 1024), (31, 1536), (17, 2048), (47, 2048),
         (1, 3072), (17, 3072), (1, 4096), (47, 4096), (1025, 4096),
         (17, 448), (17, 576), (17, 2560), (17, 3584),                        # no instance of their own
         (1, 8192), (31, 8192), (17, 12288), (17, 10240), (33, 9216), (17, 8704), (15, 16384)]


@pytest.mark.parametrize("M,K", CASES)
@pytest.mark.parametrize("folded", [False, True])
def test_widths(M, K, folded):
    print(f"composite width M={M} K={K} folded={folded}", flush=True)
    x16, _, perm, r16 = _operands(6100 + M + K, M, 96, K)
    p, rt = _device(perm, r16)
    xin = np.ascontiguousarray(x16[:, perm]) if folded else x16
    # Rows in a wider buffer, codes into a sentinel-padded one.
    buf = torch.full((M, K + 8), 3.0, dtype=torch.float16, device=DEV)
    buf[:, :K] = torch.from_numpy(xin).to(DEV)
    out = torch.full((M + 1, K // 2), 0x55, dtype=torch.uint8, device=DEV)
    Xq, xs = oq.rotate_quantize_act_composite(buf[:, :K], None if folded else p, rt, Xq=out[:M])
    torch.cuda.synchronize()
    q_o, xs_o, r_o = composite.rotate_quantize_composite(x16, perm, r16.astype(np.float64))
    tau = _tau(x16, perm, r16)
    parity.check_codes(parity.unpack_int4(Xq.cpu().numpy()), q_o, r_o, tau)
    rel = np.abs(xs.cpu().numpy().astype(np.float64) - xs_o) / np.where(xs_o > 0, xs_o, 1.0)
    assert np.all(rel <= tau / 7 + 4 * U32)
    assert torch.all(out[M] == 0x55).item()


def test_single_width_calls_overlap_on_streams():
    """Rows of one chunk use no workspace: calls on two streams do not disturb each other."""
    M, K = 900, 2048
    x16, _, perm, r16 = _operands(6200, M, 96, K)
    p, rt = _device(perm, r16)
    X = torch.from_numpy(x16).to(DEV)
    ref, rs = oq.rotate_quantize_act_composite(X, p, rt)
    reff, rsf = oq.rotate_quantize_act_composite(X, None, rt)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    got = []
    for i in range(8):
        with torch.cuda.stream(streams[i & 1]):
            got.append(oq.rotate_quantize_act_composite(X, p if i % 4 < 2 else None, rt))
    torch.cuda.synchronize()
    for i, (q, s) in enumerate(got):
        a, b = (ref, rs) if i % 4 < 2 else (reff, rsf)
        assert torch.equal(q, a) and torch.equal(s, b)
