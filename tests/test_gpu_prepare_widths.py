"""The weight preparation at the widths where its kernels change (GPU): the channel
energies' column split (16, 32 and 64 columns a workgroup: K below and at 2048 and 6144),
with ragged columns and row counts around a round of a workgroup's rows, and the Gram
matrices' split (six workgroups a block up to K = 2048, one above); the zigzag's split of
its count; and the precision of a single Jacobi rotation."""
import numpy as np
import pytest
import torch

import paper_2605_28803_amd as oq
from oracle import composite
from tests.test_gpu_prepare import _weight

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
EPS = 2.0 ** -52


@pytest.mark.parametrize("N,K", [(511, 2040), (512, 2047), (33, 2048), (257, 2049), (1, 6143), (129, 6144), (130, 6150)])
def test_channel_energy_column_split(N, K):
    """fp64 sums in another order (within N * 2^-52 relative); equal columns have equal energies bit for bit, wherever
    they lie in a workgroup."""
    print(f"channel_energy N={N} K={K}", flush=True)
    w16 = _weight(6300 + N + K, N, K)
    for j in (1, 15, 16, 31, 63, 64, K - 1):
        w16[:, j] = w16[:, 0]
    wide = torch.zeros((N, K + 3), dtype=torch.float16, device=DEV)
    wide[:, :K] = torch.from_numpy(w16).to(DEV)
    e = oq.channel_energy(wide[:, :K]).cpu().numpy()
    ref = composite.channel_energy(w16.astype(np.float64))
    assert np.all(np.abs(e - ref) <= 2 * N * EPS * ref)
    assert np.all(e[[1, 15, 16, 31, 63, 64, K - 1]] == e[0])


@pytest.mark.parametrize("K,block", [(64, 64), (36, 4), (15 * 4, 4), (16 * 64, 64), (2048, 64), (2052, 4), (2112, 64),
                                     (4096 + 192, 64)])
def test_zigzag_count_split(K, block):
    """The 16 waves' shares of up to 2048 energies, whole and uneven, with few distinct values (ties go to the lower
    index): equal to the oracle."""
    print(f"zigzag K={K} block={block}", flush=True)
    rng = np.random.default_rng(6600 + K)
    for e in (rng.integers(0, 7, K).astype(np.float64), np.zeros(K), rng.standard_normal(K) ** 2):
        perm = oq.zigzag_permutation(torch.from_numpy(e).to(DEV), block).cpu().numpy()
        assert np.array_equal(perm, composite.zigzag_permutation(e, K // block))


@pytest.mark.parametrize("N,K", [(1, 2048), (257, 2048), (1, 2112), (63, 2112), (65, 3072), (1025, 4096)])
def test_block_svd_gram_split(N, K):
    """U_b diag(sigma_b^2) U_b^T is the block's Gram matrix.  The fp64 products are exact and their N-term sums within
    N * 2^-53 of sum |w_i w_j|; the eigendecomposition's backward error is a few hundred roundings (64 sweeps of pairs)
    of the matrix's norm."""
    print(f"block_svd N={N} K={K}", flush=True)
    w16 = _weight(6400 + N + K, N, K)
    perm = np.random.default_rng(K).permutation(K).astype(np.int32)
    wide = torch.full((N, K + 5), 9.0, dtype=torch.float16, device=DEV)
    wide[:, :K] = torch.from_numpy(w16).to(DEV)
    U, lam = oq.block_svd(wide[:, :K], torch.from_numpy(perm).to(DEV))
    U, lam = U.cpu().numpy(), lam.cpu().numpy()
    wb = w16.astype(np.float64)[:, perm].reshape(N, K // 64, 64)
    for b in range(K // 64):
        G = wb[:, b].T @ wb[:, b]
        assert np.linalg.norm((U[b] * lam[b]) @ U[b].T - G) <= (N + 640) * EPS * np.trace(G)


@pytest.mark.parametrize("seed,spread", [(0, 0.0), (1, 0.0), (2, 2.0), (3, 4.0)])
def test_block_svd_single_rotations(seed, spread):
    """A block whose channels overlap only in pairs takes one rotation a pair, so its angle's own error shows.  A
    vector of a 2 x 2 block G is good to a few roundings: |G v - (v G v) v| <= 8 * 2^-53 |G| |v| (angle, sine and cosine,
    one product each, all within 2 ulp).  An angle of 2^-46 whose remainder is dropped leaves 100 times that."""
    rng = np.random.default_rng(6500 + seed)
    w16 = np.zeros((64, 64), np.float16)
    order = rng.permutation(64)
    for i in range(32):
        w16[2 * i:2 * i + 2, order[2 * i:2 * i + 2]] = rng.standard_normal((2, 2)) * 2.0 ** rng.uniform(-spread, spread)
    U, lam = oq.block_svd(torch.from_numpy(w16).to(DEV), torch.arange(64, dtype=torch.int32, device=DEV))
    U, lam = U.cpu().numpy()[0].astype(np.longdouble), lam.cpu().numpy()[0]
    w = w16.astype(np.longdouble)
    G = w.T @ w
    for i in range(64):
        v = U[:, i]
        assert np.count_nonzero(v) <= 2
        scale = np.linalg.norm((np.abs(G) @ np.abs(v)).astype(np.float64))
        assert np.linalg.norm((G @ v - (v @ G @ v) * v).astype(np.float64)) <= 8 * 2.0 ** -53 * scale
        assert abs(float(v @ G @ v) - lam[i]) <= 16 * 2.0 ** -53 * scale
