"""The percentile's two routes at the edges of the rule between them (GPU).

The high-percentile route (maxima of row groups, then only the groups above the
m-th largest maximum) and the radix route must both return the exact nearest-rank
element, whatever the order of the rows: random, sorted (all large values in one
group), constant columns, ties across the rank, infinities and NaN (ordered above
+inf), row counts around a group's edges, and the limits m <= groups and
(m - 1) * rows per group <= 2048."""
import numpy as np
import pytest
import torch

import paper_2605_28803_amd as oq

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")

# n, K, p: one row; one group per row; the first two-row groups; 99.9% at the listed
# sizes; the last n the first route takes at 99.9% (22528: m = 23, 88 rows a group) and the next
# ones; ranks m = groups and m = groups + 1; the maximum; the median.
CASES = [(1, 8, 99.9), (255, 36, 50.0), (256, 64, 0.1), (257, 64, 99.0), (513, 260, 60.0), (1000, 100, 74.5),
         (8160, 512, 99.9), (16384, 256, 99.9), (22528, 64, 99.9), (23000, 64, 99.9), (24000, 64, 99.9),
         (512, 64, 50.2), (512, 64, 50.0), (40000, 64, 100.0), (3001, 128, 50.0)]


def _ref(y, p):
    n = y.shape[0]
    k = min(max(-(-int(round(p * 1e6)) * n // 100000000), 1), n)
    bits = np.sort(y.view(np.uint32) & 0x7FFFFFFF, axis=0)[k - 1]
    return bits.view(np.float32)


@pytest.mark.parametrize("n,K,p", CASES)
@pytest.mark.parametrize("aligned", [True, False])
def test_percentile_exact(n, K, p, aligned):
    print(f"percentile n={n} K={K} p={p} aligned={aligned}", flush=True)
    rng = np.random.default_rng(n + K)
    y = (rng.standard_normal((n, K)) * np.exp(rng.standard_normal(K))).astype(np.float32)
    y[:, 0] = np.sort(y[:, 0])
    y[:, 1] = -np.sort(-np.abs(y[:, 1]))
    y[:, 2] = 0.0
    y[:, 3] = np.where(np.arange(n) % 3 == 0, -2.5, 2.5)
    y[:, 4] = np.round(y[:, 4])
    y[n // 2, 5] = np.inf
    y[: n // 4, 6] = -np.inf
    y[:, 7] = -0.0
    y[n // 3, 7] = np.nan
    if aligned:
        Y = torch.from_numpy(y).to(DEV)
    else:  # an odd row stride and a base that is not 16-byte aligned
        big = torch.zeros((n, K + 3), dtype=torch.float32, device=DEV)
        Y = big[:, 1:K + 1]
        Y.copy_(torch.from_numpy(y))
    d = oq.calibrate_step_scales(Y, p=p, qmax=1.0).cpu().numpy()
    ref = _ref(np.ascontiguousarray(y), p)
    assert np.array_equal(d, ref, equal_nan=True)
    d7 = oq.calibrate_step_scales_noalloc(Y, p=p, qmax=7.0).cpu().numpy()
    assert np.array_equal(d7, (ref.astype(np.float64) / 7.0).astype(np.float32), equal_nan=True)
