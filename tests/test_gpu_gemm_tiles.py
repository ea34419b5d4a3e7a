"""Every tiling of the M > 64 product at its edges (GPU).

The launcher picks one of seven W4A4 and three W4A8 tilings from an estimate
of their times; each shape below takes the one named beside it (test_gemm_rules
asks the launcher's rule, on the host), with rows and columns that are not a
multiple of its tile, a last K stage that is partly empty (K % 64 == 0 is all
that is asked), a single stage, and in the deep cases every K group ending on a
short stage.  int32 accumulators are exact;
fp16 / bf16 outputs are one rounding of an fp32 value (2^-11, 2^-8 of the
value, plus the fp32 epilogue's few ulp), against the float64 oracle.  The
residual outputs of the same tilings run through a DiT block (oracle on the
library's own site values)."""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2605_28803_amd as oq
from oracle import dit as odit
from oracle import linear
from tests import dit_parity, parity
from workloads import configs, dit_inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")

W4A4 = [
    (4000, 4092, 4160),                    # 256 x 256; 64 codes in the last 256-code stage
    (4000, 4092, 4288),                    # 256 x 256; 192 codes
    (2000, 4092, 1344), (816, 2560, 2112),  # 128 x 128; 64 codes
    (1000, 6100, 1600), (1100, 8200, 1344),  # 128 x 64; 64 codes
    (520, 1000, 6208), (130, 4100, 4160),  # 64 x 64, four K groups; 64 codes in the last 512-code stage
    (992, 1536, 6528),                     # 64 x 64, four K groups; 384 codes
    (1000, 1544, 576), (300, 520, 320),    # 64 x 64; tails
    (70, 100, 64), (65, 100, 192), (1000, 2500, 256),  # 64 x 64, 128-code stages; one half full, one and a half, two
    (1000, 4100, 64), (3010, 2052, 192),   # 128 x 64, 128-code stages
]
# Few rows: 16 | 17 and 8192 | 8193 columns (the small-M kernel and the 64 x 64 tilings), one row block deep and wide, and
# the small-M kernel's rounds of no whole unit (K = 64), one, two and more units per wave (K = 2048 and its neighbours,
# both widths), and a 20-row product of more than 8192 columns that stays on it (K = 576).
FEW = [(16, 8256, 1088), (17, 8192, 1088), (17, 8200, 1088), (64, 8200, 4160), (1, 16384, 8256), (16, 16392, 8192),
       (5, 4100, 2048), (5, 4096, 2048), (16, 4100, 2112), (3, 2560, 2112), (5, 5000, 1984), (40, 5000, 1984),
       (1, 104, 64), (2, 100, 64), (50, 4100, 64), (20, 8232, 576)]
W4A8 = [
    (4000, 4092, 4160),                    # 256 x 256; half a 128-code stage
    (1000, 6100, 1600), (816, 2560, 2112),  # 128 x 128
    (70, 100, 64), (300, 520, 320), (1000, 1544, 576),  # 64 x 64, two K groups
    (1000, 9000, 192),                     # 128 x 128; short K
]


def _run(M, N, K, a8):
    rng = np.random.default_rng(M + 5 * N + 11 * K)
    q = rng.integers(-127, 128, size=(M, K)) if a8 else rng.integers(-7, 8, size=(M, K))
    qw = rng.integers(-7, 8, size=(N, K))
    A = torch.from_numpy(q.astype(np.int8) if a8 else parity.pack_int4(q)).to(DEV)
    W = torch.from_numpy(parity.pack_int4(qw)).to(DEV)
    xs = rng.uniform(0.01, 2.0, M).astype(np.float32)
    ws = rng.uniform(1e-4, 1e-2, N).astype(np.float32)
    bias = (rng.standard_normal(N) * 0.1).astype(np.float16)
    acc = linear.int_gemm(q, qw)
    got = (oq.w4a8_gemm_i32 if a8 else oq.w4a4_gemm_i32)(A, W)
    assert np.array_equal(got.cpu().numpy().astype(np.int64), acc)
    ref = linear.dequant(acc, xs, ws, bias.astype(np.float64))
    ldy = (N + 7) // 8 * 8 + 16
    for out, dt, ulp in ((oq.OUT_F16, torch.float16, 2.0 ** -11), (oq.OUT_BF16, torch.bfloat16, 2.0 ** -8)):
        buf = torch.full((M + 1, ldy), 7.0, dtype=dt, device=DEV)
        (oq.w4a8_linear if a8 else oq.w4a4_linear)(A, torch.from_numpy(xs).to(DEV), W, torch.from_numpy(ws).to(DEV),
                                                   bias=torch.from_numpy(bias).to(DEV), out_dtype=out,
                                                   Y=buf[:M, :N])
        y = buf[:M, :N].float().cpu().numpy().astype(np.float64)
        # |acc xs ws| enters the fp32 sum with the bias: three roundings of at
        # most 2^-24 of either term, then the output's.
        prod = np.abs(ref - bias.astype(np.float64))
        bound = ulp * np.abs(ref) + 2.0 ** -22 * (prod + np.abs(ref)) + 2.0 ** -24
        assert (np.abs(y - ref) <= bound).all()
        assert torch.all(buf[M] == 7.0).item() and torch.all(buf[:, N:] == 7.0).item()


@pytest.mark.parametrize("M,N,K", W4A4)
def test_w4a4_tilings(M, N, K):
    print(f"w4a4 tiling M={M} N={N} K={K}", flush=True)
    _run(M, N, K, False)


@pytest.mark.parametrize("a8", [False, True])
@pytest.mark.parametrize("M,N,K", FEW)
def test_few_rows(M, N, K, a8):
    print(f"few rows M={M} N={N} K={K} a8={a8}", flush=True)
    _run(M, N, K, a8)


@pytest.mark.parametrize("M,N,K", W4A8)
def test_w4a8_tilings(M, N, K):
    print(f"w4a8 tiling M={M} N={N} K={K}", flush=True)
    _run(M, N, K, True)


# Residual (and GELU) outputs: o and ff2 of 2000 rows take the 128 x 64 and 128 x 128
# tilings, ff0 the 128 x 128 one; 8192 rows of a 2048-wide model the 256 x 256 one;
# a 256-wide model the two of short K (1008 rows 64 x 64, 12816 rows 128 x 64).
RESID = {
    "gr00t_2000": (dataclasses.replace(configs.DIT_GR00T, name="gr00t_2000", n_blocks=2, batch=125, prefix=20), (0, 1)),
    "pi_8192": (dataclasses.replace(configs.DIT_PI, name="pi_8192", n_blocks=1, batch=128, tokens=64, hidden=2048,
                                    mlp=2048, n_heads=16, head_dim=128, prefix=16, steps=2), (0,)),
    "gr00t_narrow": (dataclasses.replace(configs.DIT_GR00T, name="gr00t_narrow", n_blocks=1, batch=63, hidden=256, mlp=256,
                                         n_heads=4, head_dim=64, prefix=5, steps=2), (0,)),
    "gr00t_narrow_801": (dataclasses.replace(configs.DIT_GR00T, name="gr00t_narrow_801", n_blocks=1, batch=801, hidden=256,
                                             mlp=256, n_heads=4, head_dim=64, prefix=5, steps=2), (0,)),
}


@pytest.mark.parametrize("name", sorted(RESID))
def test_residual_tilings(name):
    cfg, layers = RESID[name]
    inp = dit_inputs.make_dit_inputs(cfg, n_blocks=cfg.n_blocks, batch=cfg.batch)
    model = oq.DiT(cfg, inp, device="cuda:0")
    try:
        r = odit.in_projection(inp["w"], inp["x0"])
        for l in layers:
            print(f"{name}: block {l}", flush=True)
            r = dit_parity.assert_block(cfg, inp, model, l, 0, r)
    finally:
        model.close()
