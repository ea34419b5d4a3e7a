"""Performance cases of the W4A4 rotated linear library.

Each case is work that a program built on the library has it do, through the
Python binding: single rotated linears from one decoded token to a 16384-token
prefill in every quantization mode, the four linears of a backbone layer, the
offline calibration and weight preparation, and denoising steps of the two DiT
action heads.  Inputs are seeded and synthetic (activations with outlier
channels, Gaussian weights), made on the GPU.
"""
import math
import zlib

import numpy as np
import torch

import paper_2605_28803_amd as oq

DEV = "cuda:0"

# The two DiT action heads (the Pi-0.5 action expert and a GR00T-N1.5 style
# head): hidden size, MLP, heads x head_dim, Euler steps, action channels.
PI = {"arch": "pi", "hidden": 1024, "mlp": 4096, "n_heads": 8, "head_dim": 128, "steps": 10, "action_dim": 32}
GR00T = {"arch": "gr00t", "hidden": 1536, "mlp": 6144, "n_heads": 32, "head_dim": 48, "steps": 4, "action_dim": 32}


def listed():
    return [
        # One rotated linear of the Pi-0.5 action expert (a DiT-sized batch of
        # action tokens): two launches, where latency is everything.
        {"name": "linear_64x1024x1024", "kind": "linear", "mode": "tiled", "M": 64, "K": 1024, "N": 1024,
         "out": "f16", "bias": False},
        # Decoding a few sequences through the backbone's gate|up: the weight
        # stream of a single pass.
        {"name": "decode_gate_up_5", "kind": "linear", "mode": "token", "M": 5, "K": 2048, "N": 32768, "out": "bf16",
         "bias": False},
        # Backbone prefill of one prompt (816 image and text tokens): the four
        # linears of a Gemma-2B-shaped layer.
        {"name": "prefill_layer_816", "kind": "layer", "M": 816, "hidden": 2048, "kv": 256, "ffn": 16384},
        # An ordinary prefill linear with bias, rows not a multiple of a tile.
        {"name": "linear_4000x4096x4096", "kind": "linear", "mode": "token", "M": 4000, "K": 4096, "N": 4096,
         "out": "bf16", "bias": True},
        # A large batched prefill.
        {"name": "linear_16384x8192x8192", "kind": "linear", "mode": "token", "M": 16384, "K": 8192, "N": 8192,
         "out": "f16", "bias": False},
        # The paper's deployment mode (8-bit tokens, int4 weights) at the
        # backbone's gate|up.
        {"name": "w4a8_gate_up_816", "kind": "linear", "mode": "token8", "M": 816, "K": 2048, "N": 32768, "out": "f16",
         "bias": False},
        # The full composite rotation (zigzag permutation and U_b H_64) online
        # in front of the backbone's down linear, a batch of five prompts.
        {"name": "composite_down_4080", "kind": "linear", "mode": "composite", "M": 4080, "K": 16384, "N": 2048,
         "out": "f16", "bias": False},
        # Static per-channel steps at the GR00T head's second MLP linear, a
        # batch of 62 samples of 16 action tokens.
        {"name": "static_ff2_992", "kind": "linear", "mode": "static", "M": 992, "K": 6144, "N": 1536, "out": "f16",
         "bias": True},
        # Calibration of static steps: rotation to fp32 and the exact 99.9th
        # percentile of every channel over ten prompts' tokens.
        {"name": "calibrate_8160x2048", "kind": "calibrate", "M": 8160, "K": 2048},
        # Offline preparation of a backbone q|k|v weight for the composite
        # rotation.
        {"name": "prepare_qkv_2560x2048", "kind": "prepare", "N": 2560, "K": 2048},
        # One denoising step of the Pi-0.5 action expert: 50 action tokens
        # against a prefix of 816.
        {"name": "pi_step", "kind": "dit", "arch": "pi", "n_blocks": 18, "batch": 1, "tokens": 50, "prefix": 816},
        # One denoising step of the GR00T-style head over a batch of 64
        # samples, 300 conditioning tokens each.
        {"name": "gr00t_step", "kind": "dit", "arch": "gr00t", "n_blocks": 16, "batch": 64, "tokens": 16,
         "prefix": 300},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["linear"] * 9 + ["layer", "calibrate", "prepare", "dit", "dit"])
    if kind == "linear":
        mode = rng.choice(["token", "token", "token", "tiled", "token8", "composite", "folded", "static"])
        while True:
            # Input sizes of the models and their neighbours: powers of two and
            # three times one.
            K = rng.choice([1, 1, 1, 3]) * 2 ** rng.randint(8, 14)
            if not 512 <= K <= 16384:
                continue
            M = _log(rng, 1, 64 if mode == "tiled" else 16384)
            N = 8 * _log(rng, 64, 4096)
            if M * N * K <= 16384 * 8192 * 8192 and (mode not in ("composite", "folded") or M * K <= 2 ** 26):
                break
        return {"kind": "linear", "mode": mode, "M": M, "K": K, "N": N, "out": rng.choice(["f16", "bf16"]),
                "bias": rng.random() < 0.5}
    if kind == "layer":
        return {"kind": "layer", "M": _log(rng, 128, 3000), "hidden": 2048, "kv": 256, "ffn": 16384}
    if kind == "calibrate":
        return {"kind": "calibrate", "M": _log(rng, 400, 16384), "K": rng.choice([1024, 1536, 2048, 4096])}
    if kind == "prepare":
        return {"kind": "prepare", "N": 8 * _log(rng, 64, 1024), "K": rng.choice([1024, 1536, 2048, 4096])}
    if rng.random() < 0.5:
        return {"kind": "dit", "arch": "pi", "n_blocks": rng.randint(4, 18), "batch": rng.choice([1, 1, 2, 4]),
                "tokens": rng.randint(10, 64), "prefix": rng.randint(256, 900)}
    return {"kind": "dit", "arch": "gr00t", "n_blocks": 2 * rng.randint(2, 8), "batch": _log(rng, 4, 64),
            "tokens": 16, "prefix": rng.randint(100, 300)}


# ---------------------------------------------------------------------------
# Seeded inputs, the same for the library and for the 64-bit reference.
# ---------------------------------------------------------------------------


class _Draw:
    """Named tensors drawn on the GPU, each from a stream of its own."""

    def __init__(self, seed):
        self.seed = seed

    def _gen(self, name):
        g = torch.Generator(device=DEV)
        g.manual_seed((self.seed * 1000003 + zlib.crc32(name.encode())) & 0x7FFFFFFFFFFF)
        return g

    def normal(self, name, *shape, std=1.0, mean=0.0):
        return torch.randn(shape, generator=self._gen(name), device=DEV).mul_(std).add_(mean)

    def uniform(self, name, *shape, lo=0.0, hi=1.0):
        return torch.rand(shape, generator=self._gen(name), device=DEV).mul_(hi - lo).add_(lo)

    def order(self, name, n):
        return torch.randperm(n, generator=self._gen(name), device=DEV)

    def tokens(self, name, M, K, share=0.01, factor=50.0):
        """fp16 activation rows with a share of outlier channels."""
        x = self.normal(name, M, K)
        x[:, self.order(name + "/outliers", K)[: max(1, round(share * K))]] *= factor
        return x.half()

    def weight(self, name, N, K):
        return self.normal(name, N, K, std=0.02).half()


def _block(K):
    return K & -K


def _linear_inputs(case, seed):
    d = _Draw(seed)
    M, K, N = case["M"], case["K"], case["N"]
    i = {"x": d.tokens("x", M, K), "w": d.weight("w", N, K), "b": _block(K),
         "bias": d.normal("bias", N).half() if case["bias"] else None}
    if case["mode"] in ("composite", "folded"):
        i["perm"] = d.order("perm", K).int() if case["mode"] == "composite" else None
        q, r = np.linalg.qr(d.normal("u", K // 64, 64, 64).double().cpu().numpy())
        i["u"] = torch.from_numpy(q * np.sign(np.diagonal(r, axis1=1, axis2=2))[:, None, :]).to(DEV)
    if case["mode"] == "static":
        # Steps near the 99.9th percentile of a rotated channel over q_max.
        rms = i["x"].float().square().mean().sqrt().item()
        i["delta"] = torch.exp(d.normal("delta", K, std=0.1)) * (3.3 * rms / 7.0)
    return i


def _prepare_linear(case, seed):
    i = _linear_inputs(case, seed)
    M, K, N = case["M"], case["K"], case["N"]
    s = {"mode": case["mode"], "x": i["x"], "b": i["b"], "bias": i["bias"],
         "dt": oq.OUT_F16 if case["out"] == "f16" else oq.OUT_BF16}
    s["y"] = torch.empty((M, N), dtype=torch.float16 if case["out"] == "f16" else torch.bfloat16, device=DEV)
    s["xs"] = torch.empty((M,), dtype=torch.float32, device=DEV)
    if case["mode"] == "tiled":
        s["xq"] = torch.empty((oq.tiled_bytes(M, K),), dtype=torch.uint8, device=DEV)
    elif case["mode"] == "token8":
        s["xq"] = torch.empty((M, K), dtype=torch.int8, device=DEV)
    else:
        s["xq"] = torch.empty((M, K // 2), dtype=torch.uint8, device=DEV)
    if case["mode"] in ("composite", "folded"):
        s["perm"], s["rt"] = i["perm"], oq.block_rotations(i["u"])
        s["wq"], s["ws"] = oq.rotate_quantize_act_composite(i["w"], i["perm"], s["rt"])
    elif case["mode"] == "static":
        s["delta"] = i["delta"]
        s["wq"], s["ws"] = oq.quantize_weights_step(i["w"], i["b"], i["delta"])
    else:
        s["wq"], s["ws"] = oq.quantize_weights(i["w"], i["b"])
    return s


def _run_linear(s):
    mode = s["mode"]
    if mode == "tiled":
        oq.rotate_quantize_act_tiled(s["x"], s["b"], Xt=s["xq"], x_scale=s["xs"])
        return oq.w4a4_linear_tiled(s["xq"], s["xs"], s["wq"], s["ws"], s["bias"], s["dt"], Y=s["y"])
    if mode == "token8":
        oq.rotate_quantize_act_i8(s["x"], s["b"], Xq8=s["xq"], x_scale=s["xs"])
        return oq.w4a8_linear(s["xq"], s["xs"], s["wq"], s["ws"], s["bias"], s["dt"], Y=s["y"])
    if mode in ("composite", "folded"):
        oq.rotate_quantize_act_composite(s["x"], s["perm"], s["rt"], Xq=s["xq"], x_scale=s["xs"])
    elif mode == "static":
        oq.rotate_quantize_act_static(s["x"], s["b"], s["delta"], Xq=s["xq"], x_scale=s["xs"])
    else:
        oq.rotate_quantize_act(s["x"], s["b"], Xq=s["xq"], x_scale=s["xs"])
    return oq.w4a4_linear(s["xq"], s["xs"], s["wq"], s["ws"], s["bias"], s["dt"], Y=s["y"])


def _layer_cases(case):
    """The four linears of a backbone layer as linear cases."""
    d, kv, f = case["hidden"], case["kv"], case["ffn"]
    return [{"mode": "token", "M": case["M"], "K": K, "N": N, "out": "f16", "bias": False}
            for K, N in ((d, d + 2 * kv), (d, d), (d, 2 * f), (f, d))]


class _Config:
    """Sizes of a DiT handle (the attributes that oq.DiT reads)."""

    def __init__(self, case):
        self.__dict__.update(PI if case["arch"] == "pi" else GR00T)
        self.tokens, self.prefix = case["tokens"], case["prefix"]


def _dit_inputs(case, seed):
    """The dict oq.DiT takes, with the arrays as fp16 tensors on the GPU."""
    c, d = _Config(case), _Draw(seed)
    L, B, D, F, A = case["n_blocks"], case["batch"], c.hidden, c.mlp, c.action_dim
    pi = case["arch"] == "pi"

    def gain(name):
        g = d.normal(name, D, std=0.05, mean=1.0)
        g[d.order(name + "/outliers", D)[: round(0.01 * D)]] *= 50.0
        return g.half()

    blocks = []
    for l in range(L):
        p = "blk%d/" % l
        blk = {"g1": gain(p + "g1"), "wo": d.weight(p + "wo", D, D)}
        if pi:
            blk.update(g2=gain(p + "g2"), wqkv=d.weight(p + "wqkv", 3 * D, D), wgu=d.weight(p + "wgu", 2 * F, D),
                       wd=d.weight(p + "wd", D, F))
        else:
            blk.update(g3=gain(p + "g3"), beta3=d.normal(p + "beta3", D, std=0.02).half(),
                       wff0=d.weight(p + "wff0", F, D), wff2=d.weight(p + "wff2", D, F))
            if l % 2 == 0:
                blk.update(wq=d.weight(p + "wq", D, D), wkv=d.weight(p + "wkv", 2 * D, D))
            else:
                blk.update(wqkv=d.weight(p + "wqkv", 3 * D, D))
        blocks.append(blk)
    w = {"w_in": d.normal("w_in", D, A, std=A ** -0.5).half(), "b_in": d.normal("b_in", D, std=0.02).half(),
         "w_out": d.normal("w_out", A, D, std=0.02).half(), "b_out": d.normal("b_out", A, std=0.02).half(),
         "g_f": d.normal("g_f", D, std=0.05, mean=1.0).half(), "blocks": blocks}
    names = ("sc1", "sh1", "gt1", "sc2", "sh2", "gt2") if pi else ("sc1", "sh1")
    mod = {nm: d.normal("mod/" + nm, L, c.steps, D, std=0.1, mean=1.0 if nm.startswith("gt") else 0.0).half()
           for nm in names}
    s_table = np.random.default_rng(seed).uniform(np.log(0.5), np.log(4.0), (L, c.steps, 4))
    inp = {"w": w, "mod": mod, "s_table": np.exp(s_table).astype(np.float32), "n_blocks": L, "batch": B,
           "x0": d.normal("x0", B, c.tokens, A)}
    if pi:
        inp["kp"] = d.normal("kp", L, B, case["prefix"], D).half()
        inp["vp"] = d.normal("vp", L, B, case["prefix"], D).half()
    else:
        inp["cond"] = d.tokens("cond", B * case["prefix"], D).view(B, case["prefix"], D)
    return c, inp


def _prepare_dit(case, seed):
    c, inp = _dit_inputs(case, seed)

    def host(v):
        if isinstance(v, torch.Tensor):
            return v.cpu().numpy()
        if isinstance(v, dict):
            return {k: host(x) for k, x in v.items()}
        return [host(x) for x in v] if isinstance(v, list) else v

    x0 = inp.pop("x0")
    inp = host(inp)
    mod = inp["mod"]
    inp["mod"] = [[{nm: mod[nm][l, t] for nm in mod} for t in range(c.steps)] for l in range(case["n_blocks"])]
    return {"dit": oq.DiT(c, inp), "x0": x0, "x": torch.empty_like(x0), "t": seed % c.steps}


def prepare(case, seed):
    kind = case["kind"]
    if kind == "linear":
        return {"kind": kind, "s": _prepare_linear(case, seed)}
    if kind == "layer":
        return {"kind": kind, "s": [_prepare_linear(c, 4 * seed + k) for k, c in enumerate(_layer_cases(case))]}
    if kind == "calibrate":
        M, K = case["M"], case["K"]
        return {"kind": kind, "x": _Draw(seed).tokens("x", M, K), "b": _block(K),
                "y": torch.empty((M, K), dtype=torch.float32, device=DEV),
                "delta": torch.empty((K,), dtype=torch.float32, device=DEV),
                "work": torch.empty((oq.calibrate_workspace_bytes(K),), dtype=torch.uint8, device=DEV)}
    if kind == "prepare":
        return {"kind": kind, "w": _prepare_weight(case, seed)}
    return {"kind": kind, "s": _prepare_dit(case, seed)}


def _prepare_weight(case, seed):
    """A weight whose channel energies spread, with outlier columns."""
    d = _Draw(seed)
    w = d.normal("w", case["N"], case["K"], std=0.02) * torch.exp(d.normal("energy", case["K"], std=0.3))
    w[:, d.order("outliers", case["K"])[: max(1, case["K"] // 100)]] *= 5.0
    return w.half()


def run(state):
    kind = state["kind"]
    if kind == "linear":
        return _run_linear(state["s"])
    if kind == "layer":
        return [_run_linear(s) for s in state["s"]]
    if kind == "calibrate":
        oq.rotate_act_f32(state["x"], state["b"], Y=state["y"])
        return oq.calibrate_step_scales(state["y"], delta=state["delta"], work=state["work"]), state["y"]
    if kind == "prepare":
        perm, rt, wq, ws = oq.prepare_weights_composite(state["w"])
        return {"perm": perm, "rt": rt.view(torch.float16), "wq": wq, "ws": ws}
    s = state["s"]
    s["x"].copy_(s["x0"])
    return s["dit"].step(s["x"], s["t"])


# ---------------------------------------------------------------------------
# What a pass cannot do without.
# ---------------------------------------------------------------------------


def _linear_work(c):
    M, K, N, mode = c["M"], c["K"], c["N"], c["mode"]
    b = 2 * M * K + N * K // 2 + 4 * N + 2 * M * N + (2 * N if c["bias"] else 0)
    f = 2 * M * N * K
    if mode in ("composite", "folded"):
        b += 128 * K + (4 * K if mode == "composite" else 0)
        f += 128 * M * K
    else:
        f += M * K * int(math.log2(_block(K)))
    if mode == "static":
        b += 4 * K
    return b, f


def work(case):
    kind = case["kind"]
    if kind == "linear":
        b, f = _linear_work(case)
    elif kind == "layer":
        b, f = (sum(v) for v in zip(*(_linear_work(c) for c in _layer_cases(case))))
    elif kind == "calibrate":
        M, K = case["M"], case["K"]
        b, f = 6 * M * K + 4 * K, M * K * int(math.log2(_block(K)))
    elif kind == "prepare":
        N, K = case["N"], case["K"]
        # The weight in, codes, scales, permutation and block matrices out; the
        # 64 x 64 Gram matrices and the fold's products.
        b, f = 2 * N * K + N * K // 2 + 4 * N + 4 * K + 128 * K, 2 * 64 * N * K + 128 * N * K
    else:
        c = _Config(case)
        L, B, S, P, D, F = case["n_blocks"], case["batch"], case["tokens"], case["prefix"], c.hidden, c.mlp
        M = B * S
        if case["arch"] == "pi":
            lin = L * (3 * D * D + D * D + 2 * F * D + D * F)
            kv, att = L * B * P * 2 * D, L * 4 * M * (P + S) * D
        else:
            n_cross = (L + 1) // 2
            lin = L * (D * D + 2 * F * D) + n_cross * D * D + (L - n_cross) * 3 * D * D
            kv, att = n_cross * B * P * 2 * D, n_cross * 4 * M * P * D + (L - n_cross) * 4 * M * S * D
        b, f = lin // 2 + 2 * kv + 8 * M * c.action_dim, 2 * M * lin + att
    return {"bytes": int(b), "flops": int(f)}


def tolerance(case):
    kind = case["kind"]
    if kind in ("linear", "layer"):
        # The products are exact; a code at a rounding boundary may move by
        # one, and the output is rounded to 16 bits.
        return {"rel": 8e-3 if case.get("out") == "bf16" else 2e-3, "max": 0.2}
    if kind == "calibrate":
        return {"rel": 2e-6, "max": 1e-4}
    if kind == "prepare":
        # Block matrices rounded once to fp16, from singular vectors in fp64.
        return {"rel": 1e-4, "max": 2e-2, "differ": 1e-3}
    # A whole step: one code that flips in an early block moves every later
    # one, which leaves room for little but the same roundings at every site.
    return {"rel": 0.03, "max": 0.5}


# ---------------------------------------------------------------------------
# The same outputs in 64 bits, from the definitions.
# ---------------------------------------------------------------------------


def _fwht(x, b):
    """x . BlockDiag(H_b) / sqrt(b) along the last axis."""
    h = torch.ones((1, 1), dtype=torch.float64, device=x.device)
    n = min(b, 128)
    while h.shape[0] < n:
        h = torch.cat([torch.cat([h, h], 1), torch.cat([h, -h], 1)], 0)
    y = (x.double().reshape(-1, n) @ h).reshape(x.shape)
    if b > n:
        y = y.reshape(-1, b // n, n).transpose(1, 2).contiguous()
        y = _fwht(y, b // n) * math.sqrt(b // n)
        y = y.transpose(1, 2).reshape(x.shape)
    return y / math.sqrt(b)


def _quantize(z, qmax=7):
    delta = z.abs().amax(-1, keepdim=True) / qmax
    return torch.clamp(torch.round(z / torch.where(delta > 0, delta, torch.ones_like(delta))), -qmax, qmax), delta


def _w4a4(x, w, s=1.0, qmax=7):
    """The rotated, quantized linear of x [M, K] and w [N, K] in 64 bits."""
    b = _block(x.shape[-1])
    q, d = _quantize(_fwht(x, b), qmax)
    qw, dw = _quantize(_fwht(w, b))
    return (q @ qw.T) * d * dw.T


def _block_rotations(u):
    h = _fwht(torch.eye(64, dtype=torch.float64, device=u.device), 64)
    return (u @ h).half().double()


def _composite(x, perm, r):
    xp = x.double() if perm is None else x.double()[:, perm.long()]
    return torch.matmul(xp.reshape(x.shape[0], -1, 64).transpose(0, 1).contiguous(), r).transpose(0, 1).reshape(x.shape)


def _exact_linear(case, seed):
    i = _linear_inputs(case, seed)
    if case["mode"] in ("composite", "folded"):
        r = _block_rotations(i["u"])
        q, d = _quantize(_composite(i["x"], i["perm"], r))
        qw, dw = _quantize(_composite(i["w"], i["perm"], r))
        y = (q @ qw.T) * d * dw.T
    elif case["mode"] == "static":
        delta = i["delta"].double()
        q = torch.clamp(torch.round(_fwht(i["x"], i["b"]) / delta), -7, 7)
        qw, dw = _quantize(_fwht(i["w"], i["b"]) * delta)
        y = (q @ qw.T) * dw.T
    else:
        y = _w4a4(i["x"], i["w"], qmax=127 if case["mode"] == "token8" else 7)
    return y if i["bias"] is None else y + i["bias"].double()


def _exact_prepare(case, seed):
    w = _prepare_weight(case, seed).double()
    K, nb = case["K"], case["K"] // 64
    order = torch.argsort(w.square().sum(0), descending=True, stable=True)
    rank = torch.arange(K, device=DEV)
    rnd, p = rank // nb, rank % nb
    perm = torch.empty(K, dtype=torch.int64, device=DEV)
    perm[torch.where(rnd % 2 == 0, p, nb - 1 - p) * 64 + rnd] = order
    wp = w[:, perm].reshape(case["N"], nb, 64).transpose(0, 1).contiguous()
    gram = torch.matmul(wp.transpose(1, 2).contiguous(), wp).cpu().numpy()
    u = np.linalg.eigh(gram)[1][:, :, ::-1]
    top = np.take_along_axis(u, np.abs(u).argmax(1)[:, None, :], 1)
    r = _block_rotations(torch.from_numpy(u * np.where(top < 0, -1.0, 1.0)).to(DEV))
    ws = torch.matmul(wp, r).transpose(0, 1).reshape(case["N"], K).abs().amax(-1) / 7
    return {"perm": perm.int(), "rt": r.transpose(1, 2).contiguous(), "wq": None, "ws": ws}


def exact(case, seed):
    kind = case["kind"]
    if kind == "linear":
        return _exact_linear(case, seed)
    if kind == "layer":
        return [_exact_linear(c, 4 * seed + k) for k, c in enumerate(_layer_cases(case))]
    if kind == "calibrate":
        M, K = case["M"], case["K"]
        y = _fwht(_Draw(seed).tokens("x", M, K), _block(K))
        k = min(max(-(-999 * M // 1000), 1), M)
        return y.abs().sort(0).values[k - 1] / 7.0, y
    if kind == "prepare":
        return _exact_prepare(case, seed)
    # A DiT step has no 64-bit value to be held to: one code of one block that
    # rounds the other way (sites are stored in fp16) moves every later code,
    # and the trajectories of two correct steps part within a few blocks.
    return None
