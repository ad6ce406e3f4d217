"""The work this library is measured on: single gated-MLP blocks at decode
batch sizes, a decoder stack's MLP half, the per-token top-k variant, CATS on
a projection's input, and the offline calibration, each through the public
calls of ``paper_2404_08763_amd`` with the caller's buffers kept between calls.

Shapes are those of ``paper_2404_08763_amd/workloads.py`` (C1..C5, QKV) and,
for the widest and the ragged cases, sizes the library accepts in general.
Weights are N(0, 0.02^2); activations follow the configurations: normal, 1%
outlier channels scaled x20, or a Laplace scale mixture.

Every cutoff t is a quantile of the case's own |SiLU(x W_gate)|, moved within
one percent of its rank to the middle of the widest gap between two of those
magnitudes, so that which neurons are kept does not hang on rounding.
"""
import math

import torch

import paper_2404_08763_amd as P

STD = 0.02
EPS = 1e-5
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _mlp(name, d, m, B, k, dtype="bf16", x="normal", op="forward", **kw):
    c = {"name": name, "op": op, "d": d, "m": m, "B": B, "k": k, "dtype": dtype, "x": x}
    c.update(kw)
    return c


def listed():
    return [
        # one token of a tiny fp32 block: launches and host path
        _mlp("tiny_f32", 256, 688, 1, 0.5, dtype="f32"),
        # batch-1 decode, the headline: a Llama2-7B-shaped block, half the neurons kept
        _mlp("decode_7b_k50", 4096, 11008, 1, 0.5, x="outliers"),
        # and a Mistral-7B-shaped block at the highest sparsity the benchmark times
        _mlp("decode_mistral_k90", 4096, 14336, 1, 0.9, x="laplace_mix"),
        # small-batch decode where sparsity still pays
        _mlp("batch4_7b_k70", 4096, 11008, 4, 0.7),
        # the largest batch of one call, at the widest matrix-core shape in use
        _mlp("batch16_13b_k50", 5120, 13824, 16, 0.5),
        # the widest supported rows, dense (the comparison baseline, and the largest block)
        _mlp("dense8_wide", 8192, 28672, 8, 0.0, op="dense"),
        # a width and neuron count that divide nothing, an odd batch
        _mlp("ragged_b11", 2856, 7001, 11, 0.5),
        # per-token top-k at batch 1
        _mlp("topk_7b_k50", 4096, 11008, 1, 0.5, x="outliers", op="topk"),
        # CATS in front of a Mistral-7B-shaped fused Q/K/V projection (m is the output width)
        _mlp("qkv_k50", 4096, 6144, 1, 0.5, x="laplace_mix", op="sparse_input"),
        # one token through the MLP half of a 40-layer Llama2-13B-shaped decoder
        _mlp("stack_13b_k50", 5120, 13824, 1, 0.5, op="stack", L=40),
        # one block's cutoff from 2048 calibration vectors
        _mlp("calibrate_7b", 4096, 11008, 2048, 0.5, x="outliers", op="calibrate"),
        # per-layer cutoffs of a stack, the vectors propagated densely
        _mlp("calibrate_stack_7b", 4096, 11008, 1024, 0.5, op="calibrate_stack", L=4),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["forward"] * 8 + ["dense"] * 3 + ["topk"] * 2 + ["sparse_input"] * 2 + ["stack"] * 2
                    + ["calibrate"] * 2 + ["calibrate_stack"] + ["pack"])
    x = rng.choice(["normal", "outliers", "laplace_mix"])
    k = rng.choice([0.0, 0.3, 0.5, 0.7, 0.9])
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    # half the widths are those models have (multiples of 512), half are any multiple of 8
    wide = 4096 if dtype == "f32" else 8192
    d = 512 * rng.randint(1, wide // 512) if rng.random() < 0.5 else 8 * _logint(rng, 32, wide // 8)
    m = _logint(rng, 512, 28672)
    if rng.random() < 0.5:
        m = max(512, m // 64 * 64)
    B = rng.choice([1, 1, 1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 13, 16])
    c = {"op": op, "d": d, "m": m, "B": B, "k": k, "dtype": dtype, "x": x}
    if op == "dense":
        c["k"] = 0.0
    elif op == "sparse_input":
        c["dtype"] = "bf16"
        c["d"] = min(max(d + rng.randint(-7, 7), 256), 8192)  # any number of input channels
        c["m"] = m // 8 * 8
    elif op == "stack":
        c["L"] = rng.randint(2, 8)
    elif op in ("calibrate", "calibrate_stack"):
        c["B"] = _logint(rng, 64, 2048)
        c["k"] = rng.choice([0.3, 0.5, 0.7, 0.9])
        if op == "calibrate_stack":
            c.update(B=_logint(rng, 64, 1024), L=rng.randint(2, 4), d=min(d, 4096), m=min(m, 11008))
        if dtype == "f32":
            c.update(B=min(c["B"], 512))
    elif op == "pack":
        c.update(B=1, k=0.0, x="normal")
    return c


# ---- inputs -----------------------------------------------------------------


def _gen(seed, dev):
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    return g


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _weight(rows, cols, dtype, seed):
    dev = _device()
    return (torch.randn((rows, cols), generator=_gen(seed, dev), device=dev) * STD).to(dtype)


def _x(case, seed):
    """[B, d] fp32 activations of the case's distribution."""
    dev = _device()
    B, d = case["B"], case["d"]
    g = _gen(seed * 1000003 + 11, dev)
    if case["x"] == "laplace_mix":
        u = torch.rand((B, d), generator=g, device=dev, dtype=torch.float64) - 0.5
        u = u.clamp(-0.5 + 1e-12, 0.5 - 1e-12)
        x = -torch.sign(u) * torch.log1p(-2.0 * u.abs())
        s = torch.tensor([0.25, 0.5, 1.0], device=dev, dtype=torch.float64)
        pick = torch.randint(0, 3, (B,), generator=g, device=dev)
        return (x * s[pick][:, None]).float()
    x = torch.randn((B, d), generator=g, device=dev)
    if case["x"] == "outliers":
        n = int(round(0.01 * d))
        x[:, torch.randperm(d, generator=_gen(13, dev), device=dev)[:n]] *= 20.0
    return x


def _blocks(case, seed):
    """Neuron-major (W_gate^T, W_up^T, W_down), each [m, d], of the case's layers."""
    dt = DTYPES[case["dtype"]]
    return [tuple(_weight(case["m"], case["d"], dt, seed * 1000003 + 1000 * (l + 1) + i) for i in range(3))
            for l in range(case.get("L", 1))]


def _silu(z):
    return z / (1.0 + torch.exp(-z))


def _gap_cutoff(mag, k):
    """The k-quantile of mag moved to the middle of the widest relative gap
    within one percent of its rank, as the fp32 value it is passed as."""
    if k == 0.0:
        return 0.0
    s = torch.sort(mag.reshape(-1)).values
    n = s.numel()
    r = _rank(n, k)
    lo, hi = max(r - 1 - n // 100, 0), min(r - 1 + n // 100 + 1, n - 1)
    if hi <= lo:
        return float(s[r - 1].float())
    a, b = s[lo:hi], s[lo + 1:hi + 1]
    i = int(torch.argmax((b - a) / b.clamp_min(1e-30)))
    return float(((a[i] + b[i]) * 0.5).float())


def _quantile(mag, k):
    s = torch.sort(mag.reshape(-1)).values
    return s[_rank(s.numel(), k) - 1]


def _rms(x):
    return x / torch.sqrt((x * x).mean(dim=-1, keepdim=True) + EPS)


def _mlp64(w, x, t=None, k=None):
    """Rows x [B, d] (64 bits) through one block at cutoff t (or its own
    k-quantile's gap, or t_b per row).  Returns y and the cutoff."""
    g = _silu(x @ w[0].double().t())
    mag = g.abs()
    if t is None:
        t = _gap_cutoff(mag, k)
    h = torch.where(mag >= t, g * (x @ w[1].double().t()), torch.zeros_like(g))
    return h @ w[2].double(), t


def _rank(n, k):
    return min(max(int(math.ceil(k * n - 1e-6)), 1), n)


def _clear_rows(case, seed, w):
    """B rows for the per-row cutoff: of four times as many, those whose r-th
    smallest |v| stands clearest of the one below it."""
    B, k, m = case["B"], case["k"], case["m"]
    x = _x({**case, "B": 4 * B}, seed)
    r = _rank(m, k)
    if k == 0.0 or r < 2:
        return x[:B].contiguous()
    s = torch.sort(_silu(x.double() @ w[0].double().t()).abs(), dim=1).values
    gap = (s[:, r - 1] - s[:, r - 2]) / s[:, r - 1]
    return x[torch.topk(gap, B).indices.sort().values].contiguous()


def _residual(case, seed):
    return torch.randn((case["B"], case["d"]), generator=_gen(seed * 1000003 + 17, _device()), device=_device())


def _inputs(case, seed):
    """Everything the call takes, made with torch alone (t: the cutoffs)."""
    op = case["op"]
    if op == "pack":
        dt = DTYPES[case["dtype"]]
        return {"math": [_weight(case["d"], case["m"], dt, seed * 1000003 + i) for i in range(2)]
                + [_weight(case["m"], case["d"], dt, seed * 1000003 + 2)]}
    x = _x(case, seed)
    if op == "sparse_input":
        t = 0.0 if case["k"] == 0.0 else float(_quantile(x.abs(), case["k"]))
        return {"x": x, "t": t, "w": _weight(case["d"], case["m"], torch.bfloat16, seed * 1000003 + 5000)}
    blocks = _blocks(case, seed)
    s = {"x": _clear_rows(case, seed, blocks[0]) if op == "topk" else x, "w": blocks}
    if op == "forward":
        s["t"] = _gap_cutoff(_silu(x.double() @ blocks[0][0].double().t()).abs(), case["k"])
    if op == "stack":
        cur, s["t"] = x.double(), []
        for w in blocks:
            y, t = _mlp64(w, _rms(cur), k=case["k"])
            cur = cur + y
            s["t"].append(t)
    if op in ("forward", "dense", "topk"):
        s["residual"] = _residual(case, seed)
    return s


# ---- the calls --------------------------------------------------------------


def prepare(case, seed):
    op, d, m, B = case["op"], case["d"], case["m"], case["B"]
    s = _inputs(case, seed)
    s["op"], s["k"] = op, case["k"]
    if op == "pack":
        return s
    if op == "sparse_input":
        s["ws"] = P.sparse_input_workspace(d, m, B)
        s["out"] = torch.empty((B, m), device="cuda")
        return s
    layers = [P.Layer(*w) for w in s["w"]]
    s["layer"] = layers[0]
    if op in ("stack", "calibrate_stack"):
        s["stack"] = P.Stack(layers, s.get("t"))
    if op == "calibrate":
        s["ws"] = P.workspace(d, m, 1, B * m)
    elif op == "calibrate_stack":
        s["ws"] = torch.zeros(P.raw().cats_calibrate_stack_workspace_bytes(d, m, B), dtype=torch.uint8, device="cuda")
    elif op == "topk":
        s["ws"] = torch.zeros(P.raw().cats_topk_workspace_bytes(d, m, B), dtype=torch.uint8, device="cuda")
    else:
        s["ws"] = P.workspace(d, m, B)
    if op in ("forward", "dense", "topk", "stack"):
        s["out"] = torch.empty((B, d), device="cuda")
    return s


def run(s):
    op = s["op"]
    if op == "forward":
        return P.mlp_forward(s["layer"], s["x"], s["t"], residual=s["residual"], out=s["out"], ws=s["ws"])
    if op == "dense":
        return P.mlp_dense(s["layer"], s["x"], residual=s["residual"], out=s["out"], ws=s["ws"])
    if op == "topk":
        return P.mlp_forward_topk(s["layer"], s["x"], s["k"], residual=s["residual"], out=s["out"], ws=s["ws"])
    if op == "sparse_input":
        return P.sparse_input_gemv(s["w"], s["x"], s["t"], out=s["out"], ws=s["ws"])
    if op == "stack":
        return P.stack_forward(s["stack"], s["x"], eps=EPS, out=s["out"], ws=s["ws"])
    if op == "calibrate":
        return P.calibrate_threshold(s["layer"], s["x"], s["k"], ws=s["ws"])
    if op == "calibrate_stack":
        return P.calibrate_stack(s["stack"], s["x"], s["k"], eps=EPS, ws=s["ws"])
    if op == "pack":
        layer = P.layer_from_math(*s["math"])
        return [layer.w_gate_t, layer.w_up_t]
    raise ValueError(op)


# ---- what a pass cannot do without, and what it should give -----------------


def work(case):
    op, d, m, B, k, L = case["op"], case["d"], case["m"], case["B"], case["k"], case.get("L", 1)
    sw = 4 if case["dtype"] == "f32" else 2
    if op == "pack":
        return {"bytes": 4 * d * m * sw, "flops": 0}
    keep = 1.0 - k
    union = 1.0 - k ** B if k > 0 else 1.0  # share of rows some batch row keeps
    if op == "sparse_input":
        return {"bytes": sw * d * m * union + 4 * B * (d + m), "flops": 2.0 * B * d * m * keep}
    if op == "calibrate":
        return {"bytes": sw * d * m + 4.0 * B * d, "flops": 2.0 * B * d * m}
    if op == "calibrate_stack":  # the last layer needs its gate alone
        return {"bytes": (3 * L - 2.0) * sw * d * m + 4.0 * B * d, "flops": 2.0 * B * d * m * (3 * L - 2)}
    rows = 8 if op == "stack" else 12  # x, y and the residual
    return {"bytes": L * (sw * d * m * (1.0 + 2.0 * union) + rows * B * d),
            "flops": L * 2.0 * B * d * m * (1.0 + 2.0 * keep)}


def tolerance(case):
    # Measured against exact(): 1e-7 .. 5e-7 where x enters in fp32, up to 4e-6
    # where it enters the matrix cores as two bf16 parts (16 of its 24 bits);
    # 2e-6 after 40 layers.  A stack's errors add up over its layers.
    if case["op"] == "pack":
        return "exact"
    if case["op"] == "stack":
        return {"rel": 5e-5, "max": 5e-4}
    return {"rel": 2e-5, "max": 2e-4}


def exact(case, seed):
    op, k = case["op"], case["k"]
    s = _inputs(case, seed)
    if op == "pack":
        return [w.t().contiguous() for w in s["math"][:2]]
    x = s["x"].double()
    if op == "sparse_input":
        return torch.where(x.abs() >= s["t"], x, torch.zeros_like(x)) @ s["w"].double()
    if op == "calibrate":
        return float(_quantile(_silu(x @ s["w"][0][0].double().t()).abs(), k))
    if op == "calibrate_stack":
        out = []
        for l, w in enumerate(s["w"]):
            xn = _rms(x)
            out.append(float(_quantile(_silu(xn @ w[0].double().t()).abs(), k)))
            if l + 1 < len(s["w"]):
                x = x + _mlp64(w, xn, t=0.0)[0]
        return out
    if op == "stack":
        for w, t in zip(s["w"], s["t"]):
            x = x + _mlp64(w, _rms(x), t=t)[0]
        return x
    w, res = s["w"][0], s["residual"].double()
    if op == "topk":
        if k == 0.0:
            t = torch.zeros((case["B"], 1), device=x.device, dtype=torch.float64)
        else:
            r = _rank(case["m"], k)
            t = torch.sort(_silu(x @ w[0].double().t()).abs(), dim=1).values[:, r - 1:r]
        return _mlp64(w, x, t=t)[0] + res, t[:, 0]
    return _mlp64(w, x, t=s.get("t", 0.0))[0] + res
