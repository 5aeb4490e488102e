"""The work that programs using this library have it do, as cases that can be timed and compared.

Every case goes through the public binding (`binding.Calibrator`, `binding.score_rows_static`).  Kinds:

  rotate       Y = X R_op: folding a learned rotation into a weight matrix (its rows as X), or rotating activations
  rotate_quant the rotated and fake-quantised rows a quantised linear layer receives; with a few rows the call of a
               token-by-token loop
  evaluate     what a calibration run reads off a batch to judge its rotation: both quantiser scores and the row diagnostics
  score_static the two scores of rows that are rotated already, left on the device
  calibrate    the calibration loop on one site: `batches` statistics steps, one Procrustes update, and the new rotation
               put to use (folded into a matrix of `fold` rows).  `score`: the batch is also scored before the update, as an
               online run does.  `quantise`: the step is the quantisation-aware one.  `layers` > 1: one context carries the
               per-head rotations of several layers, every layer's batch goes to its own range of heads

Inputs follow the value recipe of `inputs.py` (log-normal channel scales, a few outlier channels, Student-t token
magnitudes), drawn on the GPU.
"""
import math

import numpy as np
import torch

from paper_2605_10793_amd import binding as B
from paper_2605_10793_amd import inputs as I

DEV = "cuda:0"


def _c(name, kind, d, T, heads=1, dtype="bf16", lam=0.0, **more):
    c = dict(kind=kind, d=d, heads=heads, dtype=dtype, tokens=T, lam=lam)
    if name:
        c["name"] = name
    c.update(more)
    return c


def listed():
    return [
        # a serving loop's step: a handful of tokens through the rotation and the quantiser before a linear layer
        _c("rows16_d4096", "rotate_quant", 4096, 16, zero_point=True),
        # a rotation folded into an MLP-sized weight matrix
        _c("fold_d4096", "rotate", 4096, 11008),
        # fp32 activations (the width of the fp32 calibration tests is small; this one is ragged in both directions)
        _c("rotate_f32_d1040", "rotate", 1040, 777, dtype="f32"),
        # judging a rotation on one batch (d = 3072, the mid-size residual stream)
        _c("evaluate_d3072", "evaluate", 3072, 2048),
        # rows already rotated, scored inside a capture-safe loop
        _c("static_d4096", "score_static", 4096, 16384),
        # the fp32 calibration configuration: d = 256, 2048 tokens, the paper's own update
        _c("online_f32_d256", "calibrate", 256, 2048, dtype="f32", batches=1, fold=256),
        # several mini-batches pooled before one update
        _c("pooled_d3072", "calibrate", 3072, 2048, lam=0.1, batches=8, fold=3072),
        # the configuration of the headline figure: step, int4 score, update at d = 4096
        _c("online_d4096", "calibrate", 4096, 2048, lam=0.1, batches=1, fold=2048, score=True),
        # per-head rotations of a layer: 32 heads of width 128
        _c("heads_32x128", "calibrate", 4096, 2048, heads=32, batches=1, fold=512),
        # the same for a model with narrower heads
        _c("heads_32x64", "calibrate", 2048, 2048, heads=32, batches=1, fold=512),
        # quantisation-aware calibration of a site whose width and token count fit no tile
        _c("aware_d1104", "calibrate", 1104, 1500, lam=0.1, batches=1, fold=333, quantise=True),
        # the widest rotation, 4096 tokens a batch
        _c("online_d8192", "calibrate", 8192, 4096, lam=0.1, batches=1, fold=1024, score=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["rotate", "rotate_quant", "evaluate", "score_static", "calibrate", "calibrate", "heads", "heads"])
    if kind == "heads":
        dh = rng.choice([128, 128, 64, 16 * rng.randint(2, 16)])
        layers = rng.choice([1, 2, 4]) if dh == 128 else 1
        heads = rng.choice([8, 16, 24, 32])
        T, n = _log(rng, 200, 3000), rng.choice([1, 1, 2])
        # the paper's own update (lam = 0) where its rows outnumber the width well enough to determine the rotation
        return _c(None, "calibrate", dh * heads * layers, T, heads=heads * layers, lam=0.0 if n * T >= 8 * dh else 0.1,
                  batches=n, fold=rng.randint(32, 600), layers=layers)
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    d = 16 * _log(rng, 12, 64 if dtype == "f32" else 300)
    if kind == "calibrate":
        c = _c(None, kind, d, _log(rng, 100, 4096), dtype=dtype, lam=0.1, batches=rng.choice([1, 1, 2, 5]), fold=rng.randint(64, d))
        if rng.random() < 0.4:
            c["quantise"] = True
        else:
            c["score"] = rng.random() < 0.5
        return c
    T = _log(rng, 1, 256) if kind == "rotate_quant" and rng.random() < 0.6 else _log(rng, 64, 12000)
    if kind == "rotate_quant":
        return _c(None, kind, d, T, dtype=dtype, zero_point=rng.random() < 0.5)
    return _c(None, kind, d, T, dtype=dtype)


# ---------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _activations(case, seed, rows, cols, heads):
    g = _gen(seed)
    s = torch.exp(0.5 * torch.randn(cols, generator=g, device=DEV))
    per, n = cols // heads, (8 if heads == 1 else 2)
    idx = torch.rand((heads, per), generator=g, device=DEV).argsort(dim=1)[:, :n] + per * torch.arange(heads, device=DEV)[:, None]
    s[idx.reshape(-1)] *= 50.0 + 50.0 * torch.rand(idx.numel(), generator=g, device=DEV)
    x = torch.randn((rows, cols), generator=g, device=DEV) * s
    z = torch.randn((rows, 5), generator=g, device=DEV)
    x *= (z[:, 0] / (z[:, 1:] ** 2).mean(dim=1).sqrt()).abs()[:, None]      # Student-t with 4 degrees of freedom
    return x.to(torch.bfloat16) if case["dtype"] == "bf16" else x


def _weights(case, seed, rows):
    w = torch.randn((rows, case["d"]), generator=_gen(seed), device=DEV) / math.sqrt(case["d"])
    return w.to(torch.bfloat16) if case["dtype"] == "bf16" else w


def _rotation(case, seed):
    """A dense orthogonal start per head: the Kronecker product of two small Haar rotations, columns' signs random."""
    dh, heads = case["d"] // case["heads"], case["heads"]
    a = max(k for k in range(1, int(math.isqrt(dh)) + 1) if dh % k == 0)
    out = np.empty((heads, dh, dh), dtype=np.float32)
    for h in range(heads):
        q = [I.random_orthogonal(k, 7919 * seed + 2 * h + j) for j, k in enumerate((a, dh // a))]
        sign = np.where(np.random.default_rng([seed, h]).random(dh) < 0.5, -1.0, 1.0)
        out[h] = np.kron(q[0].astype(np.float32), q[1].astype(np.float32)) * sign.astype(np.float32)[None, :]
    return out


def _inputs(case, seed):
    """Every input of the case as device tensors (the rotation as a numpy array): made from the seed alone."""
    kind, layers = case["kind"], case.get("layers", 1)
    r = {}
    if kind == "score_static":
        g = _gen(100 * seed + 1)      # rotated rows: close to Gaussian, the tokens' magnitudes kept
        y = torch.randn((case["tokens"], case["d"]), generator=g, device=DEV) * torch.exp(torch.randn((case["tokens"], 1), generator=g, device=DEV))
        r["Y"] = y.to(torch.bfloat16) if case["dtype"] == "bf16" else y
        return r
    r["R0"] = _rotation(case, seed)
    if kind == "rotate":
        r["X"] = _weights(case, 100 * seed + 2, case["tokens"])
    elif kind == "calibrate":
        cols, heads = case["d"] // layers, case["heads"] // layers
        r["X"] = [[_activations(case, 100 * seed + 10 + 16 * b + l, case["tokens"], cols, heads) for l in range(layers)]
                  for b in range(case["batches"])]
        r["W"] = _weights(case, 100 * seed + 3, case["fold"])
    else:
        r["X"] = _activations(case, 100 * seed + 4, case["tokens"], case["d"], case["heads"])
    return r


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.case = case
    vars(s).update(_inputs(case, seed))
    if case["kind"] == "score_static":
        s.out = torch.empty((2, 2), dtype=torch.float64, device=DEV)
        return s
    rows = max(case["tokens"], case.get("fold", 0))
    s.cal = B.Calibrator(case["d"], case["heads"], case["dtype"], s.R0, max_tokens=rows, prox_lambda=case["lam"])
    first = s.W if case["kind"] == "calibrate" else s.X
    s.Y = torch.empty((first.shape[0], case["d"]), dtype=first.dtype, device=DEV)
    if case.get("quantise"):
        s.Yq = torch.empty((case["tokens"], case["d"]), dtype=first.dtype, device=DEV)
    del s.R0
    return s


# ---------------------------------------------------------------- one pass

def run(s):
    case, kind = s.case, s.case["kind"]
    if kind == "score_static":
        B.score_rows_static(s.Y, s.out[0], 4, False)
        B.score_rows_static(s.Y, s.out[1], 4, True, 0.9)
        return s.out
    cal = s.cal
    if kind == "rotate":
        return cal.rotate(s.X, s.Y)
    if kind == "rotate_quant":
        return cal.rotate_quant(s.X, 4, case["zero_point"], 0.9, s.Y)
    if kind == "evaluate":
        sym, zp = cal.quant_error(s.X, 4), cal.quant_error_zp(s.X, 4, 0.9)
        pr, rho = cal.row_diagnostics(s.X)
        return {"sym": sym, "zp": zp, "pr": pr, "rho": rho}
    out = {}
    layers = case.get("layers", 1)
    per = case["heads"] // layers
    for batch in s.X:
        if case.get("quantise"):
            out["Yq"] = cal.step_batch_quant(batch[0], 4, True, 0.9, s.Yq)
        elif layers == 1:
            cal.step_batch(batch[0])
        else:
            for l, x in enumerate(batch):
                cal.step_batch_heads(x, l * per, per)
        if case.get("score"):
            out["score"] = cal.quant_error(batch[0], 4)
    _, st = cal.update_rotation()
    for k in ("inner", "m_fro"):
        out[k] = np.array([h[k] for h in st])
    out["Y"] = cal.rotate(s.W, s.Y)
    return out


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    d, T, h, e = case["d"], case["tokens"], case["heads"], 4 if case["dtype"] == "f32" else 2
    dh, kind, layers = d // case["heads"], case["kind"], case.get("layers", 1)
    rop = h * dh * dh * e                              # the rotation operand
    if kind == "score_static":
        return {"bytes": 2.0 * T * d * e, "flops": 2 * 8.0 * T * d}
    if kind in ("rotate", "rotate_quant"):
        return {"bytes": 2.0 * T * d * e + rop, "flops": 2.0 * T * d * dh}
    if kind == "evaluate":
        return {"bytes": 3.0 * T * d * e + 3 * rop + 8 * T, "flops": 3 * 2.0 * T * d * dh}
    n = case["batches"]
    score = 1 if case.get("score") else 0
    flops = n * (4 + 2 * score) * float(T) * d * dh + 2.0 * case["fold"] * d * dh
    # the polar factor by matrix products: singular values from the bottom the proximal term guarantees up to 1 at the
    # largest growth a cubic gives (2.6 a step), three steps to settle; a symmetric product (half of 2 dh^3) and a full one each
    l0 = max(case["lam"], 2.0 ** -20) / (2.0 * math.sqrt(dh))
    flops += 3.0 * dh ** 3 * h * (math.ceil(math.log(1.0 / l0) / math.log(2.6)) + 3)
    bytes_ = n * (1 + score) * T * d * e + 2.0 * case["fold"] * d * e + h * dh * dh * (4.0 + 4.0) + (n + 1) * rop
    if case.get("quantise"):
        bytes_ += n * T * d * e
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    """About four times the distance from exact() measured over the listed and some drawn cases."""
    kind, f32 = case["kind"], case["dtype"] == "f32"
    if kind == "score_static":
        return {"rel": 1e-5}
    if kind == "rotate":                # bf16: one rounding of every entry (0.0017); fp32: the split-precision products (2e-7)
        return {"rel": 1e-6} if f32 else {"rel": 0.007}
    if kind == "rotate_quant":          # an entry of Y an ulp off may take the neighbouring level (0.0016 to 0.005)
        return {"rel": 0.02}
    if kind == "evaluate":              # a row whose extreme entry is an ulp off moves its ratio by up to 2^-6
        return {"rel": 6e-4, "max": 0.03}
    # the rotation after an update in 16-bit products, then one rounding: 0.0024 to 0.0045; where nothing holds M's weak
    # directions (lam = 0) up to 0.01
    return {"rel": 0.018 if case["lam"] > 0 else 0.03}


# ---------------------------------------------------------------- the same in 64 bits

def _round(x, case):
    return x.to(torch.bfloat16).double() if case["dtype"] == "bf16" else x.to(torch.float32).double()


def _mul(x, R):
    """Rows of width h dh times the block-diagonal rotation R [h][dh][dh], in fp64."""
    h, dh = R.shape[0], R.shape[1]
    if h == 1:
        return x @ R[0]
    return torch.bmm(x.reshape(-1, h, dh).transpose(0, 1).contiguous(), R).transpose(0, 1).reshape(x.shape[0], h * dh)


def _levels(y, zero_point, clip):
    """The level values of the 4-bit quantisers, per row."""
    if zero_point:
        lo, hi = clip * y.min(1, keepdim=True).values, clip * y.max(1, keepdim=True).values
        D = (hi - lo) / 15
        z = -torch.round(lo / D)
        return D * (torch.clamp(torch.round(y / D) + z, 0, 15) - z)
    D = y.abs().max(1, keepdim=True).values / 7
    return D * torch.clamp(torch.round(y / D), -7, 7)


def _score(y, zero_point, clip=1.0):
    return (float(((y - _levels(y, zero_point, clip)) ** 2).sum()), float((y * y).sum()))


def _polar(A):
    X = A / torch.linalg.matrix_norm(A)[:, None, None]
    eye = torch.eye(A.shape[1], dtype=A.dtype, device=A.device)
    for _ in range(120):
        G = torch.bmm(X.transpose(1, 2).contiguous(), X)
        if float((G - eye).abs().max()) < 1e-13:
            break
        X = 1.5 * X - 0.5 * torch.bmm(X, G)
    return X


def exact(case, seed):
    v, kind = _inputs(case, seed), case["kind"]
    if kind == "score_static":
        y = v["Y"].double()
        return torch.tensor([_score(y, False), _score(y, True, 0.9)], dtype=torch.float64)
    R = torch.from_numpy(v["R0"]).to(DEV).double()
    Rop = _round(R, case)
    if kind == "rotate":
        return _mul(v["X"].double(), Rop)
    if kind == "rotate_quant":
        return _levels(_round(_mul(v["X"].double(), Rop), case), case["zero_point"], 0.9)
    if kind == "evaluate":
        y = _round(_mul(v["X"].double(), Rop), case)
        n2 = (y * y).sum(1)
        return {"sym": _score(y, False), "zp": _score(y, True, 0.9), "pr": n2 ** 2 / (y.shape[1] * (y ** 4).sum(1)),
                "rho": (y * y).max(1).values / n2}
    h, dh, T = case["heads"], case["d"] // case["heads"], case["tokens"]
    out = {}
    M = torch.zeros_like(R)
    for batch in v["X"]:
        x = torch.cat([b.double() for b in batch], dim=1)
        y = _mul(x, Rop)
        xh = x.reshape(T, h, dh).transpose(0, 1)
        xh = xh / torch.linalg.vector_norm(xh, dim=2, keepdim=True)
        c = torch.where(y >= 0, 1.0, -1.0).double().reshape(T, h, dh).transpose(0, 1).contiguous() / math.sqrt(dh)
        M += torch.bmm(xh.transpose(1, 2).contiguous(), c)
        if case.get("quantise"):
            out["Yq"] = _levels(_round(y, case), True, 0.9)
        if case.get("score"):
            out["score"] = _score(_round(y, case), False)
        del x, y, xh, c
    fro = torch.linalg.matrix_norm(M)
    lam = max(case["lam"], 2.0 ** -20)
    P = _polar(M + (lam / math.sqrt(dh)) * fro[:, None, None] * R)
    out["inner"] = (P * M).sum((1, 2))
    out["m_fro"] = fro
    out["Y"] = _mul(v["W"].double(), _round(P, case))
    return out
