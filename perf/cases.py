"""The work a program does with the LC-VQ linear layer, as cases to be timed.

Five kinds of pass, each through the package's public calls:

  train    one optimisation step's work on one weight matrix: the forward that saves
           its state, the backward that reads it, and, as options, the 2-bit codes of
           the step, the differentiable estimator, the Xavier domain and AdamW of Z,
           A and b
  accum    two micro-batches through the plain calls (no saved state), the second
           one's gradients added to the first's, dZ held in fp32
  eval     the forward alone, from the latents
  f32      forward and backward of an fp32 layer
  packed   the layer output from packed 2-bit codes, up and down matrices of an MLP
           in turn: decode at few tokens, prefill at many
  convert  a dense weight into codes, the codes into initial latents, and back into
           the dense weight they stand for

Shapes are the Llama-shaped matrices of the repository's workloads, or generic.
Latents are uniform over the code range and a little beyond it (so that both masks
matter), activations and upstream gradients standard normal, the map close to a
scaled identity: the recipe of the repository's benchmark.
"""
from __future__ import annotations

import math

import torch

import paper_2606_10531_amd as lc

_BF16 = torch.bfloat16
_LR, _BETA1, _BETA2, _EPS = 1e-4, 0.9, 0.999, 1e-8
_DGE_K, _DGE_CAP = 5.0, 3.0


def listed():
    return [
        # a layer of a toy model in fp32: latency and the number of launches
        dict(name="f32_256x256_16", kind="f32", N=16, m=256, n=256, d=8),
        # fp32 training of a small layer, out-features and tokens not whole tiles
        dict(name="f32_1376x1024_500", kind="f32", N=500, m=1376, n=1024, d=4),
        # the benchmarked layer: attention projection of a 7B model, 4096 tokens
        dict(name="train_4096x4096_4096", kind="train", N=4096, m=4096, n=4096, d=8, pack=True, dge=False, adam=False),
        # the same layer fine-tuned on short batches
        dict(name="train_4096x4096_256", kind="train", N=256, m=4096, n=4096, d=8, pack=False, dge=False, adam=False),
        # down projection with the differentiable estimator in the Xavier domain,
        # and the optimiser's update of Z, A and b
        dict(name="train_4096x11008_2048", kind="train", N=2048, m=4096, n=11008, d=8, pack=False, dge=True, adam=True),
        # up projection of a 70B model, 4096 tokens, with the 2-bit codes
        dict(name="train_28672x8192_4096", kind="train", N=4096, m=28672, n=8192, d=8, pack=True, dge=False, adam=False),
        # gradient accumulation over two ragged micro-batches, groups of four
        dict(name="accum_11008x4096_1000", kind="accum", N=1000, m=11008, n=4096, d=4),
        # validation of a short sequence between training steps
        dict(name="eval_4096x11008_333", kind="eval", N=333, m=4096, n=11008, d=8),
        # one token through eight MLPs of a 7B model, compressed weights
        dict(name="decode_11008x4096_1", kind="packed", N=1, m=11008, n=4096, d=8, layers=8, noalloc=False),
        # sixteen sequences decoded together through two MLPs of a 70B model
        dict(name="decode_28672x8192_16", kind="packed", N=16, m=28672, n=8192, d=8, layers=2, noalloc=True),
        # a prompt of 512 tokens through one MLP of a 7B model
        dict(name="prefill_11008x4096_512", kind="packed", N=512, m=11008, n=4096, d=4, layers=1, noalloc=False),
        # the initialisation of a 70B matrix from its dense weight
        dict(name="convert_28672x8192", kind="convert", m=28672, n=8192, d=8),
    ]


def _log_int(rng, lo, hi, step=1):
    """A multiple of step in [lo, hi], spread over its logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))
    return max(lo, min(hi, int(v) // step * step)) // step * step


def draw(rng):
    kind = rng.choice(["train", "train", "accum", "eval", "f32", "packed", "packed", "convert"])
    d = rng.choice([4, 8, 8])
    if kind == "f32":
        return dict(kind=kind, N=_log_int(rng, 1, 1024), m=_log_int(rng, 64, 2048), n=_log_int(rng, 64, 2048, 8), d=d)
    if kind == "convert":
        return dict(kind=kind, m=_log_int(rng, 512, 28672, 8), n=_log_int(rng, 512, 8192, 8), d=d)
    if kind == "packed":
        m, n = _log_int(rng, 1024, 28672, 64), _log_int(rng, 1024, 8192, 64)
        N = rng.choice([_log_int(rng, 1, 16), _log_int(rng, 17, 2048)])
        layers = max(1, min(16, (1 << 28) // (m * n))) if N <= 16 else 1
        return dict(kind=kind, N=N, m=m, n=n, d=d, layers=layers, noalloc=rng.choice([False, True]))
    m, n = _log_int(rng, 512, 28672, 8), _log_int(rng, 512, 28672, 8)
    if kind == "eval":
        return dict(kind=kind, N=min(_log_int(rng, 1, 4096), (1 << 39) // (m * n)), m=m, n=n, d=d)
    N = max(64, min(_log_int(rng, 64, 16384), (1 << 39) // (m * n)))
    if kind == "accum":
        return dict(kind=kind, N=max(64, N // 2), m=m, n=n, d=d)
    return dict(kind=kind, N=N, m=m, n=n, d=d, pack=rng.choice([False, True]), dge=rng.choice([False, True]),
                adam=rng.choice([False, True]))


# ---------------------------------------------------------------- preparation --

def _draws(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _map(g, d):
    A = 0.02 * (torch.eye(d, device="cuda") + 0.1 * torch.randn((d, d), device="cuda", generator=g))
    return A, 0.005 * torch.randn((d,), device="cuda", generator=g)


def _normal(g, shape, dtype):
    return torch.randn(shape, device="cuda", generator=g).to(dtype)


def _latent(g, m, n, dtype):
    return torch.empty((m, n), device="cuda").uniform_(-0.75, 3.75, generator=g).to(dtype)


def _packed_mats(case):
    return [(case["m"], case["n"]), (case["n"], case["m"])] * case["layers"]


def prepare(case, seed):
    g, kind, d = _draws(seed), case["kind"], case["d"]
    m, n, N = case["m"], case["n"], case.get("N", 0)
    s = dict(case=case)
    if kind == "convert":
        s["A"], s["b"] = _map(g, d)
        v = 1.5 + 1.1 * torch.randn((m * n // d, d), device="cuda", generator=g)
        s["W"] = (v @ s["A"].T + s["b"]).reshape(m, n).to(_BF16)
        return s
    if kind == "packed":
        s["layers"] = []
        for mm, nn in _packed_mats(case):
            A, b = _map(g, d)
            s["layers"].append(dict(
                P=torch.randint(0, 256, (mm, nn // 4), dtype=torch.uint8, device="cuda", generator=g), A=A, b=b,
                X=_normal(g, (N, nn), _BF16), out=torch.empty((N, mm), dtype=_BF16, device="cuda")))
        if not case["noalloc"]:
            need = max(lc.workspace_bytes(lc.OP_FWD_PACKED, N, mm, nn, d, _BF16) for mm, nn in _packed_mats(case))
            s["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda")
        return s
    s["A"], s["b"] = _map(g, d)
    if kind == "f32":
        s["Z"] = _latent(g, m, n, torch.float32)
        s["X"], s["dY"] = _normal(g, (N, n), torch.float32), _normal(g, (N, m), torch.float32)
        return s
    s["Z"] = _latent(g, m, n, _BF16)
    if kind == "eval":
        s["X"] = _normal(g, (N, n), _BF16)
        return s
    if kind == "accum":
        s["X"] = [_normal(g, (N, n), _BF16) for _ in range(2)]
        s["dY"] = [_normal(g, (N, m), _BF16) for _ in range(2)]
        s["dZ"] = torch.empty((m, n), dtype=torch.float32, device="cuda")
        s["dA"] = torch.empty((d, d), dtype=torch.float32, device="cuda")
        s["db"] = torch.empty((d,), dtype=torch.float32, device="cuda")
        return s
    s["X"], s["dY"] = _normal(g, (N, n), _BF16), _normal(g, (N, m), _BF16)
    s["q"] = (1.0, 0.0)
    master = s["Z"].float()
    if case["dge"]:  # latents in the Xavier domain: W_p = (Z - t) / q_scale
        s["q"] = lc.xavier_quantizer(m, n)
        master = (master - s["q"][1]) / s["q"][0]
        s["Z"] = master.to(_BF16)
    if case["adam"]:
        s["step"] = 0
        for name, p in (("Z", master), ("A", s["A"]), ("b", s["b"])):
            s["theta_" + name] = p.clone()
            s["m1_" + name], s["m2_" + name] = torch.zeros_like(p), torch.zeros_like(p)
    s["wsf"] = torch.empty(lc.workspace_bytes(lc.OP_FWD, N, m, n, d, _BF16), dtype=torch.uint8, device="cuda")
    s["wsb"] = torch.empty(lc.workspace_bytes(lc.OP_BWD, N, m, n, d, _BF16), dtype=torch.uint8, device="cuda")
    s["saved"] = lc.new_saved(N, m, n, d, _BF16, "cuda")
    s["Y"], s["dX"] = torch.empty((N, m), dtype=_BF16, device="cuda"), torch.empty((N, n), dtype=_BF16, device="cuda")
    s["dZ"] = torch.empty((m, n), dtype=_BF16, device="cuda")
    s["dA"] = torch.empty((d, d), dtype=torch.float32, device="cuda")
    s["db"] = torch.empty((d,), dtype=torch.float32, device="cuda")
    s["packed"] = torch.empty((m, n // 4), dtype=torch.uint8, device="cuda") if case["pack"] else None
    return s


# ------------------------------------------------------------------- one pass --

def _run_train(s):
    case = s["case"]
    d, (qs, qb) = case["d"], s["q"]
    lc.linear_fwd(s["Z"], s["A"], s["b"], s["X"], d, packed_out=s["packed"], workspace=s["wsf"], out=s["Y"],
                  q_scale=qs, q_shift=qb, saved=s["saved"])
    grads = dict(dX=s["dX"], dZ=s["dZ"], dA=s["dA"], db=s["db"], workspace=s["wsb"], q_scale=qs, q_shift=qb,
                 saved=s["saved"])
    if case["dge"]:
        lc.linear_bwd_dge(s["Z"], s["A"], s["b"], s["X"], s["dY"], d, k=_DGE_K, cap=_DGE_CAP, **grads)
    else:
        lc.linear_bwd(s["Z"], s["A"], s["b"], s["X"], s["dY"], d, **grads)
    out = {k: s[k] for k in ("Y", "dX", "dZ", "dA", "db")}
    if case["pack"]:
        out["packed"] = s["packed"]
    if case["adam"]:
        s["step"] += 1
        for name, grad, shadow in (("Z", s["dZ"], s["Z"]), ("A", s["dA"], s["A"]), ("b", s["db"], s["b"])):
            lc.adamw_step(s["theta_" + name], grad, s["m1_" + name], s["m2_" + name], s["step"], _LR, _BETA1, _BETA2,
                          _EPS, shadow=shadow)
            out["theta_" + name], out["m1_" + name] = s["theta_" + name], s["m1_" + name]
            out["m2_" + name], out["new_" + name] = s["m2_" + name], shadow
    return out


def run(s):
    case = s["case"]
    kind, d = case["kind"], case["d"]
    if kind == "train":
        return _run_train(s)
    if kind == "accum":
        out = {}
        for i in range(2):
            out["Y%d" % i] = lc.linear_fwd(s["Z"], s["A"], s["b"], s["X"][i], d)
            out["dX%d" % i] = lc.linear_bwd(s["Z"], s["A"], s["b"], s["X"][i], s["dY"][i], d, accumulate=i > 0,
                                            dz_dtype=torch.float32, dZ=s["dZ"], dA=s["dA"], db=s["db"])[0]
        return dict(out, dZ=s["dZ"], dA=s["dA"], db=s["db"])
    if kind == "eval":
        return lc.linear_fwd(s["Z"], s["A"], s["b"], s["X"], d)
    if kind == "f32":
        Y = lc.linear_fwd(s["Z"], s["A"], s["b"], s["X"], d)
        dX, dZ, dA, db = lc.linear_bwd(s["Z"], s["A"], s["b"], s["X"], s["dY"], d)
        return dict(Y=Y, dX=dX, dZ=dZ, dA=dA, db=db)
    if kind == "packed":
        if case["noalloc"]:
            return [lc.linear_fwd_packed_noalloc(x["P"], x["A"], x["b"], x["X"], d, out=x["out"]) for x in s["layers"]]
        return [lc.linear_fwd_packed(x["P"], x["A"], x["b"], x["X"], d, workspace=s["ws"], out=x["out"])
                for x in s["layers"]]
    codes, packed = lc.encode(s["W"], s["A"], s["b"], d, codes=True, packed=True)
    Wp = lc.xavier_init(codes, case["m"], case["n"], out_dtype=_BF16)
    W_hat = lc.dequant(packed, s["A"], s["b"], d, n=case["n"], src_kind=lc.SRC_PACKED2)
    return dict(codes=codes, packed=packed, W_p=Wp, W_hat=W_hat)


# ------------------------------------------------------- what a pass must move --

def work(case):
    kind, m, n, N = case["kind"], case["m"], case["n"], case.get("N", 0)
    mn, xn, ym = m * n, N * n, N * m
    if kind == "convert":  # W; codes, packed, W_p, W_hat; d fma per element each way
        return dict(bytes=mn * (2 + 1 + 0.25 + 2 + 2), flops=2.0 * mn * case["d"] * 2)
    if kind == "packed":
        return dict(bytes=sum(a * b / 4 + 2 * N * (a + b) for a, b in _packed_mats(case)),
                    flops=2.0 * N * mn * 2 * case["layers"])
    if kind == "eval":
        return dict(bytes=2.0 * (mn + xn + ym), flops=2.0 * N * mn)
    if kind == "f32":  # Z, X, dY; Y, dX, dZ
        return dict(bytes=4.0 * (2 * mn + 2 * xn + 2 * ym), flops=6.0 * N * mn)
    if kind == "accum":  # Z; per micro-batch X, dY, Y, dX; dZ once
        return dict(bytes=2.0 * mn + 2 * 4.0 * (xn + ym) + 4.0 * mn, flops=12.0 * N * mn)
    b = 2.0 * mn + 4.0 * (xn + ym) + 2.0 * mn + (mn / 4 if case["pack"] else 0)
    if case["adam"]:  # theta, m1, m2 read and written, the new latents written
        b += 26.0 * mn
    return dict(bytes=b, flops=6.0 * N * mn)


def tolerance(case):
    """fp32: sums of up to 2048 terms in another order (measured 2e-7 to 6e-7 against fp64).
    bf16: operands and results rounded to bf16 (measured 1.7e-3 to 2.4e-3 against fp64, and
    up to twice that in squares of a rounded gradient).  Codes may differ only where a weight
    lies within fp32 rounding of a decision boundary."""
    if case["kind"] == "f32":
        return dict(rel=5e-6)
    if case["kind"] == "convert":
        return dict(rel=1e-2, differ=2e-6)
    return dict(rel=1e-2)


# ------------------------------------------------------- the same in 64 bits --

def _decode64(codes, A, b, d):
    m, n = codes.shape
    return ((codes.reshape(-1, d) @ A.T) + b).reshape(m, n)


def _grads64(codes, W, A, d, X, dY):
    """dX, dW blockdiag(A), dA, db for fp64 codes and W_hat."""
    dW = dY.T @ X
    g = dW.reshape(-1, d)
    return dY @ W, (g @ A).reshape(dW.shape), g.T @ codes.reshape(-1, d), g.sum(0)


def _adam64(theta, g):
    m1, m2 = (1 - _BETA1) * g, (1 - _BETA2) * g * g
    return theta - _LR * g / (g.abs() + _EPS), m1, m2


def _pack(codes):
    c = codes.to(torch.uint8).reshape(codes.shape[0], -1, 4)
    return c[..., 0] | c[..., 1] << 2 | c[..., 2] << 4 | c[..., 3] << 6


def exact(case, seed):
    s, kind, d = prepare(case, seed), case["kind"], case["d"]
    f = torch.float64
    if kind == "packed":
        out = []
        for x in s["layers"]:
            codes = torch.stack([(x["P"] >> (2 * i)) & 3 for i in range(4)], -1).reshape(x["P"].shape[0], -1)
            out.append(x["X"].to(f) @ _decode64(codes.to(f), x["A"].to(f), x["b"].to(f), d).T)
        return out
    A, b = s["A"].to(f), s["b"].to(f)
    if kind == "convert":
        v = (s["W"].to(f).reshape(-1, d) - b) @ torch.linalg.inv(A).T
        codes = v.round().clamp(0, 3).reshape(s["W"].shape)
        a = math.sqrt(6.0 / (case["m"] + case["n"]))
        return dict(codes=codes.to(torch.uint8), packed=_pack(codes), W_p=(2 * a / 3) * (codes - 1.5),
                    W_hat=_decode64(codes, A, b, d))
    qs, qb = s.get("q", (1.0, 0.0))
    z = s["Z"].to(f)
    if (qs, qb) != (1.0, 0.0):
        z = (z * qs + qb).float().to(f)  # the quantiser rounds the fp32 value
    codes = z.round().clamp(0, 3)
    W = _decode64(codes, A, b, d)
    if kind == "eval":
        return s["X"].to(f) @ W.T
    mask = ((z.round() >= 0) & (z.round() <= 3)).to(f)
    if kind == "accum":
        out, total = {}, None
        for i in range(2):
            X, dY = s["X"][i].to(f), s["dY"][i].to(f)
            out["Y%d" % i] = X @ W.T
            out["dX%d" % i], *g = _grads64(codes, W, A, d, X, dY)
            total = g if total is None else [p + q for p, q in zip(total, g)]
        return dict(out, dZ=mask * total[0], dA=total[1], db=total[2])
    X, dY = s["X"].to(f), s["dY"].to(f)
    dX, G, dA, db = _grads64(codes, W, A, d, X, dY)
    if kind == "train" and case["dge"]:  # capped slope of the surrogate, mask of the latent itself
        w = (2 * (z - z.floor()) - 1).abs()
        slope = (w ** (1 / _DGE_K - 1) / _DGE_K).clamp(max=_DGE_CAP)
        mask = ((z >= 0) & (z <= 3)).to(f) * slope * qs
    out = dict(Y=X @ W.T, dX=dX, dZ=mask * G, dA=dA, db=db)
    if kind == "f32":
        return out
    if case["pack"]:
        out["packed"] = _pack(codes)
    if case["adam"]:
        for name, g in (("Z", out["dZ"]), ("A", dA), ("b", db)):
            out["theta_" + name], out["m1_" + name], out["m2_" + name] = _adam64(s["theta_" + name].to(f), g)
            out["new_" + name] = out["theta_" + name]
    return out
