"""What a user of this library has it do, as cases that can be timed and compared.

A case is a dict of plain values.  `kind` names the piece of work:

  layer        one linear layer through the five calibration stages (the loop body of Algorithm 1)
  block        the attention projections of one block (q, k, v on one input, o on another) in one
               aser_calibrate_layers call on three contexts
  gram         the statistics of one input, streamed in chunks of tokens
  whiten       the Cholesky factor of a smoothed Gram matrix
  reconstruct  the rank-r factors from T and S
  forward      the compensated layer at inference: the per-token activation quantizer, then the product
               (prefill: thousands of tokens; decode: one token or a small batch of them)
  spectrum     all singular values of T S, the rank for a threshold and the effective rank (Eq. 9, Eq. 3)
  output_error the layer-output error of Sec. 5.3 on a sample of tokens

Inputs follow the statistics of the seeded synthetic layers (aser_synth.py): Gaussian or post-SiLU
activations with a few large channels, Gaussian weights with 0.1 % heavy-tailed entries.  The number of planted
channels, of extracted ones and the rank agree (f = r), so that the singular values have a gap behind the
r-th and the rank-r correction L_A L_B is determined; the single columns of L_A and L_B are determined up to a
sign only, which is why the cases return the product.
"""
import math

import numpy as np
import torch

import paper_2411_07762_amd as aser

DEV = "cuda:0"


def listed():
    return [
        # the smallest layer of the tests and of the smoke run: all fp32, latency and launches
        {"name": "layer_256_f32", "kind": "layer", "m": 256, "n": 256, "tokens": 1024, "x": "f32", "dist": "gauss", "bits": 4, "r": 8},
        # the headline layer: a 4096 x 4096 attention projection, 32768 calibration tokens, W4
        {"name": "layer_4096", "kind": "layer", "m": 4096, "n": 4096, "tokens": 32768, "x": "bf16", "dist": "gauss", "bits": 4, "r": 64},
        # an MLP down projection with post-SiLU activations, the largest layer calibrated here in one go
        {"name": "layer_down_11008", "kind": "layer", "m": 4096, "n": 11008, "tokens": 65536, "x": "bf16", "dist": "silu", "bits": 4, "r": 64},
        # the attention projections of a Llama-3-8B-shaped block in one call, several layers in flight
        {"name": "block_attention", "kind": "block", "hidden": 4096, "kv": 1024, "tokens": 16384, "bits": 4, "r": 64},
        # calibration data that arrives in chunks, with a ragged last one
        {"name": "gram_4096_chunks", "kind": "gram", "n": 4096, "tokens": 30011, "chunks": 4, "x": "bf16"},
        # the whitening factor of a 4096-channel input
        {"name": "whiten_4096", "kind": "whiten", "n": 4096, "tokens": 32768},
        # the factors of a gate projection
        {"name": "reconstruct_gate", "kind": "reconstruct", "m": 14336, "n": 4096, "tokens": 32768, "r": 64},
        # W4A8 inference on a prompt of a few thousand tokens
        {"name": "prefill_w4a8", "kind": "forward", "rows": 8192, "n": 4096, "m": 4096, "r": 64, "bits": 4, "split": False},
        # W4A8 decoding, one token, up projection
        {"name": "decode_1_w4a8", "kind": "forward", "rows": 1, "n": 4096, "m": 14336, "r": 64, "bits": 4, "split": False},
        # W8A8 decoding of a small ragged batch, down projection, fp32-class rank-r branch
        {"name": "decode_19_w8a8", "kind": "forward", "rows": 19, "n": 11008, "m": 4096, "r": 64, "bits": 8, "split": True},
        # the rank rule of Eq. 9 on the headline layer: every singular value
        {"name": "spectrum_4096", "kind": "spectrum", "m": 4096, "n": 4096, "tokens": 32768, "r": 64},
        # the remaining layer-output error on one calibration sample of 2048 tokens, W4A8
        {"name": "output_error_2048", "kind": "output_error", "rows": 2048, "m": 4096, "n": 4096, "r": 64, "bits": 4, "act_bits": 8},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """A layer width: mostly the multiples that models have, now and then an odd one."""
    v = _log(rng, lo, hi)
    step = rng.choice([1, 8, 32, 128, 128, 256, 256])
    return max(lo, v // step * step)


def draw(rng):
    kind = rng.choice(["layer", "layer", "block", "gram", "whiten", "reconstruct", "forward", "forward", "forward", "spectrum", "output_error"])
    r = rng.choice([8, 16, 32, 64])
    if kind == "layer":
        m, n = _size(rng, 192, 8192), _size(rng, 192, 8192)
        x = rng.choice(["bf16", "bf16", "f32"]) if n <= 2048 else "bf16"
        return {"kind": kind, "m": m, "n": n, "tokens": _log(rng, max(1024, 4 * n), 65536), "x": x,
                "dist": rng.choice(["gauss", "silu"]), "bits": rng.choice([4, 4, 8]), "r": r}
    if kind == "block":
        h = rng.choice([1024, 1536, 2048, 2560, 3072, 4096])
        return {"kind": kind, "hidden": h, "kv": h // rng.choice([1, 2, 4]), "tokens": _log(rng, 4 * h, 16384), "bits": rng.choice([4, 8]), "r": r}
    if kind == "gram":
        return {"kind": kind, "n": _size(rng, 256, 14336), "tokens": _log(rng, 1000, 40000), "chunks": rng.choice([1, 2, 4, 8]),
                "x": rng.choice(["bf16", "bf16", "bf16", "f32"])}
    if kind == "whiten":
        n = _size(rng, 256, 11008)
        return {"kind": kind, "n": n, "tokens": 4 * n + _log(rng, 100, 30000)}
    if kind == "reconstruct":
        m, n = _size(rng, 512, 14336), _size(rng, 512, 8192)
        return {"kind": kind, "m": m, "n": n, "tokens": 4 * n + _log(rng, 100, 30000), "r": rng.choice([16, 32, 64, 64, 128])}
    if kind == "forward":
        return {"kind": kind, "rows": rng.choice([_log(rng, 1, 16), _log(rng, 2, 256), _log(rng, 128, 16384)]), "n": 32 * _log(rng, 16, 448),
                "m": _size(rng, 512, 14336), "r": rng.choice([0, 16, 40, 64, 64, 128]), "bits": rng.choice([4, 8]), "split": rng.choice([False, True])}
    if kind == "spectrum":
        return {"kind": kind, "m": _size(rng, 256, 4096), "n": _size(rng, 512, 4096), "tokens": 32768, "r": r}
    return {"kind": kind, "rows": _log(rng, 128, 4096), "m": _size(rng, 512, 6144), "n": _size(rng, 512, 6144), "r": rng.choice([0, 16, 64]),
            "bits": rng.choice([4, 8]), "act_bits": rng.choice([0, 6, 8])}


# ------------------------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32)


def _rand(g, *shape):
    return torch.rand(shape, generator=g, device=DEV, dtype=torch.float32)


def _weight(g, m, n):
    """N(0, 0.02^2) with 0.1 % of the entries drawn from Student-t(3) * 0.1."""
    w = _randn(g, m, n) * 0.02
    k = max(1, m * n // 1000)
    pos = torch.unique(torch.randint(0, m * n, (k,), generator=g, device=DEV))
    t = _randn(g, pos.numel()) / torch.sqrt(_randn(g, 3, pos.numel()).square().sum(0) / 3.0)
    w.view(-1)[pos] = 0.1 * t
    return w


def _channels(g, n, count):
    """Which channels are large, and the factor of every channel."""
    idx = torch.randperm(n, generator=g, device=DEV)[:count]
    fac = torch.ones(n, device=DEV)
    fac[idx] = 20.0 + 40.0 * _rand(g, count)
    return idx, fac


def _activations(g, tokens, n, dist, dtype, fac):
    out = torch.empty((tokens, n), dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device=DEV)
    for a in range(0, tokens, 8192):
        b = min(tokens, a + 8192)
        x = _randn(g, b - a, n)
        if dist == "silu":
            z = _randn(g, b - a, n)
            x *= z * torch.sigmoid(z)
        out[a:b] = x * fac
    return out


def _bartlett(g, n, tokens, scale):
    """The lower Cholesky factor, in fp64, of X^T X for `tokens` Gaussian tokens with channel factors `scale` (Bartlett
    decomposition; the chi-distributed diagonal by its normal approximation)."""
    L = torch.tril(_randn(g, n, n).double(), -1)
    i = torch.arange(n, device=DEV, dtype=torch.float64)
    L.diagonal().copy_(torch.sqrt(tokens - i - 0.5) + 0.7071 * _randn(g, n).double())
    return scale.double()[:, None] * L


def _smoothing(g, n, f):
    """Outlier set in descending score order (here: of the factor), M, and the channel factors of X."""
    idx, fac = _channels(g, n, f)
    idx = idx[torch.argsort(fac[idx], descending=True)]
    md = torch.ones(n, device=DEV)
    md[idx] = fac[idx] / fac[idx].min()
    return idx.to(torch.int32), md, fac


def _target(g, m, n, idx, md):
    """T of Eq. 12: rounding errors of a 4-bit quantizer, the scaled weight itself in the outlier columns."""
    step = 0.012 + 0.02 * _rand(g, m, 1)
    T = (_rand(g, m, n) - 0.5) * step
    cols = idx.long()
    T[:, cols] = 0.02 * _randn(g, m, cols.numel()) * md[cols]
    return T


def _quantized_layer(g, m, n, r, bits):
    """Codes, scales and factors as a calibrated layer has them."""
    q = torch.clamp(torch.round(_randn(g, m, n) * (2.0 if bits == 4 else 36.0)), -(2 ** (bits - 1) - 1), 2 ** (bits - 1) - 1).to(torch.int8)
    packed = bits == 4 and n % 2 == 0
    codes = ((q[:, 0::2] & 15) | (q[:, 1::2] << 4)).view(torch.uint8).contiguous() if packed else q
    scales = (0.02 + 0.01 * _rand(g, m)) / (2 ** (bits - 1) - 1)
    L_A = _randn(g, m, r) * 0.3 if r else None
    L_B = _randn(g, r, n) * (0.02 / math.sqrt(max(r, 1))) if r else None
    return q, codes, (aser.ASER_CODES_INT4_PACKED if packed else aser.ASER_CODES_INT8), scales, L_A, L_B


def _layer_inputs(case, g, m, n, x=None):
    if x is None:
        _, fac = _channels(g, n, case["r"])
        x = _activations(g, case["tokens"], n, case.get("dist", "gauss"), case.get("x", "bf16"), fac)
    return _weight(g, m, n), x


def _new_buffers(case, m, n):
    return aser.LayerBuffers(m, n, case["r"], case["r"], case["bits"], packed=(case["bits"] == 4 and n % 2 == 0))


BLOCK = (("q", "hidden", 0), ("k", "kv", 0), ("v", "kv", 0), ("o", "hidden", 1))


def _block_inputs(case, g):
    h = case["hidden"]
    xs = [_activations(g, case["tokens"], h, "gauss", "bf16", _channels(g, h, case["r"])[1]) for _ in range(2)]
    return [(name, _weight(g, case[rows], h), xs[s]) for name, rows, s in BLOCK]


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    s = {"kind": kind, "case": dict(case)}
    if kind == "block":
        s["layers"] = _block_inputs(case, g)
        s["bufs"] = [_new_buffers(case, W.shape[0], W.shape[1]) for _, W, _ in s["layers"]]
        s["streams"] = [torch.cuda.Stream() for _ in range(6)]
        st, pick = aser.aser_pick_concurrent_streams([t.cuda_stream for t in s["streams"]], 3)
        assert st == aser.ASER_OK
        s["streams"] = [s["streams"][i] for i in pick]
        s["ctxs"] = [aser.Context(0, t.cuda_stream) for t in s["streams"]]
        s["descs"] = [aser.layer_desc(W, b, X=None if name in "kv" else X, clear_stats=name not in "kv", stats_from=0 if name in "kv" else None)
                      for (name, W, X), b in zip(s["layers"], s["bufs"])]
        need = max(aser.aser_layer_workspace_bytes(d) for d in s["descs"])
        for c in s["ctxs"]:
            c.ensure_workspace(need)
        torch.cuda.synchronize()
        return s
    ctx = s["ctx"] = aser.Context(0)
    if kind == "layer":
        m, n, r = case["m"], case["n"], case["r"]
        s["W"], s["X"] = _layer_inputs(case, g, m, n)
        s["buf"] = _new_buffers(case, m, n)
        ctx.ensure_workspace(aser.aser_workspace_bytes(m, n, r))
    elif kind == "gram":
        n = case["n"]
        s["X"] = _activations(g, case["tokens"], n, "gauss", case["x"], _channels(g, n, 16)[1])
        s["G"] = torch.zeros((n, n), dtype=torch.float32, device=DEV)
        s["abs_sum"] = torch.zeros(n, dtype=torch.float64, device=DEV)
        s["count"] = torch.zeros(1, dtype=torch.int64, device=DEV)
    elif kind == "whiten":
        n = case["n"]
        _, s["md"], fac = _smoothing(g, n, 32)
        L = _bartlett(g, n, case["tokens"], fac)
        s["G"] = (L @ L.T).float()
        s["S"] = torch.empty((n, n), dtype=torch.float32, device=DEV)
        ctx.ensure_workspace(aser.aser_workspace_bytes(n, n, 0))
    elif kind in ("reconstruct", "spectrum"):
        m, n, r = case["m"], case["n"], case["r"]
        s["idx"], md, fac = _smoothing(g, n, r)
        s["T"] = _target(g, m, n, s["idx"], md)
        s["S"] = _bartlett(g, n, case["tokens"], fac / md).float()
        if kind == "reconstruct":
            s["L_A"] = torch.empty((m, r), dtype=torch.float32, device=DEV)
            s["L_B"] = torch.empty((r, n), dtype=torch.float32, device=DEV)
            s["sigma"] = torch.empty(r, dtype=torch.float32, device=DEV)
            ctx.ensure_workspace(aser.aser_workspace_bytes(m, n, r))
        else:
            s["sigma"] = torch.empty(min(m, n), dtype=torch.float64, device=DEV)
            ctx.ensure_workspace(aser.aser_spectrum_workspace_bytes(m, n, True))
    elif kind == "forward":
        rows, n, m, r = case["rows"], case["n"], case["m"], case["r"]
        _, s["md"], fac = _smoothing(g, n, 32)
        s["X"] = _activations(g, rows, n, "gauss", "bf16", fac)
        s["q"], s["codes"], s["layout"], s["scales"], s["L_A"], s["L_B"] = _quantized_layer(g, m, n, r, case["bits"])
        s["xq"] = torch.empty((rows, n), dtype=torch.int8, device=DEV)
        s["xs"] = torch.empty(rows, dtype=torch.float32, device=DEV)
        s["Y"] = torch.empty((rows, m), dtype=torch.float32, device=DEV)
        ctx.ensure_workspace(aser.aser_forward_workspace_bytes(rows, n, m, r))
    elif kind == "output_error":
        rows, n, m, r = case["rows"], case["n"], case["m"], case["r"]
        s["W"] = _weight(g, m, n)
        _, s["md"], fac = _smoothing(g, n, 32)
        s["X"] = _activations(g, rows, n, "gauss", "bf16", fac)
        s["q"], s["codes"], s["layout"], s["scales"], s["L_A"], s["L_B"] = _quantized_layer(g, m, n, r, case["bits"])
        ctx.ensure_workspace(aser.aser_output_error_workspace_bytes(m, n, rows, r))
    else:
        raise ValueError(kind)
    return s


# ------------------------------------------------------------------------------------ one pass
def _layer_out(b):
    return {"codes": b.codes, "scales": b.scales, "idx": b.idx, "mdiag": b.mdiag, "sigma": b.sigma, "err": b.err, "correction": b.L_A @ b.L_B}


def run(s):
    kind, case = s["kind"], s["case"]
    if kind == "layer":
        s["buf"].reset_statistics()
        aser.calibrate_layer(s["ctx"], s["W"], s["X"], s["buf"])
        return _layer_out(s["buf"])
    if kind == "block":
        for t in s["streams"]:
            t.wait_stream(torch.cuda.current_stream())
        st = aser.aser_calibrate_layers(s["ctxs"], s["descs"])
        assert st == aser.ASER_OK, s["ctxs"][0].last_error()
        for b, d in zip(s["bufs"], s["descs"]):
            b.err = d.err
        return [_layer_out(b) for b in s["bufs"]]
    ctx = s["ctx"]
    if kind == "gram":
        s["G"].zero_(), s["abs_sum"].zero_(), s["count"].zero_()
        per = -(-case["tokens"] // case["chunks"])
        for a in range(0, case["tokens"], per):
            ctx.check(aser.aser_gram_accumulate(ctx, s["X"][a:a + per], s["G"], s["abs_sum"], s["count"]))
        return {"G": s["G"].tril_(), "abs_sum": s["abs_sum"], "count": s["count"]}       # only the lower triangle is defined
    if kind == "whiten":
        st, info = aser.aser_whiten(ctx, s["G"], s["md"], 0.0, s["S"])
        ctx.check(st)
        return {"S": s["S"], "info": info}
    if kind == "reconstruct":
        st, err, _ = aser.aser_error_reconstruct(ctx, s["T"], s["S"], case["r"], s["L_A"], s["L_B"], s["sigma"], idx=s["idx"], f=case["r"])
        ctx.check(st)
        return {"sigma": s["sigma"], "err": err, "correction": s["L_A"] @ s["L_B"]}
    if kind == "forward":
        ctx.check(aser.aser_quantize_act_rtn(ctx, s["X"], s["md"], 8, s["xq"], s["xs"]))
        ctx.check(aser.aser_compensated_forward(ctx, s["xq"], s["xs"], s["codes"], s["layout"], s["scales"], s["L_A"], s["L_B"], case["r"],
                                                case["split"], s["Y"]))
        return {"codes": s["xq"], "scales": s["xs"], "Y": s["Y"]}
    if kind == "spectrum":
        ctx.check(aser.aser_singular_values(ctx, s["T"], s["S"], s["sigma"]))
        st, r, share = aser.aser_select_rank(ctx, s["sigma"], 0.5)
        ctx.check(st)
        st, erank = aser.aser_effective_rank(ctx, s["sigma"])
        ctx.check(st)
        return {"sigma": s["sigma"], "rank": r, "share": list(share), "erank": erank}
    st, err, ref = aser.aser_layer_output_error(ctx, s["W"], s["X"], s["md"], s["codes"], s["layout"], s["scales"], s["L_A"], s["L_B"], case["r"],
                                                case["act_bits"])
    ctx.check(st)
    return {"err": err, "ref": ref}


# ------------------------------------------------------------------------------------ what a pass cannot do without
def _layer_work(m, n, tokens, esz, bits, r, gram=True):
    b = 4 * m * n + m * n * bits / 8 + 4 * r * (m + n)
    f = n ** 3 / 3 + m * n * (n + 1) + 4 * m * n * r
    if gram:
        b += tokens * n * esz
        f += tokens * n * (n + 1)
    return b, f


def work(case):
    kind = case["kind"]
    if kind == "layer":
        b, f = _layer_work(case["m"], case["n"], case["tokens"], 2 if case["x"] == "bf16" else 4, case["bits"], case["r"])
    elif kind == "block":
        b = f = 0.0
        for name, rows, _ in BLOCK:
            db, df = _layer_work(case[rows], case["hidden"], case["tokens"], 2, case["bits"], case["r"], gram=name in "qo")
            b, f = b + db, f + df
    elif kind == "gram":
        n, t = case["n"], case["tokens"]
        b, f = t * n * (2 if case["x"] == "bf16" else 4) + 2 * n * (n + 1), t * n * (n + 1)
    elif kind == "whiten":
        n = case["n"]
        b, f = 2 * n * (n + 1) + 4 * n * n, n ** 3 / 3
    elif kind == "reconstruct":
        m, n, r = case["m"], case["n"], case["r"]
        b, f = 4 * m * n + 2 * n * (n + 1) + 4 * r * (m + n), m * n * (n + 1) + 4 * m * n * r
    elif kind == "forward":
        rows, n, m, r = case["rows"], case["n"], case["m"], case["r"]
        b = 2 * rows * n + m * n * case["bits"] / 8 + 4 * r * (m + n) + rows * n + 4 * rows * m
        f = 2 * rows * n * m + 2 * rows * r * (m + n)
    elif kind == "spectrum":
        m, n = case["m"], case["n"]
        k = min(m, n)
        b, f = 4 * m * n + 2 * n * (n + 1) + 8 * k, m * n * (n + 1) + m * n * k + 4 * k ** 3 / 3
    else:
        rows, n, m, r = case["rows"], case["n"], case["m"], case["r"]
        b, f = 2 * rows * n + 4 * m * n + m * n * case["bits"] / 8 + 4 * r * (m + n), 4 * rows * n * m + 2 * m * n * r
    return {"bytes": b, "flops": f}


def tolerance(case):
    """About four times what two correct evaluations differ by: fp32 sums in another order and 2^-16 per fp32 product, as the
    library's products carry; codes, indices and counts are the same."""
    kind = case["kind"]
    if kind in ("layer", "block", "reconstruct"):
        return {"rel": 4e-5, "max": 4e-3, "differ": 0.0}
    if kind == "gram":
        return {"rel": 2e-6, "max": 2e-5, "differ": 0.0}
    if kind == "whiten":
        return {"rel": 1e-5, "max": 1e-3, "differ": 0.0}
    if kind == "forward":
        if not case["r"]:
            return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}
        return {"rel": 2e-5 if case["split"] else 8e-3, "max": 4e-4 if case["split"] else 0.1, "differ": 0.0}
    if kind == "spectrum":
        return {"rel": 1e-5, "max": 1e-3, "differ": 0.0}
    return {"rel": 1e-5, "max": 1e-4}


# ------------------------------------------------------------------------------------ the same in 64 bits
def _exact_rtn(W, idx, bits):
    Ws = W.cpu().clone()
    Ws[:, idx.cpu().long()] = 0.0
    amax = Ws.abs().amax(dim=1)
    scales = amax / np.float32(2 ** (bits - 1) - 1)
    scales[amax == 0] = 1.0
    return torch.round(Ws / scales[:, None]), scales


def _truncated(A, r):
    """The r largest singular values of A, their left vectors, and the norm of what is left."""
    g = _gen(1)
    Q = torch.linalg.qr(torch.randn((A.shape[0], min(r + 32, min(A.shape))), generator=g, device=A.device, dtype=torch.float64).cpu())[0].to(A.device)
    for _ in range(16):
        Q = torch.linalg.qr((A @ (A.T @ Q)).cpu())[0].to(A.device)
    U, sg, _ = torch.linalg.svd((Q.T @ A).cpu(), full_matrices=False)
    U = Q @ U[:, :r].to(A.device)
    err = float(torch.linalg.norm(A - U @ (U.T @ A)))
    return U, sg[:r].to(A.device), err


def _exact_gram(X):
    n = X.shape[1]
    G = torch.zeros((n, n), dtype=torch.float64, device=DEV)
    a = torch.zeros(n, dtype=torch.float64, device=DEV)
    for i in range(0, X.shape[0], 16384):
        x = X[i:i + 16384].double()
        G += x.T @ x
        a += x.abs().sum(0)
    return G, a


def _exact_layer(W, X, stats, r, bits):
    G, a = stats if stats is not None else _exact_gram(X)
    m, n = W.shape
    xbar = a / X.shape[0]
    score = xbar * W.double().abs().mean(0)
    idx = torch.argsort(score, descending=True, stable=True)[:r]
    md = torch.ones(n, dtype=torch.float64, device=DEV)
    md[idx] = xbar[idx] / xbar[idx].min()
    md32 = md.float()
    codes, scales = _exact_rtn(W, idx, bits)
    T = W.double() * md32.double() - codes.to(DEV).double() * scales.to(DEV).double()[:, None]
    Gs = G / (md32.double()[:, None] * md32.double()[None, :])
    S = torch.linalg.cholesky(Gs.cpu()).to(DEV)
    U, sg, err = _truncated(T @ S, r)
    return {"codes": None, "scales": scales.double(), "idx": None, "mdiag": md, "sigma": sg, "err": err, "correction": U @ (U.T @ T)}


def _exact_act(X, md, bits):
    x = X.float().cpu() / md.cpu()
    amax = x.abs().amax(dim=1)
    scales = amax / np.float32(2 ** (bits - 1) - 1)
    scales[amax == 0] = 1.0
    return torch.round(x / scales[:, None]).to(DEV).double(), scales.to(DEV).double()


def exact(case, seed):
    kind = case["kind"]
    if kind == "layer":
        if case["n"] > 12000:
            return None
        W, X = _layer_inputs(case, _gen(seed), case["m"], case["n"])
        return _exact_layer(W, X, None, case["r"], case["bits"])
    if kind == "block":
        layers = _block_inputs(case, _gen(seed))
        stats = {}
        for _, _, X in layers:
            if X.data_ptr() not in stats:
                stats[X.data_ptr()] = _exact_gram(X)
        return [_exact_layer(W, X, stats[X.data_ptr()], case["r"], case["bits"]) for _, W, X in layers]
    s = prepare(case, seed)
    if kind == "gram":
        G, a = _exact_gram(s["X"])
        return {"G": G.tril_(), "abs_sum": a, "count": None}
    if kind == "whiten":
        G = torch.tril(s["G"].double())
        G = G + torch.tril(G, -1).T
        md = s["md"].double()
        return {"S": torch.linalg.cholesky((G / (md[:, None] * md[None, :])).cpu()), "info": None}
    if kind == "reconstruct":
        T = s["T"].double()
        U, sg, err = _truncated(T @ s["S"].double(), case["r"])
        return {"sigma": sg, "err": err, "correction": U @ (U.T @ T)}
    if kind == "spectrum":
        A = s["T"].double() @ s["S"].double()
        B = (A @ A.T if case["m"] <= case["n"] else A.T @ A).cpu()
        sg = torch.linalg.eigvalsh(B).clamp_min(0).sqrt().flip(0)
        c = torch.cumsum(sg, 0) / sg.sum()
        r = max(1, int((c < 0.5).sum()))
        p = sg / sg.sum() + 1e-12
        return {"sigma": sg, "rank": None, "share": [float(sg.sum()), float(c[r - 1]), float(c[r])], "erank": float(torch.exp(-(p * torch.log(p)).sum()))}
    Wq = s["q"].double() * s["scales"].double()[:, None]
    low = (s["L_A"].double() @ s["L_B"].double()) if case["r"] else 0.0
    if kind == "forward":
        q, xs = _exact_act(s["X"], s["md"], 8)
        return {"codes": None, "scales": xs, "Y": (q * xs[:, None]) @ (Wq + low).T}
    if case["act_bits"]:
        q, xs = _exact_act(s["X"], s["md"], case["act_bits"])
        xq = q * xs[:, None]
    else:
        xq = s["X"].double() / s["md"].double()
    Y = s["X"].double() @ s["W"].double().T
    return {"err": float(torch.linalg.norm(Y - xq @ (Wq + low).T)), "ref": float(torch.linalg.norm(Y))}
