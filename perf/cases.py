"""The calls whose speed this library is measured by, with their inputs, the work they cannot do without, what another
correct implementation may differ by, and their results in 64 bits.

A case is one call of a public entry point on inputs of the kind the library meets in use: rows of logits as an
image-token model emits them (``workloads.py`` has the recipes of which these are the GPU-made relatives), drafted tokens
drawn from them, and for the verifier rows the same logits moved by noise.  Programs that decode keep their output
buffers and their workspace from call to call, so the states here hold them wherever the entry point takes them.
"""
from __future__ import annotations

import math

import torch

import paper_2603_25463_amd as ciar
from paper_2603_25463_amd import binding

_DTYPE = {"float32": torch.float32, "bfloat16": torch.bfloat16}
_TAU = 0.01                                    # both outcomes of the threshold occur on rows like these
_LOSS = {"lambda_v": 1.0, "lambda_p": 0.5, "lambda_beta": 0.25, "alpha": 0.5}
_FLOATS = ("p_lo", "p_mid", "p_hi", "omega", "sigma", "score")
_CHUNK_TOKENS = 1 << 25                        # tokens of a tensor that are made, or checked, at a time


def listed() -> list[dict]:
    return [
        # One drafted window of one image in a tight decoding loop: the smallest call there is, all latency.
        _case("window", "fused_static", rows=8, vocab=16384, window=8),
        # All 16 x 16 tokens of one image verified at once (short windows): fewer rows than the chip has room for.
        _case("image", "fused", rows=256, vocab=16384, window=4),
        # Eight images in flight, the repository's benchmark shape.
        _case("batch", "fused", rows=2048, vocab=16384, window=8),
        # Sixteen 32 x 32 images with bf16 logits.
        _case("batch_bf16", "fused", rows=16384, vocab=16384, dtype="bfloat16", window=8, sigma=0.5),
        # A large vocabulary and many images, bf16: the largest call.
        _case("vocab64k", "fused", rows=32768, vocab=65536, dtype="bfloat16", window=8, sigma=0.4, zipf=True),
        # Device side alone: the quantifier with the radius tensor that the Interval Head emits; a ragged vocabulary and
        # a number of rows that divides into nothing.
        _case("device", "quantify", rows=1531, vocab=12345, radius=True),
        # Cloud side alone: the accept test and the draws; bf16, ragged in rows, vocabulary and window.
        _case("cloud", "verify", rows=4099, vocab=32003, dtype="bfloat16", window=7, sigma=0.5),
        # Three Interval Heads that vote, each with its radius tensor, bf16.
        _case("voting", "voting", rows=2048, vocab=16384, dtype="bfloat16", heads=3, radius=True),
        # Three Interval Heads whose intervals are averaged, each with its radius tensor.
        _case("ensemble", "ensemble", rows=2048, vocab=16384, heads=3, radius=True),
        # The training loss of a batch (forward), radius tensor included.
        _case("loss", "loss", rows=2048, vocab=16384, radius=True, sigma=0.5),
        # From hidden states to scores for eight images: the head's two linear maps, then the quantifier.
        _case("head", "head", rows=2048, vocab=16384, hidden=1280),
        # The same for one drafted window: the weights are read for eight rows.
        _case("head_window", "head", rows=8, vocab=16384, hidden=1280),
    ]


def _case(name, op, *, rows, vocab, dtype="float32", window=8, sigma=0.3, radius=False, heads=1, hidden=0, zipf=False):
    c = {"op": op, "rows": rows, "vocab": vocab, "dtype": dtype, "window": window, "sigma": sigma, "radius": radius,
         "heads": heads, "hidden": hidden, "zipf": zipf}
    return {"name": name, **c} if name else c


def draw(rng) -> dict:
    """One more case of the same ranges: every entry point, both dtypes and radius modes, odd sizes."""
    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["fused", "fused", "quantify", "verify", "voting", "ensemble", "loss", "head"])
    window = rng.choice([1, 2, 4, 5, 8, 8, 16, 31])
    if op == "head":
        # vocabularies and depths that the head's contraction is made for
        vocab = 128 * spread(16, 128)
        return _case(None, op, rows=min(spread(1, 4096), (1 << 26) // vocab), vocab=vocab, window=window,
                     hidden=64 * spread(8, 64))
    dtype = rng.choice(["float32", "bfloat16"])
    vocab = spread(1024, 32768 if dtype == "float32" else 65536)
    if rng.random() < 0.5:
        vocab = max(1024, vocab // 1024 * 1024)
    radius = rng.random() < (0.35 if op == "fused" else 0.0 if op == "verify" else 0.6)
    heads = rng.randint(2, 5) if op in ("voting", "ensemble") else 1
    tensors = heads * (1 + radius) + (op in ("fused", "verify", "loss"))
    most = 1.6e9 / (tensors * vocab * (4 if dtype == "float32" else 2))
    return _case(None, op, rows=min(spread(1, 32768), int(most)), vocab=vocab, dtype=dtype, window=window,
                 sigma=rng.choice([0.2, 0.3, 0.5]), radius=radius, heads=heads, zipf=rng.random() < 0.25)


# ---- inputs -------------------------------------------------------------------------------------------------------

def _stride(case) -> int:
    """Elements between rows: the next multiple of 16 bytes."""
    per = 4 if case["dtype"] == "float32" else 8
    return -(-case["vocab"] // per) * per


def _params(case) -> "ciar.Params":
    # with a radius tensor the head's radius as it is (scale 1), without one the radius of a 90 % interval
    if case["radius"] or case["op"] == "head":
        return ciar.Params(radius_scale=1.0, tau=_TAU, window=case["window"])
    return ciar.Params(confidence=0.9, tau=_TAU, window=case["window"])


def _inputs(case, seed) -> dict:
    """The tensors a call reads, from the seed alone."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 1000003 + 17)

    def rand(*shape):
        return torch.rand(shape, generator=gen, device="cuda")

    def randn(*shape):
        return torch.randn(shape, generator=gen, device="cuda")

    def uniform24(n):
        return torch.randint(0, 1 << 24, (n,), generator=gen, device="cuda", dtype=torch.int32).float() / (1 << 24)

    N, V, H, op = case["rows"], case["vocab"], case["heads"], case["op"]
    if op == "head":
        D = case["hidden"]
        bias = torch.zeros(2 * V, device="cuda")
        bias[V:] = -1.0                                        # radii of about 0.3 at a raw radius of 0
        return {"hidden": randn(N, D).bfloat16(), "weight": (randn(2 * V, D) * (2.0 / math.sqrt(D))).bfloat16(),
                "bias": bias, "ids": torch.randint(0, V, (N,), generator=gen, device="cuda", dtype=torch.int32)}
    dtype, stride = _DTYPE[case["dtype"]], _stride(case)
    two = op in ("fused", "fused_static", "verify", "loss")
    got = {"draft": torch.empty((H, N, stride), dtype=dtype, device="cuda")[:, :, :V]}
    if two:
        got["target"] = torch.empty((N, stride), dtype=dtype, device="cuda")[:, :V]
    if case["radius"]:
        got["radius"] = torch.empty((H, N, stride), dtype=dtype, device="cuda")[:, :, :V]
    ids = torch.empty(N, dtype=torch.int32, device="cuda")
    profile = -1.1 * torch.log1p(torch.randperm(V, generator=gen, device="cuda").float()) if case["zipf"] else 0.0
    step = max(1, _CHUNK_TOKENS // V)
    for lo in range(0, N, step):
        n = min(step, N - lo)
        # rows of their own spread, 60 % of them with one token well above the others
        scale = 1.0 if case["zipf"] else 0.5 + 2.5 * rand(n, 1)
        row = randn(n, V) * scale + profile
        at = torch.randint(0, V, (n, 1), generator=gen, device="cuda")
        row.scatter_add_(1, at, 8.0 * (rand(n, 1) < 0.6))
        for h in range(H):                                     # several heads: the same row, each with noise of its own
            own = row if H == 1 else row + 0.3 * randn(n, V)
            got["draft"][h, lo:lo + n] = own
            if case["radius"]:
                got["radius"][h, lo:lo + n] = randn(n, V) + (2.0 * rand(n, 1) - 1.0)
        if two:
            got["target"][lo:lo + n] = row + case["sigma"] * randn(n, V)
        # the drafted token: a draw from the first head's row (Gumbel-max)
        noise = rand(n, V).clamp_(min=1e-30).log_().neg_().clamp_(min=1e-30).log_()
        ids[lo:lo + n] = torch.argmax(got["draft"][0, lo:lo + n].float() - noise, dim=1)
        del row, noise
    got["ids"] = ids
    if H == 1:
        got["draft"] = got["draft"][0]
        if case["radius"]:
            got["radius"] = got["radius"][0]
    if op in ("fused", "fused_static", "verify"):
        got["u_accept"], got["u_resample"] = uniform24(N), uniform24(N)
    return got


def prepare(case, seed) -> dict:
    s = _inputs(case, seed)
    s["op"], s["params"] = case["op"], _params(case)
    N, V, op = case["rows"], case["vocab"], case["op"]
    W = -(-N // case["window"])
    out = {}
    if op in ("fused", "fused_static", "quantify", "head"):
        for k in _FLOATS:
            out[k] = torch.empty(N, dtype=torch.float32, device="cuda")
        out["flags"] = torch.empty(N, dtype=torch.uint8, device="cuda")
    if op in ("fused", "fused_static", "verify"):
        out["accept"] = torch.empty(N, dtype=torch.uint8, device="cuda")
        out["row_id"] = torch.empty(N, dtype=torch.int32, device="cuda")
        out["accept_len"] = torch.empty(W, dtype=torch.int32, device="cuda")
        out["resampled_id"] = torch.empty(W, dtype=torch.int32, device="cuda")
    s["out"] = out
    nbytes = 0
    if op in ("fused", "quantify", "verify"):
        nbytes = binding.workspace_bytes(N, s["params"].to_c(s["draft"]))
    elif op == "head":
        nbytes = binding.interhead_workspace_bytes(N, binding.head_params(s["hidden"], s["weight"], s["bias"], s["params"],
                                                                          None)[3])
    elif op in ("voting", "ensemble"):
        cp = s["params"].to_c(s["draft"][0])
        nbytes = int(ciar.lib().ciar_multihead_workspace_bytes(N, case["heads"], cp))
    s["workspace"] = torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None
    return s


def run(s):
    op, P, out, ws = s["op"], s["params"], s["out"], s["workspace"]
    if op == "fused_static":
        return ciar.quantify_verify_static(s["draft"], s["target"], s["ids"], s["u_accept"], s["u_resample"], P, out,
                                           radius=s.get("radius"))
    if op == "fused":
        return ciar.quantify_verify(s["draft"], s["target"], s["ids"], s["u_accept"], s["u_resample"], P, out=out,
                                    workspace=ws, radius=s.get("radius"))
    if op == "quantify":
        return ciar.quantify(s["draft"], s["ids"], P, out=out, workspace=ws, radius=s.get("radius"))
    if op == "verify":
        return ciar.verify(s["draft"], s["target"], s["ids"], s["u_accept"], s["u_resample"], P, out=out, workspace=ws)
    if op in ("voting", "ensemble"):
        return ciar.quantify_multihead(s["draft"], s["ids"], P, ciar.VOTING if op == "voting" else ciar.ENSEMBLE,
                                       radius_heads=s.get("radius"), workspace=ws)
    if op == "loss":
        return ciar.interdro_loss(s["draft"], s.get("radius"), s["target"], P, **_LOSS)
    return ciar.interhead_quantify(s["hidden"], s["weight"], s["bias"], s["ids"], P, out=out, workspace=ws)


# ---- what a call costs at least, and how exact it is --------------------------------------------------------------

def work(case) -> dict:
    """Each input read once, each output written once; flops only where the path is a contraction."""
    N, V, H, op = case["rows"], case["vocab"], case["heads"], case["op"]
    W = -(-N // case["window"])
    if op == "head":
        D = case["hidden"]
        return {"bytes": 2 * N * D + 2 * 2 * V * D + 4 * 2 * V + (4 + 25) * N, "flops": 2 * N * 2 * V * D}
    rows = H * (1 + case["radius"]) + (op in ("fused", "fused_static", "verify", "loss"))
    small = {"fused": 12 + 30, "fused_static": 12 + 30, "verify": 12 + 5, "quantify": 4 + 25, "voting": 4 + 1 + 25 * H,
             "ensemble": 4 + 25, "loss": 32}[op]
    return {"bytes": rows * N * V * (4 if case["dtype"] == "float32" else 2) + small * N + 8 * W, "flops": 0}


def tolerance(case) -> dict:
    # 32-bit exponentials and reciprocals, 64-bit sums, results rounded to 32 bits.  The threshold, the accept test and
    # the draw are decisions on such numbers: one that lies within rounding of its boundary may fall either way.
    if case["op"] == "head":
        # the logits are 32-bit sums of `hidden` products: their order moves a logit by ~1e-6 (seen against 64 bits: 1.1e-6)
        return {"rel": 5e-6, "max": 1e-4, "differ": 0.005}
    # (seen against 64 bits: 3e-7 of a few rows' bounds, 1e-7 of many)
    return {"rel": 1.2e-6, "max": 3e-5, "differ": 0.005}


# ---- the results in 64 bits, in plain torch -----------------------------------------------------------------------

def _interval(c, raw, case):
    """(p_lo, p, p_hi) of rows of centre logits, caps applied; raw: the radius tensor's rows or None."""
    x = torch.softmax(c.double(), dim=1)
    if raw is None:
        z = math.sqrt(2.0) * torch.erfinv(torch.tensor(float(torch.tensor(0.9, dtype=torch.float32)), dtype=torch.float64))
        r = torch.full((1, 1), min(float(z), 10.0), dtype=torch.float64, device=c.device)
    else:
        r = torch.nn.functional.softplus(raw.double(), threshold=700.0).clamp(max=10.0)
    up, dn = torch.exp(r), torch.exp(-r)
    rest = 1.0 - x
    lo, hi = dn * x / (rest + dn * x), up * x / (rest + up * x)
    lo = lo * torch.clamp(float(torch.tensor(0.99)) / lo.sum(1, keepdim=True), max=1.0)
    hi = hi * torch.clamp(float(torch.tensor(1.01)) / hi.sum(1, keepdim=True), min=1.0)
    return lo, x, hi


def _scores(lo, mid, hi, ids):
    at = ids.long()[:, None]
    width = hi - lo
    omega, sigma = width.sum(1), width.std(1, unbiased=False)
    return {"p_lo": lo.gather(1, at)[:, 0], "p_mid": mid.gather(1, at)[:, 0], "p_hi": hi.gather(1, at)[:, 0],
            "omega": omega, "sigma": sigma, "score": omega * sigma}


def _loss_terms(c, raw, t, case):
    if raw is None:
        r = torch.zeros((1, 1), dtype=torch.float64, device=c.device)   # a constant radius cancels in both softmaxes
    else:
        r = torch.nn.functional.softplus(raw.double(), threshold=700.0).clamp(max=10.0)
    c, q = c.double(), torch.softmax(t.double(), dim=1)
    logs = [torch.log_softmax(o, dim=1) for o in (c, c + r, c - r)]
    terms = [(l.exp() - q).abs().sum(1) for l in logs] + [-(q * l).sum(1) for l in logs]
    terms.append((q * (torch.log_softmax(t.double(), dim=1) - logs[0])).sum(1))
    return torch.stack(terms)


def exact(case, seed):
    s = _inputs(case, seed)
    N, V, H, op = case["rows"], case["vocab"], case["heads"], case["op"]
    whole = {"fused": ("flags", "accept", "row_id", "accept_len", "resampled_id"), "quantify": ("flags",),
             "verify": ("accept", "row_id", "accept_len", "resampled_id"), "voting": ("flags", "head_flags"),
             "ensemble": ("flags",), "head": ("flags",)}
    whole["fused_static"] = whole["fused"]
    if op == "verify":
        return None                                            # its outputs are whole numbers
    parts = []
    step = max(1, _CHUNK_TOKENS // V)
    for lo in range(0, N, step):
        k = slice(lo, min(lo + step, N))
        if op == "loss":
            parts.append(_loss_terms(s["draft"][k], s["radius"][k] if case["radius"] else None, s["target"][k], case))
            continue
        if op == "head":
            z = s["hidden"][k].double() @ s["weight"].double().T + s["bias"].double()
            curves = [_interval(z[:, :V], z[:, V:], case)]
        else:
            c = s["draft"] if H > 1 else s["draft"][None]
            r = (s["radius"] if H > 1 else s["radius"][None]) if case["radius"] else [None] * H
            curves = [_interval(c[h, k], r[h][k] if case["radius"] else None, case) for h in range(H)]
        ids = s["ids"][k]
        if op == "voting":
            each = [_scores(*cv, ids) for cv in curves]
            parts.append({f: torch.stack([e[f] for e in each]) for f in _FLOATS})
        elif op == "ensemble":
            parts.append(_scores(*[sum(cv[i] for cv in curves) / H for i in range(3)], ids))
        else:
            parts.append(_scores(*curves[0], ids))
        del curves
    if op == "loss":
        terms = torch.cat(parts, dim=1)
        l1, ce = terms[0:3], terms[3:6]
        w = torch.softmax(_LOSS["alpha"] * ce[2], dim=0)
        side = _LOSS["lambda_v"] * l1.mean(1) + _LOSS["lambda_p"] * ce.mean(1)
        center = side[0] + _LOSS["lambda_beta"] * terms[6].mean()
        dro = (w * ce[2]).sum()
        return {"terms": terms, "weights": w,
                "losses": torch.stack([center, side[1], side[2], dro, center + side[1] + side[2] + dro])}
    got = {f: torch.cat([p[f] for p in parts], dim=-1) for f in _FLOATS}
    got.update({f: None for f in whole[op]})
    return got
