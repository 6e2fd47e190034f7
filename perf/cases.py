"""The attention calls whose speed is watched, as a program that uses this
package makes them.

A case names one call pattern and its sizes.  ``run`` goes through the public
binding only: a forward (``fwd``), a forward into buffers the caller keeps
(``noalloc``), a training step's attention, forward then backward (``step``),
and the same with quadratic-term dropout, whose keep bits are drawn afresh on
every step (``dropout``).

Inputs follow the recipe of the package's synthetic workloads: q, k, v and the
upstream gradient are standard normal; the long non-causal sequence has 5% of
its tokens multiplied by four.
"""
import math

import torch

from paper_2402_07901_amd import fastmax as fm

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def _case(call, B, H, N, D, p, causal, dtype, scale=1.0, rate=0.0, outliers=False):
    return {"call": call, "B": B, "H": H, "N": N, "D": D, "p": p, "causal": causal,
            "dtype": dtype, "scale": scale, "rate": rate, "outliers": outliers}


def listed():
    cases = {
        # the explicit-matrix cross-check size: one short float32 head, where
        # only latency counts
        "small_noncausal_f32": _case("fwd", 1, 1, 256, 16, 2, False, "f32"),
        # a prompt of odd length through a 12-head layer, into kept buffers
        # (serving, graph capture)
        "prompt_causal_bf16": _case("noalloc", 1, 12, 777, 64, 2, True, "bf16"),
        # Long Range Arena training (head size 32, about 2000 tokens), first
        # order with unit-norm scores, and second order
        "lra_step_p1_f32": _case("step", 2, 4, 2048, 32, 1, True, "f32", scale=1.0 / 32),
        "lra_step_p2_f32": _case("step", 2, 4, 2048, 32, 2, True, "f32"),
        # linear attention (first order, unit-norm scores) in a bf16 training
        # step over sequences of odd length
        "linear_step_p1_bf16": _case("step", 4, 16, 3001, 64, 1, True, "bf16", scale=1.0 / 64),
        # a GPT-style layer's forward: the headline
        "gpt_causal_bf16": _case("fwd", 4, 16, 8192, 64, 2, True, "bf16"),
        # a layer's training step, with the causal mask and without
        "step_causal_bf16": _case("step", 8, 12, 4096, 64, 2, True, "bf16"),
        "step_noncausal_bf16": _case("step", 8, 12, 4096, 64, 2, False, "bf16"),
        # long-range encoding: eight heads over 131072 tokens
        "long_noncausal_bf16": _case("fwd", 1, 8, 131072, 64, 2, False, "bf16", outliers=True),
        # long-context prefill: eight causal heads over 65536 tokens
        "long_causal_bf16": _case("fwd", 1, 8, 65536, 64, 2, True, "bf16"),
        # a training step at the Llama-2 head size
        "step_d128_causal_bf16": _case("step", 1, 8, 4096, 128, 2, True, "bf16"),
        # a training step with quadratic-term dropout at softmax's temperature
        "dropout_step_bf16": _case("dropout", 8, 12, 4096, 64, 2, True, "bf16", scale=0.125,
                                   rate=0.1),
    }
    return [dict(c, name=name) for name, c in cases.items()]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """A case of one of the families above; the bound on its token-heads keeps
    it below the largest listed case."""
    family = rng.choice(["f32_fwd", "f32_step", "bf16_fwd", "bf16_step", "bf16_step", "bf16_long",
                         "p1_step", "d128", "dropout"])
    causal = rng.random() < 0.6
    B, H = rng.choice([1, 2, 3, 4, 8]), rng.choice([1, 4, 5, 8, 12, 16])

    def tokens(lo, hi, most):
        return _log_int(rng, lo, max(lo, min(hi, most // (B * H))))

    if family == "f32_fwd":
        D = rng.choice([16, 32, 64])
        return _case("fwd", B, H, tokens(64, 4096, 131072), D, 2, causal, "f32")
    if family == "f32_step":
        D = rng.choice([16, 32, 64])
        return _case("step", B, H, tokens(200, 4096, 65536), D, rng.choice([1, 2]), causal, "f32",
                     scale=1.0 / D)
    if family == "bf16_fwd":
        return _case(rng.choice(["fwd", "noalloc"]) if B * H <= 12 else "fwd", B, H,
                     tokens(64, 8192, 524288 if B * H > 12 else 40000), 64, 2, causal, "bf16")
    if family == "bf16_step":
        return _case("step", B, H, tokens(64, 4096, 393216), 64, 2, causal, "bf16",
                     scale=rng.choice([1.0, 0.125]))
    if family == "bf16_long":
        B, H = 1, rng.choice([1, 2, 4, 8])
        return _case("fwd", B, H, tokens(16384, 131072, 524288), 64, 2, causal, "bf16",
                     outliers=not causal)
    if family == "p1_step":
        return _case("step", B, H, tokens(200, 8192, 196608), 64, 1, causal, "bf16",
                     scale=1.0 / 64)
    if family == "d128":
        B = rng.choice([1, 2])
        return _case(rng.choice(["fwd", "step"]), B, H, tokens(128, 4096, 32768), 128, 2, causal,
                     "bf16")
    return _case("dropout", B, H, tokens(200, 4096, 131072), rng.choice([32, 64]), 2, causal,
                 "bf16", scale=0.125, rate=rng.choice([0.1, 0.2]))


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    shape = (case["B"], case["H"], case["N"], case["D"])
    names = ["q", "k", "v"] + (["dout"] if case["call"] in ("step", "dropout") else [])
    x = {n: torch.randn(shape, generator=gen, device="cuda") for n in names}
    if case["outliers"]:
        grow = 1.0 + 3.0 * (torch.rand(shape[:3], generator=gen, device="cuda") < 0.05)
        for n in ("q", "k", "v"):
            x[n] = x[n] * grow.unsqueeze(-1)
    return {n: t.to(DTYPES[case["dtype"]]).contiguous() for n, t in x.items()}


def prepare(case, seed):
    state = _inputs(case, seed)
    state["case"] = case
    state["scale"] = None if case["scale"] == 1.0 else case["scale"]
    state["mask_seed"] = 1000 + seed
    if case["call"] == "noalloc":
        state["out"] = torch.empty_like(state["q"])
        state["g"] = torch.empty(state["q"].shape[:3], dtype=torch.float32, device="cuda")
    return state


def run(state):
    c = state["case"]
    q, k, v = state["q"], state["k"], state["v"]
    kw = {"causal": c["causal"], "scale": state["scale"]}
    if c["call"] == "noalloc":
        o, g = fm.fastmax_fwd_noalloc(q, k, v, state["out"], state["g"], p=c["p"], **kw)
        return {"o": o, "g": g}
    if c["call"] == "dropout":
        bits = fm.dropout_mask(c["B"], c["H"], c["N"], c["D"], c["rate"], state["mask_seed"])
        o, g = fm.fastmax_fwd_dropout(q, k, v, bits, c["rate"], **kw)
        dq, dk, dv = fm.fastmax_bwd_dropout(q, k, v, o, state["dout"], g, bits, c["rate"], **kw)
        return {"bits": bits, "o": o, "g": g, "dq": dq, "dk": dk, "dv": dv}
    o, g = fm.fastmax_fwd(q, k, v, p=c["p"], **kw)
    if c["call"] == "fwd":
        return {"o": o, "g": g}
    dq, dk, dv = fm.fastmax_bwd(q, k, v, o, state["dout"], g, p=c["p"], **kw)
    return {"o": o, "g": g, "dq": dq, "dk": dk, "dv": dv}


def work(case):
    """Bytes: every input read once, every output written once.  Flops: per
    token and head the fewer of the two exact formulations, the moments
    (2 P (D + 1) to build them and as many to contract them, P features with
    the symmetric packing) and the pairs (scores and weighted values, 4 D per
    key seen); their gradients likewise (for the pairs five products of 2 D).
    A masked quadratic feature has no pair form of that size."""
    B, H, N, D, p = (case[n] for n in "BHNDp")
    rows = B * H * N
    P = 1 + D + (D * (D + 1) // 2 if p == 2 else 0)
    keys = (N + 1) / 2 if case["causal"] else N
    moments, pairs = 4 * P * (D + 1), 4 * D * keys
    # the gradient: forward-direction state and dq, reverse state and dk, and
    # the reverse dv
    if p == 2:
        grad = 2 * (2 * P * (D + 1) + 2 * D * D * (D + 1) + 2 * P * D)
    else:
        grad = 2 * (4 * P * (D + 1) + 2 * P * D)
    masked = case["call"] == "dropout"
    flops = moments if masked else min(moments, pairs)
    size = 4 if case["dtype"] == "f32" else 2
    nbytes = rows * (4 * D * size + 4)
    if case["call"] in ("step", "dropout"):
        flops += grad if masked else min(grad, 10 * D * keys)
        nbytes += rows * 4 * D * size
    if masked:
        nbytes += rows * 4 * ((D * (D + 1) // 2 + 31) // 32)
    return {"bytes": float(nbytes), "flops": float(flops * rows)}


def tolerance(case):
    """About four times what the paths show against ``exact`` over these
    ranges.  float32: 4e-7 in the norm (1e-5 is what 32-bit sums in another
    order may show), 1.6e-5 in the worst entry.  bf16: 2e-3 in the norm, the
    rounding of the outputs, up to 5e-2 in the worst entry of a forward.  The
    gradients of the causal second-order step at D = 64 add over queries whose
    1/G spans four decades, in 16-bit operands: 1.3e-2 at 4096 tokens, and
    0.4 in the worst entry (the late tokens' gradients are small)."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    if case["call"] in ("step", "dropout") and case["causal"]:
        wide = case["call"] == "step" and case["D"] == 64 and case["p"] == 2
        return {"rel": 3e-2 if wide else 1e-2, "max": 0.9}
    return {"rel": 1e-2, "max": 0.2}


# ---------------------------------------------------------------------------
# The same outputs in 64 bits, from the definition (O = F / G with explicit
# weights), one head and one block of rows at a time.
# ---------------------------------------------------------------------------
def _standardise(x):
    x = x - x.mean(-1, keepdim=True)
    return x / x.square().mean(-1, keepdim=True).sqrt()


def _philox_keep(case, seed):
    """Keep bits of the package's documented generator (Philox4x32-10, Salmon
    et al., SC 2011) for every head, as [heads, N, features] booleans."""
    B, H, N, D = (case[n] for n in "BHND")
    feats = D * (D + 1) // 2
    quads = (feats + 3) // 4
    low = 0xFFFFFFFF

    def mul(m, x):
        # high and low words of a 32 by 32 bit product, without leaving int64
        a, b = m * (x >> 16), m * (x & 0xFFFF)
        lo = (((a & 0xFFFF) << 16) + b)
        return ((a >> 16) + (lo >> 32)) & low, lo & low

    for h in range(B * H):
        c0 = torch.arange(N, device="cuda", dtype=torch.int64).unsqueeze(1).expand(N, quads)
        c1 = torch.arange(quads, device="cuda", dtype=torch.int64).unsqueeze(0).expand(N, quads)
        c2, c3 = torch.full_like(c0, h), torch.zeros_like(c0)
        k0, k1 = seed & low, (seed >> 32) & low
        for _ in range(10):
            h0, l0 = mul(0xD2511F53, c0)
            h1, l1 = mul(0xCD9E8D57, c2)
            c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
            k0, k1 = (k0 + 0x9E3779B9) & low, (k1 + 0xBB67AE85) & low
        words = torch.stack([c0, c1, c2, c3], -1).reshape(N, 4 * quads)[:, :feats]
        rate = float(torch.tensor(case["rate"], dtype=torch.float32))
        yield words >= int(rate * 4294967296.0)


def _pack(keep, words):
    pad = torch.zeros((keep.shape[0], 32 * words), dtype=torch.int64, device=keep.device)
    pad[:, :keep.shape[1]] = keep
    packed = (pad.reshape(-1, words, 32) << torch.arange(32, device=keep.device)).sum(-1)
    return torch.where(packed >= 1 << 31, packed - (1 << 32), packed).to(torch.int32)


def _exact_rows(q, k, v, causal, p, rows):
    """F / G of one head, `rows` query rows at a time."""
    N = q.shape[0]
    o = torch.empty_like(q)
    g = torch.empty(N, dtype=q.dtype, device=q.device)
    for i0 in range(0, N, rows):
        i1 = min(N, i0 + rows)
        n = i1 if causal else N
        s = q[i0:i1] @ k[:n].T
        w = 1 + s if p == 1 else 1 + s + 0.5 * s * s
        if causal:
            w = w.tril(i0)
        g[i0:i1] = w.sum(1)
        o[i0:i1] = (w @ v[:n]) / g[i0:i1, None]
    return o, g


def _exact_moments(q, k, v, rows):
    """The non-causal second-order case of a long head through its moments."""
    D = q.shape[1]
    m, l = torch.triu_indices(D, D, device=q.device)
    half = torch.where(m == l, 0.5, 1.0).to(q.dtype)
    v1 = torch.cat([v, torch.ones_like(v[:, :1])], 1)

    def phi(x):
        return torch.cat([torch.ones_like(x[:, :1]), x, x[:, m] * x[:, l]], 1)

    state = sum(phi(k[i:i + rows]).T @ v1[i:i + rows] for i in range(0, k.shape[0], rows))
    state[1 + D:] *= half[:, None]
    f = torch.cat([phi(q[i:i + rows]) @ state for i in range(0, q.shape[0], rows)])
    return f[:, :D] / f[:, D:], f[:, D]


def exact(case, seed):
    x = {n: t.double() for n, t in _inputs(case, seed).items()}
    B, H, N, D, p = (case[n] for n in "BHNDp")
    heads = {n: t.reshape(B * H, N, D) for n, t in x.items()}
    step = case["call"] in ("step", "dropout")
    masked = case["call"] == "dropout"
    causal, scale = case["causal"], case["scale"]
    out = {n: [] for n in ["o", "g"] + (["dq", "dk", "dv"] if step else [])}
    if masked:
        m, l = torch.triu_indices(D, D, device="cuda")
        weight = torch.where(m == l, 0.5, 1.0).double() / (1.0 - case["rate"])
        keeps = _philox_keep(case, 1000 + seed)
    for h in range(B * H):
        q, k, v = (heads[n][h] for n in ("q", "k", "v"))
        if not step:
            qs, ks = scale * _standardise(q), _standardise(k)
            if N > 32768 and not causal:
                o, g = _exact_moments(qs, ks, v, 8192)
            else:
                o, g = _exact_rows(qs, ks, v, causal, p, 4096)
        else:
            q, k, v = (t.clone().requires_grad_() for t in (q, k, v))
            qs, ks = scale * _standardise(q), _standardise(k)
            s = qs @ ks.T
            if masked:
                keep = next(keeps)
                feat = ks[:, m] * ks[:, l] * (keep * weight)
                w = 1 + s + (qs[:, m] * qs[:, l]) @ feat.T
            else:
                w = 1 + s if p == 1 else 1 + s + 0.5 * s * s
            if causal:
                w = w.tril()
            g = w.sum(1)
            o = (w @ v) / g[:, None]
            grads = torch.autograd.grad((o * heads["dout"][h]).sum(), (q, k, v))
            for n, t in zip(("dq", "dk", "dv"), grads):
                out[n].append(t)
            o, g = o.detach(), g.detach()
        out["o"].append(o)
        out["g"].append(g)
    shape = (B, H, N, D)
    res = {n: torch.stack(t).reshape(shape if n != "g" else shape[:3]) for n, t in out.items()}
    if masked:
        # the keep bits are whole numbers: they have no 64-bit value
        res = {"bits": None, **res}
    return res
