"""The pair kernels (fm_pairs_fwd.hip, fm_pairs_bwd*.hip): explicit 32 x 32
weight tiles for short sequences.

Every workgroup shape of the plan, at sizes that straddle its tiles (32 keys,
32 queries, the keys staged per step, the queries of a workgroup), against the
oracle's explicit matrix; and the value scale's second attempt, which only a
late token far above the first tile's values reaches.  Tolerances are the
suite's (1e-4 for float32 rows, 2e-2 for bf16), per head and per row; float32
rows, whose operands carry 24 bits at any magnitude, are also held entry by
entry to a bound from the data.
"""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2402_07901_amd import fastmax as fm
from paper_2402_07901_amd.inputs import bf16_bits_to_f64, f32_to_bf16_bits, make_inputs

from gpu_util import TOL, max_rel, say, to_dev, to_f64


LINEAR, PAIRS, CAUSAL, NONCAUSAL, FLOAT32 = range(5)     # enum Kernels of fm_internal.h


def route(BH, N, D, causal, dt, backward=False, p=2, scale=1.0):
    """(kernels, shape) that the library picks for a call."""
    f = fm.lib().fm_route
    f.argtypes = [ctypes.c_int] * 5 + [ctypes.c_float] + [ctypes.c_int] * 2
    r = f(BH, N, D, p, int(causal), scale, fm.BF16 if dt == "bf16" else fm.F32, int(backward))
    assert r >= 0
    return divmod(r, 16)


def plan(BH, N, D, causal, dt, backward=False):
    """The pair kernels' shape for a call of order 2 (-1: other kernels)."""
    kernels, shape = route(BH, N, D, causal, dt, backward)
    return shape if kernels == PAIRS else -1


def segments(BH, N):
    """Segments of the many-segment scan (0: not cut so)."""
    return fm.lib().fm_scan_segments(BH, N)


# (heads, N, D, dtype): sizes around the edges of each shape's tiles
CASES = [
    (1, 1, 16, "f32"), (2, 31, 16, "f32"), (1, 257, 16, "f32"), (16, 1000, 16, "f32"),
    (64, 1601, 16, "f32"), (64, 700, 32, "f32"), (3, 33, 16, "bf16"),
    (16, 1000, 16, "bf16"), (64, 1601, 16, "bf16"), (96, 1025, 16, "bf16"), (2, 255, 32, "f32"), (8, 1030, 32, "f32"),
    (64, 1500, 32, "f32"), (5, 129, 32, "bf16"), (8, 1030, 32, "bf16"), (64, 1290, 32, "bf16"),
    (3, 65, 64, "f32"),
    (24, 700, 64, "f32"), (64, 1025, 64, "f32"), (64, 2049, 64, "f32"), (2, 32, 128, "f32"), (16, 513, 128, "f32"),
    (64, 1025, 128, "f32"), (96, 2049, 128, "f32"), (1, 127, 128, "bf16"), (16, 1025, 128, "bf16"),
    (64, 1023, 128, "bf16"),
    (1, 1, 64, "bf16"), (2, 64, 64, "bf16"), (5, 127, 64, "bf16"), (1, 700, 64, "bf16"),
    (16, 515, 64, "bf16"), (24, 1300, 64, "bf16"), (48, 1025, 64, "bf16"), (96, 2305, 64, "bf16"),
    (200, 512, 64, "bf16"), (96, 4700, 64, "bf16"),
]


BWD_CASES = [
    (1, 1, 16, "f32"), (2, 257, 16, "f32"), (16, 300, 16, "f32"), (64, 801, 16, "f32"),
    (3, 33, 16, "bf16"), (1, 513, 16, "bf16"), (4, 513, 16, "bf16"), (64, 801, 16, "bf16"), (16, 513, 16, "bf16"), (2, 257, 32, "bf16"),
    (5, 801, 32, "bf16"), (64, 700, 32, "bf16"), (1, 255, 32, "f32"), (1, 2047, 32, "f32"), (8, 1030, 32, "f32"),
    (64, 700, 32, "f32"), (5, 129, 32, "bf16"), (3, 65, 64, "f32"), (24, 700, 64, "f32"),
    (64, 900, 64, "f32"), (3, 129, 64, "f32"), (64, 257, 64, "f32"), (8, 1029, 64, "f32"), (2, 32, 128, "f32"), (16, 513, 128, "f32"), (64, 1025, 128, "f32"),
    (1, 127, 128, "bf16"), (64, 1023, 128, "bf16"), (1, 1, 64, "bf16"), (2, 64, 64, "bf16"),
    (1, 700, 64, "bf16"), (16, 515, 64, "bf16"), (24, 1300, 64, "bf16"), (96, 1025, 64, "bf16"),
    (96, 2305, 64, "bf16"),
]


def test_every_shape_is_reached():
    want = {(16, "f32"): 3, (32, "f32"): 3, (64, "f32"): 3, (128, "f32"): 1, (16, "bf16"): 3,
            (32, "bf16"): 3, (128, "bf16"): 2, (64, "bf16"): 4}
    for (D, dt), n in want.items():
        got = {plan(BH, N, D, c, dt, True) for BH, N, d, t in BWD_CASES if (d, t) == (D, dt)
               for c in (True, False)}
        assert set(range(n)) <= got, ("backward", D, dt, got)
    want = {(16, "f32"): 3, (32, "f32"): 3, (64, "f32"): 3, (128, "f32"): 3, (16, "bf16"): 3,
            (32, "bf16"): 3, (128, "bf16"): 3, (64, "bf16"): 6}
    for (D, dt), n in want.items():
        got = {plan(BH, N, D, c, dt) for BH, N, d, t in CASES if (d, t) == (D, dt)
               for c in (True, False)}
        assert set(range(n)) <= got, (D, dt, got)


def test_plan_keeps_the_moments_for_long_sequences():
    """Linear in N where the pairs' quadratic cost is the larger one."""
    assert plan(64, 8192, 64, True, "bf16") == -1
    assert plan(8, 131072, 64, False, "bf16") == -1
    assert plan(8, 65536, 64, True, "bf16") == -1
    assert plan(64, 8192, 64, True, "bf16", True) == -1
    for D in (16, 32, 64, 128):
        for back in (False, True):
            assert plan(4, 1 << 20, D, True, "f32", back) == -1


def test_plan_stays_within_the_workspace():
    """The scratch a shape takes never exceeds what the call asks for, whose
    size is the moment path's."""
    for D in (16, 32, 64, 128):
        for dt in ("f32", "bf16"):
            for causal in (True, False):
                for BH, N in ((1, 1), (1, 127), (7, 100), (96, 64), (96, 127), (300, 33), (96, 777)):
                    code = fm.BF16 if dt == "bf16" else fm.F32
                    have = fm.workspace_bytes(1, BH, N, D, 2, causal, code, True)
                    half = dt == "bf16" and D == 64 and (causal or N >= 128)
                    if plan(BH, N, D, causal, dt, True) >= 0:
                        assert have >= BH * N * (656 if half else 8 * D + 8)
                    have = fm.workspace_bytes(1, BH, N, D, 2, causal, code, False)
                    if half and plan(BH, N, D, causal, dt) == 4:
                        assert have >= BH * N * 128


def heads_of(inp, sel):
    return [inp[n + "64"].reshape(-1, *inp[n + "64"].shape[2:])[sel] for n in ("q", "k", "v")]


def check(inp, dt, causal, label):
    q, k, v = (to_dev(inp[n], dt) for n in ("q", "k", "v"))
    o, g = fm.fastmax_fwd(q, k, v, p=2, causal=causal)
    o, g = to_f64(o), g.cpu().numpy().astype(np.float64)
    BH = o.shape[0] * o.shape[1]
    o, g = o.reshape(BH, *o.shape[2:]), g.reshape(BH, -1)
    for h in sorted({0, BH // 2, BH - 1}):
        q64, k64, v64 = heads_of(inp, h)
        ro, rg = oracle.fwd_brute(q64[None, None], k64[None, None], v64[None, None], 2, causal)
        eo = max(max_rel(o[h], ro[0, 0]), row_rel(o[h], ro[0, 0]))
        eg = float((np.abs(g[h] - rg[0, 0]) / np.abs(rg[0, 0])).max())
        say(f"{label} head {h}: E_O={eo:.2e} E_G={eg:.2e}")
        assert eo <= TOL[dt] and eg <= TOL[dt], (label, h, eo, eg)
        if "D64 bf16 cFalse" in label and N_of(inp) < 128:
            # float32-grade operands: 2^-22 a product, G of at most 127 keys
            assert eg <= 1e-5, (label, h, eg)


def row_rel(x, ref):
    """The largest error of a row over the largest entry of that row."""
    den = np.abs(ref).max(-1)
    return float((np.abs(x - ref).max(-1) / np.where(den > 0, den, np.inf)).max())


def N_of(inp):
    return inp["q"].shape[2]


@pytest.mark.gpu
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("BH,N,D,dt", CASES)
def test_shapes_against_explicit_matrix(BH, N, D, dt, causal):
    inp = make_inputs(1, BH, N, D, 7100 + N, dt)
    check(inp, dt, causal, f"BH{BH} N{N} D{D} {dt} c{causal} shape {plan(BH, N, D, causal, dt)}")


def group_rel(x, ref, edges):
    """The largest error of a group of rows (between edges) over the largest entry
    of that group."""
    out = 0.0
    for a, b in zip((0, *edges), (*edges, len(ref))):
        den = np.abs(ref[a:b]).max()
        err = np.abs(x[a:b] - ref[a:b]).max()
        out = max(out, float(err / den) if den > 0 else float(err))
    return out


def check_bwd(inp, dt, causal, scale, label, edges=()):
    BH, N, D = inp["q64"].shape[1:]
    q, k, v, do = (to_dev(inp[n], dt) for n in ("q", "k", "v", "dout"))
    o, g = fm.fastmax_fwd(q, k, v, p=2, causal=causal, scale=scale)
    grads = fm.fastmax_bwd(q, k, v, o, do, g, p=2, causal=causal, scale=scale)
    again = fm.fastmax_bwd(q, k, v, o, do, g, p=2, causal=causal, scale=scale)
    if plan(BH, N, D, causal, dt, True) >= 0:
        # one owner per output row: the same bits every time
        assert all(torch.equal(a, b) for a, b in zip(grads, again)), label
    grads = [to_f64(x).reshape(BH, N, D) for x in grads]
    for h in sorted({0, BH // 2, BH - 1}):
        q64, k64, v64 = heads_of(inp, h)
        d64 = inp["dout64"].reshape(BH, N, D)[h]
        ref = oracle.bwd_brute(*(x[None, None] for x in (q64, k64, v64, d64)), 2, causal,
                               scale=scale)
        # entries are held to the largest of the head's gradient, or of
        # |dO| |v| sqrt(D) where the exact gradient vanishes (one key: dq = dk = 0)
        floor = np.abs(d64).max() * np.abs(v64).max() * np.sqrt(D) if N == 1 else 0.0
        for name, x, r in zip(("dq", "dk", "dv"), grads, ref):
            den = max(np.abs(r).max(), floor if name != "dv" else 0.0)
            e = float(np.abs(x[h] - r[0, 0]).max() / den)
            if edges:
                e = max(e, group_rel(x[h], r[0, 0], edges))
            say(f"{label} head {h} {name}: {e:.2e}")
            assert e <= TOL[dt], (label, h, name, e)


@pytest.mark.gpu
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("BH,N,D,dt", BWD_CASES)
def test_backward_shapes_against_explicit_gradient(BH, N, D, dt, causal):
    inp = make_inputs(1, BH, N, D, 7400 + N, dt, with_dout=True)
    check_bwd(inp, dt, causal, 1.0, f"bwd BH{BH} N{N} D{D} {dt} c{causal} shape "
              f"{plan(BH, N, D, causal, dt, True)}")


@pytest.mark.gpu
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("D,dt", [(64, "bf16"), (128, "bf16"), (32, "f32"), (64, "f32")])
@pytest.mark.parametrize("kind", ["late", "zeros", "tau", "huge", "tiny"])
def test_backward_scales(D, dt, causal, kind):
    """Rows of v and dO that differ by large powers of two, rows of zeros, a
    small score scale, and values near the ends of the range.  Rows on either
    side of a jump are held to the largest entry of their own."""
    N = 300
    f = np.ones(N)
    if kind == "late":
        f[200:] = 2.0 ** 12
    elif kind == "zeros":
        f[:150] = 0.0
    elif kind != "tau":
        f[:] = 2.0 ** (55 if kind == "huge" else -55)
    inp = scale_values(make_inputs(1, 3, N, D, 7500, dt, with_dout=True), dt, f)
    inp = scale_values(inp, dt, f[::-1] if kind == "late" else f, "dout")
    check_bwd(inp, dt, causal, 1.0 / D if kind == "tau" else 1.0, f"bwd {kind} D{D} {dt} c{causal}",
              edges=(100, 200) if kind == "late" else (150,) if kind == "zeros" else ())


@pytest.mark.gpu
@pytest.mark.parametrize("D", [16, 32, 128])
def test_bf16_rows_beside_far_larger_ones(D):
    """One row of v and one of dO at 2^30: the causal rows that never meet it
    keep their own magnitude, O and gradients alike."""
    N = 300
    f = np.ones(N)
    f[N // 2] = 2.0 ** 30
    edges = sorted({N - 1 - N // 2, N - N // 2, N // 2, N // 2 + 1})
    inp = scale_values(make_inputs(1, 3, N, D, 7500, "bf16", with_dout=True), "bf16", f)
    inp = scale_values(inp, "bf16", f[::-1], "dout")
    q, k, v = (to_dev(inp[n], "bf16") for n in ("q", "k", "v"))
    assert plan(3, N, D, True, "bf16") >= 0 and plan(3, N, D, True, "bf16", True) >= 0
    o = to_f64(fm.fastmax_fwd(q, k, v, p=2, causal=True)[0])
    for h in range(3):
        ref = oracle.fwd_brute(*(x[None, None] for x in heads_of(inp, h)), 2, True)[0][0, 0]
        e = group_rel(o[0, h], ref, edges)
        say(f"D{D} head {h} O: {e:.2e}")
        assert e <= TOL["bf16"], (h, e)
    check_bwd(inp, "bf16", True, 1.0, f"bwd far D{D}", edges)


def scale_values(inp, dt, factor, name="v"):
    """Rows of v (or dout) times factor [N] (powers of two: exact)."""
    v = inp[name + "64"] * factor[None, None, :, None]
    out = dict(inp)
    if dt == "bf16":
        out[name] = f32_to_bf16_bits(v.astype(np.float32))
        out[name + "64"] = bf16_bits_to_f64(out[name])
    else:
        out[name] = v.astype(np.float32)
        out[name + "64"] = out[name].astype(np.float64)
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("D,dt", [(64, "bf16"), (128, "bf16"), (32, "f32"), (64, "f32")])
@pytest.mark.parametrize("kind", ["late", "zeros", "prefix", "huge", "tiny"])
def test_value_scale(D, dt, causal, kind):
    """Values that outgrow the first tile's scale (a second attempt), a first
    tile of zeros before values of 1 and (prefix) of 2^-24, and values near the
    ends of the float range."""
    N = 420
    f = np.ones(N)
    if kind == "late":
        f[300:] = 2.0 ** 14
    elif kind in ("zeros", "prefix"):
        f[:280] = 0.0
        f[280:] = 1.0 if kind == "zeros" else 2.0 ** -24
    else:
        f[:] = 2.0 ** (110 if kind == "huge" else -110)
    inp = scale_values(make_inputs(1, 3, N, D, 7200, dt), dt, f)
    check(inp, dt, causal, f"{kind} D{D} {dt} c{causal}")


def entry_bound(q64, k64, v64, causal, scale=1.0):
    """sum_n w_in |v_nd| / G_i of one head: what every rounding of the forward
    is relative to, entry by entry (all weights of order 2 are positive)."""
    s = scale * oracle.standardize(q64)[0] @ oracle.standardize(k64)[0].T
    w = 1.0 + s + 0.5 * s * s
    if causal:
        w = np.tril(w)
    return w @ np.abs(v64) / w.sum(1)[:, None]


@pytest.mark.gpu
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("kind", ["row", "far row", "column", "plain"])
@pytest.mark.parametrize("D,N", [(16, 420), (32, 420), (64, 420), (128, 420), (32, 33)])
def test_float32_entries_keep_their_own_magnitude(D, N, kind, causal):
    """float32 values next to far larger ones that an output does not see: a row
    of 2^20 or 2^60 inside the first staged tile (causal rows before it), and a
    column of 2^20.  A score is a sum of D products and a weight, a sum of
    weights and an output take a few roundings more: (D + 32) 2^-24."""
    f = np.ones(N)
    if "row" in kind:
        f[N - 20 if N < 100 else 200] = 2.0 ** (60 if kind == "far row" else 20)
    inp = scale_values(make_inputs(1, 3, N, D, 7250, "f32"), "f32", f)
    if kind == "column":
        inp["v"][..., 3] *= np.float32(2.0 ** 20)
        inp["v64"] = inp["v"].astype(np.float64)
    q, k, v = (to_dev(inp[n], "f32") for n in ("q", "k", "v"))
    assert plan(3, N, D, causal, "f32") >= 0
    o = to_f64(fm.fastmax_fwd(q, k, v, p=2, causal=causal)[0])
    for h in range(3):
        h64 = heads_of(inp, h)
        ref = oracle.fwd_brute(*(x[None, None] for x in h64), 2, causal)[0][0, 0]
        e = float((np.abs(o[0, h] - ref) / entry_bound(*h64, causal)).max())
        say(f"{kind} D{D} N{N} c{causal} head {h}: {e:.2e}")
        assert e <= (D + 32) * 2.0 ** -24, (h, e)


def gradient_bounds(q64, k64, v64, d64, causal, scale=1.0):
    """Per entry of dq, dk and dv of one head: the sums of the gradient's terms
    without their cancellation, which every rounding is relative to."""
    (qh, _, sq), (kh, _, sk) = oracle.standardize(q64), oracle.standardize(k64)
    s = scale * qh @ kh.T
    keep = np.tril(np.ones_like(s)) if causal else 1.0
    w = keep * (1.0 + s + 0.5 * s * s)
    g = w.sum(1)[:, None]
    a = keep * (1.0 + scale * np.abs(qh) @ np.abs(kh).T) / g * (np.abs(d64) @ np.abs(v64).T
                                      + (np.abs(d64) * (w @ np.abs(v64) / g)).sum(1)[:, None])

    def back(b, xh, sd):
        return (b + b.mean(1)[:, None] + np.abs(xh) * (b * np.abs(xh)).mean(1)[:, None]) / sd.reshape(-1, 1)

    return (back(scale * a @ np.abs(kh), qh, sq), back(scale * a.T @ np.abs(qh), kh, sk),
            w.T @ (np.abs(d64) / g))


def check_gradient_entries(inp, p, causal, scale, bounds, bar, label):
    BH, N, D = inp["q64"].shape[1:]
    q, k, v, do = (to_dev(inp[n], "f32") for n in ("q", "k", "v", "dout"))
    o, g = fm.fastmax_fwd(q, k, v, p=p, causal=causal, scale=scale)
    grads = fm.fastmax_bwd(q, k, v, o, do, g, p=p, causal=causal, scale=scale)
    for h in sorted({0, BH // 2, BH - 1}):
        h64 = heads_of(inp, h) + [inp["dout64"].reshape(BH, N, D)[h]]
        ref = oracle.bwd_brute(*(x[None, None] for x in h64), p, causal, scale=scale)
        for name, x, r, b in zip(("dq", "dk", "dv"), grads, ref, bounds(*h64, causal, scale)):
            d = np.abs(to_f64(x)[0, h] - r[0, 0])
            assert not d[b == 0].any(), (label, h, name)
            e = float((d / np.where(b > 0, b, np.inf)).max())
            say(f"{label} head {h} {name}: {e:.2e}")
            assert e <= bar, (label, h, name, e)


def outlier_inputs(BH, N, D, kind):
    """Rows or columns of v and dO far above what other rows or columns meet."""
    f = np.ones(N)
    inp = make_inputs(1, BH, N, D, 7550, "f32", with_dout=True)
    if kind == "v row":
        f[N - 20 if N < 100 else 200] = 2.0 ** 40
        inp = scale_values(inp, "f32", f)
    elif kind == "dout row":
        f[N // 3] = 2.0 ** 40
        inp = scale_values(inp, "f32", f, "dout")
    elif kind == "columns":
        # what the outputs of one column weigh, another's must not hide
        inp["v"][..., 3] *= np.float32(2.0 ** 20)
        inp["dout"][..., 3] = 0.0
        inp["dout"][..., 5] *= np.float32(2.0 ** 20)
        inp["v"][..., 5] = 0.0
        for n in ("v", "dout"):
            inp[n + "64"] = inp[n].astype(np.float64)
    return inp


@pytest.mark.gpu
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("kind", ["v row", "dout row", "columns", "plain"])
@pytest.mark.parametrize("D,N", [(16, 420), (32, 420), (64, 420), (128, 420), (32, 33)])
def test_float32_gradient_entries_keep_their_own_magnitude(D, N, kind, causal):
    """Gradients next to far larger rows and columns that they do not see.  A
    term holds products of D terms, cut per 16 of them, and O's and G's own
    error, an entry sums N of them 32 at a time: (D + N / 32 + 64) 2^-24."""
    assert plan(3, N, D, causal, "f32", True) >= 0
    check_gradient_entries(outlier_inputs(3, N, D, kind), 2, causal, 1.0, gradient_bounds,
                           (D + N / 32 + 64) * 2.0 ** -24, f"{kind} D{D} N{N} c{causal}")


@pytest.mark.gpu
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("D", [16, 32, 64, 128])
def test_bf16_rows_beside_a_large_value(D, causal):
    """bf16 values are held under one power of two per 8 columns of the staged
    tile: causal rows before a row of 2^12 in the same tile keep the suite's
    bar, row by row."""
    N = 300
    f = np.ones(N)
    f[100] = 2.0 ** 12
    inp = scale_values(make_inputs(1, 3, N, D, 7260, "bf16"), "bf16", f)
    check(inp, "bf16", causal, f"large row D{D} c{causal}")


@pytest.mark.gpu
@pytest.mark.parametrize("D,dt", [(64, "bf16"), (16, "f32")])
def test_constant_row_and_infinite_value_stay_in_their_rows(D, dt):
    """A constant k row (std 0) makes the rows that see it non-finite and no
    others; so does an infinite value, up to the 32-key tile it shares."""
    N, n = 400, 200
    inp = make_inputs(1, 2, N, D, 7300, dt)
    q, k, v = (to_dev(inp[x], dt) for x in ("q", "k", "v"))
    k[0, 0, n] = 1.0
    v[0, 1, n, 3] = float("inf")
    o, g = fm.fastmax_fwd(q, k, v, p=2, causal=True)
    torch.cuda.synchronize()
    assert torch.isfinite(o[0, 0, :n]).all() and torch.isfinite(g[0, 0, :n]).all()
    assert not torch.isfinite(o[0, 0, n:]).any()
    assert torch.isfinite(o[0, 1, :n - n % 32]).all() and torch.isfinite(g[0, 1]).all()
    assert not torch.isfinite(o[0, 1, n:, 3]).any()


@pytest.mark.gpu
@pytest.mark.parametrize("BH,N", [(1, 40000), (5, 24577), (16, 26111), (21, 24700)])
def test_many_segment_scan(BH, N):
    """Few heads over a long sequence: the causal scan cut into many segments
    (a ragged last one among them) against the oracle's sampled rows, every
    segment's edge rows included."""
    S = segments(BH, N)
    assert S >= 3 and plan(BH, N, 64, True, "bf16") == -1
    inp = make_inputs(1, BH, N, 64, 7600 + BH, "bf16")
    q, k, v = (to_dev(inp[n], "bf16") for n in ("q", "k", "v"))
    o, g = fm.fastmax_fwd(q, k, v, p=2, causal=True, scale=0.125)
    o, g = to_f64(o).reshape(-1, 64), g.cpu().numpy().astype(np.float64).reshape(-1)
    nch = (N + 127) // 128
    cseg = (-(-nch // S) + 1) & ~1
    edges = [e for s in range(1, S) for e in (s * cseg * 128 - 1, s * cseg * 128)]
    local = sorted({0, 127, 128, N - 1, *edges, *np.random.default_rng(1).integers(0, N, 12).tolist()})
    rows = [h * N + i for h in {0, BH - 1} for i in local if i < N]
    ro, rg = oracle.fwd_rows(inp["q64"], inp["k64"], inp["v64"], 2, True, rows, scale=0.125)
    eo = float((np.abs(o[rows] - ro).max(-1) / np.abs(ro).max()).max())
    eg = float((np.abs(g[rows] - rg) / rg).max())
    say(f"BH{BH} N{N} S{S}: E_O={eo:.2e} E_G={eg:.2e}")
    assert eo <= TOL["bf16"] and eg <= TOL["bf16"]


# queries (keys) per workgroup of each shape
QB_FWD = {16: (32, 64, 256), 32: (32, 64, 256), 64: (64, 128, 256), 128: (64, 128, 256),
          "half": (32, 64, 128, 128, 256, 512)}
QB_BWD = {(16, "f32"): (32, 32, 256), (32, "f32"): (32, 64, 256), (64, "f32"): (64, 128, 256),
          (128, "f32"): (128,), (16, "bf16"): (32, 32, 256), (32, "bf16"): (32, 64, 256),
          (64, "bf16"): (64, 128, 256, 256), (128, "bf16"): (128, 256)}


@pytest.mark.parametrize("D", [16, 32, 64, 128])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_plans_refuse_no_size(D, dt):
    """A launch holds 2^32 threads at most: where a shape's grid is larger (many
    short heads), the call goes to a shape or a kernel that fits."""
    for BH in (1 << 17, 1 << 19, 700000, 1 << 20):
        for N in (1, 33, 100, 161, 257, 300, 600, 1100, 2500):
            for causal in (True, False):
                half = dt == "bf16" and D == 64 and (causal or N >= 128)
                s = plan(BH, N, D, causal, dt)
                if s >= 0:
                    qb = QB_FWD["half" if half else D][s]
                    assert BH * -(-N // qb) * 512 < 2 ** 32, (BH, N, s)
                s = plan(BH, N, D, causal, dt, True)
                if s >= 0:
                    qb = QB_BWD[(D, dt)][s]
                    assert 3 * BH * -(-N // qb) * 512 < 2 ** 32, (BH, N, s)
                for back in (False, True):
                    if linear_plan(BH, N, D, causal, 1.0 / D, back, dt=dt):
                        assert (3 if back else 1) * BH * -(-N // 256) * 512 < 2 ** 32, (BH, N, back)


def test_many_segments_refuse_no_size():
    """At the dispatch limit (2^32 threads a launch) the many-segment scan's
    blocks of 32 tokens per head can be one launch too many where the plain
    scan's blocks of 32 rows fit: such a call is left to the latter."""
    most = (2 ** 32 - 1) // 256             # workgroups of 256 threads
    BH = 20
    N = 32 * (most // BH) + 1
    assert BH * -(-N // 32) > most >= -(-BH * N // 32)
    assert segments(BH, N) == 0 and segments(BH, N - 33) >= 3


@pytest.mark.gpu
def test_scan_modes_agree_where_the_scan_serves():
    """The segment modes of the causal scan give the same bits at a size that
    the plan leaves to it."""
    assert plan(64, 8192, 64, True, "bf16") == -1
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    q, k, v = (torch.randn((4, 16, 8192, 64), generator=gen, device="cuda").to(torch.bfloat16)
               for _ in range(3))
    ref = fm.fastmax_fwd(q, k, v, p=2, causal=True)
    old = fm.set_scan_segments(fm.SCAN_SEGMENTS_AUTO)
    try:
        for mode in (fm.SCAN_SEGMENTS_OFF, fm.SCAN_SEGMENTS_ON, fm.SCAN_SEGMENTS_REBUILD):
            fm.set_scan_segments(mode)
            o, g = fm.fastmax_fwd(q, k, v, p=2, causal=True)
            assert torch.equal(o, ref[0]) and torch.equal(g, ref[1]), mode
    finally:
        fm.set_scan_segments(old)


# ---------------------------------------------------------------------------
# First order over blocks with linear states (fm_linear.hip): tau D <= 1, bf16
# forward and backward, float32 backward
# ---------------------------------------------------------------------------
def linear_plan(BH, N, D, causal, scale, backward, dt="bf16", p=1):
    return route(BH, N, D, causal, dt, backward, p, scale)[0] == LINEAR


LINEAR_CASES = [(64, 1, 64), (48, 255, 64), (32, 257, 64), (24, 1281, 64), (64, 900, 32),
                (64, 511, 16), (64, 520, 128), (3, 700, 128)]


def test_linear_plan():
    """Signed weights, second order and the float32 forward stay with the other
    kernels, as do few heads of many tokens; every head size has a case."""
    assert not linear_plan(64, 1024, 64, True, 1.0, True)
    assert not linear_plan(64, 1024, 64, True, 1.0 / 64, False, dt="f32")
    assert linear_plan(64, 1024, 64, True, 1.0 / 64, True, dt="f32")
    assert not linear_plan(64, 1024, 64, True, 1.0 / 64, True, p=2)
    assert not linear_plan(1, 65536, 64, True, 1.0 / 64, False)
    for back in (False, True):
        for D in (16, 32, 64, 128):
            took = any(linear_plan(BH, N, D, c, 1.0 / D, back) for BH, N, d in LINEAR_CASES if d == D
                       for c in (True, False))
            assert took == (back or D > 16)
    # the scans are faster at D = 16 whatever the size
    assert not any(linear_plan(BH, N, 16, c, 1.0 / 16, False) for BH in (1, 16, 256, 4096, 1 << 20)
                   for N in (1, 256, 2048, 60000) for c in (True, False))


@pytest.mark.gpu
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("BH,N,D", LINEAR_CASES)
@pytest.mark.parametrize("kind,dt", [("plain", "bf16"), ("late", "bf16"), ("zeros", "bf16"),
                                     ("prefix", "bf16"), ("far", "bf16"), ("plain", "f32"),
                                     ("late", "f32"), ("prefix", "f32"), ("far", "f32")])
def test_linear_against_explicit_gradient(BH, N, D, causal, kind, dt):
    """O, G and the gradients against the oracle (the suite's bars; G, whose weights
    are non-negative sums of operands good to 2^-22, to 1e-5), with rows of v
    and dO that jump by 2^12, rows of zeros before values of 1 and (prefix) of
    2^-24, and (far) one row each of v and dO at 2^40.  Rows between the jumps are
    held to the largest entry of their own."""
    scale = 1.0 / D
    inp = make_inputs(1, BH, N, D, 7700 + N, dt, with_dout=True)
    if kind != "plain":
        if N < 200:
            pytest.skip("one step of rows")
        f = np.ones(N)
        f[2 * N // 3:] = 2.0 ** 12 if kind == "late" else 1.0
        edges = (N - 2 * N // 3, 2 * N // 3)
        if kind == "far":
            f[N // 2] = 2.0 ** 40
            edges = tuple(sorted({N - 1 - N // 2, N - N // 2, N // 2, N // 2 + 1}))
        if kind in ("zeros", "prefix"):
            f[:N // 3] = 0.0
            f[N // 3:] *= 1.0 if kind == "zeros" else 2.0 ** -24
        inp = scale_values(scale_values(inp, dt, f), dt, f[::-1] if kind in ("late", "far") else f, "dout")
    q, k, v, do = (to_dev(inp[n], dt) for n in ("q", "k", "v", "dout"))
    o, g = fm.fastmax_fwd(q, k, v, p=1, causal=causal, scale=scale)
    grads = fm.fastmax_bwd(q, k, v, o, do, g, p=1, causal=causal, scale=scale)
    if linear_plan(BH, N, D, causal, scale, True, dt):
        again = fm.fastmax_bwd(q, k, v, o, do, g, p=1, causal=causal, scale=scale)
        assert all(torch.equal(a, b) for a, b in zip(grads, again))
    for h in sorted({0, BH // 2, BH - 1}):
        q64, k64, v64 = heads_of(inp, h)
        d64 = inp["dout64"].reshape(BH, N, D)[h]
        four = [x[None, None] for x in (q64, k64, v64)]
        ro, rg = oracle.fwd_brute(*four, 1, causal, scale=scale)
        eo = max(max_rel(to_f64(o).reshape(BH, N, D)[h], ro[0, 0]),
                 group_rel(to_f64(o).reshape(BH, N, D)[h], ro[0, 0], edges) if kind != "plain" else 0.0)
        gg = g.cpu().numpy().astype(np.float64).reshape(BH, N)[h]
        eg = float((np.abs(gg - rg[0, 0]) / np.abs(rg[0, 0]).max()).max())
        assert eo <= TOL[dt] and eg <= 1e-5, (h, eo, eg)
        ref = oracle.bwd_brute(*four, d64[None, None], 1, causal, scale=scale)
        floor = np.abs(d64).max() * np.abs(v64).max() * np.sqrt(D) if N == 1 else 0.0
        for name, x, r in zip(("dq", "dk", "dv"), grads, ref):
            den = max(np.abs(r).max(), floor if name != "dv" else 0.0)
            e = float(np.abs(to_f64(x).reshape(BH, N, D)[h] - r[0, 0]).max() / den)
            if kind in ("late", "far"):
                e = max(e, group_rel(to_f64(x).reshape(BH, N, D)[h], r[0, 0], edges))
            say(f"linear {kind} BH{BH} N{N} D{D} c{causal} head {h} {name}: {e:.2e}")
            # far: dk is a sum of dO.O times q^ that nearly cancels, and O is rounded
            # to bf16 (the float32 scans show the same 2.9e-2)
            assert e <= TOL[dt] * (2 if kind == "far" and dt == "bf16" else 1), (h, name, e)


def gradient_bounds_p1(q64, k64, v64, d64, causal, scale):
    """As gradient_bounds, first order: the weights' parts may cancel in w and in
    G, so both count by magnitude."""
    (qh, _, sq), (kh, _, sk) = oracle.standardize(q64), oracle.standardize(k64)
    keep = np.tril(np.ones((len(q64),) * 2)) if causal else np.ones((len(q64),) * 2)
    g = (keep * (1.0 + scale * qh @ kh.T)).sum(1)[:, None]
    wa = keep * (1.0 + scale * np.abs(qh) @ np.abs(kh).T)
    kappa = wa.sum(1)[:, None] / g
    a = keep * kappa / g * (np.abs(d64) @ np.abs(v64).T
                            + (np.abs(d64) * (wa @ np.abs(v64) / g)).sum(1)[:, None])

    def back(b, xh, sd):
        return (b + b.mean(1)[:, None] + np.abs(xh) * (b * np.abs(xh)).mean(1)[:, None]) / sd.reshape(-1, 1)

    return (back(scale * a @ np.abs(kh), qh, sq), back(scale * a.T @ np.abs(qh), kh, sk),
            wa.T @ (kappa * np.abs(d64) / g))


@pytest.mark.gpu
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("kind", ["v row", "dout row", "columns", "plain"])
@pytest.mark.parametrize("D,N", [(16, 600), (32, 600), (64, 600), (128, 600), (64, 33)])
def test_float32_first_order_gradient_entries(D, N, kind, causal):
    """The same for the float32 rows of the first-order block backward."""
    assert linear_plan(8, N, D, causal, 1.0 / D, True, dt="f32")
    check_gradient_entries(outlier_inputs(8, N, D, kind), 1, causal, 1.0 / D, gradient_bounds_p1,
                           (D + N / 32 + 64) * 2.0 ** -24, f"p1 {kind} D{D} N{N} c{causal}")


@pytest.mark.gpu
@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("D", [16, 64])
def test_first_order_row_without_weight(D, dt):
    """tau D = 1 and q^ = -k^ in the first row: its G is zero (here exactly), its
    gradient not finite.  Keys past the 32-row tile that it shares do not see it
    and keep theirs."""
    BH, N = 48, 700
    assert linear_plan(BH, N, D, True, 1.0 / D, True, dt=dt)
    inp = make_inputs(1, BH, N, D, 7900, dt, with_dout=True)
    q, k, v, do = (to_dev(inp[n], dt) for n in ("q", "k", "v", "dout"))
    o, g = fm.fastmax_fwd(q, k, v, p=1, causal=True, scale=1.0 / D)
    ref = fm.fastmax_bwd(q, k, v, o, do, g, p=1, causal=True, scale=1.0 / D)
    g[:, :, 0] = 0.0
    got = fm.fastmax_bwd(q, k, v, o, do, g, p=1, causal=True, scale=1.0 / D)
    for name, a, b in zip(("dq", "dk", "dv"), got, ref):
        assert row_rel(to_f64(a)[0, :, 32:], to_f64(b)[0, :, 32:]) <= TOL[dt], name
