"""The pair kernels (fm_pairs_fwd.hip): explicit 32 x 32 weight tiles for short
sequences.

Every workgroup shape of the plan, at sizes that straddle its tiles (32 keys,
32 queries, the keys staged per step, the queries of a workgroup), against the
oracle's explicit matrix; and the value scale's second attempt, which only a
late token far above the first tile's values reaches.  Tolerances are the
suite's: the kernels' operands carry 22 bits (float32 grade) or 11 (bf16,
D = 64), the bars 1e-4 and 2e-2.
"""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2402_07901_amd import fastmax as fm
from paper_2402_07901_amd.inputs import bf16_bits_to_f64, f32_to_bf16_bits, make_inputs

from gpu_util import TOL, max_rel, say, to_dev, to_f64


def plan(BH, N, D, causal, dt):
    """The shape the library picks (-1: the moment kernels)."""
    f = getattr(fm.lib(), "_ZN2fm14pairs_fwd_planEiiiiiim")
    f.restype = ctypes.c_int
    code = fm.BF16 if dt == "bf16" else fm.F32
    ws = fm.workspace_bytes(1, BH, N, D, 2, causal, code)
    return f(BH, N, D, 2, int(causal), int(dt == "bf16"), ctypes.c_size_t(ws))


# (heads, N, D, dtype): sizes around the edges of each shape's tiles
CASES = [
    (1, 1, 16, "f32"), (2, 31, 16, "f32"), (1, 257, 16, "f32"), (16, 1000, 16, "f32"),
    (64, 1601, 16, "f32"), (64, 700, 32, "f32"), (3, 33, 16, "bf16"), (2, 255, 32, "f32"), (8, 1030, 32, "f32"),
    (64, 1500, 32, "f32"), (5, 129, 32, "bf16"), (64, 1290, 32, "bf16"), (3, 65, 64, "f32"),
    (24, 700, 64, "f32"), (64, 1025, 64, "f32"), (64, 2049, 64, "f32"), (2, 32, 128, "f32"), (16, 513, 128, "f32"),
    (64, 1025, 128, "f32"), (1, 127, 128, "bf16"), (16, 1025, 128, "bf16"),
    (64, 1023, 128, "bf16"),
    (1, 1, 64, "bf16"), (2, 64, 64, "bf16"), (1, 700, 64, "bf16"), (16, 515, 64, "bf16"),
    (24, 1300, 64, "bf16"), (48, 1025, 64, "bf16"), (96, 2305, 64, "bf16"),
    (200, 512, 64, "bf16"), (96, 4700, 64, "bf16"),
]


def test_every_shape_is_reached():
    want = {(16, "f32"): 3, (32, "f32"): 3, (64, "f32"): 3, (128, "f32"): 3, (128, "bf16"): 3,
            (64, "bf16"): 6}
    for (D, dt), n in want.items():
        got = {plan(BH, N, D, c, dt) for BH, N, d, t in CASES if (d, t) == (D, dt)
               for c in (True, False)}
        assert set(range(n)) <= got, (D, dt, got)


def test_plan_keeps_the_moments_for_long_sequences():
    """Linear in N where the pairs' quadratic cost is the larger one."""
    assert plan(64, 8192, 64, True, "bf16") == -1
    assert plan(8, 131072, 64, False, "bf16") == -1
    assert plan(8, 65536, 64, True, "bf16") == -1
    for D in (16, 32, 64, 128):
        assert plan(4, 1 << 20, D, True, "f32") == -1


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
        eo = max_rel(o[h], ro[0, 0])
        eg = float((np.abs(g[h] - rg[0, 0]) / np.abs(rg[0, 0])).max())
        say(f"{label} head {h}: E_O={eo:.2e} E_G={eg:.2e}")
        assert eo <= TOL[dt] and eg <= TOL[dt], (label, h, eo, eg)


@pytest.mark.gpu
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("BH,N,D,dt", CASES)
def test_shapes_against_explicit_matrix(BH, N, D, dt, causal):
    inp = make_inputs(1, BH, N, D, 7100 + N, dt)
    check(inp, dt, causal, f"BH{BH} N{N} D{D} {dt} c{causal} shape {plan(BH, N, D, causal, dt)}")


def scale_values(inp, dt, factor):
    """v rows times factor [N] (a power of two: exact)."""
    v = inp["v64"] * factor[None, None, :, None]
    out = dict(inp)
    if dt == "bf16":
        out["v"] = f32_to_bf16_bits(v.astype(np.float32))
        out["v64"] = bf16_bits_to_f64(out["v"])
    else:
        out["v"] = v.astype(np.float32)
        out["v64"] = out["v"].astype(np.float64)
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("D,dt", [(64, "bf16"), (128, "bf16"), (32, "f32"), (64, "f32")])
@pytest.mark.parametrize("kind", ["late", "zeros", "huge", "tiny"])
def test_value_scale(D, dt, causal, kind):
    """Values that outgrow the first tile's scale (a second attempt), a first
    tile of zeros, and values near the ends of the float range."""
    N = 420
    f = np.ones(N)
    if kind == "late":
        f[300:] = 2.0 ** 14
    elif kind == "zeros":
        f[:280] = 0.0
    else:
        f[:] = 2.0 ** (110 if kind == "huge" else -110)
    inp = scale_values(make_inputs(1, 3, N, D, 7200, dt), dt, f)
    check(inp, dt, causal, f"{kind} D{D} {dt} c{causal}")


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
