"""The search that evaluates only the factors next to each stored scale, against the search over every pair.

On the CPU a numpy model of the rule (which factors are evaluated, when the walk outwards may end, who wins a tie)
is compared with the plain double loop; on the GPU the kernels' two search modes are compared with each other, over
the orders, grids, magnitudes and inputs that the rule accepts.  Everything has to be equal bit for bit.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_12245_amd import binding as B

F = np.float32
DEV = "cuda:0"


# ------------------------------------------------------------------ CPU: the rule itself
def grid_of(n, lo, hi):
    return [F(F(F(lo) * F(n - 1 - k)) + F(F(hi) * F(k))) / F(n - 1) for k in range(n)]


def codes_at(w, t):
    with np.errstate(all="ignore"):
        return oracle.e2m1_nibble_many(w * (F(1.0) / t))


VALUES = np.array([0, .5, 1, 1.5, 2, 3, 4, 6, -0., -.5, -1, -1.5, -2, -3, -4, -6], dtype=np.float64)


def error_of(w, nib, s):
    """the ascending fused chain (binary64 operations rounded to binary32 stand in for the fused ones)"""
    err = F(0.0)
    for x, q in zip(w, VALUES[nib]):
        e = F(float(x) - q * float(s))
        err = F(float(e) * float(e) + float(err))
    return err


def plain_loop(w, base, grid, scales):
    best = None
    for k, beta in enumerate(grid):
        nib = codes_at(w, F(base * beta))
        for c, s in enumerate(scales):
            e = error_of(w, nib, s)
            if best is None or e < best[0]:
                best = (e, c, tuple(nib))
    return best


def excluded(s, t, e):
    rounding = F(1.0e-5)
    distance = F(abs(F(s - t)) - F(2.0 ** -22) * max(s, t))
    return s < F(2.0 ** 60) and F(s * distance) > F(float(rounding) * float(e) + 2.0 ** -98)


def nearest(w, base, grid, scales, offset):
    """offset: how far off the estimate of the enclosing pair is (the result must not depend on it)"""
    n, best, count = len(grid), None, 0

    def pair(k, c, s):
        nonlocal best, count
        t = F(base * grid[k])
        nib = tuple(codes_at(w, t))
        e = error_of(w, np.array(nib), s)
        count += 1
        if best is None or e < best[0] or (e == best[0] and k < best[3] and nib != best[2]):
            best = (e, c, nib, k)
        return t, e

    for c, s in enumerate(scales):
        km = min(range(n), key=lambda k: abs(float(base) * float(grid[k]) - float(s)))
        km = min(max(km + offset, 0), n - 1)
        split = km + (1 if F(base * grid[km]) <= s else 0)
        ka, kb = max(split - 1, 0), min(split, n - 1)
        t, e = pair(ka, c, s)
        while ka > 0 and not (t <= s and excluded(s, t, e)):
            ka -= 1
            t, e = pair(ka, c, s)
        t, e = pair(kb, c, s)
        while kb < n - 1 and not (t >= s and excluded(s, t, e)):
            kb += 1
            t, e = pair(kb, c, s)
    return best[:3], count


@pytest.mark.parametrize("n,lo,hi", [(101, 0.5, 1.5), (4, 0.9, 1.1), (21, 0.3, 0.7), (33, 1.25, 4.0), (257, 0.95, 1.05)])
def test_rule_equals_the_plain_loop(n, lo, hi):
    rng = np.random.default_rng(n)
    grid = grid_of(n, lo, hi)
    assert all(a <= b for a, b in zip(grid, grid[1:]))
    evaluated = total = 0
    for trial in range(24):
        scale = F(2.0 ** rng.integers(-30, 30))
        kind = trial % 6
        w = rng.standard_t(4, 16).astype(np.float32)
        if kind == 1:
            w = rng.integers(-6, 7, 16).astype(np.float32)              # exact ties at and between the thresholds
        elif kind == 2:
            w = rng.choice(np.array([0, .25, .75, 1.25, 1.75, 2.5, 3.5, 5], np.float32), 16)   # on the thresholds
        elif kind == 3:
            w[3] = 40.0                                                 # far beyond the largest code
        elif kind == 4:
            w[rng.random(16) < 0.8] = 0.0
        elif kind == 5:
            w[:] = 0.0
            w[rng.integers(0, 16)] = -0.0
        w = (w * scale).astype(np.float32)
        base = F(scale * F(1.0 if kind in (1, 2) else rng.uniform(0.3, 1.2)))
        for scales in ([F(base * F(0.9375)), F(base * F(1.0))], [base, F(base * F(0.5)), F(base * F(2.0))], [F(base * F(0.25)), F(base * F(8.0))]):
            want = plain_loop(w, base, grid, scales)
            for offset in (0, -1, 1) if trial % 4 == 0 else (0,):
                got, count = nearest(w, base, grid, scales, offset)
                assert got[0] == want[0] and got[1] == want[1] and got[2] == want[2], (trial, kind, scales, offset)
                if offset == 0:
                    evaluated, total = evaluated + count, total + n * len(scales)
    assert evaluated < total / (2 if n > 20 else 1)


# ------------------------------------------------------------------ GPU: the two search modes of the kernels
def inputs(dtype, cols):
    g = torch.Generator(device="cpu").manual_seed(cols)
    r = lambda rows: torch.randn(rows, cols, generator=g)  # noqa: E731
    sparse = r(37) * (torch.rand(37, cols, generator=g) < 0.1)
    sparse[5] = 0.0
    outlier = r(19) * 0.02
    outlier[::3, ::7] *= 300.0
    return [(n, w.to(dtype).to(DEV)) for n, w in (
        ("normal", r(130) * 0.02), ("integers", torch.randint(-6, 7, (33, cols), generator=g).float()),
        ("thresholds", torch.randint(-12, 13, (21, cols), generator=g).float() * 0.25), ("sparse", sparse), ("outliers", outlier),
        ("constant", torch.full((3, cols), 0.75)), ("small", r(9) * 2.0 ** -40), ("large", r(9) * 2.0 ** 62))]


def same(a, b, what):
    for f in ("codes", "scales", "global_scale", "sse", "status", "iters_run"):
        x, y = getattr(a, f), getattr(b, f)
        assert x is None or torch.equal(x, y), (what, f)
    if a.sse_trace is not None:
        assert torch.equal(a.sse_trace.nan_to_num(-1.0), b.sse_trace.nan_to_num(-1.0)), what


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("kw", [
    dict(), dict(n_beta=4), dict(n_beta=5, beta_lo=0.9, beta_hi=1.1), dict(n_beta=129), dict(n_beta=1000),
    dict(n_beta=33, beta_lo=0.25, beta_hi=0.8), dict(n_beta=33, beta_lo=1.2, beta_hi=3.0),
    dict(n_beta=8, beta_lo=1.0, beta_hi=1.0000005), dict(n_beta=16, beta_lo=1.0, beta_hi=1.0),
    dict(dd_mode=B.SOAR_DD_WINDOW, dss_radius=0), dict(dd_mode=B.SOAR_DD_WINDOW, dss_radius=5, n_beta=41),
    dict(arm=B.SOAR_METHOD_DSS_ONLY, dss_radius=1), dict(arm=B.SOAR_METHOD_DSS_ONLY, dss_radius=3, n_beta=17),
], ids=lambda kw: "-".join(f"{k}{v}" for k, v in kw.items()) or "paper")
def test_nvfp4_search_modes_agree(kw, dtype):
    kw = dict(kw)
    arm = kw.pop("arm", None)
    for cols in (16, 272):
        for name, w in inputs(dtype, cols):
            out = []
            for mode in (B.SOAR_SEARCH_AUTO, B.SOAR_SEARCH_FULL):
                p = B.soar_arm_params(arm, iters=3, early_stop_rel=0.0, **kw) if arm else \
                    B.soar_paper_params(iters=3, early_stop_rel=0.0, **kw)
                p.search_mode = mode
                out.append(B.quantize_iter(w, p))
            torch.cuda.synchronize()
            same(*out, (name, cols, kw))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("kw", [dict(), dict(n_beta=4), dict(n_beta=1000, radius=2), dict(n_beta=33, beta_lo=0.25, beta_hi=0.8),
                                dict(n_beta=33, beta_lo=1.2, beta_hi=3.0, radius=3), dict(n_beta=8, beta_lo=1.0, beta_hi=1.0000005),
                                dict(n_beta=64, radius=0)],
                         ids=lambda kw: "-".join(f"{k}{v}" for k, v in kw.items()) or "default")
def test_mxfp4_search_modes_agree(kw, dtype):
    for cols in (32, 288):
        for name, w in inputs(dtype, cols):
            out = [B.mx_quantize(w, B.soar_mx_default_params(single_pass=single, **kw)) for single in (False, True)]
            torch.cuda.synchronize()
            same(*out, (name, cols, kw))
