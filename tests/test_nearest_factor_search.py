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


# Both sides of the lines at which AUTO changes from the factors next to a candidate to the changes of the codes (radius
# 48; fewer than eight factors: 2 to 8), the widest window, and grids around the 128 factors that are looked through at once
WIDE = [dict(n_beta=4, dss_radius=2), dict(n_beta=4, dss_radius=3), dict(n_beta=5, dss_radius=3), dict(n_beta=6, dss_radius=5),
        dict(n_beta=6, dss_radius=6), dict(n_beta=7, dss_radius=8), dict(n_beta=7, dss_radius=9), dict(n_beta=8, dss_radius=48),
        dict(n_beta=8, dss_radius=49), dict(dss_radius=48), dict(dss_radius=49), dict(dss_radius=125), dict(n_beta=32, dss_radius=125),
        dict(n_beta=33, dss_radius=60), dict(n_beta=127, dss_radius=60), dict(n_beta=128, dss_radius=60), dict(n_beta=129, dss_radius=60),
        dict(n_beta=161, beta_lo=0.01, beta_hi=30.0, dss_radius=60), dict(n_beta=300, dss_radius=125)]


def ends_of_the_range(dtype, cols, low, high):
    """rows whose largest magnitudes run through the powers of two around both ends of a range"""
    g = torch.Generator(device="cpu").manual_seed(cols + 1)
    return [("low end", torch.cat([torch.randn(4, cols, generator=g) * 2.0 ** e for e in range(low - 3, low + 4)]).to(dtype).to(DEV)),
            ("high end", torch.cat([torch.randn(4, cols, generator=g) * 2.0 ** e for e in range(high - 3, high + 4)]).to(dtype).to(DEV))]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("kw", WIDE, ids=lambda kw: "-".join(f"{k}{v}" for k, v in kw.items()))
def test_nvfp4_wide_windows_and_ends_of_the_range_agree(kw, dtype):
    # the global scale, about 1/2688 of the maximum, leaves the nearest search at 2^-35 and 2^50; the maximum at 2^60
    tensors = inputs(dtype, 272) + ends_of_the_range(dtype, 48, -24, 58) + [(f"2^{e}", inputs(dtype, 48)[0][1] * 2.0 ** e) for e in (-18, -19, -20)]
    for arm in (None, B.SOAR_METHOD_DSS_ONLY):
        for name, w in tensors:
            out = []
            for mode, resident in ((B.SOAR_SEARCH_AUTO, 0), (B.SOAR_SEARCH_AUTO, 1), (B.SOAR_SEARCH_FULL, 0)):
                k = dict(kw, iters=2, early_stop_rel=0.0)
                p = B.soar_arm_params(arm, **k) if arm else B.soar_paper_params(dd_mode=B.SOAR_DD_WINDOW, **k)
                p.search_mode, p.resident = mode, resident
                out.append(B.quantize_iter(w, p))
            torch.cuda.synchronize()
            same(out[0], out[2], (name, kw, arm))
            same(out[1], out[2], (name, kw, arm))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("kw", [dict(n_beta=n, radius=r) for n, r in ((4, 1), (4, 2), (5, 2), (5, 3), (7, 4), (7, 5), (8, 5), (8, 6), (101, 5), (101, 6),
                                                                      (101, 8), (101, 16), (101, 127), (128, 16), (129, 16), (31, 127), (300, 127))],
                         ids=lambda kw: "-".join(f"{k}{v}" for k, v in kw.items()))
def test_mxfp4_wide_windows_and_ends_of_the_range_agree(kw, dtype):
    # block scales leave the nearest search below 2^(67 - 127) and above 2^(186 - 127), that is maxima below 2^-58 and above 2^61
    for name, w in inputs(dtype, 288) + ends_of_the_range(dtype, 96, -59, 60) + ends_of_the_range(dtype, 96, -118, 120):
        out = [B.mx_quantize(w, B.soar_mx_default_params(single_pass=single, **kw)) for single in (False, True)]
        torch.cuda.synchronize()
        same(*out, (name, kw))


def milliseconds(run):
    run()
    times = []
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record(); run(); b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b))
    return min(times)


@pytest.mark.gpu
def test_the_default_search_is_not_the_slower_one():
    """whatever the radius, the grid and the magnitudes: evaluating every pair takes no less time (half as long again is
    allowed for noise; wide windows and short grids took several times as long with the nearest-factor search alone)"""
    w = inputs(torch.bfloat16, 4096)[0][1].repeat(4, 1)
    for n, r in ((4, 1), (4, 16), (101, 1), (101, 8), (101, 16), (101, 127), (400, 32)):
        auto, every = (milliseconds(lambda: B.mx_quantize(w, B.soar_mx_default_params(n_beta=n, radius=r, single_pass=s))) for s in (False, True))
        assert auto <= 1.5 * every, ("mxfp4", n, r, auto, every)
    for f in (1.0, 2.0 ** -30):
        for n, r in ((4, 1), (4, 16), (16, 1.0), (101, 2), (101, 64), (101, 125), (400, 32)):
            out = []
            for mode in (B.SOAR_SEARCH_AUTO, B.SOAR_SEARCH_FULL):
                p = B.soar_paper_params(iters=2, early_stop_rel=0.0, n_beta=n, dd_mode=B.SOAR_DD_WINDOW, dss_radius=int(r),
                                        **(dict(beta_lo=1.0, beta_hi=1.0) if r == 1.0 and n == 16 else {}))
                p.search_mode = mode
                out.append(milliseconds(lambda: B.quantize_iter(w * f, p)))
            assert out[0] <= 1.5 * out[1], ("nvfp4", f, n, r, out)
