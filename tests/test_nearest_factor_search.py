"""The search that evaluates only the factors next to each stored scale, against the search over every pair.

On the CPU a numpy model of the rule (which factors are evaluated, when the walk outwards may end, who wins a tie)
is compared with the plain double loop; on the GPU the kernels' two search modes are compared with each other, over
the orders, grids, magnitudes and inputs that the rule accepts.  Everything has to be equal bit for bit.
"""
import os
import re

import numpy as np
import pytest
import torch

import oracle
from paper_2605_12245_amd import binding as B
from paper_2605_12245_amd import build

F = np.float32
DEV = "cuda:0"


# ------------------------------------------------------------------ CPU: the rule itself
SOURCE = "".join(open(os.path.join(build.HERE, "csrc", f)).read() for f in ("soar_iterated.hpp", "soar_mxfp4.hpp"))
FAR_SIDE = {n: F(re.search(rf"kFarSideRounding{n} = ([0-9.e-]+)f", SOURCE).group(1)) for n in (16, 32)}
SLACK = F(2.0 ** -21)


def grid_of(n, lo, hi):
    return np.array([F(F(F(lo) * F(n - 1 - k)) + F(F(hi) * F(k))) / F(n - 1) for k in range(n)], dtype=np.float32)


def fma(a, b, c):
    """binary64 operations rounded to binary32 stand in for the fused ones"""
    return F(float(a) * float(b) + float(c))


VALUES = np.array([0, .5, 1, 1.5, 2, 3, 4, 6, -0., -.5, -1, -1.5, -2, -3, -4, -6], dtype=np.float64)


class Block:
    """codes of a block at every factor, and errors for a stored scale by the ascending fused chain"""

    def __init__(self, w, base, grid):
        with np.errstate(all="ignore"):
            self.t = (F(base) * grid).astype(np.float32)
            self.nib = np.stack([oracle.e2m1_nibble_many((w * (F(1.0) / t)).astype(np.float32)) for t in self.t])
        self.w, self.grid, self.base = w, grid, F(base)

    def errors(self, s):
        err = np.zeros(len(self.grid), np.float32)
        with np.errstate(over="ignore"):
            for j, x in enumerate(self.w):
                e = (float(x) - VALUES[self.nib[:, j]] * float(s)).astype(np.float32).astype(np.float64)
                err = (e * e + err.astype(np.float64)).astype(np.float32)
        return err


def plain_loop(block, scales):
    """factors ascending, for each the candidates in their order, the first smallest error wins"""
    table = np.stack([block.errors(s) for s in scales], axis=1)
    k, c = divmod(int(table.reshape(-1).argmin()), len(scales))
    return table[k, c], c, tuple(block.nib[k])


def best_factor(block, err, s, ka, kb, rounding, slack):
    """the kernels' best_factor and mx_best_factor from the pair ka <= kb on: the walks outwards and their certificate"""
    last = len(block.grid) - 1
    per_error = F(s * F(F(1.0) / rounding))
    slack = F(s * F(slack * per_error))

    def far(distance, e):
        with np.errstate(over="ignore"):
            return fma(distance, per_error, -slack) > e

    t, best, k, seen = block.t, err[ka], ka, 1 + (kb != ka)
    if err[kb] < best:
        best, k = err[kb], kb
    lo, hi = ka, kb
    down = lo > 0 and not far(F(s - t[ka]), err[ka])
    up = hi < last and not far(F(t[kb] - s), err[kb])
    while down or up:
        kk = lo = lo - 1 if down else lo
        if not down:
            kk = hi = hi + 1
        seen += 1
        gone = far(F(s - t[kk]) if down else F(t[kk] - s), err[kk])
        if err[kk] < best or (err[kk] == best and kk < k):
            best, k = err[kk], kk
        if down:
            down = not gone and lo > 0
        else:
            up = not gone and hi < last
    return best, k, seen


def start_pair(block, s, off):
    """joint_search_nearest: the estimate of where s lies, off by `off`, clamped to the grid"""
    n = len(block.grid)
    per_beta = F(F(n - 1) / F(block.grid[-1] - block.grid[0]))
    at = fma(s, F(F(F(1.0) / block.base) * per_beta), -F(block.grid[0] * per_beta))
    ka = int(min(max(at, F(0.0)), F(n - 2)))
    ka = min(max(ka + off, 0), n - 2)
    return ka, ka + 1


def start_pair_mx(block, s, off):
    """mx_search_nearest: one factor where s lies below the grid, else the two around it"""
    n = len(block.grid)
    at = F(F(F(s / block.base) - block.grid[0]) * F(F(n - 1) / F(block.grid[-1] - block.grid[0])))
    lo = int(min(max(at, F(0.0)), F(n - 1)))
    lo = min(max(lo + off, 0), n - 1)
    return lo, lo if at < 0 else min(lo + 1, n - 1)


def nearest(block, scales, off=0, weaken=1.0, slack=SLACK):
    """candidates in their order; a tie goes to the smaller factor unless both give the same codes"""
    size = len(block.w)
    win, seen = None, 0
    for c, s in enumerate(scales):
        err = block.errors(s)
        ka, kb = (start_pair if size == 16 else start_pair_mx)(block, s, off)
        e, k, n = best_factor(block, err, s, ka, kb, F(FAR_SIDE[size] * F(weaken)), slack)
        seen += n
        nib = tuple(block.nib[k])
        if win is None or e < win[0] or (e == win[0] and k < win[3] and nib != win[2]):
            win = (e, c, nib, k)
    return win[:3], seen


def blocks(size, rng, trials):
    """weights and base scales: heavy-tailed, on the grid, on the thresholds, a dominating outlier, sparse, zero; magnitudes
    over the range in which the kernels take this search (global scales 2^-35 .. 2^50 times stored scales; E8M0 codes 67 .. 186)"""
    for trial in range(trials):
        kind = trial % 6
        e = int(rng.integers(-30, 30)) if trial % 3 else (int(rng.choice([-44, -43, 55, 56])) if size == 16 else int(rng.choice([-60, -59, 58, 59])))
        scale = F(2.0 ** e)
        w = rng.standard_t(4, size).astype(np.float32)
        if kind == 1:
            w = rng.integers(-6, 7, size).astype(np.float32)
        elif kind == 2:
            w = rng.choice(np.array([0, .25, .75, 1.25, 1.75, 2.5, 3.5, 5], np.float32), size)
        elif kind == 3:
            w[3] = 13.0
        elif kind == 4:
            w[rng.random(size) < 0.8] = 0.0
        elif kind == 5:
            w[:] = 0.0
            w[rng.integers(0, size)] = -0.0
        base = scale if size == 32 or kind in (1, 2) else F(scale * F(rng.uniform(0.3, 1.2)))
        yield trial, kind, (w * scale).astype(np.float32), base


@pytest.mark.parametrize("size", [16, 32])
@pytest.mark.parametrize("n,lo,hi", [(101, 0.5, 1.5), (4, 0.9, 1.1), (21, 0.3, 0.7), (33, 1.25, 4.0), (257, 0.95, 1.05)])
def test_rule_equals_the_plain_loop(n, lo, hi, size):
    grid = grid_of(n, lo, hi)
    assert all(a <= b for a, b in zip(grid, grid[1:]))
    evaluated = total = 0
    for trial, kind, w, base in blocks(size, np.random.default_rng(n + size), 24):
        block = Block(w, base, grid)
        if size == 16:
            windows = ([F(base * F(0.9375)), base], [base, F(base * F(0.5)), F(base * F(2.0))], [F(base * F(0.25)), F(base * F(8.0))],
                       [F(base * F(2.0 ** -o)) for o in range(0, 12, 3)])
        else:
            windows = ([base, F(base / 2), F(base * 2)], [base] + [F(base * F(2.0 ** o)) for k in range(1, 7) for o in (-k, k)])
        for scales in windows:
            want = plain_loop(block, scales)
            for off in (0, -1, 1, 3, -n) if size == 16 else (0,):       # the estimate may be off; the power of two is exact
                got, seen = nearest(block, scales, off)
                assert got == want, (trial, kind, scales, off)
                if off == 0 and len(scales) < 5:
                    evaluated, total = evaluated + seen, total + n * len(scales)
    assert evaluated < total / (2 if n > 20 else 1)


@pytest.mark.parametrize("size", [16, 32])
@pytest.mark.parametrize("weaken,slack,sound", [(1.0, SLACK, True), (2.0 ** -8, SLACK, False), (1.0e-20, F(0.0), False)],
                         ids=["as it is", "a 256th of the rounding", "no rounding"])
def test_certificate_is_needed_and_no_weaker_one_will_do(size, weaken, slack, sound):
    """Elements on the smallest thresholds of the factors next to a stored scale, and one that dominates the error: a factor
    further out computes to the same error although its exact one is larger, and being the earlier one it wins."""
    rng = np.random.default_rng(7)
    grid = grid_of(401, 0.95, 1.05)
    wrong = 0
    for trial in range(150):
        k = int(rng.integers(50, 350)) if size == 16 else 200
        s = F(rng.uniform(grid[k], grid[k + 1])) if size == 16 else F(1.0)
        w = (rng.choice([.25, .75], size) * rng.uniform(grid[k - 4], grid[k + 4], size)).astype(np.float32)
        w[0] = 2.0 ** rng.uniform(3.0, 8.0)
        block = Block(w, F(1.0), grid)
        wrong += nearest(block, [s], 0, weaken, slack)[0] != plain_loop(block, [s])
    assert (wrong == 0) if sound else (wrong > 0), wrong


def test_the_rule_modelled_here_is_the_one_in_the_source():
    """the constants that the model does not read, and the gates in front of the search"""
    assert FAR_SIDE[16] == F(1.0e-5) and FAR_SIDE[32] == F(1.8e-5)
    # four times twice the rounding of a chain of n elements: 2 (n + 2) units of 2^-24
    assert all(FAR_SIDE[n] > 4 * 2 * (n + 2) * 2.0 ** -24 for n in (16, 32))
    assert SOURCE.count("slack = s * (0x1p-21f * per_error)") == 2
    assert "return alpha > 0x1p-35f && alpha < 0x1p50f && f_of(amax_bits) < 0x1p60f;" in SOURCE
    assert "const bool near = (uint32_t)(e0 - 67) < 120u;" in SOURCE


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
@pytest.mark.parametrize("kw", [dict(n_beta=n, radius=r) for n, r in ((4, 2), (4, 3), (5, 3), (5, 4), (7, 5), (7, 6), (8, 6), (8, 7), (101, 5), (101, 6),
                                                                      (101, 7), (101, 16), (101, 127), (128, 16), (129, 16), (31, 127), (300, 127))],
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
