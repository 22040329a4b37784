"""The MXFP4 search of bf16 blocks: nothing above a factor that equals the candidate scale is evaluated, larger candidates only
where a block reaches beyond 6 X0, smaller ones only where its largest weight does not rule them out.

On the CPU a numpy model of the rule against the plain double loop over every (factor, candidate) pair; on the GPU the search
against the evaluation of every pair.  Equal bit for bit.  The inputs are bf16 weights whose ties with the midpoints of the grid,
saturated elements and zero blocks are what the rule has to get right.
"""
import re

import numpy as np
import pytest
import torch

from paper_2605_12245_amd import binding as B
from test_nearest_factor_search import FAR_SIDE, SLACK, SOURCE, Block, F, fma, grid_of, plain_loop, same

DEV = "cuda:0"
GRIDS = [(101, 0.5, 1.5), (4, 0.9, 1.1), (21, 0.25, 1.25), (33, 0.25, 2.25), (17, 1.0, 2.0), (33, 1.25, 4.0), (257, 0.95, 1.05), (5, 0.5, 1.0)]


TIED_ERROR, MISS_MARGIN = (F(re.search(rf"constexpr float {name} = ([0-9.]+)f", SOURCE).group(1)) for name in ("kEqualFactorError", "kMissMargin"))


def bf16(w):
    return torch.from_numpy(np.asarray(w, np.float32)).to(torch.bfloat16).float().numpy()


def best_factor(block, s, ratio):
    """mx_best_factor<true>: (error, factor, pairs evaluated)"""
    err, t, grid, last = block.errors(s), block.t, block.grid, len(block.grid) - 1
    per_error = F(s * F(F(1.0) / FAR_SIDE[32]))
    slack = F(s * F(SLACK * per_error))

    def far(distance, e):
        return fma(distance, per_error, -slack) > e

    at = F(F(ratio - grid[0]) * F(F(last) / F(grid[-1] - grid[0])))
    lo = int(min(max(at, F(0.0)), F(last)))
    hi = lo if at < 0 else min(lo + 1, last)
    if grid[lo] == ratio:
        lo, hi = max(lo - 1, 0), lo
    best, k = err[lo], lo
    if err[hi] < best:
        best, k = err[hi], hi
    seen = 1 + (hi != lo)
    down = lo > 0 and not far(F(s - t[lo]), err[lo])
    up = hi < last and not (far(F(t[hi] - s), err[hi]) or (t[hi] == s and err[hi] < TIED_ERROR * F(s * s)))
    while down or up:
        kk = lo = lo - 1 if down else lo
        if not down:
            kk = hi = hi + 1
        seen += 1
        gone = far(F(s - t[kk]) if down else F(t[kk] - s), err[kk])
        if err[kk] < best or (err[kk] == best and kk < k):
            best, k = err[kk], kk
        down, up = (not gone and lo > 0, up) if down else (down, not gone and hi < last)
    return best, k, seen


def search(block, x0, radius):
    bmax = np.abs(block.w).max()
    best, k, seen = best_factor(block, x0, F(1.0))
    code = 0
    no_larger = bool((block.grid == F(1.0)).any()) and bmax <= F(6.0) * x0
    for o in range(1, radius + 1):
        for sign in (-1, 1):
            s = F(x0 * F(2.0 ** (sign * o)))
            if sign < 0:
                miss = max(fma(s, -6.0, bmax), F(0.0))
                if MISS_MARGIN * F(miss * miss) > best:
                    continue
            elif no_larger:
                continue
            e, kk, n = best_factor(block, s, F(2.0 ** (sign * o)))
            seen += n
            if e < best or (e == best and kk < k and (block.nib[kk] != block.nib[k]).any()):
                best, k, code = e, kk, sign * o
    return best, code, tuple(block.nib[k]), seen


def bf16_blocks(rng, trials):
    for trial in range(trials):
        kind = trial % 8
        scale = F(2.0 ** int(rng.choice([-60, -59, -3, 0, 7, 58, 59])))
        w = rng.standard_t(4, 32)
        if kind == 1:
            w = rng.choice([0, .25, .75, 1.25, 1.75, 2.5, 3.5, 5], 32) * rng.choice([-1, 1], 32)        # ties under X0
        elif kind == 2:
            w = rng.choice([.5, 1.5, 2.5, 3.5, 5, 7, 3, 1], 32)                                          # ties under 2 X0
        elif kind == 3:
            w = rng.uniform(-8, 8, 32)                                                                   # saturated, large errors
        elif kind == 4:
            w = rng.choice([.25, .75, 1.25, 2.5, 5], 32) * (1 + rng.choice([-1, 0, 1], 32) * 2.0 ** -7)  # one unit beside ties
        elif kind == 5:
            w = rng.standard_normal(32) * 0.2
            w[rng.integers(32)] = rng.choice([4.0, 4.03125, 4.25, 5.0, 5.96875, 6.0, 6.03125, 7.96875])  # the two exclusions' edges
        elif kind == 6:
            w = np.zeros(32) if trial % 16 == 6 else np.where(np.arange(32) == 5, 4.0, 0.0)
        elif kind == 7:
            w = rng.integers(-6, 7, 32)
        w = bf16(np.asarray(w, np.float32) * scale)
        top = np.abs(w).max()
        x0 = F(2.0 ** (int(np.frexp(top)[1]) - 3)) if top > 0 else F(1.0)
        if F(2.0 ** -60) <= x0 < F(2.0 ** 60):
            yield trial, w, x0


@pytest.mark.parametrize("n,lo,hi", GRIDS)
def test_rule_equals_the_plain_loop(n, lo, hi):
    grid = grid_of(n, lo, hi)
    seen = blocks = 0
    for trial, w, x0 in bf16_blocks(np.random.default_rng(n), 160):
        block = Block(w, x0, grid)
        for radius in (0, 1, 2, 6):
            if radius > n - 2:
                continue
            want = plain_loop(block, [x0] + [F(x0 * F(2.0 ** o)) for k in range(1, radius + 1) for o in (-k, k)])
            best, code, nib, pairs = search(block, x0, radius)
            rank = 0 if code == 0 else 2 * abs(code) - (code < 0)
            assert (best, rank, nib) == want, (trial, radius)
            if radius == 1:
                seen, blocks = seen + pairs, blocks + 1
    if (n, lo, hi) == (101, 0.5, 1.5):
        assert seen < 3.6 * blocks, seen / blocks       # many of these blocks saturate; six before


def test_the_constants_allow_for_the_rounding():
    # a rise of 2^-10 s^2 against the rounding of two errors of 32 terms, 34 units of 2^-24 each
    assert 2.0 ** -10 > 2 * 34 * 2.0 ** -24 * TIED_ERROR and 1.0 - MISS_MARGIN > 2 * 34 * 2.0 ** -24


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("n,lo,hi", GRIDS)
def test_search_equals_every_pair_on_the_gpu(n, lo, hi, dtype):
    rows = [w for seed in range(12) for _, w, _ in bf16_blocks(np.random.default_rng([n, seed]), 160)]
    w = torch.from_numpy(np.stack(rows))
    w = torch.cat([w, w.flip(0)], dim=1).to(dtype).to(DEV)
    for radius in (0, 1, 2, 6):
        if radius > n - 2:
            continue
        kw = dict(n_beta=n, beta_lo=lo, beta_hi=hi, radius=radius)
        out = [B.mx_quantize(w, B.soar_mx_default_params(single_pass=single, **kw)) for single in (False, True)]
        torch.cuda.synchronize()
        same(*out, kw)
