"""The search's winner named by the parabola alone, where that is hardest: blocks whose best scale lies half-way between two E4M3
values, or a rounding beside it.  The same bytes as the exhaustive search, and the oracle's."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_12245_amd import binding as B
from paper_2605_12245_amd import synth

DEV = "cuda:0"
GRID = torch.tensor([0.5, 1, 1.5, 2, 3, 4, 6, -0.5, -1, -1.5, -2, -3, -4, -6])
E2M1 = torch.tensor([0, 0.5, 1, 1.5, 2, 3, 4, 6, 0, -0.5, -1, -1.5, -2, -3, -4, -6], dtype=torch.float64)
E4M3 = torch.tensor([k / 8 * 2.0 ** -6 if k < 8 else (1 + k % 8 / 8) * 2.0 ** (k // 8 - 7) for k in range(127)], dtype=torch.float64)


def half_way(rows, dtype, off):
    """Rows of 16 blocks in pairs: E2M1 values, a 6 among them, times the two midpoints beside an E4M3 value of even mantissa, which the
    first scale of both then is: what the one lacks to it in Eq. 5 the other has too much, and alpha is 1.  off: other elements are that many
    units of 2^-22 further out or in, in the second block the other way, which leaves alpha where it is."""
    gen = torch.Generator().manual_seed(rows + off)
    pairs = rows * 8
    values = GRID[torch.randint(0, len(GRID), (pairs, 16), generator=gen)]
    at_six = torch.randint(0, 16, (pairs,), generator=gen)
    values[torch.arange(pairs), at_six] = 6.0
    binade = 2.0 ** torch.randint(-5, 4, (pairs,), generator=gen)
    even = (1 + torch.randint(1, 4, (pairs,), generator=gen) / 4) * binade
    nudge = torch.randint(-off, off + 1, (pairs, 16), generator=gen) * (2.0 ** -22 * binade)[:, None]
    nudge[values.abs() == 6.0] = 0.0                        # the largest element keeps the first scale
    lower, upper = values * (even - binade / 16)[:, None] + nudge, values * (even + binade / 16)[:, None] - nudge
    w = torch.stack((lower, upper), 1).reshape(rows, 256).to(dtype)
    w[0, :32] = 0.0
    w[0, 0] = w[0, 16] = 2688.0                             # alpha0 = 1
    return w


def in_doubt(w, out):
    """the share of blocks whose two nearest scales the parabola alone cannot tell apart (search_certified)"""
    codes = out.codes.cpu().reshape(-1, 8).long()
    q = E2M1[torch.stack((codes & 15, codes >> 4), -1).reshape(-1, 16)]
    x = w.double().reshape(-1, 16)
    c = (q * q).sum(1)
    best = (x * q).sum(1) / c
    scale = E4M3 * out.global_scale.double().item()
    upper = torch.searchsorted(scale, best).clamp(2, 126)
    sa, sb = scale[upper - 1], scale[upper]
    past = 2 * best - (sa + sb)
    error = ((x - q * torch.where(past > 0, sb, sa)[:, None]) ** 2).sum(1)
    doubt = (c * (sb - sa) * (past.abs() - 2.0 ** -16 * best) <= 2.0 ** -17 * error) & (error > 0)
    return doubt.double().mean().item(), (past == 0).double().mean().item()


def same_as_the_exhaustive_search(w, check=lambda out: None):
    rows, dtype = w.shape[0], w.dtype
    d = w.to(DEV)
    host = synth.bf16_bits(w) if dtype == torch.bfloat16 else w.numpy()
    for radius in (1, 4, 8):
        ref = oracle.quantize(host, oracle.METHOD_SOAR, radius) if rows == 16 else None
        for resident in (B.SOAR_RESIDENT_AUTO, B.SOAR_RESIDENT_NEVER):
            outs = []
            for mode in (B.SOAR_SEARCH_AUTO, B.SOAR_SEARCH_FULL):
                p = B.soar_default_params(B.SOAR_METHOD_SOAR, radius, mode)
                p.resident = resident
                o = B.new_outputs(rows, 256, DEV)
                desc = B.make_desc(d, o)
                B.quantize_batch([desc], p, B.new_batch_workspace([desc], p, DEV))
                outs.append(o)
            torch.cuda.synchronize()
            for f in ("codes", "scales", "global_scale", "status"):
                assert torch.equal(getattr(outs[0], f), getattr(outs[1], f)), (radius, resident, f)
            assert outs[0].sse.item() == outs[1].sse.item()
            check(outs[0])
            if ref is not None:
                assert np.array_equal(outs[0].codes.cpu().numpy(), ref.codes) and np.array_equal(outs[0].scales.cpu().numpy(), ref.scales)


# bf16 has no values within the doubt but the midpoints themselves; 2000 units lie across its edge
@pytest.mark.gpu
@pytest.mark.parametrize("dtype,off,least,most", [(torch.bfloat16, 0, 0.99, 1.0), (torch.float32, 0, 0.99, 1.0), (torch.float32, 1, 0.99, 1.0),
                                                  (torch.float32, 3, 0.99, 1.0), (torch.float32, 2000, 0.3, 0.9)],
                         ids=["bf16", "fp32", "fp32-1", "fp32-3", "fp32-2000"])
@pytest.mark.parametrize("rows", [16, 1100])
def test_half_way_scales_equal_the_exhaustive_search(rows, dtype, off, least, most):
    w = half_way(rows, dtype, off)

    def check(out):
        doubt, ties = in_doubt(w, out)
        assert out.global_scale.item() == 1.0 and least <= doubt <= most and (off > 0 or ties >= 0.99)

    same_as_the_exhaustive_search(w, check)


def beside_half_way(rows, dtype, ulps):
    """E2M1 values times midpoints of any two neighbours, a few units of the element type off: alpha is near 1, and few blocks are in doubt"""
    gen = torch.Generator().manual_seed(rows + ulps)
    values = torch.tensor([(1 + m / 8) * 2.0 ** e for e in range(-5, 4) for m in range(8)])
    mid = (values[:-1] + values[1:]) / 2
    blocks = GRID[torch.randint(0, len(GRID), (rows, 16, 16), generator=gen)]
    w = blocks * mid[torch.randint(0, len(mid), (rows, 16, 1), generator=gen)]
    w = w.reshape(rows, 256).to(dtype)
    if ulps:
        bits = w.view(torch.int16 if dtype == torch.bfloat16 else torch.int32)
        bits += torch.randint(-ulps, ulps + 1, bits.shape, generator=gen).to(bits.dtype)
    w[0, 0] = 2688.0                                         # alpha0 = 1
    return w


@pytest.mark.gpu
@pytest.mark.parametrize("ulps", [0, 1, 3])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("rows", [16, 1100])
def test_scales_beside_half_way_equal_the_exhaustive_search(rows, dtype, ulps):
    same_as_the_exhaustive_search(beside_half_way(rows, dtype, ulps))
