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


def half_way(rows, dtype, ulps):
    """rows of 16 blocks of E2M1 values times midpoints of neighbouring E4M3 values: with alpha 1 every scale ties"""
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
def test_half_way_scales_equal_the_exhaustive_search(rows, dtype, ulps):
    w = half_way(rows, dtype, ulps)
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
            if ref is not None:
                assert np.array_equal(outs[0].codes.cpu().numpy(), ref.codes) and np.array_equal(outs[0].scales.cpu().numpy(), ref.scales)
