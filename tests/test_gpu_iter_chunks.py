"""Iterations whose tiles are dealt in chunks over the workgroups that fill the GPU once: the same results, bit for bit, as with
one chunk per workgroup (a forced number of tiles), at the numbers of tiles where the size of a chunk changes."""
import pytest
import torch

from paper_2605_12245_amd import binding as B

DEV = "cuda:0"
PLACES = 5 * 256          # of k_iter on 256 compute units; elsewhere the edges lie elsewhere and the comparison still holds


def run(weights, params):
    outs = [B.new_outputs(w.shape[0], w.shape[1], DEV, params.iters) for w in weights]
    descs = [B.make_desc(w, o) for w, o in zip(weights, outs)]
    B.quantize_batch(descs, params, B.new_batch_workspace(descs, params, DEV))
    torch.cuda.synchronize()
    return outs


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("tiles", [(1, 1), (PLACES - 1, 1), (2 * 2 * PLACES - 3, 2), (2 * 2 * PLACES - 1, 1, 1), (2 * 4 * PLACES - 70, 64, 3),
                                   (2 * 4 * PLACES, 5)], ids=str)
def test_dealt_chunks_equal_one_chunk_per_workgroup(tiles, dtype):
    gen = torch.Generator(device=DEV).manual_seed(sum(tiles))
    # the last tile of every tensor is ragged
    weights = [(torch.randn((t * 256 - 3 * k - 1, 16), generator=gen, device=DEV) * 0.02).to(dtype) for k, t in enumerate(tiles)]
    for p in (B.soar_paper_params(iters=3), B.soar_arm_params(B.SOAR_METHOD_DSS_ONLY, iters=2)):
        dealt = run(weights, p)
        p.tiles_per_wg = 4
        for a, b in zip(dealt, run(weights, p)):
            for f in ("codes", "scales", "global_scale", "sse", "status", "iters_run"):
                assert torch.equal(getattr(a, f), getattr(b, f)), f
            assert torch.equal(a.sse_trace.nan_to_num(-1.0), b.sse_trace.nan_to_num(-1.0))


@pytest.mark.gpu
def test_chunks_of_more_than_four_tiles():
    """a tensor of more than 4096 chunks of four tiles: eight tiles a chunk, the last one ragged, beside a small tensor"""
    gen = torch.Generator(device=DEV).manual_seed(8)
    weights = [(torch.randn((rows, 16), generator=gen, device=DEV) * 0.02).to(torch.bfloat16) for rows in (256 * (4 * 4096 + 13) - 7, 256 * 9 - 1)]
    p = B.soar_paper_params(iters=2)
    dealt = run(weights, p)
    for tiles_per_wg in (8, 16):
        p.tiles_per_wg = tiles_per_wg
        for a, b in zip(dealt, run(weights, p)):
            for f in ("codes", "scales", "global_scale", "sse", "status", "iters_run", "sse_trace"):
                assert torch.equal(getattr(a, f), getattr(b, f)), (tiles_per_wg, f)
