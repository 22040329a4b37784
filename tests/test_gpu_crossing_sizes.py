"""One-launch kernels at the numbers of workgroups where the way their results cross the grid changes (16 and 64 workgroups read
each other directly, 32 with fewer loads; groups of 16 and of 64, the last one ragged), against the paths of several launches."""
import pytest
import torch

from paper_2605_12245_amd import binding as B

DEV = "cuda:0"
WORKGROUPS = (1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 65, 79, 80, 81, 127, 128, 129, 193, 255, 256)     # of 256 lanes, a block each


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
def test_every_way_across_the_grid(dtype):
    gen = torch.Generator(device=DEV).manual_seed(3)
    for G in WORKGROUPS:
        w = (torch.randn((256 * G - 5, 16), generator=gen, device=DEV) * 0.02)
        w[256 * (G // 2) + 9, 3] = 1.5                      # the maximum lies in one workgroup
        w = w.to(dtype)
        for p in (B.soar_default_params(), B.soar_default_params(B.SOAR_METHOD_RTN, 0), B.soar_paper_params(iters=4, early_stop_rel=0.0, n_beta=21),
                  B.soar_arm_params(B.SOAR_METHOD_CJSO_ONLY, iters=5, early_stop_rel=0.0)):
            iterated = p.iters > 1
            out, launches = [], []
            for resident in (B.SOAR_RESIDENT_AUTO, B.SOAR_RESIDENT_NEVER):
                p.resident = resident
                ws = B.new_workspace(w.shape[0], 16, p, DEV)
                both = [B.new_outputs(w.shape[0], 16, DEV, p.iters if iterated else 0) for _ in range(2)]
                B.soar_kernel_timing_enable(True)
                for o in both:                              # twice on one workspace
                    B.quantize_batch([B.make_desc(w, o)], p, ws)
                torch.cuda.synchronize()
                launches.append(B.soar_kernel_timing_read(B.SOAR_KERNEL_RESIDENT)[1])
                B.soar_kernel_timing_enable(False)
                for f in ("codes", "scales", "global_scale", "status", "iters_run", "sse", "sse_trace"):
                    assert getattr(both[0], f) is None or torch.equal(getattr(both[0], f), getattr(both[1], f)), (G, p.method, f)
                out.append(both[0])
            assert launches == [2, 0], (G, p.method)        # the one-launch kernel against the others
            a, b = out
            for f in ("codes", "scales", "global_scale", "status", "iters_run"):
                assert getattr(a, f) is None or torch.equal(getattr(a, f), getattr(b, f)), (G, p.method, f)
            if iterated:                                    # the same tree on both paths
                assert torch.equal(a.sse, b.sse) and torch.equal(a.sse_trace, b.sse_trace), (G, p.method)
            else:                                           # binary64 sums of at most 65536 errors in another order
                assert abs(a.sse.item() - b.sse.item()) <= 1e-11 * b.sse.item(), (G, p.method)
