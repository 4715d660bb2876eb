"""The GEMM-with-unmask call without a workspace, where none is needed.

A shape whose K is not split needs no workspace, so the caller may pass NULL.  That must not change
the kernel: the bits are those of the call with a workspace, and of the fused call that forms the
masked input itself.
"""
import pytest
import torch

import paper_2609_15039_amd as sp
import workloads as WL

pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.mark.parametrize("layout", ["row", "tiled"])
@pytest.mark.parametrize("prec", [sp.SPLITEE_PREC_BF16, sp.SPLITEE_PREC_BF16X3])
@pytest.mark.parametrize("M,N,K", [(17, 640, 264), (64, 3072, 512), (100, 2560, 704), (128, 500, 520), (200, 1000, 648)])
def test_no_workspace_is_the_same_call(M, N, K, prec, layout):
    print("M=%d N=%d K=%d prec=%d %s" % (M, N, K, prec, layout), flush=True)
    assert sp.splitee_gemm_workspace_bytes(M, N, K, prec) == 0
    W = torch.from_numpy(WL.gen_w(N, K, seed=1)).to(DEV).to(torch.bfloat16)
    W = sp.tile_weights(W) if layout == "tiled" else W
    X = torch.from_numpy(WL.gen_x(M, K, seed=2)).to(DEV)
    eta = sp.noise(M, K, sp.SPLITEE_MECH_GAUSSIAN, 50.0, 1.0, 3, 4)
    C = sp.correction(W, M, sp.SPLITEE_MECH_GAUSSIAN, 50.0, 1.0, 3, 4)
    Xt = sp.mask(X, eta, prec)
    with_ws = sp.masked_linear_unmask(Xt, prec, W, C, ws=sp.workspace(M, N, K, prec, gemm_only=True))
    Y = torch.full((M, N), float("nan"), device=DEV)
    sp.splitee_masked_linear_unmask(Xt, prec, K, W, sp._wtype(W), K, C, N, Y, N, M, N, K, None, 0)
    assert torch.equal(Y, with_ws)
    fused = sp.masked_linear_fused(X, W, C, sp.SPLITEE_MECH_GAUSSIAN, 50.0, 1.0, 3, 4, prec=prec, eta_override=eta)
    assert torch.equal(fused, with_ws)
