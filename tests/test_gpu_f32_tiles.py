"""The binary32 GEMM over its tiles: every row count per tile, whole and split K, both W types.

Small integers keep every partial sum exact, so the unmasked output must equal X W^T bit for bit
with and without a split; K runs through fewer K tiles than the stages, remainders of the ring and
several accumulator chains, M and N past tile edges, N without whole 16-column blocks.
"""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2609_15039_amd as sp
import workloads as WL

pytestmark = pytest.mark.gpu

DEV = "cuda"
F32 = sp.SPLITEE_PREC_F32


@pytest.mark.parametrize("wt", ["f32", "bf16"])
@pytest.mark.parametrize("M,N,K", [(1, 4, 8), (1, 2560, 4096), (16, 500, 40), (17, 64, 96), (33, 1300, 1032), (48, 132, 2048),
                                   (64, 2052, 520), (80, 3072, 264), (96, 4100, 128), (112, 2500, 200), (128, 3072, 2056),
                                   (200, 700, 4104), (333, 2560, 1288), (333, 6144, 648), (257, 4864, 392)])
def test_f32_gemm_is_exact(M, N, K, wt):
    print("M=%d N=%d K=%d %s" % (M, N, K, wt), flush=True)
    X, W = WL.gen_int((M, K), -8, 8, M + K), WL.gen_int((N, K), -4, 4, N + K)
    C = WL.gen_int((M, N), -100, 100, M + N)
    Xd, Cd = torch.from_numpy(X).to(DEV), torch.from_numpy(C).to(DEV)
    Wd = torch.from_numpy(W).to(DEV)
    if wt == "bf16":
        Wd = Wd.to(torch.bfloat16)
    want = O.gemm64(X, W)
    ws = sp.workspace(M, N, K, F32, gemm_only=True)
    Y = torch.full((M, N), float("nan"), device=DEV)
    for _ in range(3):
        sp.masked_linear_unmask(Xd[None], F32, Wd, Cd, ws=ws, Y=Y.fill_(float("nan")))
        assert np.array_equal(Y.cpu().numpy().astype(np.float64), want - C)
    R = torch.full((M, N), float("nan"), device=DEV)
    sp.splitee_masked_linear(Xd, F32, K, Wd, sp._wtype(Wd), K, R, N, M, N, K)
    assert np.array_equal(R.cpu().numpy().astype(np.float64), want)


@pytest.mark.parametrize("M,N,K", [(16, 512, 2048), (333, 2560, 4096)])
def test_f32_infinities_and_nan_stay_in_their_rows(M, N, K):
    """A row past the tile or a k past the matrix is zeros on both sides, so an infinity or a NaN
    reaches its own row only."""
    g = torch.Generator(device=DEV)
    g.manual_seed(5)
    X, W = torch.randn((M, K), generator=g, device=DEV), torch.randn((N, K), generator=g, device=DEV)
    X[3, 7], X[M - 1, K - 1] = float("inf"), float("nan")
    ws = sp.workspace(M, N, K, F32, gemm_only=True)
    Y = sp.masked_linear_unmask(X[None], F32, W, torch.zeros((M, N), device=DEV), ws=ws)
    bad = ~torch.isfinite(Y).all(dim=1)
    assert bad.nonzero().flatten().tolist() == [3, M - 1]
    assert torch.equal(Y[3], torch.where(W[:, 7] > 0, float("inf"), -float("inf")).to(Y.dtype))
    assert torch.isnan(Y[M - 1]).all()
