"""The binary64 GEMM over its tiles: every tile height, whole and split K, both W types, both outputs.

Without noise the fused call is X W^T - C rounded to binary32: small integers make it exact,
whatever the tile, the split or the K remainder.  The correction (binary64 output) is compared
with the product of the drawn noise in binary64 to K roundings.
"""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2609_15039_amd as sp
import workloads as WL

pytestmark = pytest.mark.gpu

DEV = "cuda"
SHAPES = [(1, 5, 8), (1, 3072, 2056), (16, 100, 72), (17, 63, 4096), (33, 1000, 1288), (48, 2560, 520), (64, 4100, 104),
          (100, 3072, 1032), (130, 700, 2568), (256, 3072, 264)]


@pytest.mark.parametrize("wt", ["f32", "bf16"])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_f64_gemm_is_exact(M, N, K, wt):
    print("M=%d N=%d K=%d %s" % (M, N, K, wt), flush=True)
    X, W, C = WL.gen_int((M, K), -8, 8, M + K), WL.gen_int((N, K), -4, 4, N + K), WL.gen_int((M, N), -100, 100, M + N)
    Wd = torch.from_numpy(W).to(DEV)
    if wt == "bf16":
        Wd = Wd.to(torch.bfloat16)
    Xd, Cd = torch.from_numpy(X).to(DEV), torch.from_numpy(C).to(DEV).double()
    Y = torch.full((M, N), float("nan"), device=DEV)
    sp.masked_linear_fused_f64(Xd, Wd, Cd, sp.SPLITEE_MECH_NONE, 1.0, 1.0, 0, 0, Y=Y)
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), O.gemm64(X, W) - C)


@pytest.mark.parametrize("M,N,K", [(3, 300, 1032), (100, 3072, 1032)])
def test_f64_correction_of_every_tile(M, N, K):
    W = WL.gen_w(N, K, seed=4)
    Wd = torch.from_numpy(W).to(DEV).to(torch.bfloat16)
    C = sp.correction_f64(Wd, M, sp.SPLITEE_MECH_GAUSSIAN, 1e8, 1.0, 7, 9).cpu().numpy()
    eta = O.noise(M, K, O.MECH_GAUSSIAN, 1e8, 1.0, 7, 9, 0).astype(np.float64)
    want, scale = O.gemm64(eta, W), O.gemm64(np.abs(eta), np.abs(W))
    # K roundings on either side
    assert np.all(np.abs(C - want) <= 2 * K * 2.0 ** -53 * scale)
