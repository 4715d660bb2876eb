"""splitee_masked_linear at few tokens: K split over the waves of a workgroup.

Small integers keep every partial sum exact, so the product must equal X W^T bit for bit
whatever the tile: fewer K tiles than waves, an odd and an even number of them per wave, ragged
K and N, one to several 16-row tiles, and widths that take every column count per workgroup.
The same sizes through the row-major GEMV (1-2 rows) and past the row limit.
"""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2609_15039_amd as sp
import workloads as WL

pytestmark = pytest.mark.gpu

DEV = "cuda"
PREC = {"bf16": sp.SPLITEE_PREC_BF16, "bf16x3": sp.SPLITEE_PREC_BF16X3}


@pytest.mark.parametrize("layout", ["row", "tiled"])
@pytest.mark.parametrize("prec", ["bf16", "bf16x3"])
@pytest.mark.parametrize("M,N,K", [(1, 17, 8), (2, 40, 72), (3, 4, 520), (15, 3072, 1032), (16, 5000, 2048), (17, 33, 4096),
                                   (33, 9000, 648), (48, 17000, 264), (64, 6200, 1096), (100, 1000, 8192), (128, 3072, 1544),
                                   (129, 640, 1032), (2, 256, 20488)])
def test_product_is_exact(M, N, K, prec, layout):
    print("M=%d N=%d K=%d %s %s" % (M, N, K, prec, layout), flush=True)
    gp = PREC[prec]
    X, W = WL.gen_int((M, K), -8, 8, M + K), WL.gen_int((N, K), -4, 4, N + K)
    Wd = torch.from_numpy(W).to(DEV).to(torch.bfloat16)
    Wp = sp.tile_weights(Wd) if layout == "tiled" else Wd
    Xt = sp.mask(torch.from_numpy(X).to(DEV), torch.zeros((M, K), device=DEV), gp)
    ld = -(-N // 4) * 4
    R = torch.full((M, ld), float("nan"), device=DEV)
    sp.splitee_masked_linear(Xt, gp, K, Wp, sp._wtype(Wp), K, R, ld, M, N, K)
    got = R.cpu().numpy()
    assert np.array_equal(got[:, :N].astype(np.float64), O.gemm64(X, W))
    assert np.isnan(got[:, N:]).all()  # nothing past column N is written
