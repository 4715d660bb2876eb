"""The streamed GEMM's last K tiles, whose masked input other waves load into LDS.

A split whose K tiles fill no whole turn of the kernel's ring ends in a shorter turn,
where fewer loads follow a tile's own and the wait for it counts differently.  One plane
spends the least time per tile, so it shows a short wait first.  Small integers
(|x| <= 8, |w| <= 4, K <= 9728) keep every partial sum below 2^24: the product is exact
in any summation order, and every repeat has to equal it bit for bit.
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
# M by plan (64-row tiles, 128-row tiles, a second row of tiles); K tiles 1 .. 5 without a split
# and, at the projections' widths, split K of every remainder
@pytest.mark.parametrize("M,N,K", [(40, 256, 64), (40, 256, 128), (100, 520, 320), (291, 2560, 4096), (291, 2560, 9728),
                                   (300, 3072, 3072), (200, 700, 1032)])
def test_last_k_tiles_are_complete(M, N, K, prec, layout):
    print("M=%d N=%d K=%d %s %s" % (M, N, K, prec, layout), flush=True)
    gp = PREC[prec]
    X, W = WL.gen_int((M, K), -8, 8, M + K), WL.gen_int((N, K), -4, 4, N + K)
    Wd = torch.from_numpy(W).to(DEV).to(torch.bfloat16)
    Wp = sp.tile_weights(Wd) if layout == "tiled" else Wd
    Xt = sp.mask(torch.from_numpy(X).to(DEV), torch.zeros((M, K), device=DEV), gp)
    want = torch.from_numpy(O.gemm64(X, W)).to(DEV)
    ws = sp.workspace(M, N, K, gp, gemm_only=True)
    bad = 0
    for _ in range(20):
        Y = torch.full((M, N), float("nan"), device=DEV)
        sp.masked_linear_unmask(Xt, gp, Wp, None, ws=ws, Y=Y)
        bad += int((Y.double() != want).sum())
    assert bad == 0, "%d of %d elements differ over 20 repeats" % (bad, 20 * M * N)
