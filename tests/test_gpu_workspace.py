"""One workspace, calls of different shapes and precisions in turn.

The decode kernels split K over workgroups that meet at counters in the workspace and expect them
to be zero.  Here calls that leave partial tiles or a masked input in the workspace (binary32 and
bfloat16, K split and not) come before K-split decode calls that launch nothing which would
clear the counters; each must give the bits that it gives with a fresh workspace.
"""
import pytest
import torch

import paper_2609_15039_amd as sp
import workloads as WL

pytestmark = pytest.mark.gpu

DEV = "cuda"
G = sp.SPLITEE_MECH_GAUSSIAN
F32, BF16, X3 = sp.SPLITEE_PREC_F32, sp.SPLITEE_PREC_BF16, sp.SPLITEE_PREC_BF16X3
# (M, N, K, precision): binary32 unsplit (K < 256) and split, streamed unsplit and split
BEFORE = [(40, 3000, 200, F32), (40, 500, 2048, F32), (200, 9000, 136, X3), (40, 3072, 3072, X3), (200, 640, 2056, BF16)]
# K-split decode calls: the skinny kernel (3 .. 16 rows) and, on tiled W, the GEMV (1 row)
DECODE = [(4, 2560, 4096, X3, "rows"), (16, 2560, 4096, X3, "tiled"), (1, 2560, 4096, X3, "tiled"), (5, 700, 2048, BF16, "tiled")]


def _layer(M, N, K, seed, layout="rows"):
    W = torch.from_numpy(WL.gen_w(N, K, seed=seed)).to(DEV).to(torch.bfloat16)
    X = torch.from_numpy(WL.gen_x(M, K, seed=seed + 1)).to(DEV)
    return X, sp.tile_weights(W) if layout == "tiled" else W


def _decode(M, N, K, prec, layout, ws):
    X, W = _layer(M, N, K, 7, layout)
    eta = sp.noise(M, K, G, 100.0, 1.0, 3, 4)
    C = torch.zeros((M, N), device=DEV)
    out = []
    for call in (lambda Y: sp.masked_linear_fused(X, W, C, G, 100.0, 1.0, 3, 4, prec=prec, eta_override=eta, ws=ws, Y=Y),
                 lambda Y: sp.masked_linear_unmask(sp.mask(X, eta, prec), prec, W, C, ws=ws, Y=Y)):
        out.append(call(torch.full((M, N), float("nan"), device=DEV)))
    return out


@pytest.mark.parametrize("before", BEFORE)
@pytest.mark.parametrize("decode", DECODE)
def test_decode_after_a_call_of_another_shape(decode, before):
    print(decode, before, flush=True)
    M, N, K, prec, layout = decode
    want = _decode(M, N, K, prec, layout, None)
    assert all(bool(torch.isfinite(y).all()) for y in want)
    m, n, k, p = before
    X, W = _layer(m, n, k, 11)
    need = max(sp.splitee_fused_workspace_bytes(m, n, k, p), sp.splitee_fused_workspace_bytes(M, N, K, prec))
    ws = torch.zeros(need + 256, dtype=torch.uint8, device=DEV)
    ws = (ws[-ws.data_ptr() % 256:][:need], need)
    C = torch.zeros((m, n), device=DEV)
    for first in (lambda: sp.masked_linear_fused(X, W, C, G, 100.0, 1.0, 3, 4, prec=p, ws=ws),
                  lambda: sp.masked_linear_unmask(sp.mask(X, torch.zeros_like(X), p), p, W, C, ws=ws)):
        first()
        for got, y in zip(_decode(M, N, K, prec, layout, ws), want):
            assert torch.equal(got, y)
