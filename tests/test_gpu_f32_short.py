"""The binary32 GEMM at small K under many tiles: 128 x 128 tiles, all of K in one accumulator chain.

Small integers make every sum exact, so the outputs must equal X W^T - C and X W^T bit for bit: K of one
to four whole 32-k tiles and with remainders, one past the limit, tile counts that these tiles take (512, 483,
1520) and two that they do not (460, 288), ragged rows and columns.
"""
import pytest
import torch

import paper_2609_15039_amd as sp

pytestmark = pytest.mark.gpu

DEV = "cuda"
F32 = sp.SPLITEE_PREC_F32


def _ints(shape, hi, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return torch.randint(-hi, hi + 1, shape, generator=g, device=DEV).float()


@pytest.mark.parametrize("wt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("M,N", [(2048, 4096), (2900, 2684), (1250, 19452), (2900, 2500), (1100, 4096)])
@pytest.mark.parametrize("K", [0, 8, 32, 40, 64, 104, 128, 136])
def test_small_k_is_exact(M, N, K, wt):
    print("M=%d N=%d K=%d %s" % (M, N, K, wt), flush=True)
    ld = max(K, 8)
    X, W, C = _ints((M, ld), 8, 1), _ints((N, ld), 4, 2).to(wt), _ints((M, N), 100, 3)
    want = X[:, :K].double() @ W[:, :K].double().T
    ws = sp.workspace(M, N, K, F32, gemm_only=True)
    Y, R = torch.full((M, N), float("nan"), device=DEV), torch.full((M, N), float("nan"), device=DEV)
    sp.splitee_masked_linear_unmask(X, F32, ld, W, sp._wtype(W), ld, C, N, Y, N, M, N, K, ws[0], ws[1])
    sp.splitee_masked_linear(X, F32, ld, W, sp._wtype(W), ld, R, N, M, N, K)
    assert torch.equal(Y.double(), want - C) and torch.equal(R.double(), want)


@pytest.mark.parametrize("K", [40, 128])
def test_infinities_and_nan_stay_in_their_rows_and_columns(K):
    M, N = 2900, 2684
    X, W = _ints((M, K), 8, 4), _ints((N, K), 4, 5)
    W[W == 0] = 1.0
    X[X == 0] = 1.0
    X[M - 1, K - 1], X[3, 0], W[N - 1, 5] = float("inf"), float("nan"), float("inf")
    R = torch.zeros((M, N), device=DEV)
    sp.splitee_masked_linear(X, F32, K, W, sp.SPLITEE_F32, K, R, N, M, N, K)
    bad = ~torch.isfinite(R)
    want = torch.zeros_like(bad)
    want[3], want[M - 1], want[:, N - 1] = True, True, True
    assert torch.equal(bad, want)
