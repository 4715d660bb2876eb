"""The binary64 GEMM adds at most 128 k in one accumulator chain, also where K is not split.

X is 2^53 at one k and 1 elsewhere, W is ones, C takes 2^53 off again: next to 2^53 a 1 is lost (the spacing
of binary64 there is 2), so a row keeps the ones of every chain but that of the 2^53, which other chains
sum exactly before they are added, with a rounding of 1 at most per chain added.
"""
import pytest
import torch

import paper_2609_15039_amd as sp

pytestmark = pytest.mark.gpu

CHAIN = 128


@pytest.mark.parametrize("wt", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("M", [1, 32, 48, 64])  # 16384 columns are whole rounds of 256 tiles at any height
@pytest.mark.parametrize("K,at", [(520, 0), (1024, 300), (136, 135)])
def test_only_the_chain_of_the_large_term_loses_its_ones(M, K, at, wt):
    print("M=%d K=%d at=%d %s" % (M, K, at, wt), flush=True)
    N = 16384
    X, W = torch.ones((M, K), device="cuda"), torch.ones((N, K), device="cuda", dtype=wt)
    X[:, at] = 2.0 ** 53
    C = torch.full((M, N), 2.0 ** 53, device="cuda", dtype=torch.float64)
    Y = sp.masked_linear_fused_f64(X, W, C, sp.SPLITEE_MECH_NONE, 1.0, 1.0, 0, 0)
    chains = -(-K // 96)  # the shortest chains
    assert float(Y.min()) >= K - CHAIN - chains, float(Y.min())
    assert float(Y.max()) <= K - 1 + chains
