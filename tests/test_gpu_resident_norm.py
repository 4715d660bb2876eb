"""The power method around the steps of the kernel that holds W in registers.

Row counts on both sides of each step of rows per workgroup, column counts on both sides of each
4096-column chunk, one past the largest that fits, a workgroup count that leaves some without columns to
sum, few rounds and more.  Some run in registers and some streamed; test_gpu_norm_paths.py asserts which, and holds the
registers' results to the same bars.  Bars as in test_gpu_sensitivity.py.
"""
import numpy as np
import pytest
import torch

import oracle as O
import paper_2609_15039_amd as sp
import workloads as WL
from oracle import sensitivity as S
from tests.test_gpu_sensitivity import dev_w, first_round_bound, later_rounds_rtol, start_vector

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K,wd,iters", [
    (3, 16, "bf16", 8), (3, 16, "bf16", 7), (512, 4096, "bf16", 24), (513, 40, "bf16", 8), (1025, 40, "bf16", 8),
    (1024, 4096, "bf16", 23), (2049, 1000, "bf16", 8), (3073, 1032, "bf16", 24), (4097, 520, "bf16", 8),
    (5120, 264, "bf16", 8), (5121, 264, "bf16", 8), (10240, 136, "bf16", 8), (10241, 136, "bf16", 8),
    (513, 4104, "bf16", 24), (2560, 4104, "bf16", 8), (2561, 4104, "bf16", 8), (5120, 4104, "bf16", 8), (5121, 4104, "bf16", 8),
    (300, 8200, "bf16", 24), (3072, 8200, "bf16", 8), (3073, 8200, "bf16", 8), (2048, 12296, "bf16", 8),
    (5120, 512, "f32", 8), (5121, 512, "f32", 8), (2048, 4104, "f32", 24), (1024, 8200, "f32", 24)])
def test_rounds_match_oracle(N, K, wd, iters):
    print("N=%d K=%d %s" % (N, K, wd), flush=True)
    W = WL.gen_w(N, K, seed=N + K, dtype=wd)
    Wd, v0 = dev_w(W, wd), start_vector(K, 5, 6)
    sig, hist = sp.spectral_norm(Wd, iters, 5, 6, history=True)
    ref = S.power_iteration(W, v0, iters)
    assert sig == hist[-1]
    assert abs(hist[0] - ref[0]) <= first_round_bound(W, v0)
    np.testing.assert_allclose(hist, ref, rtol=later_rounds_rtol(W, ref[-1]), atol=0)
    assert sp.spectral_norm(Wd, iters, 5, 6, history=True)[1] == hist  # the same tree every time


@pytest.mark.parametrize("bits", [0x7F80, 0x7FC0, -1])  # infinity, NaN, the all-ones NaN
def test_a_value_that_is_no_number_ends_in_nan(bits):
    W = dev_w(WL.gen_w(600, 264, seed=3), "bf16")
    W.view(torch.int16)[17, 33] = bits
    assert np.isnan(sp.spectral_norm(W, 8, 1, 2))
