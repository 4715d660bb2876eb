"""Which kernels a spectral norm takes, and that the rounds of one that gives up are run again.

W held in registers on either side of its limits of rows, columns and rounds, among them workgroup counts
whose sums take more than 64 KB of LDS.  A poll bound of no tries (set by the caller: every workgroup
leaves normally) makes that kernel give up; the result must then be the streamed kernels', whose first
rounds a shorter, streamed call gives bit for bit.
"""
import numpy as np
import pytest
import torch

import paper_2609_15039_amd as sp
import workloads as WL
from oracle import sensitivity as S
from tests.test_gpu_sensitivity import first_round_bound, later_rounds_rtol, start_vector

pytestmark = pytest.mark.gpu

STREAMED, RESIDENT, GAVE_UP = sp.SPLITEE_PATH_STREAMED, sp.SPLITEE_PATH_RESIDENT, sp.SPLITEE_PATH_GAVE_UP


def norm(N, K, wd, iters, spins=-1, W=None):
    W = torch.from_numpy(WL.gen_w(N, K, seed=N + K, dtype=wd) if W is None else W).cuda()
    if wd == "bf16":
        W = W.to(torch.bfloat16)
    ws = sp._aligned_bytes(sp.splitee_spectral_norm_workspace_bytes(N, K, iters), "cuda")
    return sp.splitee_spectral_norm_probe(W, sp._wtype(W), K, N, K, iters, 5, 6, ws, ws.numel(), spins)


@pytest.mark.parametrize("N,K,wd,iters,path", [
    (4, 16, "bf16", 8, RESIDENT), (8192, 3072, "bf16", 8, RESIDENT), (8192, 3072, "bf16", 7, STREAMED),
    (10240, 136, "bf16", 8, RESIDENT), (10241, 136, "bf16", 8, STREAMED), (768, 3072, "bf16", 38, RESIDENT),
    (768, 3072, "bf16", 37, STREAMED), (5120, 4104, "bf16", 8, RESIDENT), (5121, 4104, "bf16", 8, STREAMED),
    (3072, 8200, "bf16", 8, RESIDENT), (3073, 8200, "bf16", 8, STREAMED), (2048, 12296, "bf16", 24, RESIDENT),
    (2048, 16384, "bf16", 24, RESIDENT), (1600, 16384, "bf16", 24, RESIDENT), (2049, 16384, "bf16", 24, STREAMED),
    (5120, 512, "f32", 12, RESIDENT), (5121, 512, "f32", 12, STREAMED), (2048, 4104, "f32", 24, RESIDENT),
    (2049, 4104, "f32", 24, STREAMED),
    # few rows of many columns: a workgroup sums too many of them (held in registers these took 1.04 to 7 times as long)
    (16, 16384, "bf16", 40, STREAMED), (16, 1024, "f32", 40, STREAMED), (64, 4096, "bf16", 64, STREAMED),
    (512, 4096, "bf16", 24, STREAMED), (512, 9728, "bf16", 40, STREAMED), (1024, 9728, "f32", 40, STREAMED)])
def test_path(N, K, wd, iters, path):
    print("N=%d K=%d %s %d rounds" % (N, K, wd, iters), flush=True)
    assert norm(N, K, wd, iters)[0] == path


# every count of rows per workgroup, by column chunks of 4096 and type, at an edge of its rows or columns
@pytest.mark.parametrize("N,K,wd,iters", [
    (512, 1024, "bf16", 8), (1024, 4096, "bf16", 32), (1025, 40, "bf16", 8), (2049, 1000, "bf16", 8), (3073, 1032, "bf16", 8),
    (10240, 136, "bf16", 8), (1024, 8192, "bf16", 24), (1536, 4104, "bf16", 17), (2048, 4104, "bf16", 13),
    (2561, 4104, "bf16", 10), (1024, 8200, "bf16", 24), (3072, 8200, "bf16", 8), (2048, 12296, "bf16", 8),
    (512, 1024, "f32", 24), (1024, 4096, "f32", 36), (1025, 520, "f32", 20), (5120, 512, "f32", 8), (2048, 4104, "f32", 24)])
def test_rounds_in_registers_match_oracle(N, K, wd, iters):
    print("N=%d K=%d %s %d rounds" % (N, K, wd, iters), flush=True)
    W, v0 = WL.gen_w(N, K, seed=N + K, dtype=wd), start_vector(K, 5, 6)
    path, hist = norm(N, K, wd, iters, W=W)
    ref = S.power_iteration(W, v0, iters)
    assert path == RESIDENT
    assert abs(hist[0] - ref[0]) <= first_round_bound(W, v0)
    np.testing.assert_allclose(hist, ref, rtol=later_rounds_rtol(W, ref[-1]), atol=0)


@pytest.mark.parametrize("N,K,wd", [(2048, 1000, "bf16"), (8192, 3072, "bf16"), (5000, 512, "f32")])
def test_a_kernel_that_gives_up_is_run_again_streamed(N, K, wd):
    print("N=%d K=%d %s" % (N, K, wd), flush=True)
    path, streamed = norm(N, K, wd, 7)
    assert path == STREAMED
    path, h = norm(N, K, wd, 16, spins=0)
    assert path == GAVE_UP and h[:7] == streamed
    path, h = norm(N, K, wd, 16)
    assert path == RESIDENT and h == pytest.approx(norm(N, K, wd, 16, spins=0)[1], rel=1e-6)
