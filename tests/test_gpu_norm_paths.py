"""Which kernels a spectral norm takes, and that the rounds of one that gives up are run again.

W held in registers on either side of its limits of rows, columns and rounds, among them workgroup counts
whose sums take more than 64 KB of LDS.  A poll bound of no tries (set by the caller: every workgroup
leaves normally) makes that kernel give up; the result must then be the streamed kernels', whose first
rounds a shorter, streamed call gives bit for bit.
"""
import pytest
import torch

import paper_2609_15039_amd as sp
import workloads as WL

pytestmark = pytest.mark.gpu

STREAMED, RESIDENT, GAVE_UP = sp.SPLITEE_PATH_STREAMED, sp.SPLITEE_PATH_RESIDENT, sp.SPLITEE_PATH_GAVE_UP


def norm(N, K, wd, iters, spins=-1):
    W = torch.from_numpy(WL.gen_w(N, K, seed=N + K, dtype=wd)).cuda()
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


@pytest.mark.parametrize("N,K,wd", [(2048, 1000, "bf16"), (8192, 3072, "bf16"), (5000, 512, "f32")])
def test_a_kernel_that_gives_up_is_run_again_streamed(N, K, wd):
    print("N=%d K=%d %s" % (N, K, wd), flush=True)
    path, streamed = norm(N, K, wd, 7)
    assert path == STREAMED
    path, h = norm(N, K, wd, 16, spins=0)
    assert path == GAVE_UP and h[:7] == streamed
    path, h = norm(N, K, wd, 16)
    assert path == RESIDENT and h == pytest.approx(norm(N, K, wd, 16, spins=0)[1], rel=1e-6)
