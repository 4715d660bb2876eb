"""Workspace queries over the edges of their arguments, and the calls that ask them (no device needed)."""
import subprocess
import sys

import pytest

import paper_2609_15039_amd as sp


def test_empty_shapes_have_a_workspace_size():
    # in a process of its own: a division by zero would end it
    code = """
import itertools, paper_2609_15039_amd as sp
lib = sp.load()
for M, N, K, prec in itertools.product((0, 1, 5, 32, 200), (0, 8), (0, 64, 4096), (0, 1, 2)):
    g, f = lib.splitee_gemm_workspace_bytes(M, N, K, prec), lib.splitee_fused_workspace_bytes(M, N, K, prec)
    assert f >= g and (g == 0 if M == 0 or N == 0 else True), (M, N, K, prec, g, f)
    assert lib.splitee_masked_linear_unmask(256, prec, K, 256, 1, K, None, 0, 256, 8, M, 0, K, None, 0, None) == 0
    assert lib.splitee_masked_linear_unmask(256, prec, K, 256, 1, K, None, 0, 256, N, 0, N, K, None, 0, None) == 0
    lib.splitee_f64_workspace_bytes(M, N, K)
"""
    p = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True)
    assert p.returncode == 0, p.stderr


@pytest.mark.parametrize("prec", (sp.SPLITEE_PREC_F32, sp.SPLITEE_PREC_BF16X3))
def test_a_bank_workspace_serves_every_chunk(prec):
    # a bank is made in chunks of 256 rows and a shorter last one, which can need more than a whole one
    lib = sp.load()
    for K in (64, 256, 512, 1024, 2048, 4096, 9728):
        for N in (4, 256, 1000, 2560, 6144, 16384, 19456):
            size = lib.splitee_bank_workspace_bytes(K, N, prec)
            assert size % 4 == 0
            for rows in range(1, 257):
                assert lib.splitee_fused_workspace_bytes(rows, N, K, prec) + 256 * N * 4 <= size, (K, N, rows)
