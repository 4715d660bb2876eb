"""Banks whose last, short chunk needs more workspace than a whole one."""
import pytest
import torch

import paper_2609_15039_amd as sp
import workloads as WL

pytestmark = pytest.mark.gpu

G = sp.SPLITEE_MECH_GAUSSIAN


# one whole chunk, then 160 rows (binary32) and 64 (three planes) whose K is split
@pytest.mark.parametrize("N,K,rows,prec", [(19456, 512, 416, sp.SPLITEE_PREC_F32), (19456, 1024, 320, sp.SPLITEE_PREC_BF16X3)])
def test_bank_with_a_short_last_chunk(tmp_path, N, K, rows, prec):
    W = torch.from_numpy(WL.gen_w(N, K, seed=2)).cuda().to(torch.bfloat16)
    path = str(tmp_path / "bank.spb")
    sp.bank_create(path, W, K, G, 1.0, 1.0, 0, 5, 0, rows, prec)
    bank = sp.splitee_bank_open(path)
    got = torch.empty((rows, N), device="cuda")
    sp.splitee_bank_load(bank, rows, got, N, True)
    sp.splitee_bank_close(bank)
    assert torch.equal(got[:256], sp.correction(W, 256, G, 1.0, 1.0, 0, 5, 0, prec))
    assert torch.equal(got[256:], sp.correction(W, rows - 256, G, 1.0, 1.0, 0, 5, 256, prec))
