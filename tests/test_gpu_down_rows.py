"""Down projection of the low-rank branch where its blocks change from 16 to
32 rows (more than 4096), with a last block of one row, K steps short of 32
and of the vector loads' 8, and more blocks than workgroups: the error bound
of the other down projection tests against the oracle, and the codes and
scale of the fused pass equal to the quantizer's alone."""
import pytest
import torch

import paper_2608_03057_amd as T
from test_gpu_lowrank import DEV, branch, check_T, dev_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,r", [(15, 40, 32), (17, 33, 16), (4096, 72, 32), (4097, 72, 16),
                                   (4112, 41, 32), (4130, 1032, 32), (16385, 16, 32)])
def test_down_rows(M, K, r):
    x, D, _ = branch((M * 7 + K) % 30011, M, K, r, 1)
    xd = x.to(DEV)
    check_T(T.lowrank_down(xd, dev_bf16(D)), x, D, f"down {M}x{K} r={r}")
    Q, p, Tq = T.quantize_activations_lowrank(xd, dev_bf16(D))
    Q1, p1 = T.quantize_activations(xd)
    torch.cuda.synchronize()
    check_T(Tq, x, D, f"fused {M}x{K} r={r}")
    assert torch.equal(Q, Q1) and torch.equal(p[:2], p1[:2]), f"fused {M}x{K}"
