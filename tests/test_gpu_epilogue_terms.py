"""Every epilogue term at once (asymmetric codes, weight zero points, low-rank
branch, bias) through the forms that stage them in their own way: K shared by
wave groups, single and in a grouped step, the other tiles of a step, and the
persistent walk over one layer and over lists.  Against the oracle's
definition, with the bar of the weight-quantizer tests: 1e-6 of the
dequantised terms' magnitude, the branch's eps, and 1e-12 of the summed
terms for the oracle's own fp64 sum."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_03057_amd as T
from paper_2608_03057_amd import inputs
from test_gpu_lowrank import branch, dev_bf16, eps_lr, lr_magnitude
from test_gpu_parity import DEV
from test_gpu_step_tiles import STEPS
from test_gpu_wquant import check_y, magnitude, quantize_w, term_abs

pytestmark = pytest.mark.gpu


class Operands:
    """One layer with every term: device operands and the oracle's inputs."""

    def __init__(self, seed, M, N, K):
        self.shape = (M, N, K)
        self.Qd, self.swd, self.zwd, self.Wc, self.sw, self.zw = quantize_w(
            inputs.weights_f32(seed, N, K))
        self.x, self.D, self.U = branch(seed + 1, M, K, 32 if seed % 2 else 16, N, "skewed")
        self.Xd, self.params, self.T = T.quantize_activations_lowrank(self.x.to(DEV),
                                                                      dev_bf16(self.D))
        self.alpha, self.z, Q = oracle.act_quant(self.x)
        self.Xc = (Q.astype(np.int16) - 128).astype(np.int8).reshape(M, K)
        self.bias = inputs.random_case(seed + 2, 1, N, 1)[3]
        self.terms = dict(act=self.params, colsums=T.weight_colsums(self.Qd),
                          lowrank=(self.T, dev_bf16(self.U)),
                          wzero=(self.zwd, T.row_sums(self.Xd)))
        self.biasd = self.bias.to(DEV)
        self.acc = torch.full((M, N), 12345, dtype=torch.int32, device=DEV)
        self.y = torch.full((M, N), -7.0, device=DEV)

    def layer(self):
        return T.make_layer(self.Xd, self.Qd, 0.0, self.swd, self.biasd, self.acc, self.y,
                            **self.terms)

    def check(self, b, where):
        M, N, K = self.shape
        # Whole tiles' edges and random entries of what the oracle would take
        # long over.
        rng = np.random.default_rng(M + N)
        rows, cols = np.arange(M), np.arange(N)
        if M * N * K > 1 << 30:
            rows = np.unique(np.concatenate([rows[::64], rows[63::64], [M - 1],
                                             rng.integers(0, M, 16)]))
            cols = np.unique(np.concatenate([cols[::32], cols[31::32], [N - 1],
                                             rng.integers(0, N, 16)]))
        Xc, Wc = self.Xc[rows], self.Wc[cols]
        sw, zw, bias = self.sw[cols], self.zw[cols], self.bias.numpy()[cols]
        ra, ry = oracle.layer_dequant(Xc, Wc, sw, b, act=(self.alpha, self.z), zw=zw, bias=bias)
        rr, cc = np.meshgrid(rows, cols, indexing="ij")
        idx = torch.as_tensor(rows, device=DEV), torch.as_tensor(cols, device=DEV)
        got = self.acc[idx[0]][:, idx[1]].cpu().numpy()
        assert np.array_equal(got, ra), where
        xr, Uc = self.x[torch.as_tensor(rows)], self.U[torch.as_tensor(cols)]
        _, lr64 = oracle.lowrank(xr, self.D, Uc)
        _, S = lr_magnitude(xr, self.D, Uc)
        R = oracle.row_sums(Xc) + K * (128.0 - self.z)
        corr = (128.0 - self.z) * oracle.weight_colsums(Wc)[b - 1].astype(np.float64)
        mag = magnitude(ra, self.alpha * sw.astype(np.float64), zw, R, corr, bias)
        check_y(self.y[idx[0]][:, idx[1]], ry + lr64, mag, where,
                eps_lr(K) * S + 1e-12 * term_abs(Xc, Wc, sw, b, 0.0, (self.alpha, self.z), zw))


# 64x64 tiles in four groups of waves and in two, 128x128 in two, the plain
# 64x64 and 128x128 tiles, the persistent walk of one to two tiles per
# workgroup (K of one K tile, of two, and several).
@pytest.mark.parametrize("M,N,K,tune", [
    (100, 130, 1152, None), (70, 33, 1153, None), (577, 1000, 1040, None),
    (1000, 900, 1153, None), (1500, 1400, 1904, None), (300, 200, 304, dict(tile=4)),
    (300, 200, 304, dict(tile=3)), (4130, 4100, 112, dict(tile=1)), (4130, 4100, 256, dict(tile=1)),
    (4000, 4000, 2064, None)])
def test_single(M, N, K, tune):
    o = Operands((M * 3 + N + K) % 30000, M, N, K)
    for b in (7, 2):
        T.masked_linear(o.Xd, o.Qd, 0.0, o.swd, b, o.biasd, acc=o.acc, y=o.y, tune=tune, **o.terms)
        torch.cuda.synchronize()
        o.check(b, f"{(M, N, K)} {tune} b={b}")


@pytest.mark.parametrize("form", STEPS)
def test_step(form):
    ops = [Operands(1700 + 10 * i, *s) for i, s in enumerate(STEPS[form])]
    layers = [o.layer() for o in ops]
    table = torch.tensor([[8, 3 + i] for i in range(len(ops))], dtype=torch.uint8)
    ws = torch.empty(T.schedule_workspace_bytes(layers), dtype=torch.uint8, device=DEV)
    T.run_schedule(layers, table, 2, 2, 0, 2, workspace=ws)
    torch.cuda.synchronize()
    for i, o in enumerate(ops):
        o.check(3 + i, f"{form} layer {i}")
