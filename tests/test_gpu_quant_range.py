"""The quantizers' two divisions (the five-operation one between 2^-60 and
2^60, the general one outside) and their clamp, where they can differ: inputs
scaled so that alpha lies on either side of both limits, denormal inputs
beside it, NaN and infinite inputs."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_03057_amd as T
from paper_2608_03057_amd import inputs
from test_gpu_act import quantize
from test_gpu_parity import DEV
from test_gpu_wquant import quantize_w

pytestmark = pytest.mark.gpu

# alpha = range / 255 (256): the limits lie between the neighbours.
SCALES = [-100, -70, -60, -55, -52, 0, 52, 55, 60, 62, 70, 100]


@pytest.mark.parametrize("e", SCALES)
@pytest.mark.parametrize("K", [515, 1152])
def test_activations(e, K):
    x = inputs.activations_f32(31, torch.arange(9), K, "skewed")
    x[2, 3:40] = torch.linspace(-1, 1, 37) * 1e-30      # quotients far below a step
    x = torch.ldexp(x, torch.tensor(e))
    x[4, 1], x[4, 2] = 1e-44, -1e-44
    quantize(x)


@pytest.mark.parametrize("e", SCALES)
@pytest.mark.parametrize("K", [515, 1152, 3001])
def test_weights(e, K):
    W = inputs.weights_f32(77, 12, K)
    W[1] = W[1].abs()                                   # one-sided rows: z near 0
    W[2] = -W[2].abs()
    W[3, 5:30] = torch.linspace(-1, 1, 25) * 1e-30
    W = torch.ldexp(W, torch.tensor(e))
    W[4, 1], W[4, 2] = 1e-44, -1e-44
    W[5] = W[5] - W[5].min()                            # minimum 0: z = 0
    quantize_w(W)


def fp32_codes(x, lo, hi, levels, rounding):
    """The definition in IEEE single precision on the CPU, NaN to code 0."""
    lo, hi = torch.tensor(lo), torch.tensor(hi)
    alpha = (hi - lo) / levels
    z = -lo / alpha
    q = torch.clamp(torch.nan_to_num(rounding(x / alpha + z), nan=0.0), 0, 255)
    return alpha, z, (q - 128).to(torch.int8)


@pytest.mark.parametrize("K", [130, 516])
def test_not_finite(K):
    """NaN is left out of the range and takes code 0; with an infinity in it
    the range, alpha and every code are those of the same arithmetic."""
    inf, nan = float("inf"), float("nan")
    for special in ([nan], [inf], [-inf], [nan, inf]):
        x = inputs.activations_f32(5, torch.arange(3), K, "skewed")
        flat = x.reshape(-1)
        for i, v in enumerate(special):
            flat[7 + 64 * i] = v
        num = flat[~torch.isnan(flat)]
        q, p = T.quantize_activations(x.to(DEV))
        torch.cuda.synchronize()
        alpha, z, want = fp32_codes(x, float(num.min()), float(num.max()), 255.0, torch.round)
        assert torch.equal(q.cpu(), want), special
        assert np.array_equal(p[:2].cpu().numpy(), torch.stack([alpha, z]).numpy(),
                              equal_nan=True), special
        W = inputs.weights_f32(9, 4, K)
        for i, v in enumerate(special):
            W[1, 5 + 64 * i] = v
        Q, a, zw, _ = T.quantize_weights(W.to(DEV))
        torch.cuda.synchronize()
        for n in range(4):
            num = W[n][~torch.isnan(W[n])]
            alpha, z, want = fp32_codes(W[n], float(num.min()), float(num.max()), 256.0,
                                        torch.floor)
            assert torch.equal(Q[n].cpu(), want), (special, n)
            assert np.array_equal(np.float32([a[n].item(), zw[n].item()]),
                                  np.float32([alpha.item(), z.item()]), equal_nan=True)
