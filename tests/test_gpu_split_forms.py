"""The library's own choice of a split layer's tile and ranges, on both sides of
the rule, ragged: linear layers and a conv in 128x128 tiles (7, 8 and 2 ranges)
and in 256x256 tiles (12, 5 and 7).  Exact products in float64 on the GPU; fp32
within 1e-6 of the dequantised magnitude."""
import pytest
import torch

import paper_2608_03057_amd as T
from test_gpu_parity import DEV

pytestmark = pytest.mark.gpu
SX = 0.02


def operands(seed, *shapes):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return [torch.randint(-128, 128, s, generator=g, device=DEV, dtype=torch.int8) for s in shapes]


def check(acc, y, ra, sw, bias, where):
    assert torch.equal(acc, ra.to(torch.int32)), where
    main = ra * (SX * sw.double())
    tol = 1e-6 * (main.abs() + bias.double().abs())
    assert bool(((y.double() - (main + bias.double())).abs() <= tol).all()), where


def masked(W, b):
    step = 2 ** (8 - b)
    return (torch.div(W.int(), step, rounding_mode="floor") * step).double()


@pytest.mark.parametrize("M,N,K", [(1000, 1030, 16400), (500, 520, 8208), (1000, 1030, 32768),
                                   (2300, 1280, 11520)])
def test_linear(M, N, K):
    X, W = operands(M + K, (M, K), (N, K))
    sw, bias = torch.rand(N, device=DEV) * 0.01, torch.rand(N, device=DEV)
    ws = torch.empty(T.workspace_bytes(M, N, K), dtype=torch.uint8, device=DEV)
    for b in (8, 3):
        acc, y = T.masked_linear(X, W, SX, sw, b, bias, workspace=ws)
        torch.cuda.synchronize()
        check(acc, y, X.double() @ masked(W, b).T.contiguous(), sw, bias, f"{(M, N, K)} b={b}")


@pytest.mark.parametrize("H,Wd,C,N", [(33, 31, 960, 520), (60, 60, 928, 1000), (39, 41, 2560, 1280)])
def test_conv(H, Wd, C, N):
    X, W = operands(H * C, (H, Wd, C), (N, 3, 3, C))
    sw, bias = torch.rand(N, device=DEV) * 0.01, torch.rand(N, device=DEV)
    ws = torch.empty(T.workspace_bytes(H * Wd, N, 9 * C), dtype=torch.uint8, device=DEV)
    acc, y = T.masked_conv3x3(X, W, SX, sw, 5, bias, workspace=ws)
    torch.cuda.synchronize()
    pad = torch.zeros((H + 2, Wd + 2, C), dtype=torch.float64, device=DEV)
    pad[1:-1, 1:-1] = X.double()
    Wb = masked(W, 5)
    ra = sum(pad[r:r + H, c:c + Wd].reshape(H * Wd, C) @ Wb[:, r, c].T.contiguous()
             for r in range(3) for c in range(3))
    check(acc.reshape(-1, N), y.reshape(-1, N), ra, sw, bias, f"conv {(H, Wd, C, N)}")


@pytest.mark.parametrize("H,Wd,C,N", [(160, 131, 16, 1030), (96, 97, 48, 2500)])
def test_packed_conv_of_many_tiles(H, Wd, C, N):
    """More 256x256 tiles than compute units on packed weights: the sums of the
    rows' kernels."""
    X, W = operands(H + C, (H, Wd, C), (N, 3, 3, C))
    sw = torch.rand(N, device=DEV) * 0.01
    want, wy = T.masked_conv3x3(X, W, SX, sw, 6)
    acc, y = T.masked_conv3x3(X, None, SX, sw, 6, packed=T.pack_weights(W))
    torch.cuda.synchronize()
    assert torch.equal(acc, want)
    assert torch.allclose(y, wy, rtol=1e-6, atol=0.0)


# Packed layers of more than one 256x256 tile per compute unit, on each side of
# the lines between 256x256 and 128x256 tiles: a deep K with 144 tiles and with
# none in the last round, with 104, and K 2048 with 144.
@pytest.mark.parametrize("M,N,K", [(4990, 5000, 2064), (4000, 8190, 2192), (4990, 4600, 2064),
                                   (4990, 5000, 2048)])
def test_packed_linear_of_many_tiles(M, N, K):
    X, W = operands(M + K, (M, K), (N, K))
    sw = torch.rand(N, device=DEV) * 0.01
    acc, y = T.masked_linear(X, None, SX, sw, 6, packed=T.pack_weights(W))
    torch.cuda.synchronize()
    ra = X.double() @ masked(W, 6).double().T.contiguous()
    assert torch.equal(acc, ra.to(torch.int32))
    ref = ra * (SX * sw.double())
    assert bool(((y.double() - ref).abs() <= 1e-6 * ref.abs()).all())
