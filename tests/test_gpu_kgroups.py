"""Single layers whose K range is shared by groups of waves, and the single
persistent walk, through the library's own choice, at the sizes where its
rules change and where groups run out of K tiles, and the walk forced on short
K: int32 bit-exact and fp32 within 1e-6 of the dequantised magnitude against
the oracle, with a bias, and a low-rank branch on some."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_03057_amd as T
from paper_2608_03057_amd import inputs
from test_gpu_bytealign import shifted
from test_gpu_parity import DEV, check_outputs, f32

pytestmark = pytest.mark.gpu
SX = f32(0.02)


def rows_cols(M, N, K, seed):
    X, W, sw, bias = inputs.random_case(seed, M, N, K)
    X[0, 0], W[0, 0] = -128, -128
    return X, W, sw, bias


# Four groups of 64x64 tiles (fewer K tiles than 4, a last group without any,
# ragged K), two groups of 64x64, two of 128x128 (an odd number of K tiles).
@pytest.mark.parametrize("M,N,K", [
    (65, 40, 900), (66, 70, 1024), (100, 130, 1153), (128, 64, 1280), (70, 33, 1168),
    (577, 1000, 1040), (1000, 900, 1153), (1500, 1400, 1904), (1664, 1280, 1793)])
def test_groups(M, N, K):
    X, W, sw, bias = rows_cols(M, N, K, 8100 + M)
    for b, off in ((8, 0), (3, 1)):
        Xd, Wd = shifted(X, off), shifted(W, off)
        acc, y = T.masked_linear(Xd, Wd, SX, sw.to(DEV), b, bias.to(DEV))
        torch.cuda.synchronize()
        ra, ry = oracle.masked_linear(X, W, SX, sw, b, bias)
        check_outputs(acc, y, ra, ry, SX, sw, bias, f"{(M, N, K)} b={b}")


@pytest.mark.parametrize("H,Wd,C,N", [(9, 8, 130, 65), (18, 25, 128, 100), (30, 20, 128, 640),
                                      (40, 52, 256, 1280)])
def test_groups_conv(H, Wd, C, N):
    X = inputs.random_case(8200 + H, H * Wd, 1, C)[0].reshape(H, Wd, C)
    _, W, sw, bias = inputs.random_case(8300 + C, 1, N, 9 * C)
    W = W.reshape(N, 3, 3, C)
    acc, y = T.masked_conv3x3(X.to(DEV), W.to(DEV), SX, sw.to(DEV), 5, bias.to(DEV))
    torch.cuda.synchronize()
    ra, ry = oracle.conv3x3(X, W, SX, sw, 5, bias)
    check_outputs(acc.reshape(-1, N), y.reshape(-1, N), np.asarray(ra).reshape(-1, N),
                  np.asarray(ry).reshape(-1, N), SX, sw, bias, f"conv {(H, Wd, C, N)}")


# Ragged in every size: the walk at the fewest tiles that take it (144, level
# with 128x128 by the estimates, 20.6 us against 20.2), 128x128 (29.6 us against
# the walk's 41.3, 37.4 / 44.0), nearly level (94.4 / 95.1), and the walk with
# one tile per workgroup (31.5 / 47.1) and with three (61.9 / 80.5), the XCDs'
# runs of unequal length.
@pytest.mark.parametrize("M,N,K", [(2300, 4000, 1152), (4100, 4090, 1040), (8200, 2305, 1168),
                                   (12000, 2816, 2064), (4000, 4000, 2064), (4200, 11100, 1040)])
@pytest.mark.parametrize("extras", [False, True])
def test_single_walk(M, N, K, extras):
    X, W, sw, bias = rows_cols(M, N, K, 8400 + M)
    kw = {}
    if extras:
        g = torch.Generator().manual_seed(M)
        Tl = torch.randn((M, 16), generator=g)
        U = (torch.randn((N, 16), generator=g) * 0.25).to(torch.bfloat16)
        kw = dict(lowrank=(Tl.to(DEV), U.to(DEV)))
    acc, y = T.masked_linear(X.to(DEV), W.to(DEV), SX, sw.to(DEV), 6, bias.to(DEV), **kw)
    torch.cuda.synchronize()
    rng = np.random.default_rng(M)
    # every tile's corners and random entries: rows x columns
    rows = np.unique(np.concatenate([np.arange(0, M, 256), np.arange(255, M, 256), [M - 1],
                                     rng.integers(0, M, 8)]))
    cols = np.unique(np.concatenate([np.arange(0, N, 256), np.arange(255, N, 256), [N - 1],
                                     rng.integers(0, N, 8)]))
    rr, cc = np.meshgrid(rows, cols, indexing="ij")
    Wb = torch.floor(W[cols].double() / 4) * 4
    ra = (X[rows].double() @ Wb.T).numpy()
    assert np.array_equal(acc.cpu().numpy()[rr, cc], ra.astype(np.int64))
    ref = ra * SX * sw.numpy().astype(np.float64)[cols] + bias.numpy().astype(np.float64)[cols]
    mag = np.abs(ra * SX * sw.numpy().astype(np.float64)[cols]) + np.abs(bias.numpy()[cols])
    tol = 1e-6 * mag
    if extras:
        # T enters as two bfloat16 parts (2^-16 of each term) and the rank-16
        # sum rounds in fp32.
        t, u = Tl[rows].double(), U[cols].double()
        ref = ref + (t @ u.T).numpy()
        tol = tol + (2.0 ** -16 + 70 * 2.0 ** -24) * (t.abs() @ u.abs().T).numpy()
    assert np.all(np.abs(y.cpu().numpy().astype(np.float64)[rr, cc] - ref) <= tol)


# The walk over two tiles per workgroup (17 x 17 of 256x256) where the stages
# and register slots turn over within a tile: one K tile, short and whole, two
# and three, with and without a remainder.  Every entry, on the GPU in float64.
@pytest.mark.parametrize("K", [16, 128, 144, 256, 272, 400])
@pytest.mark.parametrize("M,N", [(4130, 4100), (8200, 2305)])
def test_forced_walk(M, N, K):
    X, W, sw, bias = (t.to(DEV) for t in rows_cols(M, N, K, 8500 + K))
    for b in (8, 3):
        acc, y = T.masked_linear(X, W, SX, sw, b, bias, tune=dict(tile=1))
        torch.cuda.synchronize()
        step = 2 ** (8 - b)
        Wb = (torch.div(W.int(), step, rounding_mode="floor") * step).double()
        ra = X.double() @ Wb.T.contiguous()
        assert torch.equal(acc, ra.to(torch.int32)), f"K={K} b={b}"
        main = ra * (SX * sw.double())
        tol = 1e-6 * (main.abs() + bias.double().abs())
        assert bool(((y.double() - (main + bias.double())).abs() <= tol).all()), f"K={K} b={b}"
