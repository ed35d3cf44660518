"""Grouped steps whose XCDs each take an eighth of every layer: many layers of
very different depth and of 1 to 40 tiles (fewer than XCDs in some, so that a
layer has no tile for some XCDs), in every form with one workgroup per tile, on
rows and packed weights, with convs beside them.  Integer sums bit-exact against
float64 products, every tile of every layer written."""
import pytest
import torch

import paper_2608_03057_amd as T
from test_gpu_parity import DEV

pytestmark = pytest.mark.gpu


def exact(X, W, b):
    step = 2 ** (8 - b)
    Wb = (torch.div(W.int(), step, rounding_mode="floor") * step).double()
    return (X.double() @ Wb.T.contiguous()).to(torch.int32)


def exact_conv(X, W, b):
    H, Wd, C = X.shape
    pad = torch.zeros((H + 2, Wd + 2, C), dtype=torch.int8, device=DEV)
    pad[1:-1, 1:-1] = X
    cols = torch.cat([pad[r:r + H, c:c + Wd].reshape(H * Wd, C) for r in range(3)
                      for c in range(3)], 1)
    return exact(cols, W.reshape(W.shape[0], -1), b).reshape(H, Wd, -1)


def build(L, convs, packed):
    g = torch.Generator(device=DEV).manual_seed(L)
    c = torch.Generator().manual_seed(L)

    def codes(*s):
        return torch.randint(-128, 128, s, generator=g, device=DEV, dtype=torch.int8)

    def pick(lo, hi):
        return int(torch.randint(lo, hi, (1,), generator=c))

    out = []
    for i in range(L):
        M, N = pick(65, 700), pick(3, 700)
        K = 16 * (pick(1, 20) if i % 3 else pick(100, 300))
        out.append([codes(M, K), codes(N, K), torch.empty((M, N), dtype=torch.int32, device=DEV)])
    for _ in range(convs):
        H, Wd, C, N = pick(8, 30), pick(9, 30), 16 * pick(1, 12), pick(3, 300)
        out.append([codes(H, Wd, C), codes(N, 3, 3, C),
                    torch.empty((H, Wd, N), dtype=torch.int32, device=DEV)])
    layers = []
    for X, W, acc in out:
        sw = torch.empty(W.shape[0], device=DEV)        # for its size: no y is asked for
        copy = T.pack_weights(W) if packed else None
        out[len(layers)].append(copy)
        layers.append(T.make_layer(X, W, 0.02, sw, acc=acc, packed=copy))
        layers[-1].sw = None
        if packed:
            layers[-1].W = None
    return out, layers


@pytest.mark.parametrize("L", [2, 9, 40])
@pytest.mark.parametrize("packed,convs,tune", [
    (False, 0, None), (False, 0, dict(tile=4, persistent=1)), (False, 0, dict(tile=3, persistent=1)),
    (False, 0, dict(tile=1, persistent=1)), (False, 3, None), (True, 0, dict(persistent=1)),
    (True, 0, dict(packed_tile=7, persistent=1)), (True, 3, None)])
def test_every_tile(L, packed, convs, tune):
    ops, layers = build(L, convs, packed)
    table = torch.tensor([[1 + i % 8] for i in range(len(layers))], dtype=torch.uint8)
    ws = torch.empty(T.schedule_workspace_bytes(layers), dtype=torch.uint8, device=DEV)
    for noalloc in (False, True):
        for o in ops:
            o[2].fill_(77)
        if noalloc:
            T.run_schedule_noalloc(layers, table, 1, 1, 0, 1, tune=tune)
        else:
            T.run_schedule(layers, table, 1, 1, 0, 1, workspace=ws, tune=tune)
        torch.cuda.synchronize()
        for i, (X, W, acc, _) in enumerate(ops):
            want = (exact_conv if X.dim() == 3 else exact)(X, W, 1 + i % 8)
            assert torch.equal(acc, want), f"layer {i} {tuple(X.shape)} noalloc={noalloc}"
