"""Integer sums alone (no y): the per-column factors of y need not be there.
Layers with act_params but neither colsums nor sw, through every form of the
GEMM, single and grouped; bit-exact against exact products."""
import pytest
import torch

import paper_2608_03057_amd as T
from paper_2608_03057_amd import inputs
from test_gpu_parity import DEV

pytestmark = pytest.mark.gpu


def exact(X, W, b):
    """int32 sums on the GPU: below 2^53 in float64."""
    step = 2 ** (8 - b)
    Wb = (torch.div(W.int(), step, rounding_mode="floor") * step).double()
    return (X.double() @ Wb.T.contiguous()).to(torch.int32)


def operands(M, N, K):
    X, W, _, _ = inputs.random_case(4100 + M + N, M, N, K)
    act = torch.tensor([0.03, 117.0], device=DEV)
    return X.to(DEV), W.to(DEV), act, torch.full((M, N), 12345, dtype=torch.int32, device=DEV)


def layer(X, W, act, acc, **kw):
    sw = torch.empty(W.shape[0], device=DEV)        # for its size
    d = T.make_layer(X, W, 1.0, sw, acc=acc, act=act, **kw)
    d.sw = None
    return d


# One layer without a workspace is launched as a single call: few tokens, K
# shared by four and by two wave groups, 64x64, 128x128 and 256x256 tiles; the
# packed and the plane kernels; byte-aligned rows.
@pytest.mark.parametrize("M,N,K,copy,tune", [
    (16, 70, 144, "rows", None), (100, 130, 1153, "rows", None), (577, 1000, 1040, "rows", None),
    (1500, 1400, 1904, "rows", None), (300, 200, 304, "rows", dict(tile=4)),
    (300, 200, 304, "rows", dict(tile=3)), (300, 600, 304, "rows", dict(tile=1)),
    (300, 200, 304, "rows", dict(tile=5)), (300, 200, 304, "packed", dict(packed_tile=7)),
    (300, 600, 304, "packed", dict(packed_tile=1)), (300, 200, 300, "planes", None)])
def test_single(M, N, K, copy, tune):
    X, W, act, acc = operands(M, N, K)
    kw = {}
    if copy != "rows":
        kw[copy] = T.pack_weights(W) if copy == "packed" else T.pack_planes(W)
    d = layer(X, W, act, acc, **kw)
    if copy != "rows":
        d.W = None
    T.run_schedule([d], torch.tensor([[5]], dtype=torch.uint8), 1, 1, 0, 1, tune=tune)
    torch.cuda.synchronize()
    assert torch.equal(acc, exact(X, W, 5))


# Steps in one launch: weight streams, two groups of 64x64 tiles, 64x64,
# 128x128, unit lists; one workgroup per tile and the persistent runs of the
# other tiles; packed weights, by tile and persistent.
@pytest.mark.parametrize("shapes,packed,tune", [
    ([(16, 70, 144), (9, 32, 1040)], False, None),
    ([(70, 130, 1168), (66, 200, 304)], False, None),
    ([(1000, 4608, 1152), (1000, 1100, 3088)], False, None),
    ([(1000, 4608, 1152), (1000, 1100, 3088), (1111, 4999, 1168)], False, None),
    ([(1500, 5000, 656), (2000, 4700, 656), (1500, 2100, 3088)], False, None),
    ([(300, 600, 304), (520, 260, 656)], False, dict(tile=1, persistent=1)),
    ([(300, 600, 304), (520, 260, 656)], False, dict(tile=2, persistent=2)),
    ([(300, 600, 304), (520, 260, 656)], True, dict(persistent=1)),
    ([(300, 600, 304), (520, 260, 656)], True, dict(persistent=2, persistent_wgs=1))])
def test_step(shapes, packed, tune):
    ops = [operands(*s) for s in shapes]
    copies = [dict(packed=T.pack_weights(W)) if packed else {} for _, W, _, _ in ops]
    layers = [layer(*o, **kw) for o, kw in zip(ops, copies)]
    for d in layers if packed else []:
        d.W = None
    table = torch.tensor([[3 + i] for i in range(len(layers))], dtype=torch.uint8)
    ws = torch.empty(T.schedule_workspace_bytes(layers), dtype=torch.uint8, device=DEV)
    T.run_schedule(layers, table, 1, 1, 0, 1, workspace=ws, tune=tune)
    torch.cuda.synchronize()
    for i, (X, W, _, acc) in enumerate(ops):
        assert torch.equal(acc, exact(X, W, 3 + i)), f"layer {i}"
