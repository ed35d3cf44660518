"""The grouped step's forms as the library chooses them by cost: 64x64 tiles
with K shared by two wave groups, 64x64, 128x128 and 256x256 tiles walked from
lists of work units.  Layers of different depth and ragged sizes, so that
every list crosses from one layer to another and XCD rounds hold unequal
counts of tiles.  int32 against exact products, fp32 within 1e-6 of the
dequantised magnitude (at most four roundings of 2^-24 each)."""
import numpy as np
import pytest
import torch

import paper_2608_03057_amd as T
from paper_2608_03057_amd import inputs
from test_gpu_parity import DEV, check_outputs, f32

pytestmark = pytest.mark.gpu
SX = f32(0.02)

STEPS = {
    "64x64 in two groups": [(70, 130, 1168), (66, 200, 304), (130, 65, 2064)],
    "64x64": [(1000, 4608, 1152), (1000, 1100, 3088), (777, 2000, 656)],
    "128x128": [(1000, 4608, 1152), (1000, 1100, 3088), (777, 2000, 656), (1111, 4999, 1168),
                (900, 3456, 1152)],
    "lists": [(1500, 5000, 656), (2000, 4700, 656), (1500, 2100, 3088), (900, 4000, 1168)],
}


def build(shapes, lowrank=False):
    host, layers, keep = [], [], []
    for i, (M, N, K) in enumerate(shapes):
        X, W, sw, bias = inputs.random_case(9100 + 10 * i + M, M, N, K)
        bias = bias if i % 2 == 0 else None
        acc = torch.full((M, N), 12345, dtype=torch.int32, device=DEV)
        y = torch.full((M, N), -7.0, device=DEV)
        dev = [X.to(DEV), W.to(DEV), sw.to(DEV), None if bias is None else bias.to(DEV)]
        kw = {}
        if lowrank and i != 1:
            g = torch.Generator().manual_seed(i)
            up = (torch.randn((N, 16), generator=g) * 0.05).to(torch.bfloat16).to(DEV)
            kw["lowrank"] = (torch.randn((M, 16), generator=g).to(DEV), up)
        layers.append(T.make_layer(*dev[:2], SX, *dev[2:], acc, y, **kw))
        keep.append((dev, kw))
        host.append((X, W, sw, bias, acc, y))
    return host, layers, keep


def run(layers, table, ws):
    S = table.shape[1]
    T.run_schedule(layers, table, S, S, 0, S, workspace=ws)
    torch.cuda.synchronize()


@pytest.mark.parametrize("form", STEPS)
@pytest.mark.parametrize("noalloc", [False, True])
def test_step(form, noalloc):
    host, layers, keep = build(STEPS[form])
    table = torch.tensor([[3, 1 + 3 * i % 8] for i in range(len(layers))], dtype=torch.uint8)
    if noalloc:
        T.run_schedule_noalloc(layers, table, 2, 2, 0, 2)
        torch.cuda.synchronize()
    else:
        run(layers, table, torch.empty(T.schedule_workspace_bytes(layers), dtype=torch.uint8,
                                       device=DEV))
    for i, (X, W, sw, bias, acc, y) in enumerate(host):
        b = int(table[i, 1])
        step = 2 ** (8 - b)
        # Integer sums below 2^31: exact in float64.
        ra = X.double() @ (torch.div(W.int(), step, rounding_mode="floor") * step).double().T
        ra = ra.numpy().astype(np.int64)
        ry = ra * (np.float64(SX) * sw.numpy().astype(np.float64))
        if bias is not None:
            ry = ry + bias.numpy()
        check_outputs(acc, y, ra.astype(np.int32), ry, SX, sw, bias, f"{form} layer {i} b={b}")


@pytest.mark.parametrize("form", STEPS)
def test_step_lowrank(form):
    """With the low-rank branch, against the same layers launched one by one
    (each checked against the oracle elsewhere): the same integer sums, and
    fp32 outputs apart by a few roundings of terms of the outputs' size."""
    host, layers, keep = build(STEPS[form], lowrank=True)
    table = torch.tensor([[4, 2 + i] for i in range(len(layers))], dtype=torch.uint8)
    run(layers, table, None)
    want = [(acc.clone(), y.clone()) for _, _, _, _, acc, y in host]
    for _, _, _, _, acc, y in host:
        acc.fill_(12345)
        y.fill_(-7.0)
    run(layers, table, torch.empty(T.schedule_workspace_bytes(layers), dtype=torch.uint8,
                                   device=DEV))
    for i, ((a, f), h) in enumerate(zip(want, host)):
        assert torch.equal(a, h[4]), f"{form} layer {i}"
        assert torch.allclose(f, h[5], rtol=1e-6, atol=1e-6 * float(f.std())), f"{form} layer {i}"
