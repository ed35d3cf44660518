"""Schedules under graph capture: layer lists short enough for one upload
launch and too long for two (which outside a capture are copied from host
memory that does not outlive the call), with a workspace and without.  Several
replays, the inputs changed and the host's heap reused in between, each
against the eager call."""
import pytest
import torch

import paper_2608_03057_amd as T
from paper_2608_03057_amd import inputs
from test_gpu_parity import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [3, 60])
@pytest.mark.parametrize("M", [5, 70])
@pytest.mark.parametrize("noalloc", [False, True])
def test_replays(L, M, noalloc):
    S = 2
    ops, layers = [], []
    for i in range(L):
        X, W, sw, _ = inputs.random_case(6000 + i, M, 32 + 16 * (i % 3), 128 + 16 * (i % 2))
        d = [X.to(DEV), W.to(DEV), sw.to(DEV)]
        d.append(torch.empty((M, W.shape[0]), dtype=torch.int32, device=DEV))
        ops.append(d)
        layers.append(T.make_layer(d[0], d[1], 0.02, d[2], acc=d[3]))
    table = torch.tensor([[1 + i % 8, 1 + (i + 3) % 8] for i in range(L)], dtype=torch.uint8)
    ws = torch.empty(T.schedule_workspace_bytes(layers), dtype=torch.uint8, device=DEV)

    def step():
        if noalloc:
            T.run_schedule_noalloc(layers, table, S, S, 0, S)
        else:
            T.run_schedule(layers, table, S, S, 0, S, workspace=ws)

    step()                              # kernels loaded, the scratch array looked up
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for r in range(4):
        junk = [torch.full((n,), 255, dtype=torch.uint8) for n in (1 << 10, 1 << 13, 1 << 14)] * 50
        for d in ops:
            d[0].copy_(torch.roll(d[0], 1, 1))
        step()
        want = [d[3].clone() for d in ops]
        for d in ops:
            d[3].fill_(-1)
        ws.fill_(255)
        graph.replay()
        torch.cuda.synchronize()
        for i, (d, w) in enumerate(zip(ops, want)):
            assert torch.equal(d[3], w), f"replay {r} layer {i}"
        del junk
