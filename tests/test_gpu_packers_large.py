"""Packers at sizes past 32-bit offsets, against the oracle on slices: rows so
long that 32 of them pass 2 GiB (tasq_pack_planes takes any K), with channels
missing from the last block and rows at an odd address, and so many rows that
a packer takes more than one launch."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_03057_amd as T
from test_gpu_parity import DEV

pytestmark = pytest.mark.gpu


def weight(N, K, off=0):
    g = torch.Generator(device=DEV).manual_seed(N + K)
    buf = torch.randint(-128, 128, (N * K + off + 64,), generator=g, device=DEV,
                        dtype=torch.int8)
    return buf[off:off + N * K].view(N, K)


# 2^26 - 1 is the last K whose 32 rows a 2 GiB window holds.  From K = 69273667
# on, 31 rows pass 2 GiB; at 2^27 the bytes of 32 rows are 0 modulo 2^32.
@pytest.mark.parametrize("N,K,off", [(32, (1 << 26) - 1, 0), (33, 1 << 26, 1),
                                     (31, 69273667 + 130, 3), (32, 1 << 27, 0)])
def test_planes_of_long_rows(N, K, off):
    W = weight(N, K, off)
    NB, KB = (N + 31) // 32, (K + 127) // 128
    planes = T.pack_planes(W)
    torch.cuda.synchronize()
    planes = planes.view(NB, 8, KB, 128)
    blocks = sorted({0, 1, KB // 3, KB // 2, KB - 2, KB - 1})
    for kb in blocks:
        got = planes[:, :, kb].contiguous().cpu().numpy().view(np.uint32)
        want = np.asarray(oracle.pack_planes(W[:, 128 * kb:128 * (kb + 1)].contiguous().cpu()))
        assert np.array_equal(got.reshape(-1), want.view(np.uint32).reshape(-1)), (N, K, kb)


# 2^22 blocks of 32 rows fill one launch.
@pytest.mark.parametrize("pack", ["planes", "weights"])
def test_many_rows(pack):
    N, K = (1 << 27) + 32 + 7, 3
    W = weight(N, K, 1)
    NB = (N + 31) // 32
    out = (T.pack_planes if pack == "planes" else T.pack_weights)(W)
    torch.cuda.synchronize()
    out = out.view(torch.uint8).view(NB, 4096)
    for nb in (0, 1, (1 << 22) - 1, 1 << 22, NB - 1):
        rows = W[32 * nb:32 * nb + 32].contiguous().cpu()
        want = (oracle.pack_planes if pack == "planes" else oracle.pack_weights)(rows)
        want = np.ascontiguousarray(np.asarray(want)).view(np.uint8).reshape(-1)
        assert np.array_equal(out[nb].cpu().numpy(), want), (pack, nb)
