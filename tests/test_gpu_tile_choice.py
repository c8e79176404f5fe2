"""The fused GEMMs at the sizes where the tile choice and the small-tile kernel can go wrong: every tile of the choice with
ragged last tiles, contractions around the depth of the load ring (none, one short, exactly, one more whole step; with and
without a tail), segments that straddle tiles, ranks that need one or two passes and ranks that are not multiples of 8."""
import numpy as np
import pytest
import torch

from oracle import multilora_oracle as orc
from paper_2604_05426_amd import workloads as wl
from paper_2604_05426_amd.harness import DeviceLayer, to_host
from util import rel_fro, row_rel_max

pytestmark = pytest.mark.gpu

RANKS, SCALES = (8, 0, 128, 33, 70, 16), (2.0, 1.0, 0.25, 0.5, 1.0, 3.0)

# tokens, k, n: the forward contracts over k, the backward over n
SHAPES = [(70, 40, 72), (130, 64, 448), (230, 512, 136), (333, 576, 584),             # 64 x 64 tiles; ring of 8 stages
          (1100, 320, 1096), (1100, 384, 1096), (1100, 456, 1096), (1100, 1096, 392),   # 64 x 128; ring of 6
          (2900, 256, 1096), (2900, 328, 1096), (2900, 384, 1096), (2900, 1096, 328),   # 128 x 128; ring of 5
          (8100, 72, 2048), (8100, 2048, 64),                                         # 256 x 256 forward / backward
          (6900, 72, 1800), (6900, 1800, 72)]                                         # the same, fewer tiles than CUs


@pytest.mark.parametrize("T,k,n", SHAPES)
def test_every_tile_against_the_oracle(T, k, n):
    cuts = [0.0, 0.21, 0.22, 0.6, 0.6, 0.93, 1.0]
    off = [int(T * c) for c in cuts]
    w = wl.make_workload(f"tiles_{T}_{k}_{n}", "bf16", k, n, RANKS, [b - a for a, b in zip(off, off[1:])], SCALES, seed=k + n, b_sigma=0.3)
    dl = DeviceLayer(w)
    print(f"[case] tiles T={T} k={k} n={n}", flush=True)
    dl.forward(); dl.backward(); dl.sync()
    fw = orc.forward(w.X, w.W, w.A, w.B, w.scales, w.offsets)
    bw = orc.backward(w.dY, w.X, w.W, w.A, w.B, w.scales, w.offsets)
    for got, want in ((dl.Y, fw.Y), (dl.dX, bw.dX)):       # one bf16 rounding of the result and of S / dS: 1.7e-3 .. 2.4e-3
        assert rel_fro(to_host(got), want) <= 1e-2 and row_rel_max(to_host(got), want) <= 1e-2
    for i in range(w.N):
        assert rel_fro(to_host(dl.dA[i]), bw.dA[i]) <= 1e-2 and rel_fro(to_host(dl.dB[i]), bw.dB[i]) <= 1e-2
    dl.plan.destroy()


@pytest.mark.parametrize("T,k,n", [(230, 512, 136), (1100, 328, 1096), (2900, 328, 1096), (2900, 1096, 328), (8100, 72, 2048), (8100, 2048, 64)])
def test_a_diverged_adapter_stays_out_of_its_neighbours_tiles(T, k, n):
    off = [0, T // 3 + 5, 2 * T // 3 + 9, T]
    w = wl.make_workload("diverged", "bf16", k, n, (8, 100, 16), [b - a for a, b in zip(off, off[1:])], (2.0, 0.5, 1.0), seed=5, b_sigma=0.3)
    dl = DeviceLayer(w)
    print(f"[case] diverged T={T} k={k} n={n}", flush=True)
    dl.forward(); dl.backward(); dl.sync()
    Y, dX = dl.Y.clone(), dl.dX.clone()
    keep = torch.ones(T, dtype=torch.bool, device=Y.device)
    keep[off[1]:off[2]] = False
    dl.B[1][70, 3] = float("inf")
    dl.A[1][5, 40] = float("nan")
    dl.forward(); dl.backward(); dl.sync()
    assert torch.equal(Y[keep].view(torch.int16), dl.Y[keep].view(torch.int16))
    assert torch.equal(dX[keep].view(torch.int16), dl.dX[keep].view(torch.int16))
    assert not bool(torch.isfinite(dl.Y[off[1]:off[2], 3]).any()) and not bool(torch.isfinite(dl.dX[off[1]:off[2], 5]).any())
    dl.plan.destroy()
