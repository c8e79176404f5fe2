"""The general kernels (fp32; bf16 with a width that is not a multiple of 8) at the sizes where they can go wrong: tokens, widths
and contractions on both sides of a 32 and 64 tile edge and of a step, widths below a tile and below a 16-byte piece, last
tiles that start early and share rows with the one before (in place and accumulating too), ranks around 4, 16, 32, 64 and 128,
and both tile forms."""
import pytest
import torch

from oracle import multilora_oracle as orc
from paper_2604_05426_amd import binding as ml
from paper_2604_05426_amd import workloads as wl
from paper_2604_05426_amd.harness import DeviceLayer, to_host
from util import elem_excess, rel_fro, row_rel_max

pytestmark = pytest.mark.gpu

RANKS = {"low": (1, 3, 4, 0, 16), "mid": (17, 32, 7, 33, 64), "high": (65, 128, 100, 8, 127)}
SHAPES = [(33, 31, 33), (31, 65, 3), (64, 64, 63), (65, 5, 130), (257, 129, 31), (300, 127, 257), (511, 257, 65),
          (1000, 700, 515), (1300, 390, 650)]      # the last two: more than half a chip of 64 x 64 tiles, forward and backward


def _check(dl, w, dtype, two=1.0):
    tol = 1e-2 if dtype == "bf16" else 1e-5      # fp32: sums of at most 1300 products, relative error ~ sqrt(1300) 2^-24 = 2e-6
    fw = orc.forward(w.X, w.W, w.A, w.B, w.scales, w.offsets)
    bw = orc.backward(w.dY, w.X, w.W, w.A, w.B, w.scales, w.offsets)
    for got, want in ((dl.Y, fw.Y), (dl.dX, bw.dX)):
        assert rel_fro(to_host(got), want) <= two * tol and row_rel_max(to_host(got), want) <= 4 * two * tol
    for i in range(w.N):
        assert rel_fro(to_host(dl.dA[i]), bw.dA[i]) <= tol and rel_fro(to_host(dl.dB[i]), bw.dB[i]) <= tol
        assert elem_excess(to_host(dl.dA[i]), bw.dA[i], dtype) <= 1 and elem_excess(to_host(dl.dB[i]), bw.dB[i], dtype) <= 1


@pytest.mark.parametrize("ranks", sorted(RANKS))
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_general_kernels_at_their_edges(dtype, ranks):
    for T, k, n in SHAPES:
        off = [0, T // 3, T // 3 + 1, T // 3 + 1, T - T // 4, T]
        w = wl.make_workload(f"edge_{T}_{k}_{n}", dtype, k, n, RANKS[ranks], [b - a for a, b in zip(off, off[1:])],
                             (2.0, 0.5, 1.0, 0.25, 3.0), seed=T + k + n, b_sigma=0.3)
        print(f"[case] general {dtype} T={T} k={k} n={n} ranks={RANKS[ranks]}", flush=True)
        dl = DeviceLayer(w)
        dl.forward(); dl.backward(); dl.sync()
        _check(dl, w, dtype)
        for t in (dl.Y, dl.dX):
            t.fill_(float("nan"))
        for t in dl.dA + dl.dB:
            t.zero_()
        dl.forward(ml.FLAG_BASE_ONLY); dl.forward(ml.FLAG_LORA_ONLY)
        dl.backward(ml.FLAG_BASE_ONLY); dl.backward(ml.FLAG_LORA_ONLY | ml.FLAG_ACCUM_GRADS); dl.sync()
        _check(dl, w, dtype, two=2.0)       # the frozen-weight result is stored before the LoRA term is added: two roundings
        # a diverged neighbour stays out of the other segments, also where they share a tile
        dl.forward(); dl.backward(); dl.sync()
        Y, dX = dl.Y.clone(), dl.dX.clone()
        dl.A[0][k // 2, :] = float("nan")
        dl.B[0][:, n // 2] = float("inf")
        dl.forward(); dl.backward(); dl.sync()
        view = torch.int16 if dtype == "bf16" else torch.int32
        assert torch.equal(Y[off[1]:].view(view), dl.Y[off[1]:].view(view)) and torch.equal(dX[off[1]:].view(view), dl.dX[off[1]:].view(view))
        dl.plan.destroy()
