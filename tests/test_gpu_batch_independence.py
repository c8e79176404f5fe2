"""An adapter's rows of S, Y, dS and dX have the same bits whoever shares its batch: every kernel and tile that the layer may choose
for a batch sums a row in one order, which the adapter's own rank and the layer's widths fix.  One adapter's segment is run alone
and among neighbours whose tokens and ranks send the same layer to other tiles, splits and builds."""
import numpy as np
import pytest
import torch

from paper_2604_05426_amd import binding as ml
from paper_2604_05426_amd import workloads as wl
from paper_2604_05426_amd.harness import DeviceLayer

pytestmark = pytest.mark.gpu

ROWS = 150      # tokens of the adapter under test


def _run(dtype, k, n, rank, before, after, rows=ROWS, seed=11):
    """Bits of the adapter's S, Y, dS, dX, and Y, dX of the decoupled form, with `before` / `after` = (rank, tokens) of its neighbours; its own
    data depend on `seed` alone."""
    own = wl.make_workload("own", dtype, k, n, [rank], [rows], [0.7], seed=seed, b_sigma=0.3)
    ranks = [r for r, _ in before] + [rank] + [r for r, _ in after]
    lens = [t for _, t in before] + [rows] + [t for _, t in after]
    i = len(before)
    off = [0]
    for t in lens:
        off.append(off[-1] + t)
    lo, rng = off[i], np.random.default_rng(seed)
    A = [own.A[0] if j == i else np.resize(own.A[0], (k, r)) for j, r in enumerate(ranks)]
    B = [own.B[0] if j == i else np.resize(own.B[0], (r, n)) for j, r in enumerate(ranks)]
    other = rng.permutation(rows)               # the neighbours' tokens: this adapter's in another order, again and again
    X, dY = np.resize(own.X[other], (off[-1], k)), np.resize(own.dY[other], (off[-1], n))
    X[lo:lo + rows], dY[lo:lo + rows] = own.X, own.dY
    w = wl.Workload(name="batch", dtype=dtype, T=off[-1], k=k, n=n, ranks=ranks, scales=[0.7] * len(ranks), offsets=off,
                    X=X, W=own.W, A=A, B=B, dY=dY)
    dl = DeviceLayer(w)
    dl.forward(); dl.backward(); dl.sync()
    got = [dl.S_list()[i], dl.Y[lo:lo + rows].clone(), dl.dS_list()[i], dl.dX[lo:lo + rows].clone()]
    for t in (dl.Y, dl.dX):
        t.fill_(float("nan"))
    dl.forward(ml.FLAG_BASE_ONLY); dl.forward(ml.FLAG_LORA_ONLY)
    dl.backward(ml.FLAG_BASE_ONLY); dl.backward(ml.FLAG_LORA_ONLY); dl.sync()
    got += [dl.Y[lo:lo + rows].clone(), dl.dX[lo:lo + rows].clone()]
    dl.plan.destroy()
    return [np.asarray(g) if isinstance(g, np.ndarray) else g.view(torch.int16 if dtype == "bf16" else torch.int32).cpu().numpy() for g in got]


def _same_bits(dtype, k, n, rank, batches, rows=ROWS):
    want = _run(dtype, k, n, rank, [], [], rows)
    for before, after in batches:
        print(f"[case] {dtype} k={k} n={n} rank={rank} before={before} after={after}", flush=True)
        for name, a, b in zip(("S", "Y", "dS", "dX", "decoupled Y", "decoupled dX"), want, _run(dtype, k, n, rank, before, after, rows)):
            assert np.array_equal(a, b), (name, before, after, int((a != b).sum()), a.size)


@pytest.mark.parametrize("k,n", [(520, 1096), (1096, 520), (1800, 72)])
@pytest.mark.parametrize("rank", [16, 33, 100])
def test_tiles_of_the_fused_products(k, n, rank):
    """Every tile of the bf16 products (64 x 64 alone; 64 x 128, 128 x 128, 256 x 256 with more rows), contractions with and without a
    tail; ranks of one and two passes, one that is not a multiple of 8."""
    _same_bits("bf16", k, n, rank, [([(16, 37)], [(16, 930)]), ([(8, 1301)], [(64, 1500)]), ([(128, 5003)], [(16, 3000)])])


@pytest.mark.parametrize("k,n,rank", [(2048, 5120, 16), (5120, 2048, 104), (2112, 4160, 36), (2048, 2048, 100), (3072, 2048, 33)])
def test_splits_of_the_shrink(k, n, rank):
    """A contraction shared by 8, 4 and 2 work groups or done by one (3 row blocks alone, 36, 53, 110 and 150 with the neighbours), and with
    a neighbour of the wide rank class or of an odd rank, which send the layer to other builds; contractions of 32 to 80 steps, some
    that do not divide into equal pieces."""
    _same_bits("bf16", k, n, rank, [([(16, 37)], [(16, 2100)]), ([(8, 1301)], [(33, 1900)]), ([(16, 3003)], [(64, 3800)]),
                                    ([(128, 500)], [(16, 1500)]), ([(64, 5003)], [(4, 4500)])])


@pytest.mark.parametrize("dtype,k,n", [("f32", 256, 264), ("f32", 1000, 515), ("f32", 31, 700), ("f32", 128, 100), ("bf16", 1000, 515), ("bf16", 513, 260), ("bf16", 2050, 96)])
@pytest.mark.parametrize("rank,rows", [(8, 20), (16, 150), (33, 150), (100, 40)])
def test_tiles_and_builds_of_the_general_kernels(dtype, k, n, rank, rows):
    """Both tiles of the general products (32 x 32 alone, 64 x 64 with the neighbours), fewer rows than a tile, contractions with
    and without a remainder and shorter than a step, and neighbours with other ranks (the shrink's ranks per work group: test_gpu_shrink_ranks.py)."""
    _same_bits(dtype, k, n, rank, [([(4, 9)], [(16, 30)]), ([(64, 37)], [(8, 300)]), ([(8, 1301)], [(64, 1500)]), ([(128, 700)], [(16, 3000)])], rows)
