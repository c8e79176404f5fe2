"""The bf16 products and shrinks at the edges of their tiles, rings and dispatch rules: against the oracle, and bit for bit against the
form that the same rows take in another tile or batch."""
import pytest

from oracle import multilora_oracle as orc
from paper_2604_05426_amd import binding as ml
from paper_2604_05426_amd import workloads as wl
from paper_2604_05426_amd.harness import DeviceLayer, to_host
from test_gpu_batch_independence import _same_bits
from util import elem_excess, large_tiles_leave_every_bit_alone, rel_fro, row_rel_max

pytestmark = pytest.mark.gpu

RANKS = (8, 12, 33, 64, 100, 4, 0, 128)      # one and two passes, whole 16-byte pieces, 8-byte ones and none; ragged rows that start anywhere


def _layer(T, k, n, ranks):
    """Segments of T tokens with a one-token and an empty one, where there are tokens enough."""
    cuts = sorted({0, T, *(T * i // len(ranks) for i in range(len(ranks))), min(T, T // len(ranks) + 1)})
    off = (cuts + [T] * (len(ranks) + 1))[: len(ranks)] + [T]
    w = wl.make_workload("tile_edge", "bf16", k, n, ranks, [b - a for a, b in zip(off, off[1:])], [(2.0, 0.5, 1.0, 0.25)[i % 4] for i in range(len(ranks))],
                         seed=T + k + n, b_sigma=0.3)
    return w, DeviceLayer(w)


def _check(dl, w):
    # bf16 results: one rounding, 2^-9, of a sum whose rank term is a product of rounded S / dS: norms within 1e-2, rows within 4e-2
    fw = orc.forward(w.X, w.W, w.A, w.B, w.scales, w.offsets)
    bw = orc.backward(w.dY, w.X, w.W, w.A, w.B, w.scales, w.offsets)
    for got, want in ((dl.Y, fw.Y), (dl.dX, bw.dX)):
        assert rel_fro(to_host(got), want) <= 1e-2 and row_rel_max(to_host(got), want) <= 4e-2
    for i in range(w.N):
        for got, want in ((dl.S_list()[i], fw.S[i]), (dl.dS_list()[i], bw.dS[i]), (to_host(dl.dA[i]), bw.dA[i]), (to_host(dl.dB[i]), bw.dB[i])):
            assert elem_excess(got, want, "bf16") <= 1, i


# (rows, columns): 64 x 64 tiles with 1, 5 and 8 + 2 row tiles in a band, 64 x 128 with 4 and 8 + 3, 128 x 128 with 5 and 8 + 1; contractions of
# no step, one, and on both sides of the depths of the rings (rows 5 / 4 / 3 stages, weight 15 / 8 / 7), with and without a remainder
@pytest.mark.parametrize("T,cols,steps", [(40, 520, (0, 1, 4, 5, 6, 14, 15, 16, 18)), (300, 520, (1, 5, 15, 16)), (600, 520, (0, 4, 14, 17)),
                                          (250, 4104, (1, 3, 4, 5, 7, 8, 9)), (700, 1544, (0, 2, 6, 10)),
                                          (520, 4104, (1, 2, 3, 4, 6, 7, 8)), (1030, 2056, (0, 5, 9))])
def test_small_tiles(T, cols, steps):
    for i, s in enumerate(steps):
        c = 64 * s + (8, 0, 40)[i % 3] if s else 24
        for k, n in ((c, cols), (cols, c)):          # the forward product has `cols` columns, then the backward one
            print(f"[case] small tiles T={T} k={k} n={n}", flush=True)
            w, dl = _layer(T, k, n, RANKS)
            dl.forward(); dl.backward(); dl.sync()
            _check(dl, w)
            large_tiles_leave_every_bit_alone(dl)
            dl.plan.destroy()


# odd widths: products of 128 rows, 64 columns and a contraction of 64 or more take whole tiles, 64 x 64 or (2000 x 700) 128 x 64; just below, the others
@pytest.mark.parametrize("T,k,n", [(128, 64, 65), (127, 64, 65), (129, 63, 66), (191, 65, 127), (192, 319, 129), (193, 320, 321), (255, 323, 64),
                                   (257, 449, 131), (2000, 700, 333), (2001, 333, 701)])
def test_whole_tiles_of_odd_widths(T, k, n):
    for ranks in (RANKS, tuple((1, 3, 7, 16)[i % 4] for i in range(70))):        # more adapters than a wavefront has lanes
        print(f"[case] whole tiles T={T} k={k} n={n} adapters={len(ranks)}", flush=True)
        w, dl = _layer(T, k, n, ranks)
        dl.forward(); dl.backward(); dl.sync()
        _check(dl, w)
        dl.forward(ml.FLAG_BASE_ONLY); dl.backward(ml.FLAG_BASE_ONLY); dl.sync()
        for got, want in ((dl.Y, w.X.astype("f8") @ w.W.astype("f8")), (dl.dX, w.dY.astype("f8") @ w.W.T.astype("f8"))):
            assert rel_fro(to_host(got), want) <= 1e-2 and row_rel_max(to_host(got), want) <= 4e-2
        dl.plan.destroy()


@pytest.mark.parametrize("T,k,n", [(70, 520, 256), (200, 1096, 520)])
def test_small_tiles_with_more_adapters_than_lanes(T, k, n):
    w, dl = _layer(T, k, n, tuple((4, 8, 33, 64)[i % 4] for i in range(130)))
    dl.forward(); dl.backward(); dl.sync()
    _check(dl, w)
    large_tiles_leave_every_bit_alone(dl)
    dl.plan.destroy()


# one row block alone takes the halves (or shares of the contraction); with the neighbours 128 blocks do, and 129 take 64 rows
@pytest.mark.parametrize("rank", [8, 40, 64])
@pytest.mark.parametrize("k,n,rows", [(64, 512, 31), (512, 64, 33), (1984, 128, 64), (128, 1984, 65), (2112, 72, 32), (64, 4160, 150)])
def test_halves_of_row_blocks(k, n, rows, rank):
    _same_bits("bf16", k, n, rank, [([(64, 97)], [(16, 64 * 62 + 1)]), ([(40, 8192 - 128 - rows)], [(8, 1)]), ([(16, 8192)], [(64, 33)])], rows)


@pytest.mark.parametrize("k,n", [(64, 8), (128, 1984), (1984, 128), (3072, 576)])
def test_halves_of_row_blocks_against_the_oracle(k, n):
    for lens in ((1, 31, 32), (33, 63, 64), (65, 96, 127), (700, 2000, 1100)):
        print(f"[case] halves k={k} n={n} lens={lens}", flush=True)
        w = wl.make_workload("halves", "bf16", k, n, (64, 8, 40), lens, (0.5, 2.0, 1.0), seed=k + n, b_sigma=0.3)
        dl = DeviceLayer(w)
        dl.forward(); dl.backward(); dl.sync()
        _check(dl, w)
        dl.plan.destroy()
