"""The bf16 products and shrinks at the edges of their tiles, rings and dispatch rules: against the oracle, and bit for bit against the
form that the same rows take in another tile or batch."""
import pytest
import torch

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


# odd widths: 2000 and 2001 rows take whole tiles forward, 64 x 64 or 128 x 64; the others, whose tiles fill less than half of the chip, 32 x 32 tiles, and the
# backward of all goes with the weight gradients (test_whole_tiles_alone has the whole tiles' own edges)
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


def _whole(dl, rows, cols, contraction, w):
    """Whether a product of that size takes whole tiles (at least half of the chip, one round of two a CU or two steps and as many as passes)."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    tiles = -(-rows // 64) * -(-cols // 64)
    passes = sum(((b - 1) // 64 - a // 64 + 1) * -(-r // 64) for r, a, b in zip(w.ranks, w.offsets, w.offsets[1:]) if b > a) / -(-rows // 64)
    return 2 * tiles > cus and rows >= 128 and min(cols, contraction) >= 64 and (tiles <= 2 * cus or contraction / 64 >= max(2, passes))


# Products of 129 x 2, 2 x 68, 3 x 68, 129 x 6 tiles (the last: several rounds); the last tile of rows and columns whole or not; contractions of one step and
# less than two, and on both sides of the four steps that are on their way.  Backward apart: a long segment, or tables too large to join.
@pytest.mark.parametrize("T,cols,contractions", [(8200, 65, (64, 65, 127, 128)), (8256, 127, (191, 192, 193, 255)), (8193, 128, (257, 319, 321, 449)),
                                                 (128, 4289, (64, 129)), (129, 4352, (65, 323)), (192, 4290, (191, 257)), (8200, 321, (193, 387))])
@pytest.mark.parametrize("adapters", [9, 70])
def test_whole_tiles_alone(T, cols, contractions, adapters):
    # ranks below, at and above a 16-byte piece and a pass; a short, an empty and a long segment; rows of 3 that end with the buffer
    ranks = ((33, 1, 7, 100, 0, 64, 8, 2, 3) if adapters == 9 else tuple((33, 1, 3, 7, 16, 5, 100)[i % 7] for i in range(69)) + (3,))
    first = min(2100, T // 2)
    rest = T - first - 1
    lens = [first, 1, 0] + [rest // (adapters - 3)] * (adapters - 4)
    lens.append(T - sum(lens))
    for c in contractions:
        for k, n in ((c, cols), (cols, c)):
            if k % 8 == 0 and n % 8 == 0:
                continue
            print(f"[case] whole tiles alone T={T} k={k} n={n} adapters={adapters}", flush=True)
            w = wl.make_workload("whole_tiles", "bf16", k, n, ranks, lens, [(2.0, 0.5, 1.0, 0.25)[i % 4] for i in range(adapters)], seed=T + k + n, b_sigma=0.3)
            dl = DeviceLayer(w)
            assert _whole(dl, T, cols, c, w)
            dl.forward()
            dl.plan.profile_begin(64)
            dl.backward()
            kernels = {ml.KERNEL_NAMES[i] for i, _ in dl.plan.profile_end(64)}
            assert k != cols or "gemm_bwd" in kernels
            dl.sync()
            _check(dl, w)
            dl.plan.destroy()


@pytest.mark.parametrize("rank", [1, 7, 33, 100])
@pytest.mark.parametrize("k,n,rows", [(129, 65, 150), (65, 321, 70), (300, 1001, 130)])
def test_whole_tiles_leave_every_bit_alone(k, n, rows, rank):
    """An adapter by itself (32 x 32 tiles) and with neighbours whose rows make whole tiles, before and behind it and with most of the passes."""
    _same_bits("bf16", k, n, rank, [([(5, 3000)], [(3, 5300)]), ([(33, 1), (2, 8000)], []), ([], [(100, 2100)] + [(4, 100)] * 62)], rows)


def test_whole_tiles_need_a_piece_of_the_rank_rows():
    """Two rank rows of three elements: less than a piece, the launch takes the tiles that load them singly."""
    w = wl.make_workload("six_elements", "bf16", 129, 65, (0, 3), (8198, 2), (1.0, 2.0), seed=6, b_sigma=0.3)
    dl = DeviceLayer(w)
    print("[case] six rank elements", flush=True)
    dl.forward(); dl.backward(); dl.sync()
    _check(dl, w)
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
