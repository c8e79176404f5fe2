"""The backward product and the weight gradients in one launch (small batches): an odd number of weight-gradient items (a work group with
one), items of different lengths that share a work group, segments without tokens, every tile, both rank builds, split segments
with partial sums, accumulation; and a batch on the other side of the rule."""
import pytest
import torch

from oracle import multilora_oracle as orc
from paper_2604_05426_amd import binding as ml
from paper_2604_05426_amd import workloads as wl
from paper_2604_05426_amd.harness import DeviceLayer, to_host
from util import elem_excess, rel_fro, row_rel_max

pytestmark = pytest.mark.gpu


def _kernels(dl, run):
    """Names of the kernels that run() launches."""
    dl.plan.profile_begin(64)
    run()
    return {ml.KERNEL_NAMES[k] for k, _ in dl.plan.profile_end(64)}


def _apart(dl):
    """dA, dB of the same backward, written over copies of A and B: these get launches of their own."""
    A, B = [t.clone() for t in dl.A], [t.clone() for t in dl.B]
    kernels = _kernels(dl, lambda: ml.multi_lora_bwd(dl.plan, dl.dY, dl.X, dl.W, A, B, dl.S, torch.empty_like(dl.dX), A, B, dl.workspace, 0, dl.stream))
    assert "gemm_bwd" in kernels and "wgrad" in kernels and "gemm_bwd_wgrad" not in kernels
    return A + B


def _same(xs, ys):
    return all(torch.equal(x.view(torch.uint8), y.view(torch.uint8)) for x, y in zip(xs, ys))

# k, n, ranks, tokens of each adapter
CASES = [(128, 256, [16, 8, 32], [70, 1, 200]),             # 9 items; 1, 2 and 4 steps
         (384, 128, [64, 40], [129, 640]),                  # 4 panels; a segment of two chunks (partial sums)
         (264, 136, [33, 4, 0, 12, 64], [64, 65, 10, 0, 63]),   # edges of a panel, a rank of 0, no tokens
         (1024, 520, [16] * 3, [300, 250, 90]),
         (2048, 1024, [24, 64], [500, 200]),                # 64 x 128 tiles
         (2048, 640, [24, 64], [900, 700]),                 # 128 x 128 tiles
         (512, 1032, [8] * 40, [30 + i for i in range(40)])]     # 13 panels x 40 adapters: past the rule
JOINED = {0, 1, 2, 3, 4, 5}


@pytest.mark.parametrize("case", range(len(CASES)))
def test_backward_of_small_batches(case):
    k, n, ranks, lens = CASES[case]
    w = wl.make_workload(f"beside_{case}", "bf16", k, n, ranks, lens, [1.0 + 0.5 * (i % 3) for i in range(len(ranks))], seed=case, b_sigma=0.3)
    print(f"[case] side by side k={k} n={n} ranks={ranks[:6]} tokens={lens[:6]}", flush=True)
    dl = DeviceLayer(w)
    bw = orc.backward(w.dY, w.X, w.W, w.A, w.B, w.scales, w.offsets)

    def check(times):
        # bf16: tolerances of the parity tests (one rounding of dS, one of the result; accumulated: one more of the stored value)
        assert rel_fro(to_host(dl.dX), bw.dX) <= 1e-2 and row_rel_max(to_host(dl.dX), bw.dX) <= 4e-2
        for i in range(w.N):
            if w.ranks[i] and w.seg_lens[i]:
                assert rel_fro(to_host(dl.dA[i]), times * bw.dA[i]) <= 1e-2 and rel_fro(to_host(dl.dB[i]), times * bw.dB[i]) <= 1e-2
                if times == 1:
                    assert elem_excess(to_host(dl.dA[i]), bw.dA[i], "bf16") <= 1 and elem_excess(to_host(dl.dB[i]), bw.dB[i], "bf16") <= 1

    dl.forward()
    assert ("gemm_bwd_wgrad" in _kernels(dl, dl.backward)) == (case in JOINED)
    dl.sync()
    check(1)
    once = [t.clone() for t in dl.dA + dl.dB]
    assert _same(once, _apart(dl))
    # the decoupled form: the same bits
    for t in dl.dA + dl.dB:
        t.fill_(float("nan"))
    dl.backward(ml.FLAG_BASE_ONLY); dl.backward(ml.FLAG_LORA_ONLY); dl.sync()
    assert _same(once, dl.dA + dl.dB)
    dl.backward(ml.FLAG_ACCUM_GRADS); dl.sync()
    check(2)
    dl.check_guards()
    dl.plan.destroy()


# fp32: k, n, ranks, tokens; 32 x 32, 64 x 64 and 128 x 128 tiles; 16, 32 and 64 ranks per item; panels narrower than 64; more ranks than an item
F32_CASES = [(64, 96, [5, 16, 0, 3], [40, 1, 9, 0]), (40, 200, [33, 100], [70, 130]), (300, 700, [16, 32], [500, 517]), (700, 512, [64, 17, 128], [400, 16, 300]),
             (1100, 520, [48], [2100]), (130, 129, [128], [17]), (520, 515, [64, 8], [1500, 490])]
F32_JOINED = {0, 1, 2, 4, 6}      # (ranks above 32 do not go with 32 x 32 tiles)


@pytest.mark.parametrize("case", range(len(F32_CASES)))
def test_fp32_backward_of_small_batches(case):
    k, n, ranks, lens = F32_CASES[case]
    w = wl.make_workload(f"beside_f32_{case}", "f32", k, n, ranks, lens, [1.0 + 0.5 * (i % 3) for i in range(len(ranks))], seed=case, b_sigma=0.3)
    print(f"[case] fp32 side by side k={k} n={n} ranks={ranks} tokens={lens}", flush=True)
    dl = DeviceLayer(w)
    fw, bw = orc.forward(w.X, w.W, w.A, w.B, w.scales, w.offsets), orc.backward(w.dY, w.X, w.W, w.A, w.B, w.scales, w.offsets)
    dl.forward()
    assert ("gemm_bwd_wgrad" in _kernels(dl, dl.backward)) == (case in F32_JOINED)
    dl.sync()
    for got, want in ((dl.Y, fw.Y), (dl.dX, bw.dX)):
        assert rel_fro(to_host(got), want) <= 1e-5 and row_rel_max(to_host(got), want) <= 4e-5
    for i in range(w.N):
        assert rel_fro(to_host(dl.dA[i]), bw.dA[i]) <= 1e-5 and rel_fro(to_host(dl.dB[i]), bw.dB[i]) <= 1e-5
        if w.ranks[i] and w.seg_lens[i]:
            assert rel_fro(dl.S_list()[i], fw.S[i]) <= 1e-5 and rel_fro(dl.dS_list()[i], bw.dS[i]) <= 1e-5
    once = [t.clone() for t in dl.dA + dl.dB]
    assert _same(once, _apart(dl))
    for t in dl.dA + dl.dB:
        t.fill_(float("nan"))
    dl.backward(ml.FLAG_BASE_ONLY); dl.backward(ml.FLAG_LORA_ONLY); dl.sync()
    assert _same(once, dl.dA + dl.dB)
    dl.backward(ml.FLAG_ACCUM_GRADS); dl.sync()
    for i in range(w.N):
        assert rel_fro(to_host(dl.dA[i]), 2 * bw.dA[i]) <= 1e-5 and rel_fro(to_host(dl.dB[i]), 2 * bw.dB[i]) <= 1e-5
    dl.check_guards()
    dl.plan.destroy()


# bf16 rows that start at any element: k, n, ranks, tokens; 32 x 32 and 64 x 64 tiles, one and several rank items, panels with a remainder
ODD_CASES = [(65, 129, [5, 16, 0, 3], [40, 1, 9, 0]), (300, 77, [33, 100], [70, 257]), (2048, 1001, [4, 7, 33], [310, 500, 96]), (1001, 515, [16], [1100]),
             (100, 333, [64, 8], [1999, 31])]
ODD_JOINED = {0, 1, 2, 3, 4}


@pytest.mark.parametrize("case", range(len(ODD_CASES)))
def test_odd_width_backward_of_small_batches(case):
    """Against the oracle, and the same bits as with a neighbour whose tokens are too many for the one launch."""
    k, n, ranks, lens = ODD_CASES[case]
    ranks, lens = ranks + [8], lens + [2100]
    big = wl.make_workload(f"beside_odd_{case}", "bf16", k, n, ranks, lens, [1.0 + 0.5 * (i % 3) for i in range(len(ranks))], seed=case, b_sigma=0.3)
    print(f"[case] odd widths side by side k={k} n={n} ranks={ranks} tokens={lens}", flush=True)
    N, T = big.N - 1, big.offsets[-2]
    w = wl.Workload(name="part", dtype="bf16", T=T, k=k, n=n, ranks=ranks[:N], scales=big.scales[:N], offsets=big.offsets[:-1], X=big.X[:T], W=big.W,
                    A=big.A[:N], B=big.B[:N], dY=big.dY[:T])
    dl, db = DeviceLayer(w), DeviceLayer(big)
    for d in (dl, db):
        d.forward()
        assert ("gemm_bwd_wgrad" in _kernels(d, d.backward)) == (d is dl and case in ODD_JOINED)
        d.sync()
    assert _same(dl.dA + dl.dB, _apart(dl))
    bw = orc.backward(w.dY, w.X, w.W, w.A, w.B, w.scales, w.offsets)
    # bf16: tolerances of the parity tests, as above
    assert rel_fro(to_host(dl.dX), bw.dX) <= 1e-2 and row_rel_max(to_host(dl.dX), bw.dX) <= 4e-2
    assert torch.equal(dl.dX.view(torch.int16), db.dX[:T].view(torch.int16))

    def check(times):
        for i in range(N):
            if w.ranks[i]:
                assert rel_fro(to_host(dl.dA[i]), times * bw.dA[i]) <= 1e-2 and rel_fro(to_host(dl.dB[i]), times * bw.dB[i]) <= 1e-2
                for a, b in ((dl.dA[i], db.dA[i]), (dl.dB[i], db.dB[i])):
                    assert torch.equal(a.view(torch.int16), b.view(torch.int16))

    check(1)
    for d in (dl, db):
        d.backward(ml.FLAG_ACCUM_GRADS); d.sync()
    check(2)
    for d in (dl, db):
        d.check_guards()
        d.plan.destroy()


@pytest.mark.parametrize("dtype,k,n,rank,lens", [("bf16", 384, 128, 40, [129, 640]), ("f32", 300, 700, 32, [500, 517]), ("bf16", 300, 77, 33, [70, 257])])
def test_gradients_over_the_adapters(dtype, k, n, rank, lens):
    """Gradients written over the matrices they belong to, or over each other's: dX still comes from the old ones."""
    w = wl.make_workload("over", dtype, k, n, [rank] * 2, lens, [1.0, 0.5], seed=5, b_sigma=0.3)
    print(f"[case] gradients over the adapters {dtype} k={k} n={n}", flush=True)
    dl = DeviceLayer(w)
    dl.forward(); dl.backward(); dl.sync()
    want = [t.clone() for t in [dl.dX] + dl.dA + dl.dB]
    A, B = [t.clone() for t in dl.A], [t.clone() for t in dl.B]
    for order in ((0, 1), (1, 0)):
        for _ in range(3):
            for t, old in zip(dl.A + dl.B, A + B):
                t.copy_(old)
            dl.dX.fill_(float("nan"))
            dA, dB = [dl.A[j] for j in order], [dl.B[j] for j in order]
            ml.multi_lora_bwd(dl.plan, dl.dY, dl.X, dl.W, dl.A, dl.B, dl.S, dl.dX, dA, dB, dl.workspace, 0, dl.stream)
            dl.sync()
            for got, ref in zip([dl.dX] + dA + dB, want):
                assert torch.equal(got.view(torch.uint8), ref.view(torch.uint8))
    dl.check_guards()
    dl.plan.destroy()
