"""Launches of the general kernels whose work groups do not fit one dimension of a grid (2^32 work items): very many rows, very wide rows,
very many output tiles."""
import pytest
import torch

from paper_2604_05426_amd import binding as ml

pytestmark = pytest.mark.gpu


def test_rows_beyond_one_grid_dimension():
    """2^27 + 70 rows of two columns through a rank-1 adapter: 2^23 + work groups of 512 in the shrink."""
    T, k, n = (1 << 27) + 70, 2, 2
    d = dict(device="cuda", dtype=torch.float32)
    X = torch.rand((T, k), **d)
    W, A, B = (torch.tensor(v, **d) for v in ([[0.5, -1.0], [2.0, 0.25]], [[1.0], [-2.0]], [[3.0, 0.5]]))
    Y, S = torch.empty((T, n), **d), torch.full((T,), float("nan"), **d)
    plan = ml.Plan(ml.F32, T, k, n, [1], [1.0], [0, T])
    print(f"[case] general shrink T={T}", flush=True)
    ml.multi_lora_fwd(plan, X, W, [A], [B], Y, S, None)
    torch.cuda.synchronize()
    for lo in (0, T // 2, T - 4096):        # products of a few terms: exact up to one rounding each
        x = X[lo:lo + 4096].double()
        s = x @ A.double()
        assert torch.allclose(S[lo:lo + 4096].double(), s[:, 0], rtol=0, atol=1e-6)
        assert torch.allclose(Y[lo:lo + 4096].double(), x @ W.double() + s @ B.double(), rtol=0, atol=4e-6)
    assert bool(torch.isfinite(S).all())
    plan.destroy()


def test_columns_beyond_one_grid_dimension():
    """The LoRA-only backward of one token through 2^29 + 70 columns: 2^23 + panels in the weight gradient; dA = X^T dS is one product."""
    k, n = (1 << 29) + 70, 1
    d = dict(device="cuda", dtype=torch.float32)
    X, A = torch.rand((1, k), **d), torch.rand((k, 1), **d)
    B, dY, S = torch.tensor([[3.0]], **d), torch.tensor([[0.5]], **d), torch.tensor([0.25], **d)
    dX, dA, dB = torch.zeros((1, k), **d), torch.full((k, 1), float("nan"), **d), torch.zeros((1, 1), **d)
    plan = ml.Plan(ml.F32, 1, k, n, [1], [2.0], [0, 1])
    ws = torch.empty(max(plan.workspace_bytes(), 256), dtype=torch.uint8, device="cuda")
    print(f"[case] general weight gradient k={k}", flush=True)
    ml.multi_lora_bwd(plan, dY, X, None, [A], [B], S, dX, [dA], [dB], ws, ml.FLAG_LORA_ONLY)
    torch.cuda.synchronize()
    assert torch.equal(dA[:, 0], 3.0 * X[0]) and torch.equal(dX[0], 3.0 * A[:, 0])      # dS = 2 dY B = 3
    assert float(dB) == 0.25                                                            # 2 S dY
    plan.destroy()


def test_products_beyond_one_grid_dimension():
    """dX of 2^20 rows and 32769 columns: 2^23 + tiles of 64 x 64, work groups of 512.  Entries -1, 0 and 1: every sum of 65 is exact."""
    T, k, n = 1 << 20, 32769, 65
    gen = torch.Generator(device="cuda").manual_seed(1)

    def units(*shape):
        return torch.randint(-1, 2, shape, device="cuda", dtype=torch.int8, generator=gen).to(torch.bfloat16)

    W, dY = units(k, n), units(T, n)
    dX = torch.full((T, k), float("nan"), device="cuda", dtype=torch.bfloat16)
    plan = ml.Plan(ml.BF16, T, k, n, [], [], [0])
    print(f"[case] general product T={T} k={k} n={n}", flush=True)
    ml.multi_lora_bwd(plan, dY, None, W, None, None, None, dX, None, None, None, ml.FLAG_BASE_ONLY)
    torch.cuda.synchronize()
    rows = 1 << 15
    for lo in range(0, T, rows):
        assert not bool(torch.isnan(dX[lo:lo + rows]).any()), lo
    Wt = W.float().T.contiguous()
    for lo in (0, T // 2 - 100, T - 200):
        assert torch.equal(dX[lo:lo + 200].float(), dY[lo:lo + 200].float() @ Wt)
    plan.destroy()
