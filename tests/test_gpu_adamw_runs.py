"""The AdamW kernel's division into runs of 4096 elements: matrices that end on, one before and one after a run, element counts that
leave m and v at odd addresses, adapters without a rank between the others, and more adapters than one launch carries."""
import pytest
import torch

from paper_2604_05426_amd import binding as ml
from test_gpu_adamw import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("k,n,ranks", [(4096, 4095, [1, 0, 2]), (4097, 1025, [3, 1, 4]), (7, 3, [0, 1, 5, 0] * 17 + [0])])
def test_runs(dtype, k, n, ranks):
    _run(dtype, k, n, ranks, steps=2, seed=k + n)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_state_through_and_past_the_caches(dtype):
    """A plan by itself keeps a small state in the caches; with another layer over its tables, and for that layer, it goes past them: the same bits."""
    k, n, ranks = 4097, 1025, [3, 0, 8]
    off = [0, 5, 9, 40]
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(3)
    base = ml.Plan(ml.BF16 if dtype == "bf16" else ml.F32, 40, k, n, ranks, [1.0] * 3, off)
    A = [torch.randn((k, r), device="cuda", generator=gen).to(t) for r in ranks]
    B = [torch.randn((r, n), device="cuda", generator=gen).to(t) for r in ranks]
    dA = [torch.randn((k, r), device="cuda", generator=gen).to(t) for r in ranks]
    dB = [torch.randn((r, n), device="cuda", generator=gen).to(t) for r in ranks]

    def steps(plan):
        a, b = [x.clone() for x in A], [x.clone() for x in B]
        sA = [torch.empty(3 * k * r, device="cuda") for r in ranks]
        sB = [torch.empty(3 * r * n, device="cuda") for r in ranks]
        ml.multi_lora_adamw_init(plan, a, b, sA, sB)
        for i in range(1, 4):
            ml.multi_lora_adamw_step(plan, a, b, dA, dB, sA, sB, [(1e-3, 0.9, 0.99, 1e-8, 0.01, i)] * 3)
        torch.cuda.synchronize()
        return a + b + sA + sB

    alone = steps(base)
    other = ml.Plan.like(base, k, n)
    for plan in (base, other):
        assert all(torch.equal(x, y) for x, y in zip(alone, steps(plan)))
    other.destroy()
    assert all(torch.equal(x, y) for x, y in zip(alone, steps(base)))
    base.destroy()
