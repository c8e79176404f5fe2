"""The AdamW kernel's division into runs of 4096 elements: matrices that end on, one before and one after a run, element counts that
leave m and v at odd addresses, adapters without a rank between the others, and more adapters than one launch carries."""
import pytest

from test_gpu_adamw import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("k,n,ranks", [(4096, 4095, [1, 0, 2]), (4097, 1025, [3, 1, 4]), (7, 3, [0, 1, 5, 0] * 17 + [0])])
def test_runs(dtype, k, n, ranks):
    _run(dtype, k, n, ranks, steps=2, seed=k + n)
