"""More adapters in one tile than a wavefront has lanes: the products walk the candidate adapters of a tile in batches of 64, and only a
tile that meets more than that reaches the second batch.  150 adapters of 0 to 3 tokens, one batch of which has nothing to do."""
import numpy as np
import pytest

from paper_2604_05426_amd import workloads as wl
from test_gpu_parity import check_full

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("idle", ["second", "first", "none"])
@pytest.mark.parametrize("dtype,k,n", [("bf16", 320, 264), ("bf16", 72, 1096), ("f32", 96, 72), ("bf16", 100, 52)])
def test_tiles_of_150_adapters(dtype, k, n, idle):
    rng = np.random.default_rng(k + n)
    N = 150
    ranks = [int(x) for x in rng.choice([0, 4, 33, 100], size=N)]
    lens = [int(x) for x in rng.integers(0, 4, size=N)]
    for i in {"second": range(64, 128), "first": range(0, 64), "none": ()}[idle]:
        if i % 2:
            ranks[i] = 0
        else:
            lens[i] = 0
    w = wl.make_workload(f"tiny_{idle}", dtype, k, n, ranks, lens, [float(x) for x in rng.choice([0.5, 1.0, 1.7], size=N)], seed=k, b_sigma=0.3)
    check_full(w)
