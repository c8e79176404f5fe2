"""The general shrink gives a work group 16, 64 or all ranks of an adapter, by how many work groups the batch has: the same bits each way (one
adapter alone and in batches that are large enough for the other builds), and a rank on each side of a group of ranks."""
import pytest

from test_gpu_batch_independence import _same_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rank", [3, 16, 17, 33, 64, 65, 100, 128])
def test_ranks_per_work_group(dtype, rank):
    # fp32: 8700 tokens of ranks to 64 (64 at a time), 5300 with a rank of 128 (all); bf16: 2300 with 64 and 128 (64 at a time), 4600 (all)
    batches = [([(16, 37)], [(64, 8500)]), ([(8, 40)], [(128, 5100)])] if dtype == "f32" else [([(64, 37)], [(128, 2100)]), ([(8, 40)], [(128, 4400)])]
    _same_bits(dtype, 130, 201, rank, batches, rows=90)
