"""The general shrink gives a work group 16, 64 or all ranks of an adapter, by how many work groups the batch has: the same bits each way (one
adapter alone and in batches that are large enough for the other builds), and a rank on each side of a group of ranks."""
import pytest

from test_gpu_batch_independence import _same_bits

pytestmark = pytest.mark.gpu

# Neighbours that take the batch to 64 ranks a work group (in both directions with (64, 4600), fp32 (64, 6200), where the adapter's own rank is
# no wider; bf16 forward with (128, 1500), backward with (128, 2500)) and to all (128, 5100); alone it is 16.
BATCHES = {"f32": [([(16, 37)], [(64, 6200)]), ([(8, 40)], [(128, 5100)])],
           "bf16": [([(64, 37)], [(64, 4600)]), ([(8, 40)], [(128, 1500)]), ([(8, 40)], [(128, 2500)]), ([(8, 40)], [(128, 5100)])]}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rank", [3, 16, 17, 33, 64, 65, 100, 128])
def test_ranks_per_work_group(dtype, rank):
    _same_bits(dtype, 130, 201, rank, BATCHES[dtype], rows=90)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rank", [33, 100])
def test_ranks_per_work_group_of_long_contractions(dtype, rank):
    """Several pieces of the contraction per wavefront, and a remainder: the chains that take turns go past their first piece."""
    _same_bits(dtype, 1030, 2051, rank, BATCHES[dtype], rows=90)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rank", [33, 48, 100])
def test_order_of_the_rank_items(dtype, rank):
    """Three or seven items of 16 ranks: one after the other where the adapter is alone, side by side with neighbours that leave most of them empty; a
    neighbour whose rank makes their number even."""
    _same_bits(dtype, 391, 520, rank, [([(4, 500)], [(8, 300)]), ([(64 if rank < 64 else 128, 70)], [(3, 150)])], rows=90)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rank", [17, 48, 100])
def test_order_of_short_segments(dtype, rank):
    """All blocks' first 16 rows before the others: an adapter with rows in all four places among short ones that have few, and a short one by itself."""
    _same_bits(dtype, 391, 520, rank, [([(4, 2)] * 10, [(7, 3)] * 10), ([(8, 17)] + [(64, 1)] * 9, [(128, 16)] * 15)], rows=90)
    _same_bits(dtype, 391, 520, rank, [([(4, 500)], [(8, 300)]), ([], [(rank, 70)])], rows=13)
