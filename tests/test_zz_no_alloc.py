"""The entry point that allocates nothing (thc_decompress_noalloc: scratch inside the library's code object) against
thc_decompress, through the C-ABI: two calls in a row, the second on a smaller input."""
import numpy as np
import pytest
import torch

from paper_2302_08545_amd import api

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
T430 = [0, 3, 5, 7, 9, 11, 13, 14, 15, 17, 19, 21, 23, 25, 27, 30]


def _both(d, block, n, agg_bits, order, rnd, seed):
    L = api.make_params(d, block, n, 4, 30, 2.1538746, 0x5448435F53454544, T430, agg_bits, stage_order=order)
    g = torch.Generator().manual_seed(seed)
    Y = torch.randint(0, 30 * n + 1, (d,), generator=g)
    agg = (Y.to(torch.uint8) if agg_bits == 8 else Y.to(torch.int16).view(torch.uint8)).to(DEV).contiguous()
    M = (torch.rand(d // block, generator=g) * 1e-3 + 5e-4).to(DEV)
    ws = torch.zeros(api.thc_workspace_bytes(L), dtype=torch.uint8, device=DEV)
    want = torch.zeros(d, dtype=torch.float32, device=DEV)
    api.thc_decompress(L, rnd, agg, M, want, ws)
    got = torch.full((d,), float("nan"), dtype=torch.float32, device=DEV)
    api.thc_decompress_noalloc(L, rnd, agg, M, got)
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    assert float(want.abs().max()) > 0


def test_no_alloc_decompress_equals_decompress_twice_in_a_row():
    assert torch.cuda.is_available()
    # 12 blocks of 2^20: more than the 8 blocks the scratch array holds, so two groups, the second ragged
    _both(12 << 20, 1 << 20, 8, 8, 1, 5, 1)
    # then a smaller input, other block size, 16-bit sums, ascending order: the array keeps the first call's contents
    _both(3 << 14, 1 << 14, 16, 16, 0, 6, 2)
    # and a block that fills the whole array
    _both(1 << 23, 1 << 23, 4, 8, 1, 7, 3)


def test_no_alloc_rejects_blocks_beyond_the_scratch_array():
    L = api.make_params(1 << 24, 1 << 24, 2, 4, 30, 2.15, 7, T430, 8)
    z = torch.zeros(1 << 24, dtype=torch.float32, device=DEV)
    with pytest.raises(api.ThcError) as e:
        api.thc_decompress_noalloc(L, 0, z, z, z)
    assert e.value.status == -4


@pytest.mark.parametrize("order", [0, 1], ids=["ascending", "split"])
def test_no_alloc_decompress_equals_decompress_where_their_tiles_differ(order):
    """64 blocks of 2^22 in one launch take tiles of 2^15 coordinates, two blocks at a time those of 2^13."""
    _both(64 << 22, 1 << 22, 8, 8, order, 9, 4)
