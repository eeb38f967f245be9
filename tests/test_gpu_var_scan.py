"""Tile offsets of the variable-size encoder where the number of scan chunks
(8,192 tiles each) and the scan's launches change: exact prefix sums."""
import pytest
import torch

from paper_2609_24294_amd import workloads as W

pytestmark = pytest.mark.gpu

CHUNK = 8192


@pytest.mark.parametrize("ntiles", [1, 2, CHUNK - 1, CHUNK, CHUNK + 1, 5 * CHUNK, 5 * CHUNK + 1,
                                    6 * CHUNK + 17])
def test_tile_offsets(zfpx_lib, ntiles):
    nblocks = 64 * ntiles - 5
    plan = zfpx_lib.Plan.from_chunkset(W.regular_chunkset(4, 4, 4 * nblocks))
    gen = torch.Generator(device="cuda:0").manual_seed(ntiles)
    src = torch.randn(64 * nblocks, device="cuda:0", generator=gen)
    src[: src.numel() // 3] = 1.0  # constant blocks: other counts
    words, nd, off = zfpx_lib.zfpx_plan_encode_var(plan, src, 3, zfpx_lib.MINEXP_NONE, 4)
    per_tile = torch.zeros(64 * ntiles, dtype=torch.int64, device="cuda:0")
    per_tile[:nblocks] = nd.long()
    want = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda:0"),
                      per_tile.view(ntiles, 64).sum(1).cumsum(0)])
    assert nd.min() >= 1 and torch.equal(off, want)
