"""GPU coder and decoder against the CPU oracle where a bit plane's groups end
at coefficient 63, at the budget or past the 64-bit window, and where decoded
values are subnormal: bit-exact, in tiles that mix such blocks with others."""
import numpy as np
import pytest
import torch

import oracle

from _blocks import array_to_blocks, block_families, blocks_to_array

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _mixed(rng, blocks):
    """The blocks shuffled with as many ordinary ones."""
    both = np.concatenate([blocks, block_families(rng, len(blocks))])
    return np.ascontiguousarray(both[rng.permutation(len(both))])


def _subnormal(rng, n):
    scale = 2.0 ** rng.integers(-149, -119, (n, 1))
    return (rng.standard_normal((n, 64)) * scale * (rng.random((n, 64)) < 0.4)).astype(np.float32)


def _last_coefficient(rng, n):
    """One or two values per block: every coefficient significant at once."""
    v = np.zeros((n, 64), np.float32)
    for i in range(n):
        v[i, rng.integers(64)] = rng.standard_normal()
        v[i, rng.integers(64)] += rng.standard_normal() * 2.0 ** -rng.integers(0, 30)
    return v


def _check_decode(zfpx_lib, words, rate):
    nb = words.shape[0]
    out = torch.empty((4, 4, 4 * nb), dtype=torch.float32, device=DEV)
    zfpx_lib.zfpx_decode_fixed_rate(torch.from_numpy(words.reshape(-1).view(np.int64)).to(DEV),
                                    rate, out)
    got = array_to_blocks(out.cpu().numpy())
    want = np.asarray(oracle.decode_blocks(words, rate), np.float32).reshape(nb, 64)
    assert np.array_equal(got.view(np.uint32), want.view(np.uint32)), rate


@pytest.mark.parametrize("rate", [1, 4, 8, 15, 16, 32])
def test_blocks_at_the_edges(zfpx_lib, rate):
    rng = np.random.default_rng(4000 + rate)
    for make in (_subnormal, _last_coefficient):
        blocks = _mixed(rng, make(rng, 300))
        words = zfpx_lib.zfpx_encode_fixed_rate(torch.from_numpy(blocks_to_array(blocks)).to(DEV),
                                                rate)
        want = oracle.encode_blocks(blocks, rate)
        assert np.array_equal(words.cpu().numpy().view(np.uint64).reshape(-1, rate), want)
        _check_decode(zfpx_lib, want, rate)


@pytest.mark.parametrize("rate", [1, 4, 8, 15, 16, 32])
def test_streams_at_the_edges(zfpx_lib, rate):
    rng = np.random.default_rng(5000 + rate)

    def words(n):
        return rng.integers(0, 2 ** 64, (n, rate), dtype=np.uint64)

    sparse = words(300) & words(300) & words(300) & words(300)  # long scans
    dense = words(300) | words(300)                             # long runs of groups
    tiny = words(300)                                           # smallest exponents
    tiny[:, 0] &= ~np.uint64(0x1fe)
    tiny[:, 0] |= rng.integers(0, 16, 300).astype(np.uint64) << np.uint64(1)
    w = np.concatenate([sparse, dense, tiny, words(300)])
    w[:, 0] |= np.uint64(1)
    _check_decode(zfpx_lib, np.ascontiguousarray(w[rng.permutation(len(w))]), rate)
