"""Arrays with an x stride other than 1, on both sides of the launch rules (up
to 4,096 tiles and above; y closest in memory or not): GPU against the CPU
oracle, bit for bit, gaps between elements untouched."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _view(flat, layout, nz, ny, nx):
    if layout == "x2":  # x closest, every second element
        return flat[: nz * ny * nx * 2].view(nz, ny, 2 * nx)[:, :, ::2]
    if layout == "y":   # y closest
        return flat[: nz * (nx + 1) * ny].view(nz, nx + 1, ny)[:, :nx].permute(0, 2, 1)
    return flat[: nx * ny * (nz + 1)].view(nx, ny, nz + 1)[:, :, :nz].permute(2, 1, 0)


@pytest.mark.parametrize("layout", ["x2", "y", "z"])
@pytest.mark.parametrize("dims,rate", [((9, 33, 70), 16), ((8, 64, 2048), 13),
                                       ((16, 1024, 1024), 8), ((11, 519, 2691), 16)])
def test_strided_arrays(zfpx_lib, layout, dims, rate):
    nz, ny, nx = dims
    rng = np.random.default_rng(nx + len(layout))
    a = rng.standard_normal((nz, ny, nx), dtype=np.float32)
    flat = torch.zeros(2 * (nz + 1) * ny * (nx + 1), device=DEV)
    src = _view(flat, layout, *dims)
    src.copy_(torch.from_numpy(a).to(DEV))
    want = oracle.encode_regular(a, rate)
    words = zfpx_lib.zfpx_encode_fixed_rate(src, rate)
    torch.cuda.synchronize()
    assert np.array_equal(words.cpu().numpy().view(np.uint64), want)
    mark = torch.full_like(flat, 7.5)
    zfpx_lib.zfpx_decode_fixed_rate(words, rate, _view(mark, layout, *dims))
    torch.cuda.synchronize()
    back = torch.from_numpy(oracle.decode_regular(want, dims, rate)).to(DEV)
    expect = torch.full_like(flat, 7.5)
    _view(expect, layout, *dims).copy_(back)
    assert torch.equal(mark.view(torch.int32), expect.view(torch.int32))
