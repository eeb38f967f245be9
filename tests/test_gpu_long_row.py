"""A row of more than 2^31 points (8.6 GB) through the direct calls and the
serving loop, at the places where 32 bits of a position end: GPU against the
CPU oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
RATE = 2


def test_row_beyond_2_31_points(zfpx_lib):
    nx = (1 << 31) + 301
    total = torch.cuda.get_device_properties(0).total_memory
    assert total > 8 * nx * 4
    a = torch.empty(nx, device=DEV)
    rng = np.random.default_rng(231)
    tile = torch.from_numpy(rng.standard_normal(1 << 20).astype(np.float32)).to(DEV)
    for i in range(0, nx, tile.numel()):  # each stretch scaled by its own number
        n = min(tile.numel(), nx - i)
        torch.mul(tile[:n], 1.0 + i / tile.numel(), out=a[i: i + n])
    view = a.view(1, 1, nx)
    words = zfpx_lib.zfpx_encode_fixed_rate(view, RATE)
    back = torch.full((nx + 64,), float("nan"), device=DEV)
    zfpx_lib.zfpx_decode_fixed_rate(words, RATE, back[:nx].view(1, 1, nx))
    torch.cuda.synchronize()
    assert torch.isnan(back[nx:]).all()
    for at in (0, 1 << 30, (1 << 31) - 4096, 3 << 29, nx // 4 * 4 - 4096):
        x0, x1 = max(0, at - 4096), min(nx, at + 4400)
        part = a[x0:x1].cpu().numpy().reshape(1, 1, -1)
        want = oracle.encode_regular(part, RATE)
        got = words[x0 // 4 * RATE: (x1 + 3) // 4 * RATE].cpu().numpy().view(np.uint64)
        assert np.array_equal(got, want), at
        dec = oracle.decode_regular(want, part.shape, RATE)
        got = back[x0:x1].cpu().numpy()
        assert np.array_equal(got.view(np.uint32), dec.reshape(-1).view(np.uint32)), at
    served = torch.zeros_like(words)
    again = torch.zeros_like(back)
    torch.cuda.synchronize()
    sv = zfpx_lib.Server(64 << 30, max_slots=4)
    try:
        sv.submit(zfpx_lib.make_request(0, RATE, view, served))
        sv.submit(zfpx_lib.make_request(1, RATE, again[:nx].view(1, 1, nx), words))
        sv.drain(60.0)
    finally:
        sv.close()
    torch.cuda.synchronize()
    assert torch.equal(served, words)
    assert torch.equal(again[:nx], back[:nx]) and not again[nx:].any()
