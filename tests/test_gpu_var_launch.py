"""The variable-size decoder on both sides of its launch rules (workgroups of
four tiles or one, by cap; rows all on 16-byte boundaries or not, by plan and by
buffer): GPU against the CPU oracle, bit for bit, other elements untouched."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_24294_amd import workloads as W

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
NONE = -1074


@pytest.mark.parametrize("cap", [16, 23, 24, 32])
@pytest.mark.parametrize("nx,off", [(520, 0), (520, 1), (519, 0), (24, 0)])
def test_decoder_launch_rules(zfpx_lib, cap, nx, off):
    nz, ny = 7, 12  # 2 x 3 rows of blocks: whole blocks, and a level short of one
    cs = W.regular_chunkset(nz, ny, nx)
    rng = np.random.default_rng(nx + cap)
    a = (np.cumsum(rng.standard_normal((nz, ny, nx)), 2) * 0.1).astype(np.float32)
    plan = zfpx_lib.Plan.from_chunkset(cs)
    src = torch.from_numpy(a.reshape(-1)).to(DEV)
    words, nd, toff = zfpx_lib.zfpx_plan_encode_var(plan, src, 28, NONE, cap)
    torch.cuda.synchronize()
    ow, ond, otoff = oracle.pack_encode_var(cs, a, 28, NONE, cap)
    assert np.array_equal(words[: int(otoff[-1])].cpu().numpy().view(np.uint32), ow)
    assert np.array_equal(nd.cpu().numpy(), ond)
    buf = torch.full((a.size + off + 9,), 7.5, device=DEV)
    zfpx_lib.zfpx_plan_decode_var(plan, words, nd, toff, 28, NONE, cap, buf[off: off + a.size])
    torch.cuda.synchronize()
    want = np.zeros(a.size, np.float32)
    oracle.decode_unpack_var(cs, ow, ond, 28, NONE, cap, want)
    got = buf.cpu().numpy()
    assert np.array_equal(got[off: off + a.size].view(np.uint32), want.view(np.uint32))
    assert (got[:off] == 7.5).all() and (got[off + a.size:] == 7.5).all()
