"""The default launch at the rates where the workgroup size changes: GPU against
the CPU oracle, bit for bit, for tile counts around a workgroup's."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_24294_amd import workloads as W

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("rate,wg", [(16, 64), (27, 64), (28, 128), (29, 128), (30, 64)])
@pytest.mark.parametrize("nx", [250, 255 * 4, 257 * 4 + 1])
def test_default_launch(zfpx_lib, rate, wg, nx):
    cs = W.regular_chunkset(5, 4, nx)
    rng = np.random.default_rng(nx + rate)
    a = rng.standard_normal((5, 4, nx), dtype=np.float32)
    plan = zfpx_lib.Plan.from_chunkset(cs)
    assert zfpx_lib.zfpx_plan_get_config(plan, zfpx_lib.OP_ENCODE, rate) == (wg, 0)
    assert zfpx_lib.zfpx_plan_get_config(plan, zfpx_lib.OP_DECODE, rate) == (wg, 0)
    src = torch.from_numpy(a).to(DEV)
    want = oracle.encode_regular(a, rate)
    back = oracle.decode_regular(want, a.shape, rate)
    for encode, decode in (
            (lambda: zfpx_lib.zfpx_pack_encode(plan, src.view(-1), rate),
             lambda w, d: zfpx_lib.zfpx_decode_unpack(plan, w, rate, d.view(-1))),
            (lambda: zfpx_lib.zfpx_encode_fixed_rate(src, rate),
             lambda w, d: zfpx_lib.zfpx_decode_fixed_rate(w, rate, d))):
        words = encode()
        dst = torch.full_like(src, float("nan"))
        decode(words, dst)
        torch.cuda.synchronize()
        assert np.array_equal(words.cpu().numpy().view(np.uint64), want)
        assert np.array_equal(dst.cpu().numpy().view(np.uint32), back.view(np.uint32))
