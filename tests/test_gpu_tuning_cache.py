"""The autotuner's cache file: entries of these kernels are taken, entries of
other versions of the kernels are timed anew."""
import re

import pytest
import torch

from paper_2609_24294_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_entries_of_other_kernels_are_passed_over(zfpx_lib, tmp_path):
    plan = zfpx_lib.Plan.from_chunkset(W.small_chunkset())
    src = torch.randn(plan.min_buffer_elems, device="cuda:0")
    stream = torch.empty(plan.nblocks * 16, dtype=torch.int64, device="cuda:0")

    def tune(path):
        return zfpx_lib.zfpx_autotune(plan, zfpx_lib.OP_ENCODE, 16, src, stream,
                                      torch.empty_like(src), cache_path=str(path))

    path = tmp_path / "tuned"
    assert tune(path) > 0
    assert tune(path) == -1  # its own entry
    key = path.read_text().splitlines()[-1].split("|")[0]
    own = tmp_path / "own"
    own.write_text(f"{key}|256 7 1.000\n")
    assert tune(own) == -1
    assert zfpx_lib.zfpx_plan_get_config(plan, zfpx_lib.OP_ENCODE, 16) == (256, 7)
    version = re.search(r" k(\d+) ", key + " ")
    stale = ["%s|256 7 1.000" % re.sub(r" k\d+", "", key)]  # the form without a version
    if version:
        stale.append("%s|256 7 1.000" % re.sub(r" k\d+", " k%d" % (int(version[1]) - 1), key))
    for line in stale:
        other = tmp_path / "other"
        other.write_text(line + "\n")
        assert tune(other) > 0, line
        assert zfpx_lib.zfpx_plan_get_config(plan, zfpx_lib.OP_ENCODE, 16) != (256, 7)
        assert other.read_text().splitlines()[0] == line  # kept beside the new entry
        assert tune(other) == -1
