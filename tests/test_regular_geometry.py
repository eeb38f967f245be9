"""Where the kernels read and write the blocks of a regular array, over sizes
up to the largest that the entry points take (rows of more than 2^31 points
among them): the geometry's own code, built for the host under the address and
undefined-behaviour sanitizers, against 64-bit arithmetic."""
import os
import subprocess

import pytest
from test_host_sanitizers import SAN, _have_asan

pytestmark = pytest.mark.skipif(not _have_asan(), reason="gcc sanitizer runtimes not installed")

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def dump_exe(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("geo") / "regular_geo_dump")
    subprocess.run(["g++", "-std=c++17", *SAN, "-Wno-unknown-pragmas",
                    os.path.join(HERE, "host", "regular_geo_dump.cpp"), "-o", out], check=True)
    return out


def _want(nx, ny, nz, sx, sy, sz, b):
    nbx, nby = -(-nx // 4), -(-ny // 4)
    bx, by, bz = b % nbx, b // nbx % nby, b // (nbx * nby)
    pos, inside = [], 0
    for i in range(64):
        x, y, z = 4 * bx + i % 4, 4 * by + i // 4 % 4, 4 * bz + i // 16
        pos.append(min(x, nx - 1) * sx + min(y, ny - 1) * sy + min(z, nz - 1) * sz)
        inside |= int(x < nx and y < ny and z < nz) << i
    return pos, inside


B31, B32 = 1 << 31, 1 << 32


@pytest.mark.parametrize("dims", [
    (5, 9, 7), (257, 5, 3), (3, 700, 2), (1 << 20, 33, 5),
    ((1 << 30) + 3, 2, 4), (B31 - 1, 1, 1), (B31, 1, 1), (B31 + 301, 4, 4), (B32 - 2, 3, 1),
    (B32, 1, 2), (B32 + 5, 1, 1), (4 * (B31 - 1), 1, 1), (1, 4 * (B31 - 1), 1),
    (3, 1, 4 * (B31 - 1)),
])
@pytest.mark.parametrize("form", ["unit", "strided"])
def test_blocks_of_regular_arrays(dump_exe, dims, form):
    nx, ny, nz = dims
    st = (1, nx + 5, (nx + 5) * ny + 1) if form == "unit" else (-3, 3 * nx + 2, 5 * nx * ny)
    nbx = -(-nx // 4)
    nb = nbx * -(-ny // 4) * -(-nz // 4)
    assert nb < B31
    tiles = -(-nb // 64)
    near = [0, nb // 2, nb - 1, nbx - 1, nbx]
    near += [b + r * nbx for b in (1 << 28, 1 << 29, 1 << 30) if b < nbx for r in range(nb // nbx)]
    picks = sorted({min(max(b // 64 + d, 0), tiles - 1) for b in near for d in (-1, 0, 1)})
    text = " ".join(map(str, (*dims, *st)))
    text += "".join(f" {64 * t} {min(64, nb - 64 * t)}" for t in picks)
    p = subprocess.run([dump_exe], input=text, capture_output=True, text=True)
    assert p.returncode == 0, p.stderr[-2000:]
    seen, runs = 0, 0
    for line in p.stdout.splitlines():
        tag, b, *rest = line.split()
        pos, inside = _want(*dims, *st, int(b))
        assert [int(v) for v in rest] == pos + [inside], (tag, b)
        seen += tag == "b"
        runs += tag == "r"
    assert seen == sum(min(64, nb - 64 * t) for t in picks)
    if form == "unit" and nbx >= 1024:
        assert runs > 0


@pytest.mark.parametrize("dims", [(1 << 24, 1 << 24, 1 << 24), (1 << 23, 1 << 23, 1 << 23),
                                  (B32, B31, 4), ((1 << 63) - 1, 2, 2), (4 * B31, 1, 1)])
def test_more_blocks_than_an_array_may_have(dims):
    """Counts past 2^31 - 1, also where the product of the three passes 64
    bits, are refused: nothing is launched on a count that wrapped."""
    from paper_2609_24294_amd import zfpx
    nx, ny, nz = dims
    blocks = -(-nx // 4) * -(-ny // 4) * -(-nz // 4)
    L, fake = zfpx.library(), 4096  # never dereferenced
    if blocks * 8 * 16 >= 1 << 63:
        assert L.zfpx_fixed_rate_bytes(nx, ny, nz, 16) == zfpx.EINVAL
    else:
        assert L.zfpx_fixed_rate_bytes(nx, ny, nz, 16) == blocks * 8 * 16
    assert L.zfpx_encode_fixed_rate(fake, nx, ny, nz, 1, 0, 0, 16, fake, (1 << 64) - 1,
                                    None) == zfpx.EINVAL
    assert L.zfpx_decode_fixed_rate(fake, (1 << 64) - 1, nx, ny, nz, 1, 0, 0, 16, fake,
                                    None) == zfpx.EINVAL
    # no elements, whatever the other sizes: nothing to do
    assert L.zfpx_encode_fixed_rate(None, nx, 0, nz, 1, 0, 0, 16, None, 0, None) == zfpx.OK
    assert L.zfpx_fixed_rate_bytes(nx, ny, 0, 16) == 0
