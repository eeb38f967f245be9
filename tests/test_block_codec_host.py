"""The library's per-block coder and decoder, built for the host under the
address and undefined-behaviour sanitizers in slices of just the words that a
lane has on the device, against the oracle, bit for bit: any access outside the
slice fails, which on the device would silently change a neighbour's."""
import os
import subprocess

import numpy as np
import pytest
from _blocks import block_families
from test_host_sanitizers import REPORT, SAN, _have_asan

import oracle

HERE = os.path.dirname(os.path.abspath(__file__))
pytestmark = pytest.mark.skipif(not _have_asan(), reason="gcc sanitizer runtimes not installed")
NONE = -1074


@pytest.fixture(scope="module")
def check_exe(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("codec") / "block_codec_check")
    subprocess.run(["g++", "-std=c++17", *SAN, "-Wno-unknown-pragmas",
                    os.path.join(HERE, "host", "block_codec_check.cpp"), "-o", out], check=True)
    return out


def _run(exe, op, rate, built_for, var, maxprec, minexp, data):
    p = subprocess.run([exe, op, str(rate), str(built_for), str(int(var)), str(maxprec),
                        str(minexp), str(len(data))], input=data.tobytes(), capture_output=True)
    err = p.stderr.decode(errors="replace")
    assert p.returncode == 0 and not any(r in err for r in REPORT), err[-2000:]
    if op == "dec":
        return np.frombuffer(p.stdout, np.float32).reshape(-1, 64)
    n = len(data) * rate * 8
    return (np.frombuffer(p.stdout[:n], np.uint64).reshape(-1, rate),
            np.frombuffer(p.stdout[n:], np.uint32))


def _blocks(rng):
    """Value families, subnormal blocks, and blocks whose last coefficient
    becomes significant first or together with others (code words of more than
    64 bits, which are coded group by group)."""
    i = np.arange(64)
    sign = 1.0 - 2.0 * ((i + i // 4 + i // 16) % 2)
    last = sign * (1.0 + rng.standard_normal((40, 64)) * 2.0 ** -rng.integers(1, 24, (40, 1)))
    sparse = np.zeros((40, 64))
    for k in range(40):
        sparse[k, 63 - rng.integers(0, 3)] = rng.standard_normal()
        sparse[k, rng.integers(64)] += rng.standard_normal() * 2.0 ** -rng.integers(0, 30)
    tiny = (rng.standard_normal((60, 64)) * (rng.random((60, 64)) < 0.3)
            * 2.0 ** rng.integers(-150, -120, (60, 1)))
    return np.ascontiguousarray(np.concatenate(
        [block_families(rng, 180), last, sparse, tiny]).astype(np.float32))


def _streams(rng, n, rate):
    """Words that no encoder made: random, sparse and dense bits, and the
    smallest exponents (results that are subnormal)."""
    def w():
        return rng.integers(0, 2 ** 64, (n, rate), dtype=np.uint64)
    small = w()
    e = rng.integers(0, 14, n).astype(np.uint64)
    small[:, 0] = small[:, 0] & ~np.uint64(0x1ff) | np.uint64(1) | e << np.uint64(1)
    s = np.concatenate([w(), w() & w(), w() & w() & w() & w(), w() | w(), w() | w() | w(), small])
    s[n // 2:, 0] |= np.uint64(1)  # not an empty block
    return s


def _bits(a):
    return np.ascontiguousarray(a, np.float32).view(np.uint32)


@pytest.mark.parametrize("rate,built_for", [(1, 0), (2, 0), (3, 0), (5, 0), (8, 0), (8, 8), (13, 0),
                                            (16, 0), (16, 16), (24, 0), (31, 0), (32, 0),
                                            (32, 32)])
def test_fixed_rate(check_exe, rate, built_for):
    rng = np.random.default_rng(100 * rate + built_for)
    blocks = _blocks(rng)
    words, bits = _run(check_exe, "enc", rate, built_for, False, 32, NONE, blocks)
    want = oracle.encode_blocks(blocks, rate)
    assert np.array_equal(words, want)
    assert bits.min() >= 1 and bits.max() <= 64 * rate
    streams = np.concatenate([want, _streams(rng, 60, rate)])
    values = _run(check_exe, "dec", rate, built_for, False, 32, NONE, streams)
    assert np.array_equal(_bits(values), _bits(oracle.decode_blocks(streams, rate)).reshape(-1, 64))


@pytest.mark.parametrize("cap,built_for", [(1, 0), (2, 0), (8, 8), (11, 0), (16, 16), (32, 32)])
@pytest.mark.parametrize("maxprec,minexp", [(1, NONE), (9, NONE), (16, NONE), (32, NONE),
                                            (32, -7), (32, 3), (20, -130)])
def test_variable_size(check_exe, cap, built_for, maxprec, minexp):
    rng = np.random.default_rng(1000 * cap + maxprec - minexp)
    blocks = _blocks(rng)
    words, bits = _run(check_exe, "enc", cap, built_for, True, maxprec, minexp, blocks)
    streams = np.concatenate([words, _streams(rng, 20, cap)])
    values = _run(check_exe, "dec", cap, built_for, True, maxprec, minexp, streams)
    for b in range(len(blocks)):
        w, n = oracle.encode_block_var(blocks[b], maxprec, minexp, cap)
        assert n == bits[b] and np.array_equal(w[:cap], words[b]), b
    for b in range(len(streams)):
        v = oracle.decode_block_var(streams[b], maxprec, minexp, cap)
        assert np.array_equal(_bits(v), _bits(values[b])), b
