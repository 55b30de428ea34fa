"""The size of the multichannel density's scratch (host code, no GPU): work that
was captured into a graph holds its address, so no call of as many events or
fewer may replace it, whatever the process."""
import ctypes as C
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2602_06895_amd", "csrc")
LIMIT = 2 ** 28  # doubles, 2 GiB


@pytest.fixture(scope="module")
def scratch(tmp_path_factory):
    d = tmp_path_factory.mktemp("scratch")
    src = d / "s.cpp"
    src.write_text('#include "density_scratch.h"\n'
                   'extern "C" int64_t scratch(int dims, int run, int64_t n) { return msx::density_scratch(dims, run, n); }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(d / "s.so")], check=True)
    f = C.CDLL(str(d / "s.so")).scratch
    f.restype = C.c_int64
    f.argtypes = [C.c_int, C.c_int, C.c_int64]
    return f


@pytest.mark.parametrize("dims,run", [(2, 1), (10, 8), (10, 16), (22, 3), (10, 2), (60, 16)])
def test_never_falls_with_the_number_of_events(scratch, dims, run):
    rng = random.Random(dims * 100 + run)
    edge = LIMIT // (dims + 1)  # events of one channel that reach the limit
    ns = sorted({1, 2, 1000, 5000} | {max(1, edge * k // run + j) for k in range(1, run + 2) for j in (-1, 0, 1)}
                | {edge - 1, edge, edge + 1, 3 * edge} | {int(2 ** rng.uniform(0, 34)) for _ in range(300)})
    last = 0
    for n in ns:
        s = scratch(dims, run, n)
        one = (dims + 1) * n
        assert s >= last, n
        assert s >= one and s <= run * one and s <= max(one, LIMIT)
        assert s == run * one or s == max(one, LIMIT)
        last = s
