"""The buffer offsets of a 2 x 2 tile's outputs (csrc/tile_offsets.h), compiled
for the host: on outputs just below the 2^29-element limit every offset is
either its element's own or outside the buffer, also where a map of odd height
or width leaves the last tiles without a second row or column."""
import os
import subprocess

import pytest

from paper_1903_06934_amd import build

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "tile_offsets.h"
using namespace miconv;
int main(int, char **v)
{
    const long long N = atoll(v[1]), K = atoll(v[2]), P = atoll(v[3]), Q = atoll(v[4]);
    const uint32_t bytes = (uint32_t)(N * K * P * Q * 4);
    long long bad = 0, n = 0;
    // Every tile of the first and the last two planes, and a plane past the
    // last (a row of the GEMM tile that holds no channel).
    for (long long nk = 0; nk <= N * K; nk += nk == 1 && N * K > 4 ? N * K - 3 : 1)
        for (long long p = 0; p < P; p += 2)
            for (long long q = 0; q < Q; q += 2) {
                const uint32_t o = (uint32_t)(((nk * P + p) * Q + q) * 4);
                const bool in = nk < N * K;
                const TileOffsets t = tile_offsets(o, (uint32_t)Q * 4u, in, p + 1 < P, q + 1 < Q);
                for (int k = 0; k < 4; k++, n++) {
                    const long long r = p + k / 2, c = q + k % 2;
                    const bool real = in && r < P && c < Q;
                    const uint32_t want = (uint32_t)(((nk * P + r) * Q + c) * 4);
                    bad += real ? t.at[k] != want : t.at[k] < bytes;
                }
            }
    std::printf("%lld of %lld\n", bad, n);
    return bad != 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("offsets")
    src, exe = d / "main.cpp", d / "main"
    src.write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", build.CSRC, str(src), "-o", str(exe)], check=True)
    return str(exe)


@pytest.mark.parametrize("dims", [
    (1, 512, 1025, 1023),   # odd height and width, 512 elements below the limit
    (1, 4, 8191, 16386),    # odd height, even width, 8 below
    (1, 512, 1024, 1023),   # even height, odd width
    (2, 3, 7, 5),
], ids=lambda d: "x".join(map(str, d)))
def test_offsets_are_the_elements_or_outside(program, dims):
    n, k, p, q = dims
    assert n * k * p * q < 1 << 29
    r = subprocess.run([program] + [str(v) for v in dims], capture_output=True, text=True)
    assert r.returncode == 0, f"{r.stdout.strip()} offsets are wrong"
