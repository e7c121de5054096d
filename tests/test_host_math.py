"""Integer helpers of the kernels that the host prepares, run on the CPU: a small
program over csrc/common.h compares them with plain division."""
import os
import subprocess

import pytest

from paper_2609_24456_amd import build as B

pytestmark = pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="hipcc not installed")

PROGRAM = r"""
#include <cstdio>
#include "common.h"
using namespace conduit;

static unsigned long long bad = 0, seen = 0;

static void check(uint64_t got, uint64_t want, const char* what, uint64_t n, uint64_t d) {
    ++seen;
    if (got != want && bad++ < 10)
        printf("%s(%llu, %llu) = %llu, not %llu\n", what, (unsigned long long)n, (unsigned long long)d,
               (unsigned long long)got, (unsigned long long)want);
}

int main() {
    uint64_t x = 88172645463325252ull;
    auto rnd = [&] { x ^= x << 13; x ^= x >> 7; x ^= x << 17; return x; };
    // numbers below 2^31 by any divisor: around multiples of it and at the ends
    for (int k = 0; k < 200000; ++k) {
        const uint64_t d = k < 4096 ? k + 1 : (rnd() >> (33 + k % 30)) + 1;
        if (d >= 1ull << 31) continue;
        const Div31 v = make_div31((uint32_t)d);
        const uint64_t q = rnd() % (((1ull << 31) - 1) / d + 1);
        const uint64_t at[] = {0, q * d, q * d + d - 1, q * d ? q * d - 1 : 0, (1ull << 31) - 1, rnd() >> 33};
        for (uint64_t n : at)
            if (n < 1ull << 31) check(div31((uint32_t)n, v), n / d, "div31", n, d);
    }
    // planes of frames of up to 2^32 units: the ends of every plane
    for (int64_t c = 1; c <= 4; ++c)
        for (int k = 0; k < 50000; ++k) {
            const int64_t p = k < 100 ? k + 1 : k == 100 ? (1ll << 32) / c : 1 + (int64_t)((rnd() >> (32 + k % 32)) / c);
            if (c * p > 1ll << 32) continue;
            const Planes v = make_planes((int32_t)c, p);
            check(v.n, c, "planes", c, p);
            for (int64_t q = 0; q < c; ++q) {
                check(plane_of((uint32_t)(q * p), v), q, "plane_of", q * p, p);
                check(plane_of((uint32_t)(q * p + p - 1), v), q, "plane_of", q * p + p - 1, p);
            }
        }
    (void)make_planes(3, 0);  // a minibatch of columns alone
    printf("%llu compared, %llu wrong\n", seen, bad);
    return bad != 0;
}
"""


def test_divisions_against_plain_ones(tmp_path):
    src, exe = tmp_path / "math.hip", tmp_path / "math"
    src.write_text(PROGRAM)
    cmd = [B.HIPCC, "-O1", "-std=c++17", "--cuda-host-only", "-I", B.INCLUDE, "-I", B.CSRC, str(src), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
    assert " 0 wrong" in r.stdout
