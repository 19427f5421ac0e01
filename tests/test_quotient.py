"""CPU check of the kept-reciprocal quotient (csrc/bmg_quot.h), compiled for the
host: the rounded quotient, bit for bit, over random pairs of both types, over
mantissas at and next to the powers of two (where an estimate rounds the other
way most easily), and at the ends of the range that it is used in."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = next((c for c in ("/opt/rocm/llvm/bin/clang++", shutil.which("amdclang++") or "") if os.path.exists(c)), None)
SRC = r"""
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#define __device__
#define __host__
#define __forceinline__ inline
#include "bmg_quot.h"

static uint64_t state = 88172645463325252ull;
static uint64_t rnd()
{
    state ^= state << 13;
    state ^= state >> 7;
    state ^= state << 17;
    return state;
}
// a mantissa in [1, 2): random, or within four units of 1 or 2
template <typename T> static T mantissa(int bits)
{
    const uint64_t m = rnd(), n = uint64_t(1) << bits;
    uint64_t f = m % n;
    if ((m >> 60) == 0) f = (m >> 56) % 4;
    if ((m >> 60) == 1) f = n - 1 - (m >> 56) % 4;
    return T(1) + T(f) / T(n);
}
template <typename T> static long bad(int bits, int emax, long pairs)
{
    long n = 0;
    for (long k = 0; k < pairs; ++k) {
        // exponents with 1/d, r/d, r and the remainder's product in the normal range
        const int ed = int(rnd() % (emax + 1)) - emax / 2, eq = int(rnd() % (emax + 1)) - emax / 2;
        const T d = std::ldexp(mantissa<T>(bits), ed), r = std::ldexp(mantissa<T>(bits), eq + ed / 4);
        const T s = rnd() & 1 ? r : -r;
        const T want = s / d, got = hbmg::div_by(s, d, T(1) / d);
        n += std::memcmp(&want, &got, sizeof want) != 0;
    }
    return n;
}
int main()
{
    const long f = bad<float>(23, 80, 20000000), d = bad<double>(52, 800, 20000000);
    // a diagonal above 2^126 (2^1022): its reciprocal is subnormal, the quotient is not
    long e = 0;
    for (int k = 0; k < 1000000; ++k) {
        const float a = std::ldexp(mantissa<float>(23), 126), p = std::ldexp(mantissa<float>(23), 100);
        const double b = std::ldexp(mantissa<double>(52), 1022), q = std::ldexp(mantissa<double>(52), 1000);
        e += std::fabs(hbmg::div_by(p, a, 1.0f / a) - p / a) > 1.2e-7f * (p / a);
        e += std::fabs(hbmg::div_by(q, b, 1.0 / b) - q / b) > 2.3e-16 * (q / b);
    }
    std::printf("float %ld double %ld ends %ld tiny %d %d %d\n", f, d, e, hbmg::tiny_diag(0x1p-1001),
                hbmg::tiny_diag(0.0), hbmg::tiny_diag(0x1p-1000));
    return f || d || e;
}
"""


@pytest.mark.skipif(CLANG is None, reason="no clang")
def test_kept_reciprocal_quotient_is_the_rounded_one(tmp_path):
    (tmp_path / "q.cpp").write_text(SRC)
    exe = tmp_path / "q"
    subprocess.run([CLANG, "-std=c++17", "-O2", "-mfma", "-ffp-contract=off",
                    "-I", os.path.join(ROOT, "paper_1803_02481_amd", "csrc"), str(tmp_path / "q.cpp"), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "float 0 double 0 ends 0 tiny 1 0 0" in r.stdout
