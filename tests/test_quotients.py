"""The path-gradient aggregation's quotients (div_by, recip_from of k_sgm.hpp)
against the division: their source, compiled for the host, over random
mantissas, mantissas at both ends and quotients next to a rounding boundary.
The reciprocal of a mantissa of all ones alone may come out one unit low."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = r"""
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <random>
#define __device__
#define __forceinline__ inline
#define __builtin_amdgcn_div_fixup(q, b, x) (q)     // (zeros, infinities and NaN)
%s
static double bits(uint64_t u) { return __builtin_bit_cast(double, u); }
static uint64_t u64(double d) { return __builtin_bit_cast(uint64_t, d); }
int main() {
    std::mt19937_64 g(1);
    const uint64_t M = (1ull << 52) - 1;
    long bad_recip = 0, bad_div = 0;
    for (long i = 0; i < 8000000; ++i) {
        uint64_t mb = g() & M, mx = g() & M;
        const int kind = i & 7;
        if (kind == 1) mb = M - (i & 8 ? g() & 63 : 0);
        if (kind == 2) mb = g() & 63;
        if (kind == 3) mx = M - (g() & 63);
        if (kind == 4) mx = g() & 63, mb = M - (g() & 63);
        const double b = bits(mb | (1003 + g() %% 40) << 52);
        double x = bits(mx | (1003 + g() %% 40) << 52);
        if (kind == 5) x = bits(u64(bits((g() & M) | 1023ull << 52) * b) + g() %% 5 - 2);
        const double e = 1.0 / b;
        const double r = recip_from(b, bits(u64(e) + g() %% 17 - 8));
        bad_recip += r != e && !(mb == M && u64(r) + 1 == u64(e));
        bad_div += div_by(x, b, e) != x / b;
    }
    std::printf("%%ld %%ld\n", bad_recip, bad_div);
}
"""


def test_quotients_are_the_divisions(tmp_path):
    src = open(os.path.join(ROOT, "paper_2112_00821_amd", "csrc", "k_sgm.hpp")).read()
    fns = [re.search(r"__device__ __forceinline__ double %s\(.*?\n}\n" % f, src, re.S)[0] for f in ("div_by", "recip_from")]
    (tmp_path / "q.cpp").write_text(MAIN % "\n".join(f.replace("__builtin_fma", "std::fma") for f in fns))
    subprocess.run(["/opt/rocm/llvm/bin/clang++", "-std=c++17", "-O2", "-mfma", "-ffp-contract=off",
                    str(tmp_path / "q.cpp"), "-o", str(tmp_path / "q")], check=True)
    assert subprocess.run([str(tmp_path / "q")], check=True, capture_output=True, text=True).stdout.split() == ["0", "0"]
