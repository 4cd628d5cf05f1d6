"""The quotients that kernels take of sizes (csrc/quotient.h) against integer division, with reciprocals up to two units off."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2109_10060_amd", "csrc")
PROGRAM = r"""
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <initializer_list>
#include "quotient.h"
static int bad = 0;
static void check(long long n, int d) {
    if (n < 0 || n > 2147483647LL) return;
    float lo = 1.0f / d, hi = lo;
    for (int i = 0; i < 2; ++i) lo = std::nextafterf(lo, 0.f), hi = std::nextafterf(hi, 2.f);
    for (float r : {lo, 1.0f / d, hi}) {
        if (quotient((int)n, d, r) != (int)n / d && ++bad < 9) printf("%lld / %d\n", n, d);
        if (n < (1 << 22) && quotient22((int)n, d, r) != (int)n / d && ++bad < 9) printf("%lld / %d (22)\n", n, d);
    }
}
int main() {
    uint64_t s = 1;
    auto next = [&] { s = s * 6364136223846793005ull + 1442695040888963407ull; return (uint32_t)(s >> 33); };
    auto around = [&](int d) {
        for (long long k : {0ll, 1ll, 2ll, 3ll, 4194303ll / d, 4194304ll / d, 2147483647ll / d, (long long)(next() % (2147483647u / d + 1)), (long long)(next() % (4194304u / d + 1))})
            for (long long e = -2; e <= 2; ++e) check(k * d + e, d);
        for (int i = 0; i < 8; ++i) check(next() & 0x7fffffff, d), check(next() & 0x3fffff, d);
        check(2147483647ll, d);
    };
    for (int d = 1; d <= 60000; ++d) around(d);
    for (int i = 0; i < 200000; ++i) around(1 + (int)(next() >> (next() % 30)) % 2147483647);
    return bad ? 1 : 0;
}
"""


def test_quotients(tmp_path):
    src, exe = tmp_path / "q.cpp", tmp_path / "q"
    src.write_text(PROGRAM)
    # (conversions and products out of an int's range are errors, not whatever this machine makes of them)
    subprocess.run(["g++", "-O2", "-ffp-contract=off", "-std=c++17", "-fsanitize=undefined,float-cast-overflow", "-fno-sanitize-recover=all", "-I", CSRC,
                    str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr
