"""The short GELU of the transformer kernels (csrc/gelu_poly.h) against the exact one in double precision, for every fp32 value
from 2^-14 to its limit and every 4099th below: its error and the exact form's have to stay inside the slack by which it
decides a bf16 rounding."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <thread>
#include <vector>
#include "gelu_poly.h"

static float value(uint32_t b) { float x; memcpy(&x, &b, 4); return x; }
static uint32_t bits(float x) { uint32_t b; memcpy(&b, &x, 4); return b; }

static double worst(uint32_t from, uint32_t to, uint32_t step, float sign) {
    double e = 0;
    for (uint32_t b = from; b <= to; b += step) {
        const float x = sign * value(b);
        const double g = 0.5 * (double)x * (1.0 + erf((double)x * 0.70710678118654752440));
        e = std::fmax(e, std::fabs(gelu_poly(x) - g) / std::fabs((double)x));
    }
    return e;
}

int main() {
    const uint32_t lo = bits(std::ldexp(1.f, -14)), hi = bits(GELU_LIMIT), tiny = bits(std::ldexp(1.f, -100));
    const int n = 8;
    std::vector<double> e(2 * n + 2);
    std::vector<std::thread> t;
    for (int i = 0; i < 2 * n; ++i)
        t.emplace_back([&e, i, lo, hi] { e[i] = worst(lo + i / 2, hi, n, i % 2 ? -1.f : 1.f); });
    for (int i = 0; i < 2; ++i)
        t.emplace_back([&e, i, lo, tiny] { e[2 * n + i] = worst(tiny, lo, 4099, i ? -1.f : 1.f); });
    for (auto& th : t) th.join();
    double m = 0;
    for (double v : e) m = std::fmax(m, v);
    printf("%.9g %.9g\n", m, (double)GELU_SLACK);
}
"""
# 0.5 x (1 + erff(x / sqrt 2)) in fp32: the argument's rounding moves erf by at most 0.25 ulp of 1 (|t exp(-t^2)| 2 / sqrt pi < 0.5),
# erff is good to 1 ulp of 1, the sum and the product round once each: below 0.5 (0.25 + 1 + 1) 2^-24 + 2^-24 of |x|
ERF_FORM = 2.2 * 2.0 ** -24


def test_short_gelu_is_inside_its_slack(tmp_path):
    src, exe = tmp_path / "gelu.cpp", tmp_path / "gelu"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-march=native", "-ffp-contract=off", "-pthread", "-I",
                    os.path.join(ROOT, "paper_2109_10060_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    error, slack = map(float, subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split())
    assert 1e-8 < error < 1.6e-7
    # the bounds lo and hi round once each: half an ulp of a value below |x|
    assert error + ERF_FORM + 2.0 ** -24 < slack


HALVES = r"""
#include <cstdint>
#include <cstdio>
#include <cstring>
#include "gelu_poly.h"

static float value(uint32_t b) { float x; memcpy(&x, &b, 4); return x; }

int main() {
    uint32_t hi;
    const float limit = GELU_LIMIT;
    memcpy(&hi, &limit, 4);
    for (uint32_t b = 0x01000000u; b <= hi; b += b < 0x38000000u ? 997 : 7)          // from 2^-125 on
        for (int minus = 0; minus < 2; ++minus) {
            const float x = minus ? -value(b) : value(b), want = gelu_poly(x);
            float u, s, p;
            for (int l = 0; l <= GELU_TERMS; ++l) gelu_step<true>(l, 0.5f * x, u, s, p);
            if (memcmp(&p, &want, 4)) return printf("%.9g: %.9g %.9g\n", x, p, want), 1;
        }
}
"""


# transformer blocks evaluate it from half of a value (gelu_step<true>): the same bits, and nothing on the way is larger than the value
def test_halves_have_the_bits_of_the_values(tmp_path):
    src, exe = tmp_path / "halves.cpp", tmp_path / "halves"
    src.write_text(HALVES)
    subprocess.run(["g++", "-O2", "-std=c++17", "-march=native", "-ffp-contract=off", "-I",
                    os.path.join(ROOT, "paper_2109_10060_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
