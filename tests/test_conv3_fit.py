"""The input patch of a tile of the 3x3 kernel on tiled filters (csrc/conv3_fit.h): where it says that a tile of 64 or 128 pixels fits, every read of
every tap and every stored pixel stays inside the patch, wherever in its group the tile begins, for every map up to 64 x 64; and the filters' order."""
import os
import subprocess

import pytest
import torch

from paper_2109_10060_amd.net import _conv3_tiles

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2109_10060_amd", "csrc")
PROGRAM = r"""
#include <atomic>
#include <cstdio>
#include <initializer_list>
#include <thread>
#include <vector>
#include "conv3_fit.h"
std::atomic<int> fit{0}, fit2{0}, bad{0};
int width(int w) {
    for (int bm : {64, 128})
        for (int h = 1; h <= 64; ++h) {
            if (!conv3_fits(bm, w, h)) continue;
            ++fit;
            const int rows = w * h, q = w + 1, rb = w * CONV3_PITCH + CONV3_GAP;
            auto padded = [&](int m) { return conv3_padded(m / rows, m % rows / w, m % rows % w, w, h); };
            for (int g0 = 0; g0 < 2 * rows + 2 * bm; ++g0) {
                const int first = padded(g0) - (q + 1), span = padded(g0 + bm - 1) + q + 2 - first, row0 = first / q, last = first + span - 1;
                if (first < 0 || span > conv3_pixels(bm)) return printf("%d %dx%d at %d: %d pixels\n", bm, w, h, g0, span), 1;
                // the last stored pixel; the zeros behind the last row
                if (conv3_byte(last / q, last % q, row0, w) + 64 > conv3_bytes(bm) || (last / q - row0) * rb + (w + 1) * CONV3_PITCH + 64 > conv3_bytes(bm))
                    return printf("%d %dx%d at %d: behind the patch\n", bm, w, h, g0), 1;
                for (int m = g0; m < g0 + bm; ++m) {
                    const int p = padded(m) - (q + 1), at = conv3_byte(p / q, p % q, row0, w);
                    for (int u = 0; u < 3; ++u)
                        for (int v = 0; v < 3; ++v) {
                            // the tap's pixel where its row has one, else the zeros ahead of the row or behind it
                            const int t = padded(m) + (u - 1) * q + v - 1, col = m % rows % w + v;
                            const int want = conv3_byte(p / q + u, col, row0, w);
                            if (at + u * rb + v * CONV3_PITCH != want || want < 0 || want + 64 > conv3_bytes(bm)) return printf("%d %dx%d at %d: tap of %d\n", bm, w, h, g0, m), 1;
                            if (col <= w && (t < first || t > last || t / q != p / q + u || t % q != col)) return printf("%d %dx%d at %d: pixel of %d\n", bm, w, h, g0, m), 1;
                        }
                }
            }
        }
    for (int h = 1; h <= 64; ++h) {
        if (!conv3_fits2(w, h)) continue;
        ++fit2;
        const int wo = (w - 1) / 2 + 1, ho = (h - 1) / 2 + 1, rows = wo * ho, q = conv3_pitch2(w);
        auto padded = [&](int m) { return conv3_padded2(m / rows, m % rows / wo, m % rows % wo, w, h); };
        for (int g0 = 0; g0 < 2 * rows + 128; ++g0) {
            const int first = padded(g0), last = padded(g0 + 63) + 2 * q + 2;
            if (first & 1 || last - first + 1 > CONV3_PIXELS2) return printf("stride 2 %dx%d at %d: %d pixels\n", w, h, g0, last - first + 1), 1;
            for (int m = g0; m < g0 + 64; ++m)
                for (int u = 0; u < 3; ++u)
                    for (int v = 0; v < 3; ++v) {
                        const int p = padded(m) + u * q + v, at = conv3_byte2(padded(m), first) + conv3_tap2(u, v, w);
                        // the pixel's place in the patch, and its map pixel or zeros as the loader has it
                        const int iy = 2 * (m % rows / wo) + u - 1, ix = 2 * (m % rows % wo) + v - 1, s = m / rows, pr = p / q;
                        if (p < first || p > last || at != conv3_byte2(p, first) || at + 64 > CONV3_BYTES2) return printf("stride 2 %dx%d at %d: tap of %d\n", w, h, g0, m), 1;
                        const int ls = pr / (h + 1), ly = pr % (h + 1) - 1, lx = p % q - 1;
                        const bool in = iy >= 0 && iy < h && ix >= 0 && ix < w, have = lx >= 0 && lx < w && ly >= 0;
                        if (in != have || (in && (ls != s || ly != iy || lx != ix))) return printf("stride 2 %dx%d at %d: pixel of %d\n", w, h, g0, m), 1;
                    }
        }
    }
    return 0;
}
int main() {
    std::vector<std::thread> t;
    for (int i = 0; i < 8; ++i)
        t.emplace_back([i] { for (int w = 64 - i; w > 0; w -= 8) bad += width(w); });
    for (auto& th : t) th.join();
    return bad == 0 && fit > 3000 && fit2 > 3000 ? 0 : (printf("%d %d shapes\n", (int)fit, (int)fit2), 1);
}
"""


def test_a_patch_holds_what_its_taps_read(tmp_path):
    src, exe = tmp_path / "fit.cpp", tmp_path / "fit"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-pthread", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout


@pytest.mark.parametrize("n,k", [(64, 64), (40, 24), (8, 136)])
def test_order_of_the_tiled_filters(n, k):
    w = torch.randn((n, 3, 3, k)).to(torch.bfloat16)
    kc = (k + 31) // 32
    t = _conv3_tiles(w).view((n + 31) // 32, 18 * kc + 1, 2, 32, 8)
    full = torch.zeros((t.shape[0] * 32, 9, kc * 32), dtype=w.dtype)
    full[:n, :, :k] = w.reshape(n, 9, k)
    for blk in range(t.shape[0]):
        for chunk in range(kc):
            for tap in range(9):
                for half in range(2):
                    at = chunk * 32 + half * 16
                    got = t[blk, chunk * 18 + tap * 2 + half]
                    assert torch.equal(got[0], full[blk * 32:blk * 32 + 32, tap, at:at + 8])
                    assert torch.equal(got[1], full[blk * 32:blk * 32 + 32, tap, at + 8:at + 16])
