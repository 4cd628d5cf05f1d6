"""Workgroups of the tiled linear layer share its columns: what one fetches of the residual and stores of the output (run_chunk in
csrc/vit_run.h) is its own run, every column once.  With residual and output in one buffer anything else is a race."""
import os
import re
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2109_10060_amd", "csrc")
PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "vit_run.h"
int main() {
    for (int nw : {4, 8, 12})
        for (int run_blocks : {1, 2, 4, 8, 12})
            for (int total = 1; total <= 52; ++total) {
                std::vector<int> owner(4 * total, -1);
                for (int run = 0; run * run_blocks < total; ++run) {
                    const int blk0 = run * run_blocks, blk1 = total < blk0 + run_blocks ? total : blk0 + run_blocks;
                    for (int b0 = blk0; b0 < blk1; b0 += nw)
                        for (int c = 0; c < 16 * ((4 * nw + 15) / 16); ++c) {      // the lanes of a row: 16 chunks a turn
                            if (!run_chunk(c, nw, b0, blk1)) continue;
                            const int at = 4 * b0 + c;
                            if (at >= 4 * total || owner[at] >= 0) return printf("%d %d %d: chunk %d\n", nw, run_blocks, total, at), 1;
                            owner[at] = run;
                        }
                }
                for (int at = 0; at < 4 * total; ++at)
                    if (owner[at] != at / 4 / run_blocks) return printf("%d %d %d: nobody's chunk %d\n", nw, run_blocks, total, at), 1;
            }
    return 0;
}
"""


def test_a_run_touches_its_own_columns_alone(tmp_path):
    src, exe = tmp_path / "run.cpp", tmp_path / "run"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout


def test_residual_and_output_ask_the_same_question():
    kernel = open(os.path.join(CSRC, "vit_linear.hip")).read()
    for access in (r"= \*\(const uint4\*\)\(res \+", r"\*\(uint4\*\)\(y \+"):
        at = [m.start() for m in re.finditer(access, kernel)]
        assert len(at) == 1 and "run_chunk(c, NW, b0, blk1)" in kernel[at[0] - 500:at[0]], access


SEGMENTS = r"""
#include <cstdio>
#include "vit_run.h"
int main() {
    for (int nb = 1; nb <= 52; ++nb)
        for (int p = 0; p < RUN_SEGMENTS * nb; ++p)
            if (run_segment(p, nb) != p / nb) return printf("%d of %d\n", p, nb), 1;
    return run_segment(RUN_SEGMENTS, 1) == RUN_SEGMENTS;       // (one more is beyond it)
}
"""


# the segment of a block by comparisons holds for as many segments as the launcher takes
def test_segments(tmp_path):
    src, exe = tmp_path / "seg.cpp", tmp_path / "seg"
    src.write_text(SEGMENTS)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    launcher = open(os.path.join(CSRC, "vit_linear.hip")).read().split("int32_t ds_launch_vit_linear")[1]
    assert "a.n_seg > RUN_SEGMENTS) return DS_EUNSUPPORTED" in launcher.split("launch<")[0]
