"""Where lanes of a wavefront read from LDS what others of them have just written, the source says so: nothing but the order in which
the compiler leaves the accesses stands between them."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2109_10060_amd", "csrc")


def source(name):
    return re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, name)).read())


def test_a_wavefronts_line_of_biases_is_written_between_syncs():
    kernel = source("vit_tail.hip")
    assert len(re.findall(r"\bline\[[^\]]*\] *=", kernel)) == 1
    assert re.search(r"wave_sync\(\);\s*line\[l32\] = v;\s*wave_sync\(\);", kernel)
    assert "wave_sync" in source("tile_out.h") and '#include "tile_out.h"' in kernel


# of a turn's barrier a wavefront meets exactly one: the late ones theirs, the others theirs
def test_a_turn_of_the_hidden_tiles_has_one_barrier_a_wavefront():
    kernel = source("vit_tail.hip")
    loop = kernel[kernel.index("for (int hc = 0;"):kernel.index("cst = columns(b2")]
    assert len(re.findall(r"\bturn\(\)", loop)) == 2
    assert re.search(r"if \(!late\) \{\s*turn\(\);", loop) and re.search(r"if \(late\) turn\(\);", loop)
    assert re.findall(r"[^\n]*__syncthreads\(\)[^\n]*", loop) == [x for x in re.findall(r"[^\n]*__syncthreads\(\)[^\n]*", loop) if "!TWO" in x]
