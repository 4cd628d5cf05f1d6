"""The algorithmic-work model behind bench.py's roofline numerators, checked against the oracle's multiply-add
counts (which are pinned to the figures the paper prints) and against hand counts of bytes."""
import subprocess
import sys
import os

import numpy as np

import workloads as WL
from oracle import ds_oracle as O
from paper_2109_10060_amd import cost as C

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _macs(cost, kinds):
    return sum(cost[k]["flops"] for k in kinds if k in cost) / 2.0


def test_full_width_flops_equal_the_multiply_add_counts():
    B = 3
    a = WL.mbnet_arch()
    c = C.mbnet_cost(a, np.full(B, a["T"] - 1))
    want = O.madds_mbnet(a, a["cin"][-1], a["cout"][-1], int(a["cout"][-1, -1]))
    assert abs(_macs(c, ["stem", "dwconv", "gemm", "head"]) / B - want) / want < 1e-9
    r = WL.resnet_arch()
    c = C.resnet_cost(r, np.full((4, B), 3))
    want = O.madds_resnet(r, r["mid"][:, 3], r["out"][:, 3])
    assert abs(_macs(c, ["stem", "gemm", "gemm_taps", "head"]) / B - want) / want < 1e-9
    v = WL.vit_arch(routes="diag")
    c = C.vit_cost(v, np.full(B, 3))
    d_e, h, hid = (int(x) for x in v["routes"][3])
    want = O.madds_vit(v, d_e, h, hid)
    assert abs(_macs(c, ["gemm", "attention", "head"]) / B - want) / want < 1e-9


def test_sliced_routes_cost_less_and_depth_routes_skip_layers():
    r = WL.resnet_arch()
    full = C.resnet_cost(r, np.full((4, 8), 3))
    quarter = C.resnet_cost(r, np.zeros((4, 8), np.int64))
    assert quarter["gemm_taps"]["flops"] * 15.9 < full["gemm_taps"]["flops"] < quarter["gemm_taps"]["flops"] * 16.1   # r^2
    d = WL.resnet_arch(routes="depth")
    shallow = C.resnet_cost(d, np.full((4, 8), 6))       # ratio 1.0, one block fewer per stage
    deep = C.resnet_cost(d, np.full((4, 8), 7))
    assert shallow["gemm_taps"]["launches"] == deep["gemm_taps"]["launches"] - 4
    v = WL.vit_arch(routes="depth")
    c10 = C.vit_cost(v, np.full(4, 9))                    # widest route, depth - 2
    c12 = C.vit_cost(v, np.full(4, 11))
    assert c12["attention"]["launches"] - c10["attention"]["launches"] == 2
    assert abs(c12["attention"]["flops"] / c10["attention"]["flops"] - 12 / 10) < 1e-9


def test_gemm_bytes_count_each_operand_once():
    # one 1x1 layer, 2 samples of 5 rows, widths 8 -> 16 and 16 -> 32: in + out (bf16) + the union of the weight slices
    c = C.Cost()
    C._gemm(c, "gemm", 5, 5, 1, [8, 16], [16, 32])
    assert c["gemm"]["flops"] == 2 * 5 * (8 * 16 + 16 * 32)
    assert c["gemm"]["bytes"] == 2 * 5 * (8 + 16) + 2 * 5 * (16 + 32) + 2 * 16 * 32


def test_bench_refuses_more_than_one_gpu():
    p = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert p.returncode != 0 and "one GPU" in (p.stderr + p.stdout)


def test_records_add_up_to_the_class_totals_and_name_no_work_twice():
    v = WL.vit_arch()
    for arch, work, gates in ((WL.mbnet_arch(), C.mbnet_cost, 1), (WL.mbnet_pp_arch(), C.mbnet_cost, 1),
                              (WL.resnet_arch(), C.resnet_cost, 4), (v, C.vit_cost, 1),
                              (WL.vit_arch(stem_dim=24, patch=8), C.vit_cost, 1)):
        for B in (1, 64, 256):
            c = work(arch, np.stack([np.arange(B) % arch["T"]] * gates))
            for kind, total in c.items():
                mine = [r for r in c.launches if r["kind"] == kind]
                assert len(mine) == total["launches"]
                for key in ("flops", "bytes"):
                    assert abs(sum(r[key] for r in mine) - total[key]) <= 1e-9 * total[key] or kind == "inside"
    # the LayerNorms of the blocks run inside other launches and move nothing of their own; the final one reads 64 class tokens
    c = C.vit_cost(v, np.full(64, v["T"] - 1))
    assert c["layernorm"]["bytes"] == 4 * 64 * 384 and c["layernorm"]["launches"] == 1
    assert c["inside"]["bytes"] == 0 and c["inside"]["flops"] == 8 * 64 * v["tokens"] * 384 * 24


# the projection of a bottleneck block that is one launch counts with the 1x1 work, but its bytes are not those of the launch before it
def test_work_is_booked_to_the_launch_that_does_it():
    r = WL.resnet_arch()
    c = C.resnet_cost(r, np.full((4, 256), 3))
    rows = C.as_launched(c.launches)
    assert [x["kind"] for x in rows] == [x["kind"] for x in c.launches] and not any("next launch" in x["name"] for x in rows)
    first, block = (next(x for x in rows if x["name"].startswith(n)) for n in ("s0.b0.c1", "s0.b0.c2"))
    assert first["name"] == "s0.b0.c1" and "s0.b0.proj" in block["name"]
    px, m, o = 256 * 56 * 56, int(r["mid"][0, 3]), int(r["out"][0, 3])
    assert first["flops"] == 2 * px * 64 * m and first["bytes"] == 2 * px * (64 + m) + 2 * 64 * m
    assert block["flops"] >= 2 * px * (9 * m * m + m * o + 64 * o)
    for key in ("flops", "bytes"):
        assert abs(sum(x[key] for x in rows) - sum(x[key] for x in c.launches)) < 1e-9 * sum(x[key] for x in rows)


def test_the_hash_of_the_contraction_kernels_covers_their_headers():
    import re
    from paper_2109_10060_amd import profiling
    own = set(os.listdir(os.path.join(profiling.HERE, "csrc")))
    for f in profiling.KERNEL_SOURCES:
        for h in re.findall(r'#include "([^"]+)"', open(os.path.join(profiling.HERE, f)).read()):
            assert h not in own or "csrc/" + h in profiling.KERNEL_SOURCES, (f, h)
