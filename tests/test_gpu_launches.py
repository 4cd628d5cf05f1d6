"""The launches of a forward pass are the ones the work model counts: its records, class by class, are what bench.py holds
against the measured durations."""
import collections

import pytest
import torch

import workloads as WL
from paper_2109_10060_amd import cost

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
GEMM = ("gemm", "gemm_taps", "conv3", "thin", "tail", "small", "vit_linear")
PP = dict(embed=416, heads=8, head_dim=48, mlp=1664, depth=14, routes="pp", stem_dim=24, patch=8)
NETS = {
    "mbnet": (WL.mbnet_arch, WL.mbnet_params, "build_mbnet", cost.mbnet_cost, (1, 96, 256)),
    "mbnet_48": (lambda: WL.mbnet_arch(image=48), WL.mbnet_params, "build_mbnet", cost.mbnet_cost, (3,)),
    "mbnet_pp": (WL.mbnet_pp_arch, WL.mbnet_params, "build_mbnet", cost.mbnet_cost, (1, 96)),
    "resnet": (WL.resnet_arch, WL.resnet_params, "build_resnet", cost.resnet_cost, (1, 8, 33, 256)),
    "resnet_pp": (lambda: WL.resnet_arch(blocks=(3, 4, 8, 3), routes="pp"), WL.resnet_params, "build_resnet", cost.resnet_cost,
                  (9, 64, 256)),
    "resnet_half": (lambda: WL.resnet_arch(image=64, width_div=2), WL.resnet_params, "build_resnet", cost.resnet_cost, (4, 256)),
    "vit": (WL.vit_arch, WL.vit_params, "build_vit", cost.vit_cost, (1, 5, 16, 256)),
    "vit_13_heads": (lambda: WL.vit_arch(heads=13, head_dim=32, depth=2), WL.vit_params, "build_vit", cost.vit_cost, (2, 64)),
    "vit_15_heads": (lambda: WL.vit_arch(heads=15, head_dim=32, depth=2), WL.vit_params, "build_vit", cost.vit_cost, (2, 64)),
    "vit_wide": (lambda: WL.vit_arch(embed=432, mlp=1728, depth=2), WL.vit_params, "build_vit", cost.vit_cost, (2, 64)),
    "vit_pp": (lambda: WL.vit_arch(**PP), WL.vit_params, "build_vit", cost.vit_cost, (8, 64)),
}


@pytest.mark.parametrize("name", NETS)
def test_launches_follow_the_work_model(gpu_lib, name):
    make, params, build, work, batches = NETS[name]
    arch = make()
    net = getattr(gpu_lib, build)(arch, params(arch, 41), DEV)
    for B in batches:
        gen = torch.Generator(device=DEV)
        gen.manual_seed(B)
        imgs = torch.randn((B, 3, arch["image"], arch["image"]), generator=gen, device=DEV).to(torch.bfloat16)
        # the deepest route among them, so that every block has a sample
        over = (net.T - 1 - torch.arange(B, dtype=torch.int32, device=DEV) % net.T).expand(net.n_gates, B).contiguous()
        gpu_lib.ds_profile_reset()
        gpu_lib.ds_profile_enable(True)
        try:
            _, routes = gpu_lib.ds_forward(net, imgs, route_override=over)
        finally:
            gpu_lib.ds_profile_enable(False)
        got = collections.Counter("gemm" if k in GEMM else k for k, _ in gpu_lib.ds_profile_launches())
        gpu_lib.ds_profile_reset()
        want = collections.Counter("gemm" if r["kind"] in GEMM else r["kind"] for r in work(arch, routes.cpu().numpy()).launches)
        for k in ("gemm", "dwconv", "attention", "layernorm", "stem", "maxpool"):
            assert got[k] == want[k], (B, k, got, want)
