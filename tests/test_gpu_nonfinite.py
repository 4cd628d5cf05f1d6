"""What is not finite stays where it belongs: with its sample, inside a slice, within a filter's reach.  Everything else
keeps its bits."""
import numpy as np
import pytest
import torch

import workloads as WL
from oracle import ds_oracle as O
from tests.parity import relerr_max

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
PP = dict(embed=416, heads=8, head_dim=48, mlp=1664, routes="pp", stem_dim=24, patch=8)
WIDE_HEADS = dict(heads=13, head_dim=32, routes="diag")      # 416 attention channels beside an embedding of 384


def _randn(shape, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    return torch.randn(shape, generator=gen, device=DEV).to(torch.bfloat16)


def _vit(gpu_lib, kw, depth=2, seed=21):
    arch = WL.vit_arch(image=64, depth=depth, **kw)          # 17 tokens
    return arch, WL.vit_params(arch, seed)


# 13 heads of 32 beside an embedding of 384: the reduction of the projection is wider than the residual rows
@pytest.mark.parametrize("B", [5, 120, 900])
def test_vit_attention_wider_than_the_embedding(gpu_lib, B):
    arch, params = _vit(gpu_lib, WIDE_HEADS)
    net = gpu_lib.build_vit(arch, params, DEV)
    imgs = WL.images(WL.BASE_SEED + B, B, 64)
    over = (torch.arange(B, device=DEV, dtype=torch.int32) % arch["T"])[None].contiguous()
    logits, _ = gpu_lib.ds_forward(net, torch.from_numpy(imgs).to(DEV).to(torch.bfloat16), route_override=over)
    got = logits.double().cpu().numpy()
    for b in sorted({0, 1, 2, 3, B // 2, B - 2, B - 1}):
        assert relerr_max(got[b], O.forward_vit(arch, params, imgs[b], b % arch["T"])) < 2e-2, b


# Row tiles hold the rows of several samples side by side: one sample that is not finite must not reach another.  Batches for
# the few-image launches, 32-, 64- and 96-row tiles, 12 and 13 column blocks behind the attention
@pytest.mark.parametrize("kw,B", [(PP, 3), (PP, 120), (PP, 900), (PP, 2600), (WIDE_HEADS, 4), (WIDE_HEADS, 120), (WIDE_HEADS, 2600)],
                         ids=lambda v: str(v) if isinstance(v, int) else ("stem416" if "stem_dim" in v else "heads13"))
def test_vit_samples_stay_apart(gpu_lib, kw, B):
    arch, params = _vit(gpu_lib, kw)
    _samples_stay_apart(gpu_lib, gpu_lib.build_vit(arch, params, DEV), B, 64)


@pytest.mark.parametrize("B", [5, 67])
@pytest.mark.parametrize("kind", ["mbnet", "mbnet_pp", "resnet"])
def test_cnn_samples_stay_apart(gpu_lib, kind, B):
    if kind == "resnet":
        arch = WL.resnet_arch(image=64, blocks=(2, 2, 2, 2))
        net = gpu_lib.build_resnet(arch, WL.resnet_params(arch, 22), DEV)
    else:
        arch = (WL.mbnet_pp_arch if kind == "mbnet_pp" else WL.mbnet_arch)(image=64)
        net = gpu_lib.build_mbnet(arch, WL.mbnet_params(arch, 23), DEV)
    _samples_stay_apart(gpu_lib, net, B, 64)


def _samples_stay_apart(gpu_lib, net, B, image):
    imgs = _randn((B, 3, image, image), B)
    over = torch.full((net.n_gates, B), net.T - 1, dtype=torch.int32, device=DEV)
    want, _ = gpu_lib.ds_forward(net, imgs, route_override=over)
    assert torch.isfinite(want).all()
    for value in (float("nan"), float("inf"), -3e38):
        bad = sorted({1, B // 2, B - 1})
        poisoned = imgs.clone()
        poisoned[bad] = value
        got, _ = gpu_lib.ds_forward(net, poisoned, route_override=over)
        keep = torch.ones(B, dtype=torch.bool, device=DEV)
        keep[bad] = False
        assert torch.equal(got[keep], want[keep]), value


# Weights beyond a route's slice are never part of its sums, whatever they hold; slices that end inside a 16-channel step
@pytest.mark.parametrize("B", [3, 120, 900, 2600])
def test_vit_weights_outside_the_slice(gpu_lib, B):
    arch, params = _vit(gpu_lib, dict(routes="diag"))
    arch["routes"] = np.array([[200, 3, 808], [384, 6, 1536]], np.int32)
    arch["T"] = 2
    de, hd, hid = 200, 3 * arch["head_dim"], 808
    outside = {k: v.copy() for k, v in params.items()}
    for l in range(arch["depth"]):
        for name, rows, cols in [(f"l{l}.w{c}", hd, de) for c in "qkv"] + [(f"l{l}.wproj", de, hd), (f"l{l}.fc1.w", hid, de),
                                                                            (f"l{l}.fc2.w", de, hid)]:
            outside[name][rows:] = np.nan
            outside[name][:, cols:] = np.inf
    imgs = _randn((B, 3, 64, 64), B)
    over = torch.zeros((1, B), dtype=torch.int32, device=DEV)
    want, got = (gpu_lib.ds_forward(gpu_lib.build_vit(arch, p, DEV), imgs, route_override=over)[0] for p in (params, outside))
    assert torch.isfinite(want).all() and torch.equal(got, want)
