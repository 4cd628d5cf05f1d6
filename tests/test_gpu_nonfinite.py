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


# 13 heads of 32 beside an embedding of 384: the reduction of the projection is wider than the residual rows.  The few-image launches, tiles of
# 32 rows and of 64
@pytest.mark.parametrize("B", [5, 120, 900, 1000])
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
# the few-image launches, 32- and 64-row tiles, 12 and 13 column blocks behind the attention
@pytest.mark.parametrize("kw,B", [(PP, 3), (PP, 120), (PP, 900), (PP, 2600), (WIDE_HEADS, 4), (WIDE_HEADS, 120), (WIDE_HEADS, 2600)],
                         ids=lambda v: str(v) if isinstance(v, int) else ("stem416" if "stem_dim" in v else "heads13"))
def test_vit_samples_stay_apart(gpu_lib, kw, B):
    arch, params = _vit(gpu_lib, kw)
    _samples_stay_apart(gpu_lib, gpu_lib.build_vit(arch, params, DEV), B, 64)


# (300 images of a ResNet: 3x3 layers on tiled filters, of either stride)
@pytest.mark.parametrize("kind,B", [(k, B) for k in ("mbnet", "mbnet_pp", "resnet") for B in (5, 67)] + [("resnet", 300)])
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


# Depthwise filters: an output sees the pixels under its taps and no others, channel by channel
@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("H,W,C,k", [(14, 14, 72, 3), (14, 15, 40, 7), (29, 31, 24, 5), (7, 7, 136, 7), (9, 60, 8, 1)])
def test_depthwise_pixels_stay_apart(gpu_lib, H, W, C, k, stride):
    B, K, pad = 3, 7, k // 2
    x = _randn((B, H, W, C), 31 + C)
    w = _randn((K, K, C), 32 + C)
    one, zero = torch.ones((1, C), device=DEV), torch.zeros((1, C), device=DEV)
    off = torch.tensor([0, B], dtype=torch.int32, device=DEV)
    g = gpu_lib.make_groups(off, None, [C])

    def run(x, act):
        y, res = gpu_lib.ds_sliced_dwconv_spatial(x, w, one, zero, g, [k], [1], [pad], stride, act=act)
        ho, wo = res[0]
        return y[:, :ho * wo].reshape(B, ho, wo, C)

    for value in (float("nan"), float("inf"), float("-inf")):
        b, c, i, j = 1, C - 3, H // 2, W // 2
        bad = x.clone()
        bad[b, i, j, c] = value
        want, got, relu = run(x, gpu_lib.DS_ACT_NONE), run(bad, gpu_lib.DS_ACT_NONE), run(bad, gpu_lib.DS_ACT_RELU)
        oy = torch.arange(want.shape[1], device=DEV) * stride - pad
        ox = torch.arange(want.shape[2], device=DEV) * stride - pad
        reach = torch.zeros_like(want, dtype=torch.bool)
        reach[b, :, :, c] = ((oy <= i) & (i < oy + k))[:, None] & ((ox <= j) & (j < ox + k))[None, :]
        assert not torch.isfinite(got[reach]).any()
        # a strip with such a pixel is summed tap by tap: the order of a sum differs there, bits elsewhere do not
        strip = torch.zeros_like(reach)
        strip[b, :, :, c] = True
        assert torch.equal(got[~strip], want[~strip])
        near = strip & ~reach
        assert torch.allclose(got[near].float(), want[near].float(), rtol=1e-2, atol=1e-2), value
        assert torch.equal(relu[~reach], got[~reach].clamp(min=0))
        expect = got[reach].clamp(min=0)
        assert torch.equal(relu[reach], torch.where(torch.isnan(expect), torch.zeros_like(expect), expect))


# The same in the separable blocks in front of the gate: an image's pixel that overflows the stem reaches no further than the
# filters do
@pytest.mark.parametrize("pp", [False, True])
@pytest.mark.parametrize("image", [224, 66])
def test_front_block_pixels_stay_apart(gpu_lib, pp, image):
    arch = (WL.mbnet_pp_arch if pp else WL.mbnet_arch)(image=image)
    net = gpu_lib.build_mbnet(arch, WL.mbnet_params(arch, 12), DEV)
    B, half = 2, (image + 1) // 2
    imgs = _randn((B, 3, image, image), image)
    over = torch.zeros((1, B), dtype=torch.int32, device=DEV)
    sizes, r = [], half
    for _, co, s in arch["blocks"][:5]:
        r = (r - 1) // s + 1
        sizes.append((r, co, s))

    def run(x):
        taps = {i: torch.full((B, r * r, co), float("nan"), dtype=torch.bfloat16, device=DEV) for i, (r, co, _) in enumerate(sizes)}
        gpu_lib.ds_forward_taps(net, x, taps, route_override=over)
        return [taps[i].reshape(B, r, r, co) for i, (r, co, _) in enumerate(sizes)]

    want = run(imgs)
    lo, hi = image // 2, image // 2                       # image rows and columns that hold the value
    bad = imgs.clone()
    bad[1, :, lo, lo] = 3e38
    got = run(bad)
    lo, hi = lo // 2 - 1, hi // 2 + 1                     # of the stem's map: a 3x3 filter at stride 2, a little generous
    n = 5 if pp else 3
    for i, (r, co, s) in enumerate(sizes):
        assert not torch.equal(want[i], got[i])
        lo, hi = -(-(lo - n // 2) // s), (hi + n // 2) // s
        reach = torch.zeros((r, r), dtype=torch.bool, device=DEV)
        reach[max(lo, 0):hi + 1, max(lo, 0):hi + 1] = True
        assert torch.equal(want[i][0], got[i][0]), i
        a, b = want[i][1][~reach].float(), got[i][1][~reach].float()
        assert torch.isfinite(b).all() and (a - b).norm() <= 4e-3 * a.norm(), i


# Whatever is stored beyond a slice -- weights, channels of the activations, table entries -- takes no part in its results
def _outside(t, *keep):
    """t with everything beyond the leading keep[i] entries of axis i set to NaN."""
    inside = torch.zeros(t.shape, dtype=torch.bool, device=t.device)
    inside[tuple(slice(k) for k in keep)] = True
    return torch.where(inside, t, torch.full_like(t, float("nan")))


def _one_group(gpu_lib, B, k_in, k_out=None):
    off = torch.tensor([0, B], dtype=torch.int32, device=DEV)
    return gpu_lib.make_groups(off, None, [k_in], [k_out] if k_out else None)


@pytest.mark.parametrize("B,rows,K,N,k_in,k_out", [(1, 5, 384, 512, 200, 328), (3, 197, 384, 512, 200, 328), (64, 197, 384, 1536, 200, 1080),
                                                   (300, 197, 128, 256, 56, 136), (40, 197, 1536, 384, 808, 200)])
@pytest.mark.parametrize("act", [0, 2])
def test_linear_outside_the_slice(gpu_lib, B, rows, K, N, k_in, k_out, act):
    x, w, res = _randn((B, rows, K), 1), _randn((N, K), 2), _randn((B, rows, N), 3)
    bias = torch.randn(N, device=DEV)
    g = _one_group(gpu_lib, B, k_in, k_out)
    for r in (None, res):
        want = gpu_lib.ds_sliced_linear(x, w, bias, g, act=act, residual=r)
        got = gpu_lib.ds_sliced_linear(_outside(x, B, rows, k_in), _outside(w, k_out, k_in), _outside(bias, k_out), g, act=act,
                                       residual=None if r is None else _outside(r, B, rows, k_out))
        assert torch.isfinite(want).all() and torch.equal(got, want)


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("B,K,stride,H,C,N,c_in,c_out", [
    (1, 3, 1, 14, 128, 128, 72, 40), (2, 1, 1, 14, 264, 512, 136, 264), (3, 3, 2, 15, 64, 96, 24, 56), (64, 3, 1, 28, 128, 128, 72, 104),
    (64, 1, 1, 56, 64, 256, 40, 136), (33, 1, 2, 28, 256, 512, 136, 264), (2, 5, 1, 9, 32, 32, 8, 24)])
def test_conv_outside_the_slice(gpu_lib, f32, B, K, stride, H, C, N, c_in, c_out):
    if f32 and B > 4:
        B = 4
    nhwc, pad = (lambda t: t if f32 else t.permute(0, 2, 3, 1).contiguous()), K // 2
    dt = torch.float32 if f32 else torch.bfloat16
    x, w = _randn((B, C, H, H), 4).to(dt), (0.1 * _randn((N, C, K, K), 5)).to(dt)
    scale, shift = torch.randn((1, N), device=DEV), torch.randn((1, N), device=DEV)
    g = _one_group(gpu_lib, B, c_in, c_out)
    want = gpu_lib.ds_sliced_conv(nhwc(x), nhwc(w), scale, shift, g, stride, pad)
    got = gpu_lib.ds_sliced_conv(nhwc(_outside(x, B, c_in)), nhwc(_outside(w, c_out, c_in)), _outside(scale, 1, c_out),
                                 _outside(shift, 1, c_out), g, stride, pad)
    assert torch.isfinite(want).all() and want.abs().max() > 0 and torch.equal(got, want)


@pytest.mark.parametrize("B,H,C,c", [(2, 14, 72, 40), (33, 28, 136, 72), (3, 7, 1024, 520)])
def test_depthwise_and_rows_outside_the_slice(gpu_lib, B, H, C, c):
    x, w, w7 = _randn((B, H, H, C), 6), _randn((3, 3, C), 7), _randn((7, 7, C), 8)
    one, shift = torch.ones((1, C), device=DEV), torch.randn((1, C), device=DEV)
    g = _one_group(gpu_lib, B, c)
    bad = [_outside(t, *t.shape[:-1], c) for t in (x, w, w7, one, shift)]
    for stride in (1, 2):
        assert torch.equal(gpu_lib.ds_sliced_dwconv(x, w, one, shift, g, stride),
                           gpu_lib.ds_sliced_dwconv(bad[0], bad[1], bad[3], bad[4], g, stride))
        for k, l in ((3, 1), (5, 1), (7, 1), (7, 2)):
            a, b = (gpu_lib.ds_sliced_dwconv_spatial(v[0], v[2], v[3], v[4], g, [k], [l], [k // 2], stride)[0]
                    for v in ((x, w, w7, one, shift), bad))
            assert torch.equal(a, b)
    rows, beta = x.reshape(B, H * H, C), shift[0]
    assert torch.equal(gpu_lib.ds_sliced_layernorm(rows, one[0], beta, 1e-6, g),
                       gpu_lib.ds_sliced_layernorm(bad[0].reshape(B, H * H, C), bad[3][0], bad[4][0], 1e-6, g))


@pytest.mark.parametrize("B,N", [(2, 17), (33, 197)])
def test_attention_outside_the_slice(gpu_lib, B, N):
    D, H, dh, de, h = 192, 6, 48, 104, 3
    x, wqkv, wproj = _randn((B, N, D), 9), 0.1 * _randn((3, H * dh, D), 10), 0.1 * _randn((D, H * dh), 11)
    bqkv, bproj, res = torch.randn((3, H * dh), device=DEV), torch.randn(D, device=DEV), _randn((B, N, D), 12)
    g = _one_group(gpu_lib, B, de, h * dh)
    want = gpu_lib.ds_sliced_mhsa(x, wqkv, bqkv, wproj, bproj, H, dh, g, residual=res)
    got = gpu_lib.ds_sliced_mhsa(_outside(x, B, N, de), _outside(wqkv, 3, h * dh, de), _outside(bqkv, 3, h * dh),
                                 _outside(wproj, de, h * dh), _outside(bproj, de), H, dh, g, residual=_outside(res, B, N, de))
    assert torch.isfinite(want).all() and torch.equal(got, want)
