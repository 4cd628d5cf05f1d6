"""GPU parity of the kernels a dispatch picks by size, at the sizes where each can go wrong: the edges of its tiles, the
remainders of its reduction, the smallest and largest of its range.  Reference: the oracle, or torch in float64 on the CPU."""
import os
import re

import numpy as np
import pytest
import torch
import torch.nn.functional as F

import workloads as WL
from oracle import ds_oracle as O
from tests.parity import relerr, relerr_max

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2109_10060_amd", "csrc")
TOL_F32, TOL_BF16 = 1e-5, 2e-2


def dev(a, dtype=torch.float32):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV).to(dtype).contiguous()


def host(t):
    return t.detach().to(torch.float64).cpu().numpy()


def _conv_reference(x, w, bn, t, stride, pad, resid):
    y = F.conv2d(torch.from_numpy(x).double()[None], torch.from_numpy(w).double(), stride=stride, padding=pad)[0].numpy()
    co = w.shape[0]
    s = bn["gamma"][:co].astype(np.float64) / np.sqrt(bn["var"][t, :co].astype(np.float64) + 1e-5)
    y = y * s[:, None, None] + (bn["beta"][:co] - bn["mean"][t, :co] * s)[:, None, None]
    return y if resid is None else y + resid


def _conv_case(gpu_lib, B, K, stride, pad, H, W, c_in, c_out, res, f32):
    T = len(c_in)
    CI, CO = max(c_in), max(c_out)
    d = WL.nets.Draw(7000 + B + 10 * K + H + CI)
    cast = (lambda a: a) if f32 else WL.nets.as_bf16_values
    x = cast(d.normal((B, CI, H, W)))
    w = cast(d.normal((CO, CI, K, K), std=(2.0 / (CI * K * K)) ** 0.5))
    bn = WL.bn_tables(d, T, CO)
    route = d.randint(B, T)
    Ho, Wo = (H + 2 * pad - K) // stride + 1, (W + 2 * pad - K) // stride + 1
    resid = cast(d.normal((B, CO, Ho, Wo))) if res else None
    perm, inv, off = gpu_lib.ds_route_bucket(dev(route, torch.int32), T)
    scale, shift = gpu_lib.ds_bn_fold(dev(bn["gamma"]), dev(bn["beta"]), dev(bn["mean"]), dev(bn["var"]), 1e-5)
    g = gpu_lib.make_groups(off, perm, c_in, c_out)
    lay = (lambda a: dev(a)) if f32 else (lambda a: dev(a.transpose(0, 2, 3, 1), torch.bfloat16))
    y = torch.full((B, CO, Ho, Wo) if f32 else (B, Ho, Wo, CO), float("nan"), dtype=torch.float32 if f32 else torch.bfloat16,
                   device=DEV)
    gpu_lib.ds_sliced_conv(lay(x), lay(w), scale, shift, g, stride, pad, residual=lay(resid) if res else None, y=y)
    yh = host(y) if f32 else host(y).transpose(0, 3, 1, 2)
    for b in range(B):
        t = int(route[b])
        ci, co = c_in[t], c_out[t]
        want = np.maximum(_conv_reference(x[b, :ci], w[:co, :ci], bn, t, stride, pad, resid[b, :co] if res else None), 0.0)
        if not f32:
            want = O.bf16_round(want)
        assert relerr(yh[b, :co], want) < (TOL_F32 if f32 else TOL_BF16), (b, t)
        assert np.all(np.isnan(yh[b, co:]))


# fp32: the matrix-core kernel for 1x1 and 3x3 filters (slices of 8 or 16 channels, 32-pixel and 32-filter tiles, rows of
# weights that are and are not whole 16-byte pieces), the plain kernel for other filters
@pytest.mark.parametrize("B,K,stride,pad,H,W,c_in,c_out,res", [
    (1, 3, 1, 1, 1, 1, (1, 1), (1, 1), False), (5, 3, 1, 1, 8, 8, (32, 8), (32, 1), True),
    (3, 3, 1, 1, 9, 7, (33, 5), (33, 31), False), (4, 3, 2, 1, 11, 13, (64, 48), (64, 16), True),
    (2, 3, 1, 0, 10, 17, (130, 66), (70, 33), False), (3, 1, 1, 0, 5, 9, (64, 17), (40, 32), True),
    (2, 1, 2, 0, 9, 9, (3, 130), (65, 8), False), (2, 5, 1, 2, 8, 8, (12, 4), (10, 6), True)])
def test_sliced_conv_fp32(gpu_lib, B, K, stride, pad, H, W, c_in, c_out, res):
    _conv_case(gpu_lib, B, K, stride, pad, H, W, c_in, c_out, res, True)


# bf16: every tile of the small-launch kernel and the first launch beyond it.  32 x 32 tiles of a launch, 64-deep slabs:
@pytest.mark.parametrize("B,K,stride,pad,H,W,c_in,c_out,res", [
    (1, 1, 1, 0, 1, 1, (8,), (8,), False),                           # 1 tile, 1 slab
    (1, 3, 1, 1, 7, 7, (512, 128), (512, 136), False),               # 32 tiles, 72 slabs: 32 x 32, 8 shares
    (2, 1, 1, 0, 13, 13, (72, 264), (1032, 40), True),               # 363 tiles, 5 slabs: 32 x 64, 8 shares
    (1, 1, 1, 0, 28, 28, (128, 40), (512, 8), True),                 # 400 tiles, 2 slabs: 32 x 32, 4 shares
    (3, 3, 2, 1, 27, 27, (64, 24), (1000, 72), False),               # 608 tiles, 9 slabs: 32 x 32, 4 shares
    (9, 3, 1, 1, 15, 14, (256, 96), (456, 200), True),               # 900 tiles, 36 slabs: 64 x 64, 8 shares
    (5, 3, 1, 1, 28, 30, (64, 8), (200, 104), False),                # 931 tiles, 9 slabs: 32 x 64, 4 shares
    (2, 1, 1, 0, 56, 57, (64, 56), (128, 120), True),                # 796 tiles, 1 slab: two column tiles, 2 shares
    (31, 3, 2, 1, 14, 14, (160, 152), (1024, 8), False),             # 1552 tiles, 27 slabs, strided: 64 x 64, 8 shares
    (40, 1, 1, 0, 37, 37, (64, 24), (136, 128), False),              # 430 row tiles: the streaming kernel
    (40, 1, 1, 0, 37, 37, (128, 72), (264, 128), True)])             # 430 row tiles of 128 channels: not yet
def test_sliced_conv_bf16_tiles(gpu_lib, B, K, stride, pad, H, W, c_in, c_out, res):
    _conv_case(gpu_lib, B, K, stride, pad, H, W, c_in, c_out, res, False)


# few samples, bf16: tap masks of the longest filters that have them and of the first that do not, padding beyond the filter,
# maps smaller than it
@pytest.mark.parametrize("B,K,stride,pad,H,W,c_in,c_out,res", [
    (2, 15, 1, 7, 9, 5, (8, 16), (24, 8), False), (1, 16, 1, 8, 9, 6, (16, 8), (8, 8), False), (3, 5, 3, 6, 4, 7, (72, 8), (40, 16), True),
    (2, 2, 2, 0, 6, 5, (64, 136), (8, 48), False), (1, 7, 2, 3, 1, 1, (128, 64), (64, 64), True), (2, 4, 1, 1, 3, 30, (24, 40), (72, 64), False)])
def test_sliced_conv_bf16_taps(gpu_lib, B, K, stride, pad, H, W, c_in, c_out, res):
    _conv_case(gpu_lib, B, K, stride, pad, H, W, c_in, c_out, res, False)


# large launches on tiles of 128 columns: slices that end inside either half, ragged rows, a narrow group beside a wide one
@pytest.mark.parametrize("B,K,stride,pad,H,W,c_in,c_out,res", [
    (125, 1, 1, 0, 56, 56, (136, 40), (128, 72), False), (126, 1, 1, 0, 55, 57, (144, 8), (104, 8), False),
    (33, 1, 1, 0, 28, 29, (776, 40), (1240, 72), False), (64, 3, 2, 1, 55, 56, (72, 24), (136, 200), False), (130, 3, 2, 1, 57, 55, (64, 8), (72, 128), False)])
def test_sliced_conv_bf16_wide(gpu_lib, B, K, stride, pad, H, W, c_in, c_out, res):
    _conv_case(gpu_lib, B, K, stride, pad, H, W, c_in, c_out, res, False)


# more than a few samples, bf16, fewer workgroups than run at once: two and four shares of a reduction, shares without a slab of a
# narrow slice, ragged last tiles
@pytest.mark.parametrize("B,K,stride,pad,H,W,c_in,c_out,res", [
    (13, 3, 1, 1, 14, 14, (264, 40), (416, 72), True), (31, 3, 1, 1, 14, 14, (56, 40), (168, 136), False),
    (41, 3, 1, 1, 8, 7, (520, 8), (488, 64), False), (13, 1, 1, 0, 14, 14, (520, 24), (416, 72), True),
    (13, 1, 1, 0, 14, 14, (264, 136), (424, 8), False), (14, 3, 2, 1, 27, 27, (72, 16), (416, 392), False),
    (50, 1, 2, 0, 13, 14, (328, 64), (488, 480), True)])
def test_sliced_conv_bf16_shares(gpu_lib, B, K, stride, pad, H, W, c_in, c_out, res):
    _conv_case(gpu_lib, B, K, stride, pad, H, W, c_in, c_out, res, False)


# the tile records worked out from the offsets: groups without samples, one group, as many groups as lanes
@pytest.mark.parametrize("B,T,rows", [(1, 1, 1), (3, 64, 130), (70, 64, 33), (64, 5, 197), (300, 7, 128)])
def test_sliced_linear_tile_records(gpu_lib, B, T, rows):
    K, N = 72, 136
    d = WL.nets.Draw(B + T)
    x, w = WL.nets.as_bf16_values(d.normal((B, rows, K))), WL.nets.as_bf16_values(d.normal((N, K), std=0.1))
    bias = d.normal((N,))
    k_in, k_out = [8 + 8 * (t % 9) for t in range(T)], [8 + 8 * (t * 5 % 17) for t in range(T)]
    route = (d.randint(B, T) if T != 5 else np.full(B, 2)).astype(np.int32)
    perm, inv, off = gpu_lib.ds_route_bucket(dev(route, torch.int32), T)
    y = torch.full((B, rows, N), float("nan"), dtype=torch.bfloat16, device=DEV)
    gpu_lib.ds_sliced_linear(dev(x, torch.bfloat16), dev(w, torch.bfloat16), dev(bias), gpu_lib.make_groups(off, perm, k_in, k_out),
                             y=y)
    yh = host(y)
    for b in range(B):
        ki, ko = k_in[route[b]], k_out[route[b]]
        want = O.bf16_round(x[b, :, :ki].astype(np.float64) @ w[:ko, :ki].T.astype(np.float64) + bias[:ko])
        assert relerr(yh[b, :, :ko], want) < TOL_BF16
        assert np.all(np.isnan(yh[b, :, ko:]))


# one workgroup per item with and without the pool in front, channel counts that leave lanes and 16-byte pieces over
@pytest.mark.parametrize("layout,dtype,B,C,HW,hid,T", [
    ("nchw", "f32", 1, 1, 1, 1, 1), ("nchw", "f32", 5, 66, 100, 16, 64), ("nchw", "bf16", 3, 128, 77, 32, 5),
    ("nhwc", "f32", 4, 24, 49, 6, 3), ("nhwc", "bf16", 2, 512, 196, 128, 14), ("nhwc", "bf16", 3, 520, 130, 130, 4),
    ("nhwc", "bf16", 2, 8, 5, 8, 2), ("nhwc", "bf16", 1, 256, 3136, 64, 4), ("nhwc", "bf16", 2, 2056, 9, 64, 4)])
def test_gate_shapes(gpu_lib, layout, dtype, B, C, HW, hid, T):
    d = WL.nets.Draw(31 + C + HW)
    x = d.normal((B, C, HW))
    if dtype == "bf16":
        x = WL.nets.as_bf16_values(x)
    w1, b1 = d.normal((hid, C), std=C ** -0.5), d.normal((hid,), std=0.1)
    w2, b2 = d.normal((T, hid), std=hid ** -0.5), d.normal((T,), std=0.1)
    c_in = np.maximum(1, C - 8 * (np.arange(B) % 2) * (C > 8)).astype(np.int32)
    xg = x if layout == "nchw" else x.transpose(0, 2, 1)
    xg = dev(xg.reshape(B, C, HW, 1) if layout == "nchw" else xg, torch.float32 if dtype == "f32" else torch.bfloat16)
    logits, route = gpu_lib.ds_gate(xg, gpu_lib.DS_NCHW if layout == "nchw" else gpu_lib.DS_NHWC, dev(w1), dev(b1), dev(w2),
                                    dev(b2), T, c_in=dev(c_in, torch.int32))
    want = np.stack([O.gate_logits(O.gate_encoder(x[b, :c_in[b]].reshape(c_in[b], HW, 1)), w1, b1, w2, b2) for b in range(B)])
    assert relerr(host(logits), want) < TOL_F32
    assert route.cpu().numpy().tolist() == [O.gate_route(z) for z in host(logits)]


# classifier: a wavefront per output up to 8 items and 2048 channels, the 32-item tile beyond
@pytest.mark.parametrize("B,C,n_out", [(1, 8, 1), (1, 2048, 1000), (8, 520, 37), (9, 264, 66), (3, 2056, 5)])
def test_pool_head_shapes(gpu_lib, B, C, n_out):
    HW, T = 49, 2
    d = WL.nets.Draw(B + C)
    x, w = WL.nets.as_bf16_values(d.normal((B, HW, C))), WL.nets.as_bf16_values(d.normal((n_out, C), std=C ** -0.5))
    bias = d.normal((n_out,))
    k = [C, max(8, C // 2 // 8 * 8)]
    route = (np.arange(B) % T).astype(np.int32)
    perm, inv, off = gpu_lib.ds_route_bucket(dev(route, torch.int32), T)
    got = host(gpu_lib.ds_pool_head(dev(x, torch.bfloat16), dev(w, torch.bfloat16), dev(bias), gpu_lib.make_groups(off, perm, k)))
    for b in range(B):
        c = k[route[b]]
        want = x[b, :, :c].astype(np.float64).mean(axis=0) @ w[:, :c].T.astype(np.float64) + bias
        assert relerr(got[b], want) < 1e-4


# Token networks: an image's logits are the same bits in every batch size (tiles of 32 and 64 rows behind the attention, linear
# layers of 4 wavefronts and 32 rows and of 8 and 64, 12 and 13 column blocks), and with or without the weights in operand order.
@pytest.mark.parametrize("big", [False, True])
def test_vit_logits_do_not_depend_on_the_batch(gpu_lib, big):
    kw = dict(embed=416, heads=8, head_dim=48, mlp=1664, depth=2, routes="pp", stem_dim=24, patch=8) if big else dict(depth=2)
    arch = WL.vit_arch(**kw)
    net = gpu_lib.build_vit(arch, WL.vit_params(arch, 5), DEV)
    B = 225
    gen = torch.Generator(device=DEV)
    gen.manual_seed(3)
    imgs = torch.randn((B, 3, arch["image"], arch["image"]), generator=gen, device=DEV).to(torch.bfloat16)
    over = (torch.arange(B, device=DEV, dtype=torch.int32) * 7 % arch["T"])[None].contiguous()
    full, _ = gpu_lib.ds_forward(net, imgs, route_override=over)
    assert torch.isfinite(full).all() and full.abs().max() > 0
    for lo, hi in ((0, 1), (1, 2), (3, 8), (7, 10), (20, 60), (100, 190)):
        part, _ = gpu_lib.ds_forward(net, imgs[lo:hi].contiguous(), route_override=over[:, lo:hi].contiguous())
        # (the classifier sums in another order for a few images)
        assert relerr(host(part), host(full[lo:hi])) < 1e-5, (lo, hi)
    net.c_struct.n_params -= 4 * arch["depth"]
    plain, _ = gpu_lib.ds_forward(net, imgs, route_override=over)
    assert torch.equal(plain, full)


# The first block's Q/K/V of a part: up to a workgroup a compute unit through an LDS stage of 12 wavefronts (parts of 48 to 64 images,
# 72 with 13 column blocks), beyond it from registers of 8 (72 and 96 images); slices that end inside a 32-column block (five and seven
# heads of 48 channels): every row of the last block has the bits of the batch whole
@pytest.mark.parametrize("big", [False, True])
@pytest.mark.parametrize("B,parts", [(104, 2), (129, 2), (180, 2), (250, 4)])
def test_vit_parts_have_the_bits_of_the_batch(gpu_lib, big, B, parts):
    kw = dict(embed=416, heads=8, head_dim=48, mlp=1664, depth=2, routes="pp") if big else dict(depth=2)
    arch = WL.vit_arch(**kw)
    net = gpu_lib.build_vit(arch, WL.vit_params(arch, 6), DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(B)
    imgs = torch.randn((B, 3, arch["image"], arch["image"]), generator=gen, device=DEV).to(torch.bfloat16)
    over = (torch.arange(B, device=DEV, dtype=torch.int32) * 5 % arch["T"])[None].contiguous()
    N, D = arch["tokens"], arch["embed"]
    taps = {i: torch.zeros((B, N, D), dtype=torch.bfloat16, device=DEV) for i in range(2)}
    whole, _ = gpu_lib.ds_forward_taps(net, imgs, taps, route_override=over)
    ws = net.workspace(B, parts).zero_()
    shares, _ = gpu_lib.ds_forward_parts(net, imgs, parts, route_override=over, ws=ws)
    assert torch.isfinite(whole).all() and relerr(host(shares), host(whole)) < 1e-5       # (the classifier's sums, as above)
    # what every sample's last block left is still in its part's workspace: samples by route, rows of the route's width one behind the other
    last, ws, routes = [taps[i].view(torch.int16).cpu().numpy() for i in range(2)], ws.cpu().numpy(), over[0].cpu().numpy()
    h = -(-(-(-B // parts)) // 8) * 8
    for p0, space in zip(range(0, B, h), np.split(ws, -(-B // h))):
        space, at = space.view(np.int16), None
        for j, b in enumerate(p0 + np.argsort(routes[p0:p0 + h], kind="stable")):
            width, depth = (int([*arch["routes"][routes[b]], 2][i]) for i in (0, 3))
            if depth == 0:
                continue
            want = last[depth - 1][b, :, :width]
            if at is None:
                at = space.tobytes().find(want[:1].tobytes()) - j * N * D * 2
                assert at >= 0 and at % 256 == 0, p0
            assert np.array_equal(space[at // 2 + j * N * D:][:N * width].reshape(N, width), want), (p0, b)


# hidden activations inside and outside the range of GELU's polynomial: the bits of the linear layers on row-major weights
def test_gelu_rounding_matches_the_linear_layer(gpu_lib):
    arch = WL.vit_arch(depth=1)
    p = WL.vit_params(arch, 6)
    for k in ("l0.fc1.w", "l0.fc1.b"):
        p[k] = p[k] * 8.0                                   # pre-activations far beyond +-3.5 beside small ones
    net = gpu_lib.build_vit(arch, p, DEV)
    B = 48
    gen = torch.Generator(device=DEV)
    gen.manual_seed(4)
    imgs = torch.randn((B, 3, arch["image"], arch["image"]), generator=gen, device=DEV).to(torch.bfloat16)
    over = torch.arange(B, device=DEV, dtype=torch.int32)[None].contiguous()
    out = []
    for tiled in (True, False):
        if not tiled:
            net.c_struct.n_params -= 4 * arch["depth"]
        tap = torch.zeros((B, arch["tokens"], arch["embed"]), dtype=torch.bfloat16, device=DEV)
        logits, _ = gpu_lib.ds_forward_taps(net, imgs, {0: tap}, route_override=over)
        out.append((logits, tap))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


# spatial depthwise filters without dilation: rows of 14 outputs per lane, 16 or 32 channels per lane group
@pytest.mark.parametrize("B,K,stride,H,W,C", [(3, 7, 1, 1, 1, 8), (9, 7, 1, 7, 7, 640), (5, 7, 1, 14, 15, 72), (4, 5, 1, 13, 29, 288),
                                              (2, 5, 1, 112, 112, 48), (5, 7, 2, 14, 14, 288), (3, 5, 2, 29, 31, 24),
                                              (2, 3, 2, 57, 113, 96), (2, 7, 2, 224, 224, 8), (1, 7, 1, 9, 700, 40)])
def test_sliced_dwconv_spatial_pairs(gpu_lib, B, K, stride, H, W, C):
    d = WL.nets.Draw(7100 + stride + C + K + W)
    x = WL.nets.as_bf16_values(d.normal((B, C, H, W)))
    w = WL.nets.as_bf16_values(d.normal((C, 1, K, K), std=0.3))
    spec = [(k, p) for k, p in [(K, K // 2), (1, 0), (K - 2, K // 2 - 1), (K, K // 2 + 1), (3, 2), (K, K // 2 - 1)]
            if H + 2 * p >= k and W + 2 * p >= k]
    T = len(spec)
    bn = WL.bn_tables(d, T, C)
    route = np.arange(B, dtype=np.int32) % T
    cs = [max(8, C * (4 - t % 4) // 4 // 8 * 8) for t in range(T)]
    perm, _, off = gpu_lib.ds_route_bucket(dev(route, torch.int32), T)
    scale, shift = gpu_lib.ds_bn_fold(dev(bn["gamma"]), dev(bn["beta"]), dev(bn["mean"]), dev(bn["var"]), 1e-5)
    rows = max(((H + 2 * p - k) // stride + 1) * ((W + 2 * p - k) // stride + 1) for k, p in spec)
    y = torch.full((B, rows, C), float("nan"), dtype=torch.bfloat16, device=DEV)
    gpu_lib.ds_sliced_dwconv_spatial(dev(x.transpose(0, 2, 3, 1), torch.bfloat16), dev(w[:, 0].transpose(1, 2, 0), torch.bfloat16),
                                     scale, shift, gpu_lib.make_groups(off, perm, cs), [k for k, _ in spec], [1] * T,
                                     [p for _, p in spec], stride, y=y)
    yh = host(y)
    for b in range(B):
        t = int(route[b])
        k, p = spec[t]
        c = cs[t]
        want = O.bf16_round(O.relu(O.re_sbn(O.spatial_dwconv2d(x[b, :c], w, k, 1, stride, p), bn, t, 1e-5)))
        n = want.shape[1] * want.shape[2]
        assert relerr(yh[b, :n, :c].T.reshape(want.shape), want) < 1e-2, (b, spec[t])
        assert np.all(np.isnan(yh[b, :n, c:])) and np.all(np.isnan(yh[b, n:]))


# blocks in front of the gate in one kernel (pointwise filters in operand order) against the layers apart: tiles with a ragged
# last row and column, 16- and 14-column tiles, one sample to more than the workgroups at once, 3 and 5 taps, both strides
@pytest.mark.parametrize("pp", [False, True])
@pytest.mark.parametrize("image,B", [(224, 2), (150, 3), (150, 41), (66, 1), (34, 9)])
def test_mbnet_front_blocks(gpu_lib, pp, image, B):
    arch = (WL.mbnet_pp_arch if pp else WL.mbnet_arch)(image=image)
    net = gpu_lib.build_mbnet(arch, WL.mbnet_params(arch, 12), DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(image + B)
    imgs = torch.randn((B, 3, image, image), generator=gen, device=DEV).to(torch.bfloat16)
    over = (torch.arange(B, device=DEV, dtype=torch.int32) % arch["T"])[None].contiguous()

    def run():
        r, taps = (image + 1) // 2, {}
        for i, (_, co, s) in enumerate(arch["blocks"][:5]):
            r = (r - 1) // s + 1
            taps[i] = torch.full((B, r * r, co), float("nan"), dtype=torch.bfloat16, device=DEV)
        out = gpu_lib.ds_forward_taps(net, imgs, taps, route_override=over)
        return taps, out[0]

    fused, logits = run()
    net.c_struct.n_params -= len(arch["blocks"])
    apart, want = run()
    for i in range(5):
        assert torch.isfinite(apart[i]).all() and apart[i].abs().max() > 0
        # single elements may round the other way in every layer before
        a, b = host(fused[i]), host(apart[i])
        assert np.linalg.norm(a - b) < 2e-3 * np.linalg.norm(b) and relerr(a, b) < 4e-2, i
    assert relerr(host(logits), host(want)) < 1e-2


# The stem and the first two blocks in one kernel against the three launches (asked for by a tap of the first block's output):
# one strip to several, narrow ones, a ragged last one; odd maps; bands of one row, of several, of all; a pixel that overflows.
# Both sides round every layer to bf16 from fp32 sums of 9..128 products.  The stem gives the same bits; in the first depthwise layer
# strips start at other columns, so the taps of a filter row meet in other steps, and a value's last bit may flip (2^-8 of it; 30 of
# 25.7e6 outputs of 64 images with 3x3 filters, 11 of 9.6e6 with 5x5): 1e-3 of the norm is far above that.
@pytest.mark.parametrize("pp", [False, True])
@pytest.mark.parametrize("image,B", [(224, 1), (224, 35), (224, 200), (216, 3), (228, 2), (100, 9), (60, 33), (28, 2)])
def test_mbnet_first_layers_in_one_kernel(gpu_lib, pp, image, B):
    arch = (WL.mbnet_pp_arch if pp else WL.mbnet_arch)(image=image)
    net = gpu_lib.build_mbnet(arch, WL.mbnet_params(arch, 12), DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(image + B)
    imgs = torch.randn((B, 3, image, image), generator=gen, device=DEV).to(torch.bfloat16)
    over = (torch.arange(B, device=DEV, dtype=torch.int32) % arch["T"])[None].contiguous()
    r1 = (image + 1) // 2
    r2 = (r1 + 1) // 2

    def run(x, *blocks):
        shape = {0: (B, r1 * r1, arch["blocks"][0][1]), 1: (B, r2 * r2, arch["blocks"][1][1])}
        taps = {i: torch.full(shape[i], float("nan"), dtype=torch.bfloat16, device=DEV) for i in blocks}
        gpu_lib.ds_forward_taps(net, x, taps, route_override=over)
        return taps[1].reshape(B, r2, r2, -1)

    one, apart = run(imgs, 1), run(imgs, 0, 1)
    assert torch.isfinite(one).all() and one.abs().max() > 0
    assert (one.double() - apart.double()).norm() < 1e-3 * apart.double().norm()
    assert torch.equal(one, run(imgs, 1))
    # the reach of an image's pixel: 3x3 at stride 2, k x k, k x k at stride 2 (and the column left of the stem's filter)
    bad = imgs.clone()
    bad[B // 2, 1, image // 2, image // 2] = 3e38
    got, k = run(bad, 1), 5 if pp else 3
    lo = hi = image // 2
    for half, s in ((2, 2), (k // 2, 1), (k // 2, 2)):
        lo, hi = (lo - half) // s, -(-(hi + half) // s)
    reach = torch.zeros((B, r2, r2), dtype=torch.bool, device=DEV)
    reach[B // 2, max(lo, 0):hi + 1, max(lo, 0):hi + 1] = True
    assert not torch.equal(got[reach], one[reach]) and torch.isfinite(got[~reach]).all()
    near = torch.zeros_like(reach)
    near[B // 2] = True
    assert torch.equal(got[~near], one[~near])
    a, b = got[near & ~reach].double(), one[near & ~reach].double()
    assert (a - b).norm() <= 4e-3 * b.norm()


# blocks behind the gate in one kernel against the layers apart: the four tiles (32 pixels and 256 or 512 filters, 64 and 112
# pixels), maps of one row and one pixel, odd maps, a map too wide for a tile next to one that is not
@pytest.mark.parametrize("image,B", [(224, 2), (224, 20), (224, 50), (224, 70), (224, 140), (150, 33), (34, 9), (640, 1)])
def test_mbnet_sliced_blocks(gpu_lib, image, B):
    arch = WL.mbnet_arch(image=image)
    net = gpu_lib.build_mbnet(arch, WL.mbnet_params(arch, 13), DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(image + B)
    imgs = torch.randn((B, 3, image, image), generator=gen, device=DEV).to(torch.bfloat16)
    over = (torch.arange(B, device=DEV, dtype=torch.int32) % arch["T"])[None].contiguous()

    def run():
        r, taps = (image + 1) // 2, {}
        for i, (_, co, s) in enumerate(arch["blocks"]):
            r = (r - 1) // s + 1
            if i >= arch["gate_after"]:
                taps[i] = torch.full((B, r * r, co), float("nan"), dtype=torch.bfloat16, device=DEV)
        out = gpu_lib.ds_forward_taps(net, imgs, taps, route_override=over)
        return taps, out[0]

    fused, logits = run()
    net.c_struct.n_ints -= 1                                       # without the flag
    apart, want = run()
    for i, t in apart.items():
        # the pointwise sums are taken in another order, so elements may round the other way at each of up to 16 roundings before
        # (two a block): 2^-9 of an element each, 2^-9 sqrt(16) together in the 2-norm if all of them did
        n = torch.isfinite(t)
        assert torch.equal(n, torch.isfinite(fused[i])) and t[n].abs().max() > 0      # written on the slices alone
        a, b = host(torch.where(n, fused[i], 0)), host(torch.where(n, t, 0))
        assert np.linalg.norm(a - b) < 2.0 ** -7 * np.linalg.norm(b) and relerr_max(a, b) < TOL_BF16, i
    assert relerr_max(host(logits), host(want)) < TOL_BF16


# one sample is bucketed by the gate's last launch, two by the bucket kernel: every (route, previous route) pair of DS-ResNet,
# every route of the others
@pytest.mark.parametrize("which", ["mbnet", "resnet", "vit"])
def test_single_sample_bucketed_by_the_gate(gpu_lib, which):
    arch = getattr(WL, which + "_arch")()
    net = getattr(gpu_lib, "build_" + which)(arch, getattr(WL, which + "_params")(arch, 29), DEV)
    T = arch["T"]
    gen = torch.Generator(device=DEV)
    gen.manual_seed(29)
    x = torch.randn((1, 3, 224, 224), generator=gen, device=DEV).to(torch.bfloat16)
    two = x.repeat(2, 1, 1, 1).contiguous()
    stages = 4 if which == "resnet" else 1
    for q in range(T):
        for prev in range(T if which == "resnet" else 1):
            over = torch.tensor([[q if st % 2 else prev] if stages > 1 else [q] for st in range(stages)], dtype=torch.int32, device=DEV)
            one, r1 = gpu_lib.ds_forward(net, x, route_override=over)
            want, r2 = gpu_lib.ds_forward(net, two, route_override=over.repeat(1, 2).contiguous())
            assert torch.equal(r1.reshape(-1), over.reshape(-1)) and torch.equal(r2.reshape(stages, 2)[:, 0], over[:, 0])
            # the layers may be other kernels at two samples: the networks' own bound against the oracle
            assert torch.isfinite(one).all() and relerr_max(host(one), host(want)[:1]) < TOL_BF16, (q, prev)


# blocks in front of the gate with few samples (tiles of the sliced blocks' kernel) against the kernels of larger batches: both sides
# of the line at 224 (8 and 9 samples), maps of a few pixels, odd maps
@pytest.mark.parametrize("image,B", [(224, 1), (224, 8), (224, 9), (150, 3), (34, 2), (17, 5)])
def test_mbnet_unsliced_blocks_few_samples(gpu_lib, image, B):
    arch = WL.mbnet_arch(image=image)
    net = gpu_lib.build_mbnet(arch, WL.mbnet_params(arch, 17), DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(image + B)
    few = torch.randn((B, 3, image, image), generator=gen, device=DEV).to(torch.bfloat16)
    # the line is at 32 tiles for every eighth sample: a map of one tile crosses it with 257 samples
    many = few.repeat(-(-300 // B), 1, 1, 1).contiguous()

    def run(x):
        over = (torch.arange(len(x), device=DEV, dtype=torch.int32) % B % arch["T"])[None].contiguous()
        r, taps = (image + 1) // 2, {}
        for i, (_, co, s) in enumerate(arch["blocks"][:arch["gate_after"]]):
            r = (r - 1) // s + 1
            taps[i] = torch.full((len(x), r * r, co), float("nan"), dtype=torch.bfloat16, device=DEV)
        return taps, gpu_lib.ds_forward_taps(net, x, taps, route_override=over)[0]

    got, logits = run(few)
    ref, want = run(many)
    for i, t in got.items():
        # two roundings a block may go the other way, 2^-9 of an element each: 2^-9 sqrt(10) together in the 2-norm at the most
        assert torch.isfinite(t).all() and t.abs().max() > 0
        a, b = host(t), host(ref[i][:B])
        assert np.linalg.norm(a - b) < 2.0 ** -9 * 10 ** 0.5 * np.linalg.norm(b) and relerr_max(a, b) < TOL_BF16, i
    assert relerr_max(host(logits), host(want)[:B]) < TOL_BF16


# a stage's projection and first layer in one launch (few samples) against the two launches of a large batch: every kernel variant
# that pairs, stages on either side of the line, odd maps and maps of a few pixels
@pytest.mark.parametrize("image,B", [(224, 1), (224, 2), (224, 4), (150, 3), (34, 1), (34, 7)])
def test_resnet_paired_layers(gpu_lib, image, B):
    arch = WL.resnet_arch(image=image)
    net = gpu_lib.build_resnet(arch, WL.resnet_params(arch, 23), DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(image + B)
    few = torch.randn((B, 3, image, image), generator=gen, device=DEV).to(torch.bfloat16)
    many = few.repeat(-(-64 // B), 1, 1, 1).contiguous()

    def run(x):
        n = torch.arange(len(x), device=DEV, dtype=torch.int32) % B
        over = torch.stack([(n + st) % arch["T"] for st in range(4)]).contiguous()
        r, taps, block = ((image + 1) // 2 + 1) // 2, {}, 0
        for st, nb in enumerate(arch["blocks"]):
            r = r if st == 0 else (r - 1) // 2 + 1
            taps[block] = torch.full((len(x), r * r, int(arch["out"][st].max())), float("nan"), dtype=torch.bfloat16, device=DEV)
            block += nb
        return taps, gpu_lib.ds_forward_taps(net, x, taps, route_override=over)[0]

    got, logits = run(few)
    ref, want = run(many)
    for i, t in got.items():
        # up to 4 roundings a block before it may go the other way: 2^-9 sqrt(4 (i + 1)) in the 2-norm if all of them did
        n = torch.isfinite(t)
        assert torch.equal(n, torch.isfinite(ref[i][:B])) and t[n].abs().max() > 0      # written on the slices alone
        a, b = host(torch.where(n, t, 0)), host(torch.where(n, ref[i][:B], 0))
        assert np.linalg.norm(a - b) < 2.0 ** -9 * (4 * (i + 1)) ** 0.5 * np.linalg.norm(b) and relerr_max(a, b) < TOL_BF16, i
    assert relerr_max(host(logits), host(want)[:B]) < TOL_BF16


# the rest of a bottleneck block as one launch (projection inside, next block's first layer behind) against the separate launches of
# one image: both slice limits, the widest map, odd maps, maps smaller than a tile, routes of different depth, narrow networks
@pytest.mark.parametrize("which,image,B", [("width", 224, 2), ("width", 224, 60), ("width", 236, 50), ("width", 150, 130), ("width", 50, 300),
                                           ("pp", 224, 33), ("pp", 224, 60), ("pp", 129, 150), ("depth", 224, 56), ("half", 224, 60), ("half", 90, 90)])
def test_resnet_rest_of_a_block(gpu_lib, which, image, B):
    kw = {"width": {}, "pp": dict(blocks=(3, 4, 8, 3), routes="pp"), "depth": dict(routes="depth"), "half": dict(width_div=2)}[which]
    arch = WL.resnet_arch(image=image, **kw)
    net = gpu_lib.build_resnet(arch, WL.resnet_params(arch, 29), DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(image + B)
    kinds = min(B, 2 * arch["T"])
    imgs = torch.randn((kinds, 3, image, image), generator=gen, device=DEV).to(torch.bfloat16)
    n = torch.arange(kinds, device=DEV, dtype=torch.int32)
    over = torch.stack([(n + st * (not arch.get("single_gate"))) % arch["T"] for st in range(4)])
    blocks = arch["blocks"][0] + arch["blocks"][1]

    def run(which):
        taps, r = {}, ((image + 1) // 2 + 1) // 2
        for i in range(blocks):
            st = int(i >= arch["blocks"][0])
            rb = (r - 1) // 2 + 1 if st else r
            taps[i] = torch.zeros((len(which), rb * rb, int(arch["out"][st].max())), dtype=torch.bfloat16, device=DEV)
        return taps, gpu_lib.ds_forward_taps(net, imgs[which].contiguous(), taps, route_override=over[:, which].contiguous())[0]

    got, logits = run(torch.arange(B, device=DEV) % kinds)
    assert torch.isfinite(logits).all()
    for k in range(kinds):
        ref, want = run(torch.tensor([k], device=DEV))
        for i, t in got.items():
            # up to 4 roundings a block before it may go the other way: 2^-9 sqrt(4 (i + 1)) in the 2-norm if all of them did
            b = host(ref[i][0])
            for j in range(k, B, max(kinds, (B - k - 1) // kinds * kinds)):      # the image's first and last place
                a = host(t[j])
                assert np.linalg.norm(a - b) < 2.0 ** -9 * (4 * (i + 1)) ** 0.5 * np.linalg.norm(b) and relerr_max(a, b) < TOL_BF16, (i, k, j)
        assert relerr_max(host(logits[k]), host(want[0])) < TOL_BF16


# a stage's projection and first layer as one launch of the 128-row kernel, in each of its tiles (two shares, slabs of 32, 64 and 128
# channels), and where the two take different ones, against one image alone
@pytest.mark.parametrize("which,image,B", [("width", 224, 12), ("width", 224, 33), ("width", 224, 65), ("width", 90, 130), ("pp", 224, 33),
                                           ("depth", 150, 70), ("half", 224, 90)])
def test_resnet_first_layers_of_a_stage(gpu_lib, which, image, B):
    kw = {"width": {}, "pp": dict(blocks=(3, 4, 8, 3), routes="pp"), "depth": dict(routes="depth"), "half": dict(width_div=2)}[which]
    arch = WL.resnet_arch(image=image, **kw)
    net = gpu_lib.build_resnet(arch, WL.resnet_params(arch, 41), DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(image + B)
    kinds = min(B, 2 * arch["T"])
    imgs = torch.randn((kinds, 3, image, image), generator=gen, device=DEV).to(torch.bfloat16)
    n = torch.arange(kinds, device=DEV, dtype=torch.int32)
    over = torch.stack([(n + st * (not arch.get("single_gate"))) % arch["T"] for st in range(4)])

    def run(which):
        taps, r = {}, ((image + 1) // 2 + 1) // 2
        for st in range(1, 4):
            r = (r - 1) // 2 + 1
            taps[sum(arch["blocks"][:st])] = torch.zeros((len(which), r * r, int(arch["out"][st].max())), dtype=torch.bfloat16, device=DEV)
        gpu_lib.ds_forward_taps(net, imgs[which].contiguous(), taps, route_override=over[:, which].contiguous())
        return taps

    got = run(torch.arange(B, device=DEV) % kinds)
    for k in range(kinds):
        ref = run(torch.tensor([k], device=DEV))
        for i, t in got.items():
            # (as for the rest of a block)
            b = host(ref[i][0])
            for j in range(k, B, max(kinds, (B - k - 1) // kinds * kinds)):
                a = host(t[j])
                assert np.linalg.norm(a - b) < 2.0 ** -9 * (4 * (i + 1)) ** 0.5 * np.linalg.norm(b) and relerr_max(a, b) < TOL_BF16, (i, k, j)


# 7x7 stem and max-pool in one kernel: the first block passes its input on (projection the identity, residual branch zero), so its
# output is the pooled map.  Tiles of 3 x 8 pooled pixels: maps of one pixel to several tiles, ragged on both sides
@pytest.mark.parametrize("image,B", [(4, 1), (12, 3), (32, 8), (44, 5), (100, 16), (224, 9)])
def test_resnet_stem_and_pool(gpu_lib, image, B):
    arch = WL.resnet_arch(image=image)
    p = WL.resnet_params(arch, 31)
    one = {"beta": 0.0, "mean": 0.0, "var": 1.0 - arch["bn_eps"]}
    for name, gamma in (("s0.b0.proj.bn", 1.0), ("s0.b0.c3.bn", 0.0)):
        p[name] = {k: np.full_like(v, one.get(k, gamma)) for k, v in p[name].items()}
    p["s0.b0.proj.w"] = np.zeros_like(p["s0.b0.proj.w"])
    p["s0.b0.proj.w"][np.arange(64), np.arange(64), 0, 0] = 1.0
    net = gpu_lib.build_resnet(arch, p, DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(image)
    imgs = torch.randn((B, 3, image, image), generator=gen, device=DEV).to(torch.bfloat16)
    bn = p["stem.bn"]
    s = bn["gamma"].astype(np.float64) / np.sqrt(bn["var"][0].astype(np.float64) + arch["bn_eps"])
    h = bn["beta"] - bn["mean"][0] * s
    y = F.conv2d(imgs.double().cpu(), torch.from_numpy(p["stem.w"]).double(), stride=2, padding=3)
    y = F.max_pool2d(torch.relu(y * torch.from_numpy(s)[:, None, None] + torch.from_numpy(h)[:, None, None]), 3, 2, 1)
    r = y.shape[-1]
    tap = torch.zeros((B, r * r, 256), dtype=torch.bfloat16, device=DEV)
    gpu_lib.ds_forward_taps(net, imgs, {0: tap}, route_override=torch.full((4, B), arch["T"] - 1, dtype=torch.int32, device=DEV))
    want = y.permute(0, 2, 3, 1).reshape(B, r * r, 64).numpy()
    # one bf16 rounding (2^-9 of the value) of a sum over 147 products of order one in fp32
    assert np.all(np.abs(host(tap)[:, :, :64] - want) <= 2.0 ** -8 * np.abs(want) + 1e-4)


# the next block's Q/K/V behind a block, on both sides of its line and with 32 and 64 rows a workgroup, routes that end before the
# deepest one among them: the bits of the launches on the row-major weights, which have none of it
@pytest.mark.parametrize("which,B", [("cross", 8), ("cross", 9), ("cross", 80), ("pp", 19), ("pp", 20), ("pp", 90), ("depth", 12), ("depth", 77)])
def test_vit_qkv_behind_a_block(gpu_lib, which, B):
    kw = {"cross": dict(depth=3), "depth": dict(depth=4, routes="depth"),
          "pp": dict(embed=416, heads=8, head_dim=48, mlp=1664, depth=4, routes="pp")}[which]
    arch = WL.vit_arch(**kw)
    net = gpu_lib.build_vit(arch, WL.vit_params(arch, 8), DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(B)
    imgs = torch.randn((B, 3, arch["image"], arch["image"]), generator=gen, device=DEV).to(torch.bfloat16)
    over = (torch.arange(B, device=DEV, dtype=torch.int32) * 5 % arch["T"])[None].contiguous()
    got, _ = gpu_lib.ds_forward(net, imgs, route_override=over)
    net.c_struct.n_params -= 4 * arch["depth"]
    want, _ = gpu_lib.ds_forward(net, imgs, route_override=over)
    assert torch.isfinite(want).all() and torch.equal(got, want)


# parts of a batch that count their tiles of 64 rows together, on both sides of the line, parts of unequal sizes: as above
@pytest.mark.parametrize("which,B,parts", [("cross", 73, 2), ("cross", 77, 2), ("cross", 78, 4), ("pp", 79, 3), ("pp", 86, 2)])
def test_vit_blocks_of_parts(gpu_lib, which, B, parts):
    kw = {"cross": dict(depth=3), "pp": dict(embed=416, heads=8, head_dim=48, mlp=1664, depth=3, routes="pp")}[which]
    arch = WL.vit_arch(**kw)
    net = gpu_lib.build_vit(arch, WL.vit_params(arch, 9), DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(B)
    imgs = torch.randn((B, 3, arch["image"], arch["image"]), generator=gen, device=DEV).to(torch.bfloat16)
    over = (torch.arange(B, device=DEV, dtype=torch.int32) * 5 % arch["T"])[None].contiguous()
    got, _ = gpu_lib.ds_forward_parts(net, imgs, parts, route_override=over)
    net.c_struct.n_params -= 4 * arch["depth"]
    want, _ = gpu_lib.ds_forward_parts(net, imgs, parts, route_override=over)
    assert torch.isfinite(want).all() and torch.equal(got, want)


# gates that take the sums of the stage's last block (maps of whole pieces of 64 rows: the first stage's at 224 and 96 pixels), samples
# that start in the middle of a tile of 128 rows, and gates that pool the map, against a float64 mean of that block's output
@pytest.mark.parametrize("image,B", [(224, 100), (96, 100), (150, 131), (236, 97)])
def test_resnet_gates_on_the_last_blocks_sums(gpu_lib, image, B):
    arch = WL.resnet_arch(image=image)
    p = WL.resnet_params(arch, 37)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(image)
    # (images of different contrast, so that their means differ)
    imgs = (torch.randn((B, 3, image, image), generator=gen, device=DEV) * torch.linspace(0.2, 3.0, B, device=DEV)[:, None, None, None]).to(torch.bfloat16)
    over = torch.stack([(torch.arange(B, device=DEV, dtype=torch.int32) + s) % arch["T"] for s in range(4)])
    r0 = ((image + 1) // 2 + 1) // 2
    last = {0: (arch["blocks"][0] - 1, r0, 256), 1: (arch["blocks"][0] + arch["blocks"][1] - 1, (r0 - 1) // 2 + 1, 512)}

    def run(bias):
        net = gpu_lib.build_resnet(arch, p, DEV)
        taps = {i: torch.zeros((B, r * r, c), dtype=torch.bfloat16, device=DEV) for i, r, c in last.values()}
        return taps, gpu_lib.ds_forward_taps(net, imgs, taps, logit_bias=bias, route_override=None)[1]

    # the first two gates' routes are forced by their scores, the third's and second's own scores are brought to zero mean
    bias = torch.zeros((4, B, arch["T"]), device=DEV)
    bias[0].scatter_(1, over[0].long()[:, None], 1000.0)
    bias[3].scatter_(1, over[3].long()[:, None], 1000.0)
    for st in (0, 1):
        def scores(taps):
            i, r, c = last[st]
            mean = host(taps[i]).mean(1)
            w = {k: p[f"s{st + 1}.gate.{k}"].astype(np.float64) for k in ("w1", "b1", "w2", "b2")}
            return np.maximum(mean @ w["w1"].T + w["b1"], 0.0) @ w["w2"].T + w["b2"]
        z = scores(run(bias)[0])
        p[f"s{st + 1}.gate.b2"] = (p[f"s{st + 1}.gate.b2"] - z.mean(0)).astype(np.float32)
        taps, routes = run(bias)
        z = scores(taps)
        top = np.sort(z, 1)
        # fp32 sums of up to 3481 values and one bf16-free mean: 1e-5 of the scores' size is far above their error
        clear = top[:, -1] - top[:, -2] > 1e-5 * np.abs(z).max()
        got = routes[st + 1].cpu().numpy()
        assert clear.sum() > 0.9 * B and len(set(z.argmax(1)[clear])) > 1
        assert np.array_equal(got[clear], z.argmax(1)[clear])


# An image's gate scores are the same bits beside other neighbours.  The gate is made to show its pooled mean of one channel: a route's
# score is that mean, another's a threshold per image, so that bisecting over the floats finds its bits; then other orders of the batch.
@pytest.mark.parametrize("stage", [1, 2])
@pytest.mark.parametrize("image,B", [(224, 97), (96, 104), (160, 96), (208, 96), (72, 100)])
def test_resnet_gate_scores_do_not_depend_on_the_neighbours(gpu_lib, image, B, stage):
    arch = WL.resnet_arch(image=image, blocks=(2, 2, 1, 1))
    p = WL.resnet_params(arch, 43)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(image)
    # (contrast over four decades, and layers without the shifts that would hide it: a map's fp32 sum then depends on its order)
    for name in p:
        if name.endswith(".bn"):
            p[name] = {k: v * (k not in ("beta", "mean")) for k, v in p[name].items()}
    contrast = 10.0 ** (4.0 * torch.rand((B, 1, image // 4, image // 4), generator=gen, device=DEV).repeat_interleave(4, 2).repeat_interleave(4, 3) - 3.0)
    imgs = (torch.randn((B, 3, image, image), generator=gen, device=DEV) * contrast).to(torch.bfloat16)
    bias = torch.zeros((4, B, arch["T"]), device=DEV)
    for st in range(4):
        bias[st].scatter_(1, ((torch.arange(B, device=DEV) * 7 + st) % arch["T"])[:, None], 1e4)
    bias[stage] = torch.tensor([0.0, 0.0] + [-1e30] * (arch["T"] - 2), device=DEV)
    plain = torch.arange(B, device=DEV)
    orders = [plain.flip(0), plain.roll(1), *(torch.randperm(B, generator=gen, device=DEV) for _ in range(4))]
    for channel in range(5, 11):
        for k in ("w1", "b1", "w2", "b2"):
            p[f"s{stage}.gate.{k}"] = np.zeros_like(p[f"s{stage}.gate.{k}"])
        p[f"s{stage}.gate.w1"][0, channel] = p[f"s{stage}.gate.w2"][0, 0] = 1.0
        net = gpu_lib.build_resnet(arch, p, DEV)
        ws = net.workspace(B)

        def at_least(bits, order):
            b = bias[:, order].clone()
            b[stage, :, 1] = bits[order].to(torch.int32).view(torch.float32)
            return gpu_lib.ds_forward(net, imgs[order].contiguous(), logit_bias=b.contiguous(), ws=ws)[1][stage] == 0

        lo, hi = torch.zeros(B, dtype=torch.int64, device=DEV), torch.full((B,), 0x4b000000, dtype=torch.int64, device=DEV)
        while int((hi - lo).max()) > 1:
            mid = (lo + hi) // 2
            up = at_least(mid, plain)
            lo, hi = torch.where(up, mid, lo), torch.where(up, hi, mid)
        assert int((lo > 0).sum()) > B // 2
        changed = sum(int((~at_least(lo, order)).sum()) + int(at_least(hi, order).sum()) for order in orders)
        assert changed == 0, channel


# hidden layers of one column piece, of exactly a tile of 384 or 416 columns, a few columns more, two tiles and the most there are: the three
# launches of a few images (fc2 in runs of two column blocks and of four), 32 and 64 rows a workgroup behind the attention, 12 and 13 column blocks, attention wider than 12 of them: as above
@pytest.mark.parametrize("B", [3, 7, 70, 120, 1000])
@pytest.mark.parametrize("embed", [384, 416, "wide heads"])
def test_vit_hidden_tiles(gpu_lib, embed, B):
    if embed == 384:
        arch = WL.vit_arch(image=64, depth=2)                # 17 tokens
        routes = [(384, 6, 8), (384, 6, 384), (264, 4, 392), (192, 3, 768), (384, 5, 776), (384, 6, 1536)]
    elif embed == 416:
        arch = WL.vit_arch(image=64, embed=416, heads=8, head_dim=48, mlp=1664, depth=2)
        routes = [(392, 7, 8), (416, 8, 416), (416, 8, 424), (400, 8, 832), (416, 5, 840), (416, 8, 1664)]
    else:
        arch = WL.vit_arch(image=64, heads=13, head_dim=32, depth=2)
        routes = [(384, 13, 8), (384, 13, 384), (264, 12, 392), (192, 10, 768), (384, 13, 776), (384, 13, 1536)]
    arch["routes"], arch["T"] = np.array(routes, np.int32), len(routes)
    net = gpu_lib.build_vit(arch, WL.vit_params(arch, 10), DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(B)
    imgs = torch.randn((B, 3, arch["image"], arch["image"]), generator=gen, device=DEV).to(torch.bfloat16)
    over = (torch.arange(B, device=DEV, dtype=torch.int32) * 5 % arch["T"])[None].contiguous()

    def run():
        gpu_lib.ds_profile_reset()
        gpu_lib.ds_profile_enable(True)
        try:
            logits, _ = gpu_lib.ds_forward(net, imgs, route_override=over)
        finally:
            gpu_lib.ds_profile_enable(False)
        kinds = [k for k, _ in gpu_lib.ds_profile_launches()]
        gpu_lib.ds_profile_reset()
        return logits, kinds.count("tail"), kinds.count("vit_linear")

    got, tails, linears = run()
    # a launch a block, the first block's Q/K/V in one of its own (and the next one's, where it does not ride along) -- or four a block
    assert (tails, linears) == (0, 8) if B < 100 else (tails == 2 and linears in (1, 2)), (tails, linears)
    net.c_struct.n_params -= 4 * arch["depth"]
    want, tails, linears = run()
    assert (tails, linears) == (0, 0)
    assert torch.isfinite(want).all() and torch.equal(got, want)


def _line(source, pattern):
    """A line of a dispatch, as the source has it: a test that is written for one side of it does not end up on the other."""
    return int(re.search(pattern, open(os.path.join(CSRC, source)).read()).group(1))


def _in_two_workgroups(B, tokens, T):
    return (B * tokens - T) // 64 + T >= _line("vit_tail.hip", r">= (\d+)\) return ds_launch_vit_duo")


# blocks in two workgroups a compute unit, two, three and four column blocks a wavefront: embeddings that end at either side of their edges and
# inside a block, attention narrower and wider than them, hidden layers of one piece, of a tile of 128 columns, a piece more and the most
# there are, GELU far outside the polynomial's range, a sample that is not finite: the bits of the launches on the row-major weights
@pytest.mark.parametrize("embed", [384, 416, "wide heads"])
def test_vit_two_workgroups(gpu_lib, embed):
    if embed == 384:
        arch = WL.vit_arch(image=64, depth=2)                # 17 tokens
        routes = [(8, 1, 8), (136, 6, 128), (192, 3, 136), (256, 4, 384), (264, 2, 520), (320, 5, 1280), (384, 1, 264), (384, 6, 1536)]
    elif embed == 416:
        arch = WL.vit_arch(image=64, embed=416, heads=8, head_dim=48, mlp=1664, depth=2)
        routes = [(248, 8, 8), (256, 5, 1024), (288, 6, 1008), (384, 8, 256), (392, 7, 8), (400, 1, 904), (416, 5, 1160), (416, 8, 1664)]
    else:
        arch = WL.vit_arch(image=64, heads=13, head_dim=32, depth=2)
        routes = [(8, 13, 8), (224, 13, 384), (256, 1, 776), (264, 12, 392), (328, 11, 128), (384, 10, 120), (384, 13, 1400), (384, 13, 1536)]
    arch["routes"], arch["T"] = np.array(routes, np.int32), len(routes)
    p = WL.vit_params(arch, 12)
    for k in ("l1.fc1.w", "l1.fc1.b"):
        p[k] = p[k] * 8.0                                    # pre-activations far beyond +-3.5 beside small ones
    net = gpu_lib.build_vit(arch, p, DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(12)
    B = 2300                                                 # 618 tiles of 64 rows
    assert _in_two_workgroups(B, arch["tokens"], arch["T"])
    imgs = torch.randn((B, 3, arch["image"], arch["image"]), generator=gen, device=DEV).to(torch.bfloat16)
    imgs[5, 0, 0, 0], imgs[1234, 2, 9, 9] = float("nan"), float("inf")
    over = (torch.arange(B, device=DEV, dtype=torch.int32) * 5 % arch["T"])[None].contiguous()
    got, _ = gpu_lib.ds_forward(net, imgs, route_override=over)
    net.c_struct.n_params -= 4 * arch["depth"]
    want, _ = gpu_lib.ds_forward(net, imgs, route_override=over)
    odd = ~torch.isfinite(want).all(dim=1)
    assert odd.nonzero().flatten().tolist() == [5, 1234]
    assert torch.equal(torch.isnan(got[odd]), torch.isnan(want[odd])) and torch.equal(got[~odd], want[~odd])


# the same where hidden values, or their products with the weights of fc2, reach 2^127 and stay finite: nothing that a sum goes through on the way may
# be larger than it is in the launches on the row-major weights
@pytest.mark.parametrize("large", ["hidden values", "sums"])
def test_vit_two_workgroups_large_values(gpu_lib, large):
    arch = WL.vit_arch(image=64, depth=2)                    # 17 tokens
    arch["routes"], arch["T"] = np.array([(384, 6, 1536), (200, 3, 808)], np.int32), 2
    p = WL.vit_params(arch, 13)
    for l in range(2):
        b1, w2 = p[f"l{l}.fc1.b"], p[f"l{l}.fc2.w"]
        if large == "hidden values":
            b1[[3, 500, 807]], w2[:, [3, 500, 807]] = 2.5e38, 2.0 ** -125       # (2^127 is 1.7e38)
        else:
            b1[[3, 500]] = 2.0 ** 20                         # (GELU of it, rounded: the same, whatever the rows add)
            w2[:, 3], w2[:, 500] = 1.1875 * 2.0 ** 107, -1.1875 * 2.0 ** 107
    net = gpu_lib.build_vit(arch, p, DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(13)
    B = 2300                                                 # 612 tiles of 64 rows
    assert _in_two_workgroups(B, arch["tokens"], arch["T"])
    imgs = torch.randn((B, 3, arch["image"], arch["image"]), generator=gen, device=DEV).to(torch.bfloat16)
    over = (torch.arange(B, device=DEV, dtype=torch.int32) % 2)[None].contiguous()
    got, _ = gpu_lib.ds_forward(net, imgs, route_override=over)
    net.c_struct.n_params -= 4 * arch["depth"]
    want, _ = gpu_lib.ds_forward(net, imgs, route_override=over)
    assert torch.isfinite(want).all() and want.abs().max() > 0 and torch.equal(got, want)


# heads over two workgroups, four query tiles and the rest: the largest number of heads that are (128) and one sample more, as many
# wavefronts as a workgroup of one half has and one more
@pytest.mark.parametrize("dh,H,N,B", [(48, 8, 197, 16), (48, 8, 197, 17), (64, 2, 224, 3), (32, 4, 128, 32), (32, 4, 129, 32), (32, 4, 129, 33)])
def test_attention_in_two_workgroups(gpu_lib, dh, H, N, B):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(dh + B)
    D = H * dh
    x = torch.randn((B, N, D), generator=gen, device=DEV).to(torch.bfloat16)
    w = (torch.randn((4, D, D), generator=gen, device=DEV) * 0.06).to(torch.bfloat16)
    bias = 0.1 * torch.randn((4, D), generator=gen, device=DEV)
    perm, inv, off = gpu_lib.ds_route_bucket(torch.zeros(B, dtype=torch.int32, device=DEV), 1)
    g = gpu_lib.make_groups(off, perm, [D], [D])
    y = torch.empty_like(x)
    gpu_lib.ds_sliced_mhsa(x, w[:3].contiguous(), bias[:3].contiguous(), w[3].contiguous(), bias[3].contiguous(), H, dh, g, residual=x, y=y)
    bf = lambda a: a.astype(np.float32)
    xh, wh, bh, yh = host(x), host(w), host(bias), host(y)
    for b in sorted({0, 1, B // 2, B - 1}):
        att = O.sliced_mhsa(bf(xh[b]), wh[0], bh[0], wh[1], bh[1], wh[2], bh[2], wh[3], bh[3], H, dh, store="bf16")
        assert relerr(yh[b], O.bf16_round(xh[b] + att)) < TOL_BF16, b


# fp32 results with and without a residual and GELU, on every tile of the grouped GEMM: slices that end inside a tile's 64 columns and inside
# either half of them, ragged last rows.  fp32 sums of up to 776 products: at most 776 x 2^-24 = 4.6e-5 of the sum of their magnitudes
@pytest.mark.parametrize("res,act", [(False, 0), (True, 0), (False, 2), (True, 2), (True, 1)])
@pytest.mark.parametrize("B,rows,k_in,k_out", [
    (20, 131, (200, 72, 8), (488, 104, 40)),                         # 32-deep slabs
    (70, 131, (392, 136), (504, 72)),                                # 64-deep slabs
    (20, 131, (328, 40), (488, 104)),                                # two shares of the reduction
    (20, 131, (584, 8), (488, 72)),                                  # four
    (70, 131, (520, 264), (504, 40)),                                # 128-deep slabs
    (1960, 197, (136, 40), (128, 72)),                               # 128 columns, 32-deep slabs
    (134, 197, (776, 40), (1240, 72)),                               # 128 columns, 64-deep slabs
    (1, 5, (72, 8), (40, 8))])                                       # a few rows
def test_sliced_linear_fp32_results(gpu_lib, B, rows, k_in, k_out, res, act):
    T, K, N = len(k_in), max(k_in), max(k_out)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(B + K)
    rn = lambda *s: torch.randn(s, generator=gen, device=DEV)  # noqa: E731
    x, w, bias = rn(B, rows, K).to(torch.bfloat16), (rn(N, K) * K ** -0.5).to(torch.bfloat16), rn(N)
    r = rn(B, rows, N).to(torch.bfloat16) if res else None
    route = torch.arange(B, device=DEV, dtype=torch.int32) % T
    perm, inv, off = gpu_lib.ds_route_bucket(route, T)
    y = torch.full((B, rows, N), float("nan"), device=DEV)
    gpu_lib.ds_sliced_linear(x, w, bias, gpu_lib.make_groups(off, perm, k_in, k_out), act=act, residual=r, y=y)
    inside = torch.arange(N, device=DEV)[None] < torch.tensor(k_out, device=DEV)[route.long()][:, None]
    assert torch.equal(torch.isfinite(y), inside[:, None, :].expand_as(y))
    wh, bh = host(w), host(bias)
    for b in sorted({0, min(1, B - 1), B // 2, B - 1}):
        ki, ko = k_in[b % T], k_out[b % T]
        want = host(x[b])[:, :ki] @ wh[:ko, :ki].T + bh[:ko]
        if res:
            want = want + host(r[b])[:, :ko]
        want = O.gelu(want) if act == 2 else np.maximum(want, 0.0) if act == 1 else want
        assert relerr(host(y[b])[:, :ko], want) < 1e-4, b


# two workgroups a head (up to 128 heads: 21 images of six heads, 16 of eight) and one: every row of every block has the same bits
@pytest.mark.parametrize("big,B", [(False, 1), (False, 21), (True, 3), (True, 16)])
def test_attention_halves_have_the_bits_of_the_whole(gpu_lib, big, B):
    kw = dict(embed=416, heads=8, head_dim=48, mlp=1664, depth=2, routes="pp") if big else dict(depth=2)
    arch = WL.vit_arch(**kw)
    net = gpu_lib.build_vit(arch, WL.vit_params(arch, 6), DEV)
    whole = 40                                                       # 240 and 320 heads: one workgroup each
    gen = torch.Generator(device=DEV)
    gen.manual_seed(B)
    imgs = torch.randn((whole, 3, arch["image"], arch["image"]), generator=gen, device=DEV).to(torch.bfloat16)
    over = ((arch["T"] - 1 - 3 * torch.arange(whole, device=DEV, dtype=torch.int32)) % arch["T"])[None].contiguous()      # (the deepest first)

    def blocks(n):
        taps = {i: torch.zeros((n, arch["tokens"], arch["embed"]), dtype=torch.bfloat16, device=DEV) for i in range(2)}
        gpu_lib.ds_forward_taps(net, imgs[:n].contiguous(), taps, route_override=over[:, :n].contiguous())
        return taps

    few, many = blocks(B), blocks(whole)
    for i in range(2):
        assert few[i].abs().max() > 0 and torch.equal(few[i], many[i][:B]), i


# 3x3 layers on tiled filters against those on the row-major ones: tiles of 64 and of 128 pixels, of one sample's rows and across samples, stride 1 on maps
# of 7x7 to 14x14 pixels, stride 2 from 6x6 to 56x56, slices that end inside a 32-channel chunk and inside a block of 32 filters, routes that end
# early.  Filters behind the widest slice in use may hold anything.  The last entry: the blocks whose 3x3 layer runs on tiled filters, those of stride 1 with the pixels of
# a tile (the others are narrow enough for bneck_kernel, on maps whose patch does not fit, or run by no sample).
TILED = [(224, 150, "width", (1, 1, 2, 2), {2: None, 3: 128, 4: None, 5: 64}), (224, 60, "pp", (2, 2, 3, 2), {2: None, 4: None, 5: 64, 7: None, 8: 64}),
         (112, 230, "pp", (2, 3, 2, 2), {2: None, 5: None, 7: None}), (104, 33, "depth", (1, 2, 3, 2), {1: None, 2: 64}),
         (96, 300, "width", (1, 2, 2, 2), {1: None, 3: None, 4: 64, 5: None}), (224, 230, "width", (1, 1, 1, 2), {2: None, 3: None, 4: 128})]


def _tiled_case(gpu_lib, image, B, routes, blocks, exact=False):
    arch = WL.resnet_arch(image=image, blocks=blocks, routes=routes)
    p = WL.resnet_params(arch, image + B)
    T, top = arch["T"], arch["T"] - 2                     # the widest route stays out (of "depth": the deepest of the widest slices)
    rng = np.random.default_rng(B)
    for s in range(4):
        k = int(arch["mid"][s][top])
        for b in range(blocks[s]):
            w = p[f"s{s}.b{b}.c2.w"]
            if exact:
                n = w.shape[0]
                w[:] = rng.integers(-1, 2, w.shape)
                for name, gamma, beta in (("c1", 8.0, 192.0), ("c2", 1 / (192 * (6 * n) ** 0.5), None)):
                    bn = p[f"s{s}.b{b}.{name}.bn"]
                    bn["gamma"][:], bn["mean"][:], bn["var"][:] = gamma, 0, 1
                    if beta is not None:
                        bn["beta"][:] = beta
            w[k:] = np.nan
            w[:, k:] = np.inf
    net = gpu_lib.build_resnet(arch, p, DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(B)
    imgs = torch.randn((B, 3, image, image), generator=gen, device=DEV).to(torch.bfloat16)
    over = torch.stack([(torch.arange(B, device=DEV, dtype=torch.int32) * (2 * s + 1) % (T - 1)) for s in range(4)]).contiguous()
    return arch, net, imgs, over


# another order of fp32 sums in bf16 layers: up to 0.001 of the logits in 2-norm, and a single one several times that
@pytest.mark.parametrize("image,B,routes,blocks,layers", TILED)
def test_resnet_tiled_filters(gpu_lib, image, B, routes, blocks, layers):
    arch, net, imgs, over = _tiled_case(gpu_lib, image, B, routes, blocks)
    tiled, _ = gpu_lib.ds_forward(net, imgs, route_override=over)
    net.c_struct.n_params -= sum(blocks)
    plain, _ = gpu_lib.ds_forward(net, imgs, route_override=over)
    assert torch.isfinite(plain).all() and plain.abs().max() > 0
    assert (tiled - plain).norm() < 1.5e-3 * plain.norm() and relerr(host(tiled), host(plain)) < 2e-2


# The same where a 3x3 layer's sums are exact and so the same bits in any order: inputs about 192 in bf16, whole numbers but for the few below 128, and
# filters of -1, 0 and 1 (4608 products of 8 bits).  Every pixel of every block of every sample.  The kernel on tiled filters runs in the layers named and there
# alone: with a layer's tiles zeroed the logits are others.
@pytest.mark.parametrize("image,B,routes,blocks,layers", TILED)
def test_resnet_tiled_filters_exact(gpu_lib, image, B, routes, blocks, layers):
    arch, net, imgs, over = _tiled_case(gpu_lib, image, B, routes, blocks, exact=True)
    sides, r = [], (image // 2 + 1) // 2
    for s in range(4):
        r = r if s == 0 else (r + 1) // 2
        sides += [(r, 4 * arch["widths"][s])] * blocks[s]

    def run():
        taps = {i: torch.zeros((B, r * r, c), dtype=torch.bfloat16, device=DEV) for i, (r, c) in enumerate(sides)}
        logits, _ = gpu_lib.ds_forward_taps(net, imgs, taps, route_override=over)
        return [logits, *taps.values()]

    tiled = run()
    net.c_struct.n_params -= sum(blocks)
    plain = run()
    net.c_struct.n_params += sum(blocks)
    assert torch.isfinite(plain[0]).all() and all(t.abs().max() > 0 for t in plain)
    for i, (a, b) in enumerate(zip(tiled, plain)):
        assert torch.equal(a, b), i
    ran = {}
    line = _line("conv3t.hip", r"wgs > (\d+) \? launch<1, 128>")
    groups = min(B, arch["T"] ** (1 if arch.get("single_gate") else 2))
    for i in range(sum(blocks)):
        t = net.tensors[len(net.tensors) - sum(blocks) + i]
        kept = t.clone()
        t.zero_()
        logits, _ = gpu_lib.ds_forward(net, imgs, route_override=over)
        t.copy_(kept)
        if torch.equal(logits, tiled[0]):
            continue
        stage = next(st for st in range(4) if i < sum(blocks[:st + 1]))
        b, rows = i - sum(blocks[:stage]), sides[i][0] ** 2
        wide = max(int(m) for t, m in enumerate(arch["mid"][stage]) if arch.get("nblk") is None or arch["nblk"][stage][t] > b)
        wgs = ((B * rows - groups) // 128 + groups) * ((wide + 63) // 64)
        ran[i] = None if b == 0 else 128 if wgs > line else 64
    assert ran == layers


# one gate for all stages: one bucket makes the four stages' lists and the routes' four rows -- a sample bucketed by the gate itself, batches
# within and beyond the 1024 samples of a turn, parts with rows of their own, routes out of range, which come back as they were given
@pytest.mark.parametrize("B,parts", [(1, 1), (7, 1), (1100, 1), (40, 2)])
def test_resnet_single_gate_bucket(gpu_lib, B, parts):
    arch = WL.resnet_arch(image=32, blocks=(2, 2, 3, 2), routes="pp")
    net = gpu_lib.build_resnet(arch, WL.resnet_params(arch, 9), DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(B)
    imgs = torch.randn((B, 3, 32, 32), generator=gen, device=DEV).to(torch.bfloat16)
    lb = torch.zeros((4, B, arch["T"]), device=DEV)
    want = torch.arange(B, device=DEV) * 4 % arch["T"]
    lb[0].scatter_(1, want[:, None], 50.0)
    call = (lambda **k: gpu_lib.ds_forward(net, imgs, **k)) if parts == 1 else (lambda **k: gpu_lib.ds_forward_parts(net, imgs, parts, **k))
    routes = torch.full((4, B), -7, dtype=torch.int32, device=DEV)
    logits, _ = call(logit_bias=lb, routes=routes)
    assert torch.isfinite(logits).all() and all(torch.equal(routes[s], want.int()) for s in range(4))
    over = torch.full((4, B), -7, dtype=torch.int32, device=DEV)
    over[0] = want.int()
    same, r2 = call(route_override=over)
    assert torch.equal(same, logits) and torch.equal(r2, routes)
    # a sample's logits are its own
    pick = B - 1
    one, _ = gpu_lib.ds_forward(net, imgs[pick:].contiguous(), route_override=over[:, pick:].contiguous())
    assert relerr(host(one), host(logits[pick:])) < 2e-2
    if B > 4:
        over[0, 2] = arch["T"] + 3
        some, r3 = call(route_override=over)
        keep = torch.arange(B, device=DEV) != 2
        assert all(torch.equal(r3[s], over[0]) for s in range(4)) and relerr(host(some[keep]), host(logits[keep])) < 2e-2
