"""GPU parity of every C-ABI layer call against the CPU oracle on the same seeded inputs.

Tolerances: 1e-5 for fp32, 2e-2 for bf16 inputs with fp32 accumulation, asserted on the
element-wise error max_i |gpu_i - oracle_i| / max(|oracle_i|, rms(oracle)) of every compared
tensor (per sample and route slice), which bounds the stated max |gpu - oracle| / max |oracle|
from above; both are listed at the end of the run (tests/parity.py).  Integer outputs are
bit-exact, routes are exempt only where the oracle's top-2 scores are closer than 1e-6.
"""
import numpy as np
import pytest
import torch

import workloads as WL
from oracle import ds_oracle as O

pytestmark = pytest.mark.gpu

TOL_F32, TOL_BF16 = 1e-5, 2e-2
DEV = "cuda:0"


def dev(a, dtype=torch.float32):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV).to(dtype).contiguous()


from tests.parity import relerr  # noqa: E402  (element-wise form with an rms floor; never below the max form)


def host(t):
    return t.detach().to(torch.float64).cpu().numpy()


# ------------------------------------------------------------------ route bucket
@pytest.mark.parametrize("B,T,seed", [(0, 4, 0), (1, 1, 1), (7, 3, 2), (64, 4, 3), (256, 14, 4), (256, 48, 5),
                                      (256, 16, 6), (3000, 64, 7), (2049, 1024, 8)])
def test_route_bucket_bit_exact(gpu_lib, B, T, seed):
    rng = np.random.default_rng(seed)
    route = rng.integers(0, T, B).astype(np.int32)
    if B > 10:
        route[route == 1 % T] = 0          # force an empty bucket
    perm, inv, off = gpu_lib.ds_route_bucket(dev(route, torch.int32), T)
    operm, oinv, ooff = O.route_bucket(route, T)
    assert np.array_equal(perm.cpu().numpy(), operm)
    assert np.array_equal(inv.cpu().numpy(), oinv)
    assert np.array_equal(off.cpu().numpy(), ooff)


def test_route_bucket_flags_out_of_range_ids(gpu_lib):
    route = np.array([0, 5, 1, -1, 1], np.int32)
    _, _, off = gpu_lib.ds_route_bucket(dev(route, torch.int32), 2)
    assert off.cpu().numpy().tolist() == [0, 1, 3]      # offsets[T] = 3 valid ids != B


# ------------------------------------------------------------------ gate
def _check_routes(route_gpu, logits_oracle):
    for b, z in enumerate(logits_oracle):
        if O.gate_margin(z) >= 1e-6:
            assert int(route_gpu[b]) == O.gate_route(z), (b, z)


def test_gate_config1_fp32_nchw(gpu_lib):
    c = WL.config1()
    x = dev(c["x"])
    logits, route = gpu_lib.ds_gate(x, gpu_lib.DS_NCHW, dev(c["gate.w1"]), dev(c["gate.b1"]), dev(c["gate.w2"]),
                                    dev(c["gate.b2"]), c["T"])
    want = np.stack([O.gate_logits(O.gate_encoder(c["x"][b]), c["gate.w1"], c["gate.b1"], c["gate.w2"], c["gate.b2"])
                     for b in range(c["B"])])
    assert relerr(host(logits), want) < TOL_F32
    _check_routes(route.cpu().numpy(), want)


@pytest.mark.parametrize("C,HW,hid,T,B", [(256, 784, 64, 14, 33), (64, 3136, 16, 4, 9), (1024, 196, 256, 4, 17)])
def test_gate_bf16_nhwc_with_sliced_input_and_bias(gpu_lib, C, HW, hid, T, B):
    d = WL.nets.Draw(100 + C)
    x = WL.nets.as_bf16_values(d.normal((B, HW, C)))
    w1, b1 = d.normal((hid, C), std=C ** -0.5), d.normal((hid,), std=0.1)
    w2, b2 = d.normal((T, hid), std=hid ** -0.5), d.normal((T,), std=0.1)
    lb = WL.seeded_logit_bias(7, B, T)
    c_in = (8 * d.randint(B, C // 8) + 8).astype(np.int32)
    logits, route = gpu_lib.ds_gate(dev(x, torch.bfloat16), gpu_lib.DS_NHWC, dev(w1), dev(b1), dev(w2), dev(b2), T,
                                    logit_bias=dev(lb), c_in=dev(c_in, torch.int32))
    want = np.stack([O.gate_logits(O.gate_encoder(x[b].T[:c_in[b]].reshape(c_in[b], HW, 1)), w1, b1, w2, b2, lb[b])
                     for b in range(B)])
    assert relerr(host(logits), want) < TOL_F32
    _check_routes(route.cpu().numpy(), want)


def test_gate_argmax_only_ties_and_nan(gpu_lib):
    lb = np.array([[0.1, 0.7, 0.3], [0.7, 0.7, 0.3], [0.1, 0.7, 0.7], [np.nan, 0.2, 0.1], [np.nan] * 3], np.float32)
    logits, route = gpu_lib.ds_gate(None, 0, None, None, None, None, 3, logit_bias=dev(lb))
    assert route.cpu().numpy().tolist() == [O.gate_route(z) for z in lb] == [1, 0, 1, 1, 0]
    assert np.array_equal(logits.cpu().numpy(), lb, equal_nan=True)


# ------------------------------------------------------------------ double-headed gate (Eq. 23)
@pytest.mark.parametrize("C,HW,hid,T,B", [(256, 784, 64, 14, 19), (64, 3136, 16, 4, 5), (1024, 49, 256, 4, 9)])
def test_gate_double_bf16_nhwc_sliced(gpu_lib, C, HW, hid, T, B):
    d = WL.nets.Draw(300 + C)
    x = WL.nets.as_bf16_values(d.normal((B, HW, C)))
    w1, b1 = d.normal((hid, C), std=C ** -0.5), d.normal((hid,), std=0.1)
    w2, b2 = d.normal((T, hid), std=hid ** -0.5), d.normal((T,), std=0.1)
    w3, b3 = d.normal((C, hid), std=hid ** -0.5), d.normal((C,), std=0.1)
    lb = WL.seeded_logit_bias(11, B, T)
    c_in = (8 * d.randint(B, C // 8) + 8).astype(np.int32)
    y0 = torch.full((B, HW, C), float("nan"), dtype=torch.bfloat16, device=DEV)
    y, logits, route = gpu_lib.ds_gate_double(dev(x, torch.bfloat16), gpu_lib.DS_NHWC, dev(w1), dev(b1), dev(w3), dev(b3),
                                              w2=dev(w2), b2=dev(b2), T=T, logit_bias=dev(lb),
                                              c_in=dev(c_in, torch.int32), y=y0)
    yh = host(y)
    want_logits = []
    for b in range(B):
        c = int(c_in[b])
        xb = x[b].T[:c].reshape(c, HW, 1)
        want = O.bf16_round(O.gate_attention(xb, w1, b1, w3, b3))[:, :, 0].T          # [HW, c]
        assert relerr(yh[b, :, :c], want) < TOL_BF16
        # a single rounding of an fp32 product: at most one bf16 step away from the oracle anywhere
        assert np.max(np.abs(yh[b, :, :c] - want) / np.maximum(np.abs(want), 1e-30)) <= 2.0 ** -7
        assert np.all(np.isnan(yh[b, :, c:])), "channels beyond the sample's width were written"
        want_logits.append(O.gate_logits(O.gate_encoder(xb), w1, b1, w2, b2, lb[b]))
    want_logits = np.stack(want_logits)
    assert relerr(host(logits), want_logits) < TOL_F32
    _check_routes(route.cpu().numpy(), want_logits)


def test_gate_double_fp32_nchw_attention_only_in_place(gpu_lib):
    c = WL.config1()
    d = WL.nets.Draw(77)
    C, hid = c["x"].shape[1], c["gate.w1"].shape[0]
    w3, b3 = d.normal((C, hid), std=hid ** -0.5), d.normal((C,), std=0.1)
    x = dev(c["x"]).clone()
    y, logits, route = gpu_lib.ds_gate_double(x, gpu_lib.DS_NCHW, dev(c["gate.w1"]), dev(c["gate.b1"]), dev(w3), dev(b3), y=x)
    assert logits is None and route is None and y.data_ptr() == x.data_ptr()
    want = np.stack([O.gate_attention(c["x"][b], c["gate.w1"], c["gate.b1"], w3, b3) for b in range(c["B"])])
    assert relerr(host(y), want) < TOL_F32
    # zero projection: the feature map passes through bit for bit
    x2 = dev(c["x"])
    y2, _, _ = gpu_lib.ds_gate_double(x2, gpu_lib.DS_NCHW, dev(c["gate.w1"]), dev(c["gate.b1"]), dev(np.zeros_like(w3)), None)
    assert np.array_equal(host(y2), c["x"].astype(np.float32))


# ------------------------------------------------------------------ sliced linear (config 2)
def _linear_case(gpu_lib, c, y_dtype, act=0, with_res=False):
    B, N, K = c["B"], c["N"], c["K"]
    route = dev(c["route"], torch.int32)
    perm, inv, off = gpu_lib.ds_route_bucket(route, c["T"])
    g = gpu_lib.make_groups(off, perm, c["k_in"], c["k_out"])
    x, w, bias = dev(c["x"], torch.bfloat16), dev(c["w"], torch.bfloat16), dev(c["bias"])
    y = torch.full((B, N, 4 * K), float("nan"), dtype=y_dtype, device=DEV)
    res = None
    if with_res:
        res_h = WL.nets.as_bf16_values(WL.nets.Draw(9).normal((B, N, 4 * K)))
        res = dev(res_h, torch.bfloat16)
    gpu_lib.ds_sliced_linear(x, w, bias, g, act=act, residual=res, y=y)
    yh = host(y)
    worst = 0.0
    for b in range(B):
        ki, ko = int(c["k_in"][c["route"][b]]), int(c["k_out"][c["route"][b]])
        want = O.sliced_linear(c["x"][b, :, :ki], c["w"], c["bias"], ko)
        if with_res:
            want = want + res_h[b, :, :ko]
        if act == 2:
            want = O.gelu(want)
        if y_dtype == torch.bfloat16:
            want = O.bf16_round(want)
        assert np.all(np.isnan(yh[b, :, ko:])), "tail beyond the valid slice was written"
        worst = max(worst, relerr(yh[b, :, :ko], want))
    return worst


@pytest.mark.parametrize("balanced", [False, True])
@pytest.mark.parametrize("y_dtype", [torch.bfloat16, torch.float32])
def test_sliced_linear_config2(gpu_lib, balanced, y_dtype):
    c = WL.config2(balanced=balanced)
    assert _linear_case(gpu_lib, c, y_dtype) < (TOL_BF16 if y_dtype == torch.bfloat16 else 1e-4)


def test_sliced_linear_gelu_residual_ragged_small(gpu_lib):
    c = WL.config2(seed=77, B=5, N=37, K=48)          # k_in 24..48: K tails inside a 32-wide slab
    assert _linear_case(gpu_lib, c, torch.bfloat16, act=2) < TOL_BF16
    assert _linear_case(gpu_lib, c, torch.bfloat16, with_res=True) < TOL_BF16
    c = WL.config2(seed=78, B=3, N=1, K=96)
    assert _linear_case(gpu_lib, c, torch.float32) < 1e-4


# GELU of every bf16 value (identity weights: a sum is the value itself), values inside and outside the polynomial's range beside each other in a lane, the few-image
# launches and the others: the nearest bf16, but where the exact result lies closer to the middle of two than fp32's own error, 1.25e-7 of |x|
@pytest.mark.parametrize("copies", [1, 64])
@pytest.mark.parametrize("y_dtype", [torch.bfloat16, torch.float32])
def test_gelu_of_every_value(gpu_lib, copies, y_dtype):
    from scipy.special import erfc
    every = (torch.arange(1 << 16, dtype=torch.int32) << 16).view(torch.float32)
    finite = every[torch.isfinite(every)]                          # 65280 = 1020 rows of 64
    B, rows, W = 4 * copies, 256, 64
    gen = torch.Generator().manual_seed(3)
    dense = [finite[torch.randperm(finite.numel(), generator=gen)] if i else finite for i in range(copies)]
    x = torch.stack([torch.cat([d, torch.zeros(4 * W)]) for d in dense]).view(B, rows, W)
    off = torch.tensor([0, B], dtype=torch.int32, device=DEV)
    g = gpu_lib.make_groups(off, None, [W])
    eye = torch.eye(W, dtype=torch.bfloat16, device=DEV)
    for shift in (0.0, 0.0078125 / 3):                             # (the second: values that are no bf16)
        bias = torch.full((W,), shift, device=DEV)
        y = gpu_lib.ds_sliced_linear(x.to(DEV).to(torch.bfloat16), eye, bias, g, act=gpu_lib.DS_ACT_GELU, y_dtype=y_dtype)
        v = (x + bias.cpu()).double().numpy()                      # (one rounding, as in the kernel)
        want, got = 0.5 * v * erfc(v * -0.5 ** 0.5), host(y)
        most = 3.38e38                                             # (what rounds to infinity is not compared)
        ulp = 2.0 ** (np.floor(np.log2(np.maximum(np.abs(want), 2.0 ** -120))) - (8 if y_dtype == torch.bfloat16 else 24))
        ok = (np.abs(got - want) <= ulp + 1.25e-7 * np.abs(v)) | (np.abs(want) > most)
        assert ok.all(), (v[~ok][:5], got[~ok][:5], want[~ok][:5])
    # what is not finite, one a row
    odd = torch.tensor([float("inf"), float("-inf"), float("nan")])
    x = torch.zeros((B, rows, W))
    for i in range(3):
        x[:, i::3, 5 * i] = odd[i]
    y = gpu_lib.ds_sliced_linear(x.to(DEV).to(torch.bfloat16), eye, torch.zeros(W, device=DEV), g, act=gpu_lib.DS_ACT_GELU, y_dtype=y_dtype)
    # (0 times what is not finite is NaN in the row's other columns; minus infinity times an erfc of zero as well)
    got = y.float().cpu()
    assert torch.isposinf(got[:, 0::3, 0]).all() and torch.isnan(got[:, 1::3, 5]).all() and torch.isnan(got[:, 2::3, 10]).all()


def test_sliced_linear_one_bucket_gets_everything_and_empty_batch(gpu_lib):
    c = WL.config2(seed=79, B=6, N=50, K=48)
    c["route"][:] = 2
    assert _linear_case(gpu_lib, c, torch.bfloat16) < TOL_BF16
    off = torch.zeros(5, dtype=torch.int32, device=DEV)
    g = gpu_lib.make_groups(off, None, c["k_in"], c["k_out"])
    x0 = torch.zeros((0, 50, 48), dtype=torch.bfloat16, device=DEV)
    y0 = gpu_lib.ds_sliced_linear(x0, dev(c["w"], torch.bfloat16), None, g)
    assert y0.shape[0] == 0


def test_bf16_storage_rounding_is_nearest_even_bit_exact(gpu_lib):
    """With zero weights the layer stores bf16(bias): the storage rounding itself, ties included."""
    K, N, B, rows = 32, 512, 2, 3
    ulp = 2.0 ** -7
    special = [1.0 + ulp / 2, 1.0 + 3 * ulp / 2, 1.0 + ulp / 2 + 2.0 ** -20, -(1.0 + ulp / 2), 3.0e-5, 1234.567, -0.3333333]
    bias = (np.random.default_rng(3).standard_normal(N) * 3).astype(np.float32)
    bias[:len(special)] = np.array(special, np.float32)
    off = torch.tensor([0, B], dtype=torch.int32, device=DEV)
    g = gpu_lib.make_groups(off, None, [K], [N])
    x = torch.randn(B, rows, K, device=DEV).to(torch.bfloat16)
    w = torch.zeros(N, K, dtype=torch.bfloat16, device=DEV)
    y = gpu_lib.ds_sliced_linear(x, w, dev(bias), g)
    want = O.bf16_round(bias.astype(np.float64))
    assert np.array_equal(host(y)[1, 2], want)


# ------------------------------------------------------------------ config 1: gate + sliced conv + split BN + ReLU, fp32
def _config1_block(gpu_lib, c, forced=None):
    B, T = c["B"], c["T"]
    x = dev(c["x"])
    if forced is None:
        _, route = gpu_lib.ds_gate(x, gpu_lib.DS_NCHW, dev(c["gate.w1"]), dev(c["gate.b1"]), dev(c["gate.w2"]),
                                   dev(c["gate.b2"]), T)
    else:
        route = dev(np.asarray(forced, np.int32), torch.int32)
    perm, inv, off = gpu_lib.ds_route_bucket(route, T)
    bn = c["bn"]
    scale, shift = gpu_lib.ds_bn_fold(dev(bn["gamma"]), dev(bn["beta"]), dev(bn["mean"]), dev(bn["var"]), c["bn_eps"])
    g = gpu_lib.make_groups(off, perm, [c["C"]] * T, c["c_out"])
    y = torch.full((B, c["C"], c["H"], c["W"]), float("nan"), device=DEV)
    gpu_lib.ds_sliced_conv(x, dev(c["conv.w"]), scale, shift, g, c["stride"], c["pad"], act=gpu_lib.DS_ACT_RELU, y=y)
    return route.cpu().numpy(), host(y)


def _config1_oracle(c, b, t):
    co = int(c["c_out"][t])
    y = O.sliced_conv2d(c["x"][b], c["conv.w"], co, c["stride"], c["pad"])
    return O.relu(O.re_sbn(y, c["bn"], t, c["bn_eps"]))


@pytest.mark.parametrize("seed,n_routes", [(None, 1), (WL.CONFIG1_MIXED_SEEDS[0], 2), (WL.CONFIG1_MIXED_SEEDS[1], 3)])
def test_config1_free_running_block(gpu_lib, seed, n_routes):
    # the configuration's own seed routes all eight samples alike; the recorded later seeds give mixed batches from the
    # computed gate alone (no bias), every margin above 1e-3, so the routes must match the oracle exactly
    c = WL.config1() if seed is None else WL.config1(seed=seed)
    route, y = _config1_block(gpu_lib, c)
    z = [O.gate_logits(O.gate_encoder(c["x"][b]), c["gate.w1"], c["gate.b1"], c["gate.w2"], c["gate.b2"])
         for b in range(c["B"])]
    _check_routes(route, z)
    assert len(set(route.tolist())) == n_routes
    if seed is not None:
        assert min(O.gate_margin(v) for v in z) > 1e-3
        assert route.tolist() == [O.gate_route(v) for v in z]
    for b in range(c["B"]):
        t = int(route[b])
        co = int(c["c_out"][t])
        assert relerr(y[b, :co], _config1_oracle(c, b, t)) < TOL_F32
        assert np.all(np.isnan(y[b, co:]))


def test_config1_forced_routes_cover_all_ratios(gpu_lib):
    c = WL.config1()
    forced = [0, 1, 2, 3, 3, 2, 1, 0]
    _, y = _config1_block(gpu_lib, c, forced)
    for b, t in enumerate(forced):
        co = int(c["c_out"][t])
        assert relerr(y[b, :co], _config1_oracle(c, b, t)) < TOL_F32
        assert np.all(np.isnan(y[b, co:]))


# ------------------------------------------------------------------ bf16 NHWC conv (implicit GEMM)
@pytest.mark.parametrize("K,stride,pad,H,CI,CO,res", [(3, 1, 1, 14, 64, 64, False), (3, 2, 1, 15, 48, 80, False),
                                                       (1, 1, 0, 9, 96, 40, True), (1, 2, 0, 14, 64, 128, False),
                                                       (3, 1, 1, 7, 136, 24, True),
                                                       # 1x1 layers with a thin reduction and several 64-column passes: the
                                                       # streaming kernel (up to 64 input channels; up to 128 with a residual)
                                                       (1, 1, 0, 13, 64, 200, True), (1, 1, 0, 9, 40, 136, False),
                                                       (1, 1, 0, 11, 128, 264, True), (1, 1, 0, 11, 128, 264, False),
                                                       # 3x3 stride 1 on wide maps: the patch-staged kernel up to 59 pixels,
                                                       # the tap-walking kernel beyond
                                                       (3, 1, 1, 56, 32, 72, False), (3, 1, 1, 59, 32, 16, True),
                                                       (3, 1, 1, 60, 32, 16, False),
                                                       # few workgroups and 512+ channels per tap: the 128-deep slabs, with
                                                       # slices that end 8 channels into a slab
                                                       (1, 1, 0, 7, 1040, 72, True), (1, 1, 0, 7, 1040, 136, False),
                                                       (3, 2, 1, 9, 528, 40, False)])
def test_sliced_conv_bf16_nhwc(gpu_lib, K, stride, pad, H, CI, CO, res):
    B, T = 11, 4
    d = WL.nets.Draw(1000 + K * 10 + stride + CI)
    x = WL.nets.as_bf16_values(d.normal((B, CI, H, H)))
    w = WL.nets.as_bf16_values(d.normal((CO, CI, K, K), std=(2.0 / (CI * K * K)) ** 0.5))
    bn = WL.bn_tables(d, T, CO)
    route = d.randint(B, T)
    c_in = [CI * q // 4 // 8 * 8 for q in (1, 2, 3, 4)]
    c_out = [max(8, CO * q // 4 // 8 * 8) for q in (1, 2, 3, 4)]
    Ho = (H + 2 * pad - K) // stride + 1
    resid = WL.nets.as_bf16_values(d.normal((B, CO, Ho, Ho))) if res else None
    perm, inv, off = gpu_lib.ds_route_bucket(dev(route, torch.int32), T)
    scale, shift = gpu_lib.ds_bn_fold(dev(bn["gamma"]), dev(bn["beta"]), dev(bn["mean"]), dev(bn["var"]), 1e-5)
    g = gpu_lib.make_groups(off, perm, c_in, c_out)
    xg = dev(x.transpose(0, 2, 3, 1), torch.bfloat16)
    wg = dev(w.transpose(0, 2, 3, 1), torch.bfloat16)
    rg = dev(resid.transpose(0, 2, 3, 1), torch.bfloat16) if res else None
    y = torch.full((B, Ho, Ho, CO), float("nan"), dtype=torch.bfloat16, device=DEV)
    gpu_lib.ds_sliced_conv(xg, wg, scale, shift, g, stride, pad, act=gpu_lib.DS_ACT_RELU, residual=rg, y=y)
    yh = host(y).transpose(0, 3, 1, 2)
    for b in range(B):
        t = int(route[b])
        ci, co = c_in[t], c_out[t]
        want = O.re_sbn(O.sliced_conv2d(x[b, :ci], w, co, stride, pad), bn, t, 1e-5)
        if res:
            want = want + resid[b, :co]
        want = O.bf16_round(O.relu(want))
        assert relerr(yh[b, :co], want) < TOL_BF16
        assert np.all(np.isnan(yh[b, co:]))


# ------------------------------------------------------------------ depthwise conv
@pytest.mark.parametrize("stride,H,C", [(1, 14, 64), (2, 14, 96), (2, 7, 40), (1, 9, 264), (1, 57, 32), (2, 56, 24)])
def test_sliced_dwconv(gpu_lib, stride, H, C):
    B, T = 9, 5
    d = WL.nets.Draw(2000 + stride + C)
    x = WL.nets.as_bf16_values(d.normal((B, C, H, H)))
    w = WL.nets.as_bf16_values(d.normal((C, 1, 3, 3), std=0.5))
    bn = WL.bn_tables(d, T, C)
    route = d.randint(B, T)
    cs = [max(8, C * q // 5 // 8 * 8) for q in (1, 2, 3, 4, 5)]
    perm, inv, off = gpu_lib.ds_route_bucket(dev(route, torch.int32), T)
    scale, shift = gpu_lib.ds_bn_fold(dev(bn["gamma"]), dev(bn["beta"]), dev(bn["mean"]), dev(bn["var"]), 1e-5)
    g = gpu_lib.make_groups(off, perm, cs)
    Ho = (H - 1) // stride + 1
    y = torch.full((B, Ho, Ho, C), float("nan"), dtype=torch.bfloat16, device=DEV)
    gpu_lib.ds_sliced_dwconv(dev(x.transpose(0, 2, 3, 1), torch.bfloat16), dev(w[:, 0].transpose(1, 2, 0), torch.bfloat16),
                             scale, shift, g, stride, y=y)
    yh = host(y).transpose(0, 3, 1, 2)
    for b in range(B):
        t = int(route[b])
        c = cs[t]
        want = O.bf16_round(O.relu(O.re_sbn(O.sliced_dwconv2d(x[b, :c], w, stride, 1), bn, t, 1e-5)))
        assert relerr(yh[b, :c], want) < TOL_BF16
        assert np.all(np.isnan(yh[b, c:]))


# spatially sliced depthwise filter (Section 3.2, Eq. 11-13): per route a centred block of the stored 7x7 filter,
# optionally every other / every third tap at that dilation, and its own padding, hence its own output resolution
@pytest.mark.parametrize("stride,H,C,K", [(1, 14, 512, 7), (2, 14, 512, 7), (1, 28, 72, 5), (2, 9, 64, 3)])
def test_sliced_dwconv_spatial(gpu_lib, stride, H, C, K):
    B = 11
    d = WL.nets.Draw(2100 + stride + C + K)
    x = WL.nets.as_bf16_values(d.normal((B, C, H, H)))
    w = WL.nets.as_bf16_values(d.normal((C, 1, K, K), std=0.3))
    # (kernel size, dilation, padding): same-size crops, a dilated full filter, valid (unpadded) and over-padded routes
    spec = [(3, 1, 1), (5, 1, 2), (7, 1, 3), (7, 2, 3), (7, 3, 3), (3, 1, 0), (5, 2, 1), (1, 1, 0), (7, 1, 1), (3, 1, 3)]
    spec = [(k, l, p) for k, l, p in spec if k <= K and (K - k) % 2 == 0]
    T = len(spec)
    bn = WL.bn_tables(d, T, C)
    route = np.arange(B, dtype=np.int32) % T
    route = route[d.permutation(B)]
    cs = [max(8, C * (1 + t % 4) // 4 // 8 * 8) for t in range(T)]
    perm, inv, off = gpu_lib.ds_route_bucket(dev(route, torch.int32), T)
    scale, shift = gpu_lib.ds_bn_fold(dev(bn["gamma"]), dev(bn["beta"]), dev(bn["mean"]), dev(bn["var"]), 1e-5)
    g = gpu_lib.make_groups(off, perm, cs)
    res = []
    for k, l, p in spec:
        n = (k + l - 1) // l
        res.append((H + 2 * p - ((n - 1) * l + 1)) // stride + 1)
    rows_max = max(r * r for r in res)
    y = torch.full((B, rows_max, C), float("nan"), dtype=torch.bfloat16, device=DEV)
    _, got_res = gpu_lib.ds_sliced_dwconv_spatial(
        dev(x.transpose(0, 2, 3, 1), torch.bfloat16), dev(w[:, 0].transpose(1, 2, 0), torch.bfloat16), scale, shift, g,
        [s_[0] for s_ in spec], [s_[1] for s_ in spec], [s_[2] for s_ in spec], stride, y=y)
    assert [r[0] for r in got_res] == res
    yh = host(y)
    for b in range(B):
        t = int(route[b])
        k, l, p = spec[t]
        c, r = cs[t], res[t]
        want = O.bf16_round(O.relu(O.re_sbn(O.spatial_dwconv2d(x[b, :c], w, k, l, stride, p), bn, t, 1e-5)))
        assert want.shape == (c, r, r)
        got = yh[b, :r * r, :c].reshape(r, r, c).transpose(2, 0, 1)
        assert relerr(got, want) < TOL_BF16, (b, spec[t])
        assert np.all(np.isnan(yh[b, :r * r, c:])) and np.all(np.isnan(yh[b, r * r:]))
    # the plain 3x3 entry point is the K = 3, k = 3, padding 1 case of this one
    if K == 3:
        g3 = gpu_lib.make_groups(off, perm, cs)
        Ho = (H - 1) // stride + 1
        y3 = torch.full((B, Ho, Ho, C), float("nan"), dtype=torch.bfloat16, device=DEV)
        gpu_lib.ds_sliced_dwconv(dev(x.transpose(0, 2, 3, 1), torch.bfloat16), dev(w[:, 0].transpose(1, 2, 0), torch.bfloat16),
                                 scale, shift, g3, stride, y=y3)
        ys = torch.full((B, Ho * Ho, C), float("nan"), dtype=torch.bfloat16, device=DEV)
        gpu_lib.ds_sliced_dwconv_spatial(dev(x.transpose(0, 2, 3, 1), torch.bfloat16),
                                         dev(w[:, 0].transpose(1, 2, 0), torch.bfloat16), scale, shift, g3,
                                         [3] * T, [1] * T, [1] * T, stride, y=ys)
        a, b_ = host(y3).reshape(B, Ho * Ho, C), host(ys)
        assert np.array_equal(np.isnan(a), np.isnan(b_)) and relerr(np.nan_to_num(b_), np.nan_to_num(a)) < 1e-2


def test_sliced_dwconv_spatial_rejects_bad_tables(gpu_lib):
    B, C, H, K = 2, 16, 8, 7
    x = torch.zeros((B, H, H, C), dtype=torch.bfloat16, device=DEV)
    w = torch.zeros((K, K, C), dtype=torch.bfloat16, device=DEV)
    sc = torch.ones((1, C), dtype=torch.float32, device=DEV)
    off = torch.tensor([0, B], dtype=torch.int32, device=DEV)
    g = gpu_lib.make_groups(off, None, [C])
    for k, l, p in [(4, 1, 1), (9, 1, 1), (3, 0, 1), (3, 1, -1), (7, 1, 0)]:      # even crop, too large, dilation 0, negative pad, ok
        if (k, l, p) == (7, 1, 0):
            gpu_lib.ds_sliced_dwconv_spatial(x, w, sc, sc, g, [k], [l], [p], 1)
        else:
            with pytest.raises(gpu_lib.DsError):
                gpu_lib.ds_sliced_dwconv_spatial(x, w, sc, sc, g, [k], [l], [p], 1)
    xs = torch.zeros((B, 4, 4, C), dtype=torch.bfloat16, device=DEV)
    with pytest.raises(gpu_lib.DsError):                                          # no output pixel: 7 taps on a 4x4 map
        gpu_lib.ds_sliced_dwconv_spatial(xs, w, sc, sc, g, [7], [1], [0], 1, y=torch.zeros((B, 1, C), dtype=torch.bfloat16, device=DEV))


# ------------------------------------------------------------------ LayerNorm
def test_sliced_layernorm(gpu_lib):
    B, N, D, T = 13, 29, 384, 4
    d = WL.nets.Draw(3000)
    x = WL.nets.as_bf16_values(d.normal((B, N, D), std=2.0, mean=0.5))
    gm, bt = 1.0 + d.normal((D,), std=0.1), d.normal((D,), std=0.1)
    route = d.randint(B, T)
    ks = [192, 256, 320, 384]
    perm, inv, off = gpu_lib.ds_route_bucket(dev(route, torch.int32), T)
    g = gpu_lib.make_groups(off, perm, ks)
    y = torch.full((B, N, D), float("nan"), dtype=torch.bfloat16, device=DEV)
    gpu_lib.ds_sliced_layernorm(dev(x, torch.bfloat16), dev(gm), dev(bt), 1e-6, g, y=y)
    yh = host(y)
    for b in range(B):
        k = ks[route[b]]
        want = O.bf16_round(O.layernorm_sliced(x[b, :, :k], gm, bt, 1e-6))
        assert relerr(yh[b, :, :k], want) < TOL_BF16
        assert np.all(np.isnan(yh[b, :, k:]))


# ------------------------------------------------------------------ MHSA
# 224 tokens is the longest sequence the attention kernel takes, 1 token the degenerate softmax, 33 a ragged tile
@pytest.mark.parametrize("N,B", [(197, 10), (17, 7), (64, 5), (224, 4), (1, 6), (33, 3)])
def test_sliced_mhsa(gpu_lib, N, B):
    D, H, dh = 384, 6, 64
    d = WL.nets.Draw(4000 + N)
    bf = WL.nets.as_bf16_values
    x = bf(d.normal((B, N, D)))
    wq, wk, wv = (bf(d.normal((H * dh, D), std=0.06)) for _ in range(3))
    bq, bk, bv = (d.normal((H * dh,), std=0.1) for _ in range(3))
    wp, bp = bf(d.normal((D, H * dh), std=0.05)), d.normal((D,), std=0.1)
    routes = [(192, 3), (256, 4), (320, 5), (384, 6), (192, 6), (384, 3)]
    route = d.randint(B, len(routes))
    perm, inv, off = gpu_lib.ds_route_bucket(dev(route, torch.int32), len(routes))
    g = gpu_lib.make_groups(off, perm, [r[0] for r in routes], [r[1] * dh for r in routes])
    y = torch.full((B, N, D), float("nan"), dtype=torch.bfloat16, device=DEV)
    xg = dev(x, torch.bfloat16)
    gpu_lib.ds_sliced_mhsa(xg, dev(np.stack([wq, wk, wv]), torch.bfloat16), dev(np.stack([bq, bk, bv])),
                           dev(wp, torch.bfloat16), dev(bp), H, dh, g, residual=xg, y=y)
    yh = host(y)
    for b in range(B):
        de, h = routes[route[b]]
        att = O.sliced_mhsa(x[b, :, :de], wq, bq, wk, bk, wv, bv, wp, bp, h, dh, store="bf16")
        want = O.bf16_round(x[b, :, :de] + att)
        assert relerr(yh[b, :, :de], want) < TOL_BF16
        assert np.all(np.isnan(yh[b, :, de:]))


# DS-ViT++ stores 8 heads of 48 channels (Q-K-V widths 192..384 in steps of 48 with 4..8 heads); 32 is the
# other head dimension the kernel takes
@pytest.mark.parametrize("dh,H,N,B", [(48, 8, 197, 9), (48, 8, 33, 4), (32, 12, 50, 5), (32, 4, 224, 2)])
def test_sliced_mhsa_head_dims(gpu_lib, dh, H, N, B):
    D = 416
    d = WL.nets.Draw(4100 + dh + N)
    bf = WL.nets.as_bf16_values
    x = bf(d.normal((B, N, D)))
    wq, wk, wv = (bf(d.normal((H * dh, D), std=0.06)) for _ in range(3))
    bq, bk, bv = (d.normal((H * dh,), std=0.1) for _ in range(3))
    wp, bp = bf(d.normal((D, H * dh), std=0.05)), d.normal((D,), std=0.1)
    routes = [(192, H // 2), (256, H // 2 + 1), (416, H), (320, H - 1), (192, H), (416, 1)]
    route = d.randint(B, len(routes))
    perm, inv, off = gpu_lib.ds_route_bucket(dev(route, torch.int32), len(routes))
    g = gpu_lib.make_groups(off, perm, [r[0] for r in routes], [r[1] * dh for r in routes])
    y = torch.full((B, N, D), float("nan"), dtype=torch.bfloat16, device=DEV)
    xg = dev(x, torch.bfloat16)
    gpu_lib.ds_sliced_mhsa(xg, dev(np.stack([wq, wk, wv]), torch.bfloat16), dev(np.stack([bq, bk, bv])),
                           dev(wp, torch.bfloat16), dev(bp), H, dh, g, residual=xg, y=y)
    yh = host(y)
    for b in range(B):
        de, h = routes[route[b]]
        att = O.sliced_mhsa(x[b, :, :de], wq, bq, wk, bk, wv, bv, wp, bp, h, dh, store="bf16")
        want = O.bf16_round(x[b, :, :de] + att)
        assert relerr(yh[b, :, :de], want) < TOL_BF16, (b, de, h)
        assert np.all(np.isnan(yh[b, :, de:]))


def test_sliced_mhsa_rejects_other_head_dims(gpu_lib):
    D, H, dh, B, N = 128, 2, 40, 2, 16
    x = torch.zeros((B, N, D), dtype=torch.bfloat16, device=DEV)
    w = torch.zeros((3, H * dh, D), dtype=torch.bfloat16, device=DEV)
    b = torch.zeros((3, H * dh), dtype=torch.float32, device=DEV)
    wp, bp = torch.zeros((D, H * dh), dtype=torch.bfloat16, device=DEV), torch.zeros((D,), dtype=torch.float32, device=DEV)
    off = torch.tensor([0, B], dtype=torch.int32, device=DEV)
    g = gpu_lib.make_groups(off, None, [D], [H * dh])
    with pytest.raises(gpu_lib.DsError):
        gpu_lib.ds_sliced_mhsa(x, w, b, wp, bp, H, dh, g, residual=x, y=torch.empty_like(x))


def test_sliced_mhsa_rejects_sequences_beyond_224(gpu_lib):
    D, H, dh, B, N = 128, 2, 64, 2, 225
    x = torch.zeros((B, N, D), dtype=torch.bfloat16, device=DEV)
    w = torch.zeros((3, H * dh, D), dtype=torch.bfloat16, device=DEV)
    b = torch.zeros((3, H * dh), dtype=torch.float32, device=DEV)
    wp, bp = torch.zeros((D, H * dh), dtype=torch.bfloat16, device=DEV), torch.zeros((D,), dtype=torch.float32, device=DEV)
    off = torch.tensor([0, B], dtype=torch.int32, device=DEV)
    g = gpu_lib.make_groups(off, None, [D], [H * dh])
    with pytest.raises(gpu_lib.DsError):
        gpu_lib.ds_sliced_mhsa(x, w, b, wp, bp, H, dh, g, residual=x, y=torch.empty_like(x))


def test_sliced_layernorm_wide_rows_and_empty_group(gpu_lib):
    # rows wider than 512 take the wavefront-per-row kernel; group 1 is left without samples
    B, N, D, T = 6, 5, 1024, 3
    d = WL.nets.Draw(3100)
    x = WL.nets.as_bf16_values(d.normal((B, N, D), std=1.5, mean=-0.25))
    gm, bt = 1.0 + d.normal((D,), std=0.1), d.normal((D,), std=0.1)
    route = np.array([0, 2, 2, 0, 2, 0], np.int32)
    ks = [520, 768, 1024]
    perm, inv, off = gpu_lib.ds_route_bucket(dev(route, torch.int32), T)
    g = gpu_lib.make_groups(off, perm, ks)
    y = torch.full((B, N, D), float("nan"), dtype=torch.bfloat16, device=DEV)
    gpu_lib.ds_sliced_layernorm(dev(x, torch.bfloat16), dev(gm), dev(bt), 1e-6, g, y=y)
    yh = host(y)
    for b in range(B):
        k = ks[route[b]]
        want = O.bf16_round(O.layernorm_sliced(x[b, :, :k], gm, bt, 1e-6))
        assert relerr(yh[b, :, :k], want) < TOL_BF16
        assert np.all(np.isnan(yh[b, :, k:]))


def test_sliced_conv_and_dwconv_with_an_empty_group_and_one_sample(gpu_lib):
    # one sample, three of four groups empty: grids sized for the widest group must not write anything else
    B, T, H, CI, CO = 1, 4, 10, 64, 96
    d = WL.nets.Draw(5200)
    x = WL.nets.as_bf16_values(d.normal((B, CI, H, H)))
    w = WL.nets.as_bf16_values(d.normal((CO, CI, 3, 3), std=(2.0 / (CI * 9)) ** 0.5))
    wd = WL.nets.as_bf16_values(d.normal((CI, 1, 3, 3), std=0.3))
    bn, bnd = WL.bn_tables(d, T, CO), WL.bn_tables(d, T, CI)
    route = np.array([2], np.int32)
    c_in, c_out = [16, 32, 48, 64], [24, 48, 72, 96]
    perm, inv, off = gpu_lib.ds_route_bucket(dev(route, torch.int32), T)
    scale, shift = gpu_lib.ds_bn_fold(dev(bn["gamma"]), dev(bn["beta"]), dev(bn["mean"]), dev(bn["var"]), 1e-5)
    g = gpu_lib.make_groups(off, perm, c_in, c_out)
    y = torch.full((B, H, H, CO), float("nan"), dtype=torch.bfloat16, device=DEV)
    gpu_lib.ds_sliced_conv(dev(x.transpose(0, 2, 3, 1), torch.bfloat16), dev(w.transpose(0, 2, 3, 1), torch.bfloat16), scale,
                           shift, g, 1, 1, act=gpu_lib.DS_ACT_RELU, y=y)
    yh = host(y).transpose(0, 3, 1, 2)
    want = O.bf16_round(O.relu(O.re_sbn(O.sliced_conv2d(x[0, :48], w, 72, 1, 1), bn, 2, 1e-5)))
    assert relerr(yh[0, :72], want) < TOL_BF16 and np.all(np.isnan(yh[0, 72:]))
    sd, hd = gpu_lib.ds_bn_fold(dev(bnd["gamma"]), dev(bnd["beta"]), dev(bnd["mean"]), dev(bnd["var"]), 1e-5)
    gd = gpu_lib.make_groups(off, perm, c_in)
    yd = torch.full((B, H, H, CI), float("nan"), dtype=torch.bfloat16, device=DEV)
    gpu_lib.ds_sliced_dwconv(dev(x.transpose(0, 2, 3, 1), torch.bfloat16), dev(wd[:, 0].transpose(1, 2, 0), torch.bfloat16), sd, hd,
                             gd, 1, act=gpu_lib.DS_ACT_RELU, y=yd)
    ydh = host(yd).transpose(0, 3, 1, 2)
    wantd = O.bf16_round(O.relu(O.re_sbn(O.sliced_dwconv2d(x[0, :48], wd, 1, 1), bnd, 2, 1e-5)))
    assert relerr(ydh[0, :48], wantd) < TOL_BF16 and np.all(np.isnan(ydh[0, 48:]))


# ------------------------------------------------------------------ Re-SBN re-calibration
@pytest.mark.parametrize("HW,C", [(28 * 28, 512), (56 * 56, 64), (7 * 7, 1024), (112 * 112, 24)])
def test_bn_stats_streaming_recalibration(gpu_lib, HW, C):
    # three batches of different sizes streamed through the accumulators; the result must be the population
    # statistics per route over everything streamed (the oracle sees all samples at once)
    T = 4
    d = WL.nets.Draw(5000 + C)
    widths = [max(8, C * q // 4 // 8 * 8) for q in (1, 2, 3, 4)]
    acc_s = torch.zeros((T, C), dtype=torch.float64, device=DEV)
    acc_q = torch.zeros((T, C), dtype=torch.float64, device=DEV)
    cnt = torch.zeros((T,), dtype=torch.int64, device=DEV)
    samples, routes = [], []
    for B in (5, 9, 2):
        route = d.randint(B, T - 1)                      # the last route never gets a sample
        x = WL.nets.as_bf16_values(d.normal((B, HW, C), std=1.5, mean=0.3))
        perm, inv, off = gpu_lib.ds_route_bucket(dev(route, torch.int32), T)
        g = gpu_lib.make_groups(off, perm, widths)
        gpu_lib.ds_bn_stats_accumulate(dev(x, torch.bfloat16), g, acc_s, acc_q, cnt)
        for b in range(B):
            c = widths[route[b]]
            samples.append(x[b, :, :c].T.reshape(c, HW, 1))
            routes.append(int(route[b]))
    mean, var = gpu_lib.ds_bn_stats_finish(acc_s, acc_q, cnt, widths)
    want_m, want_v, want_n = O.re_sbn_recalibrate(samples, routes, T, C)
    assert cnt.cpu().numpy().tolist() == want_n.tolist()
    m, v = host(mean), host(var)
    assert np.max(np.abs(m - want_m)) < 1e-5 * max(1.0, np.max(np.abs(want_m)))
    assert np.max(np.abs(v - want_v)) < 1e-5 * np.max(np.abs(want_v))
    assert np.all(m[T - 1] == 0) and np.all(v[T - 1] == 1)
    # the new tables go straight into the fold used by every sliced layer
    scale, shift = gpu_lib.ds_bn_fold(torch.ones(C, device=DEV), torch.zeros(C, device=DEV), mean, var, 1e-5)
    assert torch.isfinite(scale).all() and torch.isfinite(shift).all()


# ------------------------------------------------------------------ pool + classifier, max-pool
@pytest.mark.parametrize("B,HW,C,n_out,T", [(37, 49, 256, 1000, 4), (9, 196, 1024, 100, 14), (3, 1, 64, 10, 2)])
def test_pool_head_sliced_input_width(gpu_lib, B, HW, C, n_out, T):
    d = WL.nets.Draw(900 + C)
    x = WL.nets.as_bf16_values(d.normal((B, HW, C)))
    w = WL.nets.as_bf16_values(d.normal((n_out, C), std=C ** -0.5))
    bias = d.normal((n_out,), std=0.1)
    route = d.randint(B, T)
    widths = [8 * max(1, (C // 8) * (t + 1) // T) for t in range(T)]
    perm, inv, off = gpu_lib.ds_route_bucket(dev(route, torch.int32), T)
    g = gpu_lib.make_groups(off, perm, widths, widths)
    logits = gpu_lib.ds_pool_head(dev(x, torch.bfloat16), dev(w, torch.bfloat16), dev(bias), g)
    lg = host(logits)
    for b in range(B):
        c = widths[route[b]]
        pooled = O.gate_encoder(x[b, :, :c].T.reshape(c, HW, 1))
        want = O.sliced_linear(pooled, w[:, :c], bias, n_out)
        assert relerr(lg[b], want) < 1e-4, b          # fp32 accumulation of bf16 values over up to 196 x 1024 terms


@pytest.mark.parametrize("B,H,W,C", [(5, 112, 112, 64), (3, 7, 9, 24), (2, 1, 1, 8)])
def test_maxpool_3x3_stride2(gpu_lib, B, H, W, C):
    d = WL.nets.Draw(950 + H)
    x = WL.nets.as_bf16_values(d.normal((B, H, W, C)))
    y = gpu_lib.ds_maxpool(dev(x, torch.bfloat16))
    yh = host(y)
    for b in range(B):
        want = O.maxpool3x3s2(x[b].transpose(2, 0, 1))          # oracle layout [C, H, W]
        assert np.array_equal(yh[b].transpose(2, 0, 1), want), b   # a maximum of bf16 values is one of them: bit-exact
