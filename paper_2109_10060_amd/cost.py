"""Algorithmic work of one ds_forward pass, per kernel class, for a given route assignment.

flops: 2 x multiply-adds the method itself must do on the valid slices (not the dense work
it avoids).  bytes: each kernel reads its valid input once and writes its valid output once
(bf16), reads a residual once where it has one, and reads the union of the weight slices
once per launch.  These are the numerators of the roofline fractions bench.py reports.

The records follow the launches: which layers run as one kernel depends on sizes, and the rules of the library's dispatch
are repeated here (_tiles, _few_samples, _separable, _front, _tail).  Work that happens inside a launch of another class (the
LayerNorms of a transformer block) is kept under "inside", without bytes or launches of its own.
"""
from __future__ import annotations

from collections import defaultdict

import numpy as np


class Cost(defaultdict):
    """Per kernel class totals (self[kind]) and, in launch order, one record per launch (self.launches)."""

    def __init__(self):
        super().__init__(lambda: {"flops": 0.0, "bytes": 0.0, "launches": 0})
        self.launches = []

    def add(self, kind, flops, nbytes, name="", shape="", merge=False, launch=True, later=False):
        """merge: the work rides along in the previous launch of this kind (a chained layer): no new launch.  later: it is counted there
        because of its class, but the contraction launched next does it (as_launched).
        launch=False: totals only, the work happens inside a launch of another kind."""
        e = self[kind]
        e["flops"] += float(flops)
        e["bytes"] += float(nbytes)
        if not launch:
            return
        if merge:
            last = next(r for r in reversed(self.launches) if r["kind"] == kind)
            last["flops"] += float(flops)
            last["bytes"] += float(nbytes)
            if later:
                last.setdefault("later", []).append({"name": name, "flops": float(flops), "bytes": float(nbytes)})
                name += " (in the next launch)"
            last["name"] += " + " + name
            return
        e["launches"] += 1
        self.launches.append({"kind": kind, "name": name, "shape": shape, "flops": float(flops), "bytes": float(nbytes)})


def as_launched(records):
    """The records with every piece of work in the launch that does it, whatever its class."""
    rows = [dict(r) for r in records]
    for i, r in enumerate(rows):
        for work in r.pop("later", ()):
            into = next(q for q in rows[i + 1:] if q["kind"] in ("gemm", "gemm_taps"))
            for key in ("flops", "bytes"):
                r[key] -= work[key]
                into[key] += work[key]
            r["name"] = r["name"].replace(f" + {work['name']} (in the next launch)", "")
            into["name"] += " + " + work["name"]
    return rows


def _osz(n, k, s, p):
    return (n + 2 * p - k) // s + 1


def _tiles(B, rows, groups, bm=128):
    """Row tiles of a launch, at most."""
    g = min(B, groups)
    return (B * rows - g) // bm + g


def _few_samples(B, rows, groups, n):
    """A 1x1 layer at stride 1 that the kernel for few samples takes (it has no layer chained behind it)."""
    return _tiles(B, rows, groups, 32) * -(-n // 32) <= 1000


def _paired(ta, tb, nk):
    """Two 1x1 layers of ta and tb 32 x 32 tiles and nk 64-deep slabs that run as one launch: the same kernel variant alone."""
    choice = lambda t: 0 if t <= 340 and nk > 2 else 1 if 340 < t <= 500 and nk >= 5 else 2 if t <= 700 else 3 if nk >= 24 else 4 if nk > 4 else 5  # noqa: E731
    big = choice(max(ta, tb))
    return ta + tb <= 1000 and big != 3 and (nk <= 1 or choice(ta) == choice(tb))


def _paired_wide(ta, na, tb, nb, k, few, strided):
    """A projection of ta and a first layer of tb row tiles, na and nb columns and k channels as one launch of the 128-row kernel."""
    def tile(t, n, conv):
        if not conv and (128 < k < 320 and 64 < n <= 128 and t >= 3000 or k >= 768 and n > 64 and t * -(-n // 128) >= 2048):
            return "wide"
        wgs, slabs = t * -(-n // 64), -(-k // 64)
        if k < 320:
            return "32"
        if slabs >= 8 and wgs <= (512 if slabs >= 32 else 256):
            return "four shares"
        return "two shares" if wgs <= 512 else "128" if k >= 512 and wgs <= 1536 else "64"
    one = tile(ta, na, strided)
    return k > 128 and few > 1000 and one == tile(tb, nb, False) and one not in ("wide", "four shares")


def _separable(r, ci, co, s, k, kfull, tiled):
    """An unsliced depthwise + pointwise block that runs as one kernel: output size, channels, stride, filter size."""
    if ci % 8 or co % 8:
        return False
    if tiled and r > 8 and k in (3, 5) and (kfull - k) % 2 == 0:
        limits = [(32, 64), (64, 128)] + ([(128, 128)] if s == 1 else []) + \
            ([(128, 256) if s == 2 else (256, 256)] if k == 3 else [])
        if any(ci <= a and co <= b for a, b in limits):
            return True
    return k == 3 and kfull == 3 and ci <= 128 and co <= 128 and r % (4 if s == 1 else 2) == 0


def _few_separable(r, ci, co, B):
    """A block in front of the gate (3x3 filters) of so few samples that the kernel of the sliced blocks runs it."""
    return _sliced_separable(r, ci) and -(-B // 8) * -(-r // (32 // r)) * -(-co // 256) <= 32


def _front(arch):
    """The stem and the first two separable blocks run as one kernel."""
    b = arch["blocks"]
    k = int(arch["ksize"][0, 0]) if "ksize" in arch else 3
    return (arch["image"] % 4 == 0 and arch["gate_after"] >= 2 and (b[0][2], b[1][2]) == (1, 2) and ("ksize" not in arch or arch["ksize"][0, 1] == k)
            and b[0][0] == arch["stem_out"] and b[1][0] == b[0][1] and b[1][1] % 8 == 0
            and (k, b[0][0], b[0][1], b[1][1] <= (128 if k == 3 else 64)) in ((3, 32, 64, True), (5, 16, 32, True)))


def _sliced_separable(r, ci):
    """A block behind the gate (3x3 filters) that runs as one kernel: output size, stored channels."""
    return r <= 32 and -(-ci // 64) * 64 <= 2048


def _gemm(cost, kind, rows_in, rows_out, kk, k_in, k_out, residual=False, out_bytes=2, chained=False, name=""):
    """k_in, k_out: per-sample arrays of valid widths.  chained: the layer runs inside the launch that
    produced its input rows, so it adds flops, its output and its weights, but no input read and no launch."""
    k_in, k_out = np.asarray(k_in, np.float64), np.asarray(k_out, np.float64)
    flops = 2.0 * rows_out * kk * np.sum(k_in * k_out)
    nbytes = (0.0 if chained else 2.0 * rows_in * np.sum(k_in)) + out_bytes * rows_out * np.sum(k_out) * (2 if residual else 1)
    nbytes += 2.0 * kk * float(np.max(k_in)) * float(np.max(k_out))
    live = k_in * k_out > 0
    shape = (f"rows {int(rows_out) * int(live.sum())} k {int(k_in[live].min()) if live.any() else 0}..{int(k_in.max())}"
             f"{'x' + str(int(kk)) if kk > 1 else ''} n {int(k_out[live].min()) if live.any() else 0}..{int(k_out.max())}")
    cost.add(kind, flops, nbytes, name=name, shape=shape, merge=chained)


def mbnet_cost(arch, routes) -> Cost:
    routes = np.asarray(routes).reshape(-1)
    B = routes.shape[0]
    c = Cost()
    r = _osz(arch["image"], 3, 2, 1)
    so = arch["stem_out"]
    if _front(arch):
        # counted as one launch of the depthwise class that reads the images and writes the second block's output
        k2 = float(arch["ksize"][0, 0]) ** 2 if "ksize" in arch else 9.0
        (c0, c1, _), (_, f, _) = arch["blocks"][:2]
        r2 = _osz(r, 3, 2, 1)
        c.add("dwconv", 2.0 * B * (r * r * (27.0 * so + k2 * c0 + c0 * c1) + r2 * r2 * (k2 * c1 + c1 * f)),
              2.0 * B * (3 * arch["image"] ** 2 + r2 * r2 * f) + 2.0 * (27 * so + c0 * c1 + c1 * f), name="stem + ds0 + ds1 fused",
              shape=f"{arch['image']}x{arch['image']}x3 -> {r2}x{r2}x{f}")
    else:
        c.add("stem", 2.0 * B * r * r * 27 * so, B * (3 * arch["image"] ** 2 * 2 + r * r * so * 2), name="stem 3x3/2")
    for i, (_ci, _co, s) in enumerate(arch["blocks"]):
        rin = r
        r = _osz(r, 3, s, 1)
        if i < 2 and _front(arch):
            continue
        ci, co = arch["cin"][routes, i].astype(np.float64), arch["cout"][routes, i].astype(np.float64)
        kk = arch["ksize"][routes, i].astype(np.float64) ** 2 if "ksize" in arch else 9.0
        cif, cof = int(_ci), int(_co)
        k = int(arch["ksize"][0, i]) if "ksize" in arch else 3
        if (_separable(r, cif, cof, s, k, arch["kfull"][i] if "ksize" in arch else 3, True)
                or "ksize" not in arch and _few_separable(r, cif, cof, B) if i < arch["gate_after"]
                else "ksize" not in arch and _sliced_separable(r, cif)):
            # a block the library runs as one kernel (depthwise map kept in LDS): counted as one launch
            # of the depthwise class that reads the block's input and writes the pointwise output
            span = lambda v: f"{int(v.min())}..{int(v.max())}" if v.min() < v.max() else f"{int(v.max())}"  # noqa: E731
            c.add("dwconv", 2.0 * r * r * (kk * ci).sum() + 2.0 * r * r * np.sum(ci * co),
                  2.0 * rin * rin * ci.sum() + 2.0 * r * r * co.sum() + 2.0 * ci.max() * co.max(), name=f"ds{i} dw+pw fused",
                  shape=f"{rin}x{rin}x{span(ci)} -> {r}x{r}x{span(co)}")
        else:
            c.add("dwconv", 2.0 * r * r * (kk * ci).sum(), 2.0 * (rin * rin + r * r) * ci.sum(), name=f"ds{i} dw",
                  shape=f"{rin}x{rin} s{s} c {int(ci.min())}..{int(ci.max())}")
            _gemm(c, "gemm", r * r, r * r, 1, ci, co, name=f"ds{i} pw")
        if i == arch["gate_after"] - 1:
            c.add("gate", 2.0 * B * (r * r * co[0]), 2.0 * B * r * r * co[0], name="gate pool + MLP")
    cl = arch["cout"][routes, -1].astype(np.float64)
    c.add("head", 2.0 * arch["num_classes"] * cl.sum(), 2.0 * r * r * cl.sum() + 2.0 * arch["num_classes"] * cl.max(),
          name="pool + classifier")
    return c


def resnet_cost(arch, routes) -> Cost:
    routes = np.asarray(routes).reshape(4, -1)
    B = routes.shape[1]
    c = Cost()
    r1 = _osz(arch["image"], 7, 2, 3)
    so = arch["stem_out"]
    r = _osz(r1, 3, 2, 1)
    pooled = so == 64 and arch["image"] % 4 == 0        # stem and max-pool in one kernel
    c.add("stem", 2.0 * B * r1 * r1 * 147 * so, B * (3 * arch["image"] ** 2 * 2 + (r * r if pooled else r1 * r1) * so * 2),
          name="stem 7x7/2" + (" + max-pool" if pooled else ""))
    if not pooled:
        c.add("maxpool", 0.0, 2.0 * B * so * (r1 * r1 + r * r), name="max-pool")
    groups = arch["T"] if arch.get("single_gate") else arch["T"] ** 2
    cprev = np.full(B, so, np.float64)
    for s, nb in enumerate(arch["blocks"]):
        mid = arch["mid"][s][routes[s]].astype(np.float64)
        out = arch["out"][s][routes[s]].astype(np.float64)
        if s == 0 or not arch.get("single_gate"):
            c.add("gate", 2.0 * r * r * cprev.sum(), 2.0 * r * r * cprev.sum(), name=f"s{s} gate pool + MLP")
        # stages with slices of at most 128 channels run a block's last convolution and the next block's first one
        # as one launch (the wide map is written once and not read back)
        mids, outs = arch["mid"][s], arch["out"][s]
        rs = r if s == 0 else _osz(r, 3, 2, 1)
        chain = bool(mids.max() <= 128 and outs.max() >= 128 and not (mids % 8).any() and not (outs % 8).any()
                     and not _few_samples(B, rs * rs, groups, int(outs.max()))
                     and _tiles(B, rs * rs, groups) >= (150 if mids.max() <= 64 else 400))
        # 3x3 layer, last convolution and the next block's first one of a stride-1 block as one launch, in the first stage's first
        # block with the projection too
        fits = lambda nb_: mids.max() <= 32 * nb_ and outs.max() <= 128 * nb_ and _tiles(B, rs * rs, groups) >= (40 if nb_ == 2 else 300)  # noqa: E731
        rest = bool(rs <= 59 and not (mids % 8).any() and not (outs % 8).any() and fits(2 if mids.max() <= 64 else 4))
        # few samples: the first layer of a stage is one launch with the projection
        paired = _paired(_tiles(B, rs * rs, groups, 32) * -(-int(outs.max()) // 32), _tiles(B, r * r, groups, 32) * -(-int(mids.max()) // 32),
                         -(-int(arch["out"][s - 1].max() if s else so) // 64))
        inside = bool(rest and s == 0 and so <= 64 and so % 8 == 0 and mids.max() <= 64 and not paired)
        # (beyond them too, where both take the same tile of the 128-row kernel)
        paired = paired or not inside and _paired_wide(_tiles(B, rs * rs, groups), int(outs.max()), _tiles(B, r * r, groups), int(mids.max()),
                                                       int(arch["out"][s - 1].max() if s else so),
                                                       min(_tiles(B, rs * rs, groups, 32) * -(-int(outs.max()) // 32),
                                                           _tiles(B, r * r, groups, 32) * -(-int(mids.max()) // 32)), s > 0)
        for b in range(nb):
            # dynamic depth: samples whose route has run its blocks of this stage contribute nothing
            on = (arch["nblk"][s][routes[s]] > b).astype(np.float64) if arch.get("nblk") is not None else np.ones(B)
            if not on.any():
                break
            stride = 2 if (b == 0 and s > 0) else 1
            ro = _osz(r, 3, stride, 1)
            cin = (cprev if b == 0 else out) * on
            m, o = mid * on, out * on
            one = rest and stride == 1
            if b == 0 and not inside:
                _gemm(c, "gemm", ro * ro, ro * ro, 1, cin, o, name=f"s{s}.b{b}.proj")      # 1x1 projection reads only the strided pixels
            behind = rest and b > (s > 0)               # the block before it was one launch, this block's first layer at its end
            _gemm(c, "gemm_taps" if behind else "gemm", r * r, r * r, 1, cin, m, chained=(behind or chain) and b > 0 or b == 0 and paired,
                  name=f"s{s}.b{b}.c1")
            if b == 0 and inside:
                c.add("gemm", 2.0 * ro * ro * np.sum(cin * o), 2.0 * r * r * np.sum(cin) + 2.0 * float(cin.max() * o.max()),
                      name=f"s{s}.b{b}.proj", merge=True, later=True)
            _gemm(c, "gemm_taps", r * r, ro * ro, 9, m, m, name=f"s{s}.b{b}.c2 3x3" + ("/2" if stride == 2 else ""))
            _gemm(c, "gemm_taps" if one else "gemm", ro * ro, ro * ro, 1, m, o, residual=not (b == 0 and inside), chained=one,
                  name=f"s{s}.b{b}.c3" + ("" if b == 0 and inside else "+res"))
            r = ro
        cprev = out
    c.add("head", 2.0 * arch["num_classes"] * cprev.sum(),
          2.0 * r * r * cprev.sum() + 2.0 * arch["num_classes"] * cprev.max(), name="pool + classifier")
    return c


def _tail(arch, live, B):
    """(Q/K/V with its LayerNorm inside, launches behind the attention: "one", "three" or "four" and a LayerNorm)."""
    de, hd, hid = live[:, 0], live[:, 1] * arch["head_dim"], live[:, 2]
    if de.max() > 416:
        return False, "four"
    if arch["mlp"] <= 1664 and _tiles(B, arch["tokens"], arch["T"], 32) <= 56:
        return True, "three"
    return True, "one" if hd.max() <= 416 and not (hd % 16).any() else "four"


def vit_cost(arch, routes) -> Cost:
    routes = np.asarray(routes).reshape(-1)
    tab = arch["routes"][routes].astype(np.float64)
    de, h, hid = tab[:, 0], tab[:, 1], tab[:, 2]
    hd = h * arch["head_dim"]
    N, B = arch["tokens"], routes.shape[0]
    c = Cost()
    C = arch.get("stem_dim", 0)
    if C:
        r = _osz(arch["image"], 7, 2, 3)
        full = np.full(B, C, np.float64)
        c.add("stem", 2.0 * B * r * r * 147 * C, B * (3 * arch["image"] ** 2 * 2 + r * r * C * 2), name="stem 7x7/2")
        for _ in range(2):
            if _separable(r, C, C, 1, 3, 3, False):
                # the block runs as one kernel (depthwise map kept in LDS): one launch of the depthwise class
                c.add("dwconv", 2.0 * B * r * r * 9 * C + 2.0 * B * r * r * C * C, 2.0 * 2 * B * r * r * C + 2.0 * C * C,
                      name="stem dw+pw fused")
            else:
                c.add("dwconv", 2.0 * B * r * r * 9 * C, 2.0 * 2 * B * r * r * C, name="stem dw")
                _gemm(c, "gemm", r * r, r * r, 1, full, full, name="stem pw")
        c.add("gate", 2.0 * B * r * r * C, 2.0 * B * r * r * C, name="gate pool + MLP")
        # the patch projection reads every pixel of the stem's map once
        taps = arch["patch"] ** 2
        _gemm(c, "gemm_taps", (N - 1) * taps, N - 1, taps, full, de, name="patch embed conv")
    else:
        kp = 3 * arch["patch"] ** 2
        c.add("index", 0.0, 2.0 * 2 * B * (N - 1) * kp, name="patch extraction")
        _gemm(c, "gemm", N - 1, N - 1, 1, np.full(B, kp), de, name="patch embed")
    full = tab[:, :3].copy()
    ahead = False                                       # this block's Q/K/V rode along with the block before it
    for l in range(arch["depth"]):
        # dynamic depth: a route that runs fewer than l + 1 blocks contributes nothing to this layer
        on = (tab[:, 3] > l).astype(np.float64) if tab.shape[1] > 3 else np.ones(B)
        if not on.any():
            break
        de, h, hid = full[:, 0] * on, full[:, 1] * on, full[:, 2] * on
        hd = h * arch["head_dim"]
        live = arch["routes"] if tab.shape[1] < 4 else arch["routes"][arch["routes"][:, 3] > l]
        fused, behind = _tail(arch, live, B)
        ln = (8.0 * N * de.sum(), 4.0 * N * de.sum())
        if fused:
            c.add("inside", ln[0], 0.0, name=f"l{l}.ln1", launch=False)
        else:
            c.add("layernorm", *ln, name=f"l{l}.ln1")
        _gemm(c, "gemm", N, N, 1, de, 3 * hd, name=("" if not fused else f"l{l}.ln1+") + f"l{l}.qkv", chained=ahead)
        ahead = behind == "one" and _tiles(B, arch["tokens"], arch["T"], 32) >= (140 if live[:, 0].max() > 384 else 60)
        c.add("attention", 4.0 * N * N * hd.sum(), 2.0 * 4 * N * hd.sum(), name=f"l{l}.attention")
        if behind == "one":
            # rows in, the residual stream read and written; both hidden maps stay in the compute unit
            w = hd.max() * de.max() + 2.0 * de.max() * hid.max()
            c.add("inside", ln[0], 0.0, name=f"l{l}.ln2", launch=False)
            c.add("gemm", 2.0 * N * (np.sum(hd * de) + 2.0 * np.sum(de * hid)), 2.0 * N * (hd.sum() + 2.0 * de.sum()) + 2.0 * w,
                  name=f"l{l}.proj+res + ln2 + fc1+gelu + fc2+res",
                  shape=f"rows {int(N) * int((de > 0).sum())} k {int(hd[de > 0].min())}..{int(hd.max())} n "
                        f"{int(de[de > 0].min())}..{int(de.max())} hidden {int(hid[de > 0].min())}..{int(hid.max())}")
            continue
        _gemm(c, "gemm", N, N, 1, hd, de, residual=True, name=f"l{l}.proj+res")
        if behind == "three":
            c.add("inside", ln[0], 0.0, name=f"l{l}.ln2", launch=False)
        else:
            c.add("layernorm", *ln, name=f"l{l}.ln2")
        _gemm(c, "gemm", N, N, 1, de, hid, name=("" if behind != "three" else f"l{l}.ln2+") + f"l{l}.fc1+gelu")
        _gemm(c, "gemm", N, N, 1, hid, de, residual=True, name=f"l{l}.fc2+res")
    de = full[:, 0]
    c.add("layernorm", 8.0 * de.sum(), 4.0 * de.sum(), name="final ln (class token)")
    c.add("head", 2.0 * arch["num_classes"] * de.sum(), 2.0 * de.sum() + 2.0 * arch["num_classes"] * de.max(), name="classifier")
    return c
