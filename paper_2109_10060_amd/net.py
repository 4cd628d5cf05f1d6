"""Network descriptors for ds_forward.

Marshalling only: parameters arrive as host arrays in the logical layouts of the
network description (conv filters [C_O, C_I, K, K], depthwise [C, 1, 3, 3], linear
[out, in]); they are moved to the device in the storage layout the kernels read
in place (channels-last filters [C_O, K, K, C_I], depthwise [3, 3, C], stem
[K*K*3, C_O], stacked Q/K/V), split batch-norm statistics are folded to per-route
scale/shift tables by the library's own ds_bn_fold kernel, and the integer
description plus the device pointers are laid out in the order include/dsnet.h
documents for each architecture.  Filters and linear weights that kernels read in operand
order are held twice, row-major and tiled, and a launch reads the copy its kernel is written
for: other weights are another Net.
"""
from __future__ import annotations

import ctypes

import numpy as np
import torch


def _dev(a, dtype, device):
    return torch.from_numpy(np.ascontiguousarray(a)).to(device).to(dtype).contiguous()


class Net:
    def __init__(self, arch_id: int, ints, tensors, num_classes: int, n_gates: int, T: int):
        from . import ds_net
        self.arch_id = arch_id
        self.tensors = list(tensors)          # keeps device memory alive
        self.num_classes = num_classes
        self.n_gates = n_gates
        self.T = T
        self._ints = (ctypes.c_int32 * len(ints))(*[int(v) for v in ints])
        self._ptrs = (ctypes.c_void_p * len(self.tensors))(*[t.data_ptr() for t in self.tensors])
        self.c_struct = ds_net(arch_id, len(ints), ctypes.cast(self._ints, ctypes.POINTER(ctypes.c_int32)),
                               len(self.tensors), ctypes.cast(self._ptrs, ctypes.POINTER(ctypes.c_void_p)))
        self.device = self.tensors[0].device

    def workspace_bytes(self, B: int, parts: int = 1) -> int:
        from . import load
        if parts == 1:
            return int(load().ds_forward_workspace(ctypes.byref(self.c_struct), B))
        return int(load().ds_forward_parts_workspace(ctypes.byref(self.c_struct), B, parts))

    def workspace(self, B: int, parts: int = 1) -> torch.Tensor:
        return torch.empty(max(self.workspace_bytes(B, parts), 256), dtype=torch.uint8, device=self.device)


def _fold(bn, eps, device):
    from . import ds_bn_fold
    f32 = torch.float32
    return ds_bn_fold(_dev(bn["gamma"], f32, device), _dev(bn["beta"], f32, device), _dev(bn["mean"], f32, device),
                      _dev(bn["var"], f32, device), eps)


def _ohwi(w, device):
    return _dev(np.transpose(w, (0, 2, 3, 1)), torch.bfloat16, device)


def _stem(w, device):
    co = w.shape[0]
    return _dev(np.transpose(w, (2, 3, 1, 0)).reshape(-1, co), torch.bfloat16, device)


def _operand_tiles(w):
    """[N, K] bf16 -> [ceil(N/32)][ceil(K/16) | 1] tiles of 32 x 16 in the order of a matrix instruction's lanes: half of the
    16 channels, row, 8 channels.  The odd number of 1 KiB tiles per row of tiles keeps the rows, which the wavefronts of a
    workgroup stream side by side, off the same L2 channels."""
    n, k = w.shape
    nb, kb = (n + 31) // 32, (k + 15) // 16 | 1
    t = torch.zeros((nb * 32, kb * 16), dtype=w.dtype, device=w.device)
    t[:n, :k] = w
    return t.view(nb, 32, kb, 2, 8).permute(0, 2, 3, 1, 4).contiguous()


def _pointwise_tiles(w):
    """[N, K] bf16 -> [ceil(N/32)][ceil(K/32) | 1] pairs of 16 x 32 tiles in the order of a matrix instruction's lanes: quarter
    of the 32 channels, row, 8 channels.  The first tile of a pair has filters 0..3 of every eight, the second 4..7, so that
    a lane ends with eight neighbouring outputs of a pixel."""
    n, k = w.shape
    nb, kb = (n + 31) // 32, (k + 31) // 32 | 1
    t = torch.zeros((nb * 32, kb * 32), dtype=w.dtype, device=w.device)
    t[:n, :k] = w
    return t.view(nb, 4, 2, 4, kb, 4, 8).permute(0, 4, 2, 5, 1, 3, 6).contiguous()


def _conv3_tiles(w):
    """[N, 3, 3, K] bf16 -> [ceil(N/32)][18 ceil(K/32) + 1] tiles of 32 x 16 in the order of a matrix instruction's lanes: of every
    32 channels the nine taps, of a tap two halves of 16 channels.  The tile at the end of a block of filters keeps the blocks,
    which the wavefronts of a workgroup stream side by side, off the same L2 channels."""
    n, _, _, k = w.shape
    nb, kc = (n + 31) // 32, (k + 31) // 32
    t = torch.zeros((nb * 32, 9, kc * 32), dtype=w.dtype, device=w.device)
    t[:n, :, :k] = w.reshape(n, 9, k)
    out = torch.zeros((nb, 18 * kc + 1, 512), dtype=w.dtype, device=w.device)
    out[:, :-1] = t.view(nb, 32, 9, kc, 2, 2, 8).permute(0, 3, 2, 4, 5, 1, 6).reshape(nb, 18 * kc, 512)
    return out


def build_mbnet(arch: dict, p: dict, device="cuda:0") -> Net:
    from . import DS_ARCH_MBNET
    bf, f32 = torch.bfloat16, torch.float32
    eps = arch["bn_eps"]
    nb, T = len(arch["blocks"]), arch["T"]
    ints = [arch["image"], arch["stem_out"], nb, arch["gate_after"], arch["gate_hidden"], T, arch["num_classes"]]
    for ci, co, s in arch["blocks"]:
        ints += [ci, co, s]
    ints += arch["cin"].reshape(-1).tolist() + arch["cout"].reshape(-1).tolist()
    if "ksize" in arch:
        ints += [int(k) for k in arch["kfull"]] + arch["ksize"].reshape(-1).tolist()
    else:
        ints.append(1)
    t = [_stem(p["stem.w"], device), *_fold(p["stem.bn"], eps, device)]
    for i in range(nb):
        t.append(_dev(np.transpose(p[f"ds{i}.dw.w"][:, 0], (1, 2, 0)), bf, device))
        t += list(_fold(p[f"ds{i}.dw.bn"], eps, device))
        t.append(_dev(p[f"ds{i}.pw.w"][:, :, 0, 0], bf, device))
        t += list(_fold(p[f"ds{i}.pw.bn"], eps, device))
    t += [_dev(p[k], f32, device) for k in ("gate.w1", "gate.b1", "gate.w2", "gate.b2")]
    t += [_dev(p["fc.w"], bf, device), _dev(p["fc.b"], f32, device)]
    # the pointwise filters once more in operand order; behind the gate only where the depthwise filters are not sliced (else the
    # entries are not read)
    t += [_pointwise_tiles(t[3 + 6 * i + 3]) if i < arch["gate_after"] or "ksize" not in arch else t[3 + 6 * i + 3] for i in range(nb)]
    return Net(DS_ARCH_MBNET, ints, t, arch["num_classes"], 1, T)


def build_resnet(arch: dict, p: dict, device="cuda:0") -> Net:
    from . import DS_ARCH_RESNET
    bf, f32 = torch.bfloat16, torch.float32
    eps = arch["bn_eps"]
    T = arch["T"]
    ints = [arch["image"], arch["stem_out"], T, arch["num_classes"], *arch["widths"], *arch["blocks"],
            *arch["gate_hidden"], *arch["mid"].reshape(-1).tolist(), *arch["out"].reshape(-1).tolist()]
    if arch.get("nblk") is not None:
        ints += [int(v) for v in arch["nblk"].reshape(-1)]
        if arch.get("single_gate"):
            ints.append(1)
    t = [_stem(p["stem.w"], device), *_fold(p["stem.bn"], eps, device)]
    for s, nb in enumerate(arch["blocks"]):
        t += [_dev(p[f"s{s}.gate.{k}"], f32, device) for k in ("w1", "b1", "w2", "b2")]
        for b in range(nb):
            pre = f"s{s}.b{b}"
            for c in ("c1", "c2", "c3") + (("proj",) if b == 0 else ()):
                t.append(_ohwi(p[f"{pre}.{c}.w"], device))
                t += list(_fold(p[f"{pre}.{c}.bn"], eps, device))
    t += [_dev(p["fc.w"], bf, device), _dev(p["fc.b"], f32, device)]
    # the 3x3 filters once more in operand order
    at = 3
    for nb in arch["blocks"]:
        at += 4
        for b in range(nb):
            t.append(_conv3_tiles(t[at + 3]))
            at += 12 if b == 0 else 9
    return Net(DS_ARCH_RESNET, ints, t, arch["num_classes"], 4, T)


def build_vit(arch: dict, p: dict, device="cuda:0") -> Net:
    from . import DS_ARCH_VIT, DS_ARCH_VIT_STEM
    bf, f32 = torch.bfloat16, torch.float32
    D = arch["embed"]
    C = arch.get("stem_dim", 0)
    ints = [arch["image"], arch["patch"], D, arch["heads"], arch["head_dim"], arch["mlp"], arch["depth"],
            arch["tokens"], arch["T"], arch["num_classes"]]
    t = []
    if C:
        eps = arch["bn_eps"]
        ints += [arch["routes"].shape[1], C, arch["gate_hidden"]]
        t += [_stem(p["stem.c0.w"], device), *_fold(p["stem.c0.bn"], eps, device)]
        for i in (1, 2):
            t.append(_dev(np.transpose(p[f"stem.ds{i}.dw.w"][:, 0], (1, 2, 0)), bf, device))
            t += list(_fold(p[f"stem.ds{i}.dw.bn"], eps, device))
            t.append(_dev(p[f"stem.ds{i}.pw.w"][:, :, 0, 0], bf, device))
            t += list(_fold(p[f"stem.ds{i}.pw.bn"], eps, device))
        t += [_dev(p[k], f32, device) for k in ("gate.w1", "gate.b1", "gate.w2", "gate.b2")]
        t.append(_ohwi(p["embed.w"], device))
    else:
        t.append(_dev(p["embed.w"].reshape(D, -1), bf, device))
    ints += arch["routes"].reshape(-1).tolist()
    t += [_dev(p["embed.b"], f32, device), _dev(p["cls"], bf, device), _dev(p["pos"], bf, device)]
    for l in range(arch["depth"]):
        q = f"l{l}"
        t += [_dev(p[q + ".ln1.g"], f32, device), _dev(p[q + ".ln1.b"], f32, device),
              _dev(np.stack([p[q + ".wq"], p[q + ".wk"], p[q + ".wv"]]), bf, device),
              _dev(np.stack([p[q + ".bq"], p[q + ".bk"], p[q + ".bv"]]), f32, device),
              _dev(p[q + ".wproj"], bf, device), _dev(p[q + ".bproj"], f32, device),
              _dev(p[q + ".ln2.g"], f32, device), _dev(p[q + ".ln2.b"], f32, device),
              _dev(p[q + ".fc1.w"], bf, device), _dev(p[q + ".fc1.b"], f32, device),
              _dev(p[q + ".fc2.w"], bf, device), _dev(p[q + ".fc2.b"], f32, device)]
    t += [_dev(p["ln.g"], f32, device), _dev(p["ln.b"], f32, device), _dev(p["head.w"], bf, device),
          _dev(p["head.b"], f32, device)]
    # the block's linear weights once more in the order in which a matrix instruction's lanes read them
    first = len(t) - 4 - 12 * arch["depth"]
    for l in range(arch["depth"]):
        t += [_operand_tiles(t[first + 12 * l + i]) for i in (4, 8, 10)]
        t.append(torch.stack([_operand_tiles(w) for w in t[first + 12 * l + 2]]))
    return Net(DS_ARCH_VIT_STEM if C else DS_ARCH_VIT, ints, t, arch["num_classes"], 1, arch["T"])
