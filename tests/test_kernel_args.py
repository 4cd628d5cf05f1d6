"""Arguments of the gate kernels as built: the table by which a network's pass of one image buckets inside its gate (256 bytes and
more) is an argument of those instances alone, not of every gate launch."""
import os
import struct

import pytest

import paper_2109_10060_amd as ds

msgpack = pytest.importorskip("msgpack")
BUNDLE, NOTE = b"__CLANG_OFFLOAD_BUNDLE__", b"AMDGPU\0\0"


def kernels():
    """name -> metadata of the kernels in libdsnet.so"""
    if not os.path.exists(ds.LIB_PATH):
        from paper_2109_10060_amd.build import build
        build(verbose=False)
    blob = open(ds.LIB_PATH, "rb").read()
    out, at = {}, blob.find(BUNDLE)
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + len(BUNDLE))
        pos = at + len(BUNDLE) + 8
        for _ in range(n):
            off, size, name = struct.unpack_from("<QQQ", blob, pos)
            code = blob[at + off:at + off + size]
            pos += 24 + name
            note = code.find(NOTE)
            if note >= 12:
                _, desc, kind = struct.unpack_from("<III", code, note - 12)
                if kind == 32:
                    meta = msgpack.unpackb(code[note + 8:note + 8 + desc])
                    out.update((k[".name"], k) for k in meta["amdhsa.kernels"])
        at = blob.find(BUNDLE, at + 1)
    return out


def test_only_gates_that_bucket_take_the_bucket():
    size = {name: max(a[".offset"] + a[".size"] for a in k[".args"] if not a[".value_kind"].startswith("hidden"))
            for name, k in kernels().items() if "gate_fused_kernel" in name or "gate_out_kernel" in name}
    with_table = {n: s for n, s in size.items() if "BucketArgs" in n}
    plain = {n: s for n, s in size.items() if n not in with_table}
    assert len(with_table) == 3 and len(plain) == 6
    assert max(plain.values()) + 256 < min(with_table.values())
