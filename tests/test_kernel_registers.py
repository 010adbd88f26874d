"""Registers spilled to scratch memory by the built kernels, as the compiler recorded them in the library: what
the kernels' speed was measured with.  (Values live through a trajectory that should not be show up here.)"""
import os
import re
import struct

import pytest

msgpack = pytest.importorskip("msgpack")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def spills():
    """{kernel name with its template arguments: spilled vector registers} of libopmm.so."""
    d = open(os.path.join(ROOT, "paper_2007_09884_amd", "libopmm.so"), "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    out = {}
    for m in re.finditer(magic, d):
        n, = struct.unpack_from("<Q", d, m.start() + 24)
        p = m.start() + 32
        for _ in range(n):
            off, size, l = struct.unpack_from("<QQQ", d, p)
            target = d[p + 24:p + 24 + l].decode()
            p += 24 + l
            if "gfx950" not in target:
                continue
            e = d[m.start() + off:m.start() + off + size]
            shoff, = struct.unpack_from("<Q", e, 40)
            shentsize, shnum = struct.unpack_from("<HH", e, 58)
            for k in range(shnum):
                s = shoff + k * shentsize
                if struct.unpack_from("<I", e, s + 4)[0] != 7:      # SHT_NOTE
                    continue
                o, _size = struct.unpack_from("<QQ", e, s + 24)
                namesz, descsz, kind = struct.unpack_from("<III", e, o)
                if kind != 32:                                      # NT_AMDGPU_METADATA
                    continue
                desc = e[o + 12 + (namesz + 3) // 4 * 4:][:descsz]
                for kern in msgpack.unpackb(desc, strict_map_key=False)["amdhsa.kernels"]:
                    name = re.search(r"([a-z][a-z_0-9]*_(?:kernel|pass))(I(?:L[a-z]-?\d+E)+E|I[fd]E)?", kern[".name"])
                    args = re.findall(r"L[a-z](-?\d+)E", name.group(2) or "")
                    out[name.group(1) + ("<%s>" % ",".join(args) if args else "")] = kern[".vgpr_spill_count"]
    return out


def test_spilled_registers():
    s = spills()
    of = lambda kernel: {k: v for k, v in s.items() if k.split("<")[0] == kernel}
    assert len(of("fit_round_kernel")) == 8 and set(of("fit_round_kernel").values()) == {0}
    for kernel in ("fit_screen_kernel", "fit_verify_kernel", "fit_persistent_kernel", "nm_kernel", "simulate_kernel",
                   "sensitivity_kernel"):
        assert of(kernel) and max(of(kernel).values()) <= 10, of(kernel)
    # dual numbers fill the file; the normal matrix's sums must not be live beside them
    assert sorted(of("polish_kernel")) == ["polish_kernel<1>", "polish_kernel<2>", "polish_kernel<3>"]
    assert max(of("polish_kernel").values()) <= 150, of("polish_kernel")
