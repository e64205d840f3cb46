"""Registers of the built kernels against the waves that a CU is meant to hold (the
metadata of this repository's own gfx950 code objects; no GPU)."""
import os
import struct

import msgpack
import pytest

import paper_0912_4255_amd as rsf

LIB = os.path.join(os.path.dirname(rsf.__file__), "librsfstat.so")


def _kernels():
    """{mangled name: metadata} from the code objects bundled in the library."""
    data = open(LIB, "rb").read()
    out, at = {}, data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + 24)
        pos = at + 32
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, pos)
            triple = data[pos + 24:pos + 24 + idlen]
            pos += 24 + idlen
            if b"gfx950" in triple and size:
                out.update(_notes(data[at + off:at + off + size]))
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)
    return out


def _notes(elf):
    shoff, = struct.unpack_from("<Q", elf, 40)
    size, count = struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        _, kind, _, _, off, length = struct.unpack_from("<IIQQQQ", elf, shoff + i * size)
        while kind == 7 and length >= 12:
            nlen, dlen, ntype = struct.unpack_from("<III", elf, off)
            if ntype == 32 and elf[off + 12:off + 18] == b"AMDGPU":
                desc = elf[off + 12 + -(-nlen // 4) * 4:][:dlen]
                return {k[".name"]: k for k in msgpack.unpackb(desc)["amdhsa.kernels"]}
            step = 12 + -(-nlen // 4) * 4 + -(-dlen // 4) * 4
            off, length = off + step, length - step
    return {}


def _waves_per_cu(k):
    """By registers alone: 512 per lane of a SIMD, allocated in eights, 4 SIMDs, whole
    workgroups, at most 8 waves per SIMD."""
    regs = max(8, -(-(k[".vgpr_count"] + k.get(".agpr_count", 0)) // 8) * 8)
    group = -(-k[".max_flat_workgroup_size"] // 64)
    per_simd = -(-group // 4)
    return min(8, 512 // regs) // per_simd * group


@pytest.mark.parametrize("name,waves", [
    ("rsf_sft_rows_kILi512E", 16),   # two workgroups of 8 waves
    ("rsf_sft_rows_kILi256E", 12),   # three of 4
    ("rsf_resample_kILb1E", 12),     # three of 4: orbits of every sample
    ("rsf_resample_run_k", 16),      # two of 8
])
def test_waves_that_registers_allow(name, waves):
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    found = {n: k for n, k in _kernels().items() if name in n}
    assert found
    for n, k in found.items():
        assert _waves_per_cu(k) >= waves, (n, k[".vgpr_count"], k[".max_flat_workgroup_size"])
