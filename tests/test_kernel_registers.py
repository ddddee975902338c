"""Registers of the attention kernels as built (the code objects' own metadata, no GPU): what rules of the launch and waves per
SIMD rest on."""
import re
import struct

import pytest

from paper_2402_11131_amd import build

msgpack = pytest.importorskip("msgpack")


def _code_objects(data):
    at = data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        p = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + n]:
                yield data[at + off:at + off + size]
            p += 24 + n
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)


def _kernels():
    """Metadata of every kernel of the library by its mangled name: the note of type 32 of each code object."""
    out = {}
    for elf in _code_objects(open(build.LIB_PATH, "rb").read()):
        table = struct.unpack_from("<Q", elf, 40)[0]
        size, count = struct.unpack_from("<HH", elf, 58)
        for i in range(count):
            _, kind, _, _, off = struct.unpack_from("<IIQQQ", elf, table + i * size)
            if kind != 7:
                continue
            name_len, desc_len, note = struct.unpack_from("<III", elf, off)
            at = off + 12 + (name_len + 3) // 4 * 4
            if note == 32:
                for k in msgpack.unpackb(elf[at:at + desc_len])["amdhsa.kernels"]:
                    out[k[".name"]] = k
    return out


def _instances(kernels):
    """(D, query tiles, few-row merge) -> registers of the instances of the kernel with 16 rows per wave, the most of each."""
    out = {}
    for name, k in kernels.items():
        m = re.match(r"_ZN2ss15msa_bf16_kernelILi(\d+)ELi(\d)ELb[01]ELb[01]ELb([01])E", name)
        if m:
            key = int(m[1]), int(m[2]), m[3] == "1"
            out.setdefault(key, []).append(k[".vgpr_count"])
    return out


def test_attention_instances():
    kernels = _kernels()
    regs = _instances(kernels)
    waves = lambda r: 512 // (-(-r // 8) * 8)   # of a SIMD's 512 registers, given out by eights
    assert len(regs) == 14
    # one query tile per wave group: the merge of three and four splits is not in the instance that the other calls take
    assert waves(max(regs[128, 1, False])) == 2 and waves(max(regs[64, 1, False])) == 3
    assert max(regs[64, 1, False]) < max(regs[64, 1, True]) and max(regs[128, 1, False]) < max(regs[128, 1, True])
    # heads of 64: at most six waves per SIMD, which the rule for the stages of the step's own rows counts with
    assert all(waves(r) <= 6 for (d, _, _), rs in regs.items() if d == 64 for r in rs)
    # sixteen waves per workgroup
    assert all(r <= 128 for (_, nw, _), rs in regs.items() if nw >= 4 for r in rs)
    assert all(k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0 for n, k in kernels.items() if "msa_bf16" in n)
