"""Registers, scratch and instructions of the built convolution kernels, from the code objects inside libdat.so (runs without
a GPU)."""
import os
import re
import struct
import subprocess

import msgpack

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2206_06257_amd", "libdat.so")


def _code_objects():
    """The gfx950 code objects bundled into the library."""
    data, pos = open(LIB, "rb").read(), 0
    while (pos := data.find(b"__CLANG_OFFLOAD_BUNDLE__", pos)) >= 0:
        entries, at = struct.unpack_from("<Q", data, pos + 24)[0], pos + 32
        for _ in range(entries):
            off, size, n = struct.unpack_from("<QQQ", data, at)
            triple, at = data[at + 24:at + 24 + n], at + 24 + n
            if b"gfx950" in triple and size:
                yield data[pos + off:pos + off + size]
        pos += 24


def _kernels():
    """Kernel metadata (AMDGPU ELF notes) of the code objects."""
    out = []
    for elf in _code_objects():
        sections, (entsize, count) = struct.unpack_from("<Q", elf, 40)[0], struct.unpack_from("<HH", elf, 58)
        for i in range(count):
            h = sections + i * entsize
            if struct.unpack_from("<I", elf, h + 4)[0] != 7:              # SHT_NOTE
                continue
            p, length = struct.unpack_from("<QQ", elf, h + 24)
            end = p + length
            while p < end:
                name, desc, kind = struct.unpack_from("<III", elf, p)
                d = p + 12 + (name + 3) // 4 * 4
                if kind == 32:                                            # NT_AMDGPU_METADATA
                    out += msgpack.unpackb(elf[d:d + desc])["amdhsa.kernels"]
                p = d + (desc + 3) // 4 * 4
    return out


def test_ordinary_convolution_launches_carry_no_class_table_and_hardly_spill():
    """The single-stage kernels in narrow tiles are held to 80 and 96 registers (six and five workgroups per CU) and keep at
    most four values of their prologue in scratch; the multi-stage kernels, alone on their CU, spill nothing."""
    conv = [k for k in _kernels() if "igemm_dma_kernel" in k[".name"] or "igemm_ring_kernel" in k[".name"]]
    plain = [k for k in conv if "IgemmClasses" not in k[".name"].split("EvNS")[0]]
    assert len(plain) >= 12 and len(conv) > len(plain)
    for k in plain:
        ring = "igemm_ring_kernel" in k[".name"]
        assert k[".vgpr_spill_count"] <= (0 if ring else 4) and k[".sgpr_spill_count"] == 0, k
        assert k[".kernarg_segment_size"] <= 256, k


def test_convolution_kernels_load_from_global_memory(tmp_path):
    """No flat loads: those go through the LDS path as well and are waited for together with it."""
    objdump = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
    seen = 0
    for i, elf in enumerate(_code_objects()):
        f = tmp_path / ("%d.o" % i)
        f.write_bytes(elf)
        text = subprocess.run([objdump, "-d", str(f)], stdout=subprocess.PIPE, check=True, text=True).stdout
        for name, body in re.findall(r"^[0-9a-f]+ <(\S+)>:\n(.*?)(?=^[0-9a-f]+ <|\Z)", text, re.S | re.M):
            if "igemm" in name or "wgrad" in name:
                seen += 1
                assert "global_load" in body or "buffer_load" in body, name
                assert "flat_load" not in body, name
    assert seen >= 40
