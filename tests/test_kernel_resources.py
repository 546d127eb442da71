"""Registers and scratch memory of the built step kernels, from the code object's own metadata."""
import os
import re
import struct
import subprocess

from paper_1707_00198_amd import lbm

ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _kernels(tmp_path):
    """{mangled name: (scratch bytes a lane, vector registers)} of the gfx950 code objects in the library."""
    blob, out, at = open(lbm.LIB_PATH, "rb").read(), {}, -1
    while (at := blob.find(MAGIC, at + 1)) >= 0:
        n, p = struct.unpack_from("<Q", blob, at + len(MAGIC))[0], at + len(MAGIC) + 8
        for _ in range(n if n < 16 else 0):
            off, size, length = struct.unpack_from("<QQQ", blob, p)
            triple = blob[p + 24:p + 24 + length].decode()
            p += 24 + length
            if not triple.endswith("gfx950") or size == 0:
                continue
            elf = tmp_path / "gfx950.elf"
            elf.write_bytes(blob[at + off:at + off + size])
            notes = subprocess.run([os.path.join(ROCM, "llvm", "bin", "llvm-readelf"), "--notes", str(elf)], capture_output=True,
                                   text=True, check=True).stdout
            for k in re.split(r"\n\s+- \.", notes):
                name = re.search(r"\.name:\s+(\S+)", k)
                scratch, vgprs = (re.search(r"\.%s:\s+(\d+)" % f, k) for f in ("private_segment_fixed_size", "vgpr_count"))
                if name and scratch and vgprs:
                    out[name.group(1)] = int(scratch.group(1)), int(vgprs.group(1))
    return out


def test_patch_kernels_hold_their_values_in_registers(tmp_path):
    """At 64 vector registers, two blocks of 16 wavefronts on a CU: no scratch memory, but for two
    registers of the plain FP64 build (12 bytes with their alignment)."""
    k = {n: v for n, v in _kernels(tmp_path).items() if "patch_kernelI" in n}
    assert len(k) == 24
    for name, (scratch, vgprs) in k.items():
        assert scratch <= (12 if "patch_kernelIdLi1ELi8E" in name and "Lb0E" in name else 0), (name, scratch, vgprs)
        assert vgprs <= 64 or "patch_kernelIdLi1ELi4E" in name, (name, vgprs)


def test_blocks_of_eight_wavefronts_keep_their_registers(tmp_path):
    """A block of 8 wavefronts puts 2 on each SIMD, so a CU holds 2 such blocks up to 128 vector
    registers and none more down to 85: a tighter bound would only push values into scratch memory."""
    k = {n: v for n, v in _kernels(tmp_path).items() if re.search(r"step_kernelI.*Li(8ELi1|4ELi2)ELb[01]E", n) and not n.endswith(".kd")}
    assert len(k) == 16
    for name, (scratch, vgprs) in k.items():
        assert scratch == 0, (name, scratch, vgprs)
        assert vgprs <= 128 or "step_kernelId" in name, (name, vgprs)
