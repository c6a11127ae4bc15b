"""Registers that the compiler spilled to scratch in the built library's
lateral FFT kernels (from the code objects' metadata). Radix 32 needs nearly
all of the 128 registers that four waves per SIMD leave; with 12 of them in
scratch the x pass over 512-point rows took 577 us where it takes 491, more
than the passes in LDS that it replaced (478 us). Two spilled registers (one
store and one load of 8 bytes per thread) stay within the noise."""
import os
import re
import shutil
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1510_01078_amd", "libpatnufft.so")
BIN = "/opt/rocm/llvm/bin"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    """The gfx950 ELF images of every offload bundle in the section."""
    at = blob.find(MAGIC)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", blob, at + 24)
        pos = at + 32
        for _ in range(count):
            off, size, idlen = struct.unpack_from("<QQQ", blob, pos)
            name = blob[pos + 24:pos + 24 + idlen]
            pos += 24 + idlen
            if b"gfx950" in name and size:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + 24)


def _spills(tmp_path):
    """Demangled kernel name -> spilled vector registers."""
    section = tmp_path / "fatbin"
    subprocess.run([f"{BIN}/llvm-objcopy", "--dump-section", f".hip_fatbin={section}", LIB, str(tmp_path / "copy.so")],
                   check=True, capture_output=True, timeout=120)
    out = {}
    for i, elf in enumerate(_code_objects(section.read_bytes())):
        f = tmp_path / f"{i}.elf"
        f.write_bytes(elf)
        notes = subprocess.run([f"{BIN}/llvm-readelf", "--notes", str(f)], check=True, capture_output=True, text=True,
                               timeout=120).stdout
        for entry in notes.split("\n  - ")[1:]:
            name = re.search(r"\.name:\s+(\S+)", entry)
            spill = re.search(r"\.vgpr_spill_count:\s+(\d+)", entry)
            if name and spill:
                out[name.group(1)] = int(spill.group(1))
    plain = subprocess.run(["c++filt"], input="\n".join(out), capture_output=True, text=True, check=True).stdout
    return {re.sub(r"\(.*", "", n): v for n, v in zip(plain.split("\n"), out.values())}


@pytest.mark.skipif(not os.path.exists(LIB), reason="library not built")
@pytest.mark.skipif(not all(shutil.which(t) for t in (f"{BIN}/llvm-objcopy", f"{BIN}/llvm-readelf", "c++filt")),
                    reason="needs ROCm's binary utilities")
def test_lateral_transforms_spill_next_to_nothing(tmp_path):
    spills = _spills(tmp_path)
    seen = 0
    for kernel in ("k_fft_x_reg", "k_fft_y_reg"):
        for t in ("float", "double"):
            for cls in (16, 20, 32):
                n = spills[f"void patk::{kernel}<{t}, {cls}>"]
                assert n <= 2, (kernel, t, cls, n)
                seen += 1
    assert seen == 12
