"""Registers of the compiled lattice passes, from the metadata of the built library: where two
workgroups of 512 threads (or four of 256) are meant to share a CU, a kernel holds 128 at most."""
import os
import re
import shutil
import struct
import subprocess

import pytest

READELF = next((c for c in ("/opt/rocm/llvm/bin/llvm-readelf", shutil.which("llvm-readelf")) if c and os.path.exists(c)),
               None)
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(path):
    """The device ELF images of a library: one bundle per source file, its entries (offset, size, target)."""
    data = open(path, "rb").read()
    for m in re.finditer(re.escape(MAGIC), data):
        at = m.start() + len(MAGIC)
        n, = struct.unpack_from("<Q", data, at)
        if n > 8:
            continue  # the text, not a bundle
        at += 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, at)
            target = data[at + 24:at + 24 + idlen].decode()
            at += 24 + idlen
            if "gfx950" in target and size:
                yield data[m.start() + off:m.start() + off + size]


def _registers(tmp_path):
    import paper_2603_24370_amd as ss
    ss.lib()
    from paper_2603_24370_amd import build as b
    out = {}
    for k, image in enumerate(_code_objects(b.LIB)):
        p = tmp_path / f"{k}.elf"
        p.write_bytes(image)
        notes = subprocess.run([READELF, "--notes", str(p)], capture_output=True, text=True, check=True).stdout
        for kernel in notes.split("- .agpr_count:")[1:]:
            name = re.search(r"\.name:\s+(\S+)", kernel).group(1)
            out[name] = tuple(int(re.search(rf"\.{k}:\s+(\d+)", kernel).group(1)) for k in ("vgpr_count", "vgpr_spill_count"))
    return out


@pytest.mark.skipif(READELF is None, reason="needs llvm-readelf")
def test_a_batch_keeps_four_waves_per_simd(tmp_path):
    """The FP32 passes of a batch on its default shapes (64 x 16 and 64 x 8 sites, two rows per thread)."""
    regs = {n: v for n, (v, _) in _registers(tmp_path).items() if re.match(r"_ZN2ss10batch_passIfLi\d+ELi\d+ELi64ELi(16|8)ELi2EE", n)}
    assert len(regs) == 2 * 2 * 11  # theories, shapes, passes
    assert {n: v for n, v in regs.items() if v > 128} == {}


# Abelian Higgs passes, and the registers that they spilled before their rows went on scalar
# bases and a batch's descriptors were held in registers
@pytest.mark.parametrize("kernel,spills", [("stage_passIdLi0ELi2ELi64ELi32ELi4EE", 25),
                                           ("stage_passIdLi0ELi3ELi64ELi32ELi4EE", 57),
                                           ("batch_passIfLi0ELi7ELi64ELi16ELi2EE", 5),
                                           ("batch_passIdLi0ELi2ELi64ELi32ELi4EE", 25),
                                           ("batch_passIdLi0ELi3ELi64ELi32ELi4EE", 69)])
@pytest.mark.skipif(READELF is None, reason="needs llvm-readelf")
def test_passes_spill_no_more_than_they_need(kernel, spills, tmp_path):
    (name, (_, n)), = ((k, v) for k, v in _registers(tmp_path).items() if kernel in k)
    assert n <= spills, name
