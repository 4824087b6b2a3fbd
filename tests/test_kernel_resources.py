"""No kernel of the built library uses private memory (CPU): the runtime would
take it from the device at a first launch, in a library whose entry points
allocate nothing, and a register spilled to it costs memory traffic in a loop.
Read from the metadata of the code objects that the build put into libecho.so."""
import os
import re
import struct
import subprocess

import pytest

from paper_2504_03651_amd import echo

LLVM = "/opt/rocm/llvm/bin"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(fatbin):
    """The gfx950 images of the offload bundles in a .hip_fatbin section."""
    at = fatbin.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", fatbin, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", fatbin, p)
            name = fatbin[p + 24:p + 24 + idlen].decode()
            p += 24 + idlen
            if "gfx950" in name:
                yield fatbin[at + off:at + off + size]
        at = fatbin.find(MAGIC, at + 1)


@pytest.mark.skipif(not os.path.exists(f"{LLVM}/llvm-readelf"), reason="needs ROCm's llvm-readelf")
def test_no_kernel_spills_or_uses_private_memory(tmp_path):
    fat = tmp_path / "fatbin"
    subprocess.run([f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={fat}", echo.LIB_PATH,
                    str(tmp_path / "copy.so")], check=True)
    kernels = {}
    for i, image in enumerate(_code_objects(fat.read_bytes())):
        obj = tmp_path / f"{i}.o"
        obj.write_bytes(image)
        notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", str(obj)], check=True,
                               capture_output=True, text=True).stdout
        for k in re.split(r"\n  - ", notes):
            name = re.search(r"\.name: +(_Z\S+)", k)
            if name:
                kernels[name[1]] = (int(re.search(r"\.private_segment_fixed_size: +(\d+)", k)[1]),
                                    int(re.search(r"\.vgpr_spill_count: +(\d+)", k)[1]))
    assert sum("prefill_kernel" in n for n in kernels) == 6 and len(kernels) > 20, sorted(kernels)
    assert {n: v for n, v in kernels.items() if v != (0, 0)} == {}
