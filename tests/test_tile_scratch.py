"""The built library's tiled kernels, by the metadata of its code objects: none of them, of whatever tile shape and
wavefront count, keeps anything in scratch memory."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2511_01884_amd import build

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
OBJCOPY = "/opt/rocm/llvm/bin/llvm-objcopy"
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def _scratch(tmp_path):
    """Kernel name -> bytes of scratch memory a lane."""
    fat = tmp_path / "fat"
    subprocess.run([OBJCOPY, "--dump-section", ".hip_fatbin=%s" % fat, build.LIB_PATH, os.devnull], check=True)
    data = fat.read_bytes()
    used = {}
    for m in re.finditer(re.escape(BUNDLE), data):
        at = m.start() + len(BUNDLE)
        (entries,) = struct.unpack_from("<Q", data, at)
        at += 8
        for _ in range(entries):
            offset, size, length = struct.unpack_from("<QQQ", data, at)
            name = data[at + 24:at + 24 + length].decode()
            at += 24 + length
            if "gfx950" not in name:
                continue
            code = tmp_path / "code"
            code.write_bytes(data[m.start() + offset:m.start() + offset + size])
            notes = subprocess.run([READELF, "--notes", str(code)], check=True, stdout=subprocess.PIPE, text=True).stdout
            names = re.findall(r"^    \.name: +(\S+)", notes, re.M)
            sizes = re.findall(r"^    \.private_segment_fixed_size: (\d+)", notes, re.M)
            assert len(names) == len(sizes)
            used.update(zip(names, map(int, sizes)))
    return used


@pytest.mark.skipif(not (shutil.which(READELF) and shutil.which(OBJCOPY)), reason="no tools for code objects")
def test_no_tile_kernel_uses_scratch_memory(tmp_path):
    used = {name: size for name, size in _scratch(tmp_path).items() if "tile_kernel" in name or "finalize_kernel" in name}
    assert any("Li2ELi2ELi4ELi4E" in name for name in used)   # 256 x 256 by four wavefronts, the tightest
    assert not {name: size for name, size in used.items() if size}
