"""What the compiler made of the kernels, read from the library as built: registers that do not fit a kernel's budget go to scratch, that
is to memory, once per lane and launch (28 bytes per lane of 480 workgroups of 1024: 14 MB written and most of them read back)."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2605_29346_amd import build


def _kernels(tmp_path):
    """Kernel metadata of the library's gfx950 code object: name -> bytes of scratch per lane, vector registers, spilled vector registers."""
    tool = next((t for t in ("/opt/rocm/llvm/bin/llvm-readelf", shutil.which("llvm-readelf")) if t and os.path.exists(t)), None)
    if tool is None:
        pytest.skip("no llvm-readelf here")
    blob, found = open(build.LIB, "rb").read(), {}
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    for at in (m.start() for m in re.finditer(magic, blob)):
        count, p = struct.unpack_from("<Q", blob, at + len(magic))[0], at + len(magic) + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", blob, p)
            target, p = blob[p + 24: p + 24 + length].decode(), p + 24 + length
            if "gfx950" not in target or not size:
                continue
            path = tmp_path / "code.o"
            path.write_bytes(blob[at + offset: at + offset + size])
            notes = subprocess.run([tool, "--notes", str(path)], check=True, capture_output=True, text=True).stdout
            for entry in notes.split("  - .agpr_count:")[1:]:
                get = lambda key: re.search(rf"\.{key}:\s+(\S+)", entry).group(1)
                found[get("name")] = (int(get("private_segment_fixed_size")), int(get("vgpr_count")), int(get("vgpr_spill_count")))
    return found


def test_no_kernel_spills_vector_registers_to_memory(tmp_path):
    kernels = _kernels(tmp_path)
    assert sum("k_hop" in k for k in kernels) == 12 and any("k_close" in k for k in kernels), sorted(kernels)
    assert {k: v for k, v in kernels.items() if v[0] or v[2]} == {}
    assert all(v[1] <= 64 for k, v in kernels.items() if "k_hop" in k)  # two workgroups of 1024 lanes on a compute unit
