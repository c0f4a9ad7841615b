"""No kernel of the built library keeps vector registers in scratch memory: the compiler has placed such stores behind a
loop's exit with no lane active, where they store nothing. Read from the kernels' own metadata. No GPU needed."""
import os
import re
import struct
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _kernels(lib, tmp):
    """name -> spilled vector registers and bytes of scratch of every gfx950 kernel of a library."""
    fat = str(tmp / "fatbin")
    subprocess.run([f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={fat}", lib, str(tmp / "copy")], check=True,
                   capture_output=True)
    data = open(fat, "rb").read()
    found = {}
    for at in (m.start() for m in re.finditer(MAGIC, data)):
        count, entry = struct.unpack_from("<Q", data, at + len(MAGIC))[0], at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, entry)
            target = data[entry + 24:entry + 24 + length].decode()
            entry += 24 + length
            if "gfx950" not in target or not size:
                continue
            code = tmp / "code"
            code.write_bytes(data[at + offset:at + offset + size])
            notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", str(code)], check=True, capture_output=True,
                                   text=True).stdout
            for block in re.split(r"\n  - \.agpr", notes)[1:]:
                field = lambda key: re.search(rf"\.{key}:\s+(\S+)", block).group(1)  # noqa: E731
                found[field("name")] = int(field("vgpr_spill_count")), int(field("private_segment_fixed_size"))
    return found


def test_no_kernel_spills_vector_registers(tmp_path):
    if not os.path.exists(f"{LLVM}/llvm-readelf"):
        pytest.skip("needs the ROCm LLVM tools")
    from paper_1710_10789_amd import build

    if not os.path.exists(build.LIB):
        build.build()
    kernels = _kernels(build.LIB, tmp_path)
    assert sum("dos_forward_kernel" in k for k in kernels) == 16 * 3 * 3  # orbitals, weight types, modes
    assert sum("chi_spline_kernel" in k for k in kernels) == 16 * 3
    assert {k: v for k, v in kernels.items() if v[0] or v[1]} == {}
