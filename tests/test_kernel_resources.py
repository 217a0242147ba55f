"""What the compiler gave the kernels of the built library, from the kernel descriptors' metadata
in its code objects: the kernels of the default paths hold everything in registers.  A spilled
register costs a trip through memory in kernels that are tuned to their register limit, and does
not show in any result."""

import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2605_01910_amd import santa as S

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"  # then u64 count and per entry u64 offset, size, id length, id


def scratch_bytes(tmp_path):
    """Scratch (private segment) bytes per lane of every kernel, by mangled name."""
    lib = open(S.LIB_PATH, "rb").read()
    out, at = {}, lib.find(MAGIC)
    while at >= 0:
        p = at + len(MAGIC) + 8
        for _ in range(struct.unpack_from("<Q", lib, p - 8)[0]):
            off, size, n = struct.unpack_from("<QQQ", lib, p)
            target = lib[p + 24:p + 24 + n]
            p += 24 + n
            if size and b"amdgcn" in target:
                obj = tmp_path / "code_object"
                obj.write_bytes(lib[at + off:at + off + size])
                notes = subprocess.run([READELF, "--notes", str(obj)], capture_output=True, text=True, check=True)
                for entry in re.split(r"\n  - ", notes.stdout):
                    m = re.search(r"\.private_segment_fixed_size:\s+(\d+)", entry)
                    name = re.search(r"\.symbol:\s+'?(\S+?)\.kd", entry)
                    if m and name:
                        out[name.group(1)] = int(m.group(1))
        at = lib.find(MAGIC, at + len(MAGIC))
    return out


@pytest.mark.skipif(not os.path.exists(READELF), reason="no llvm-readelf")
def test_default_kernels_use_no_scratch(tmp_path):
    scratch = scratch_bytes(tmp_path)
    for kernel in ("k_row_sampled", "k_row_flash", "k_stream_cdf", "k_value_heads", "k_bern_stream",
                   "k_dense_stream"):
        found = {n: b for n, b in scratch.items() if f"{len(kernel)}{kernel}I" in n}
        assert found, kernel
        assert not any(found.values()), {n: b for n, b in found.items() if b}
