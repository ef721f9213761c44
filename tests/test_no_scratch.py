"""No kernel of the library has a private segment (spilled registers, stack): the runtime would reserve
device memory for it at the kernel's first dispatch, which the library promises not to cause, and every
access to it waits for the loads in flight.  Read from the built library's own kernel metadata (CPU only)."""
import os
import re
import struct
import subprocess

import pytest

from paper_2606_13898_amd import hilo

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"

pytestmark = pytest.mark.skipif(not (os.path.exists(hilo.LIB_PATH) and os.path.exists(READELF)),
                                reason="libhilo.so not built, or no llvm-readelf")


def code_objects(blob):
    """The gfx950 ELF images of the library's offload bundles (one bundle per source file)."""
    for m in re.finditer(MAGIC, blob):
        at = m.start() + len(MAGIC)
        n, = struct.unpack_from("<Q", blob, at)
        at += 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", blob, at)
            name = blob[at + 24:at + 24 + idlen].decode()
            at += 24 + idlen
            if size and "gfx950" in name:
                yield blob[m.start() + off:m.start() + off + size]


def test_no_kernel_uses_scratch(tmp_path):
    sizes = {}
    with open(hilo.LIB_PATH, "rb") as f:
        blob = f.read()
    for i, co in enumerate(code_objects(blob)):
        path = tmp_path / f"{i}.co"
        path.write_bytes(co)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for name, size in re.findall(r"\.name:\s+(\S*k_\S+)\n.*?\.private_segment_fixed_size:\s+(\d+)", notes, re.S):
            sizes[name] = int(size)
    assert sum("k_gemm8" in n for n in sizes) == 16 and any("k_attn_bf16" in n for n in sizes), sorted(sizes)
    assert not {n: s for n, s in sizes.items() if s}
