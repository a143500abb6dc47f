"""What the compiler gave each kernel of the built libcdt.so: registers, LDS
and scratch, from the metadata of its gfx950 code objects (CPU only)."""
import os
import re
import struct
import subprocess

import pytest

_MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    """The gfx950 ELF images of the bundles in `blob`."""
    at = blob.find(_MAGIC)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", blob, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, tlen = struct.unpack_from("<QQQ", blob, p)
            triple = blob[p + 24:p + 24 + tlen]
            p += 24 + tlen
            if b"gfx950" in triple and size:
                yield blob[at + off:at + off + size]
        at = blob.find(_MAGIC, at + 24)


def kernels(tmp_path):
    """{mangled kernel name: {"vgpr_count": .., "group_segment_fixed_size": ..,
    "private_segment_fixed_size": .., ...}}."""
    from paper_2607_19490_amd import cdt
    readelf = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")
    if not os.path.exists(readelf):
        pytest.skip("llvm-readelf not found")
    with open(cdt.LIB_PATH, "rb") as f:
        blob = f.read()
    found = {}
    for i, elf in enumerate(_code_objects(blob)):
        path = str(tmp_path / f"{i}.elf")
        with open(path, "wb") as f:
            f.write(elf)
        notes = subprocess.run([readelf, "--notes", path], check=True, capture_output=True,
                               text=True).stdout
        # a kernel's own fields are indented by four, its arguments' deeper
        for entry in notes.split("\n  - .agpr_count")[1:]:
            fields = dict(re.findall(r"^    \.(\w+):\s+(\S+)$", entry, re.M))
            found[fields["name"]] = {k: int(v) for k, v in fields.items() if v.isdigit()}
    return found
