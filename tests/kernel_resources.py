"""What the compiler made of each kernel of the built libcdt.so: registers, LDS
and scratch, from the metadata of its gfx950 code objects, and its loads and
waits, from their disassembly (CPU only)."""
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


def _tool(name):
    path = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", name)
    if not os.path.exists(path):
        pytest.skip(f"{name} not found")
    return path


def _elf_files(tmp_path):
    from paper_2607_19490_amd import cdt
    with open(cdt.LIB_PATH, "rb") as f:
        blob = f.read()
    for i, elf in enumerate(_code_objects(blob)):
        path = str(tmp_path / f"{i}.elf")
        with open(path, "wb") as f:
            f.write(elf)
        yield path


def kernels(tmp_path):
    """{mangled kernel name: {"vgpr_count": .., "group_segment_fixed_size": ..,
    "private_segment_fixed_size": .., ...}}."""
    readelf = _tool("llvm-readelf")
    found = {}
    for path in _elf_files(tmp_path):
        notes = subprocess.run([readelf, "--notes", path], check=True, capture_output=True,
                               text=True).stdout
        # a kernel's own fields are indented by four, its arguments' deeper
        for entry in notes.split("\n  - .agpr_count")[1:]:
            fields = dict(re.findall(r"^    \.(\w+):\s+(\S+)$", entry, re.M))
            found[fields["name"]] = {k: int(v) for k, v in fields.items() if v.isdigit()}
    return found


def most_loads_without_a_wait(tmp_path, part):
    """{mangled kernel name with `part` in it: the longest run of 16-byte global
    loads with no wait for one of them in between}."""
    objdump = _tool("llvm-objdump")
    found = {}
    for path in _elf_files(tmp_path):
        text = subprocess.run([objdump, "-d", "--no-show-raw-insn", path], check=True,
                              capture_output=True, text=True).stdout
        for m in re.finditer(r"^[0-9a-f]+ <(\w+)>:\n(.*?)(?=^\n|\Z)", text, re.M | re.S):
            if part not in m.group(1):
                continue
            run = best = 0
            for line in m.group(2).splitlines():
                if "global_load_dwordx4" in line:
                    run += 1
                    best = max(best, run)
                elif "s_waitcnt" in line and "vmcnt" in line:
                    run = 0
            found[m.group(1)] = best
    return found
