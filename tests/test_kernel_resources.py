"""No kernel of the library keeps values in scratch memory.

A kernel with scratch makes the runtime set aside memory for it per queue at its first launch, which the allocation-free
entry point promises not to need, and its spilled values cost a memory round trip each.  The compiler states both in the
code object's metadata, which is read here from the built library.
"""
import os
import re
import struct
import subprocess

import pytest

import paper_2607_14568_amd as gdn

READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_object(path):
    """The gfx950 code object of the library's offload bundle."""
    blob = open(path, "rb").read()
    at = blob.index(MAGIC)
    (n,) = struct.unpack_from("<Q", blob, at + len(MAGIC))
    pos = at + len(MAGIC) + 8
    for _ in range(n):
        off, size, idlen = struct.unpack_from("<QQQ", blob, pos)
        ident = blob[pos + 24:pos + 24 + idlen].decode()
        pos += 24 + idlen
        if "gfx950" in ident:
            return blob[at + off:at + off + size]
    raise AssertionError("no gfx950 code object in %s" % path)


def test_no_kernel_uses_scratch(tmp_path):
    if not os.path.exists(READELF):
        pytest.skip("llvm-readelf is not installed")
    obj = tmp_path / "gdn.co"
    obj.write_bytes(_code_object(gdn.LIB_PATH))
    notes = subprocess.run([READELF, "--notes", str(obj)], capture_output=True, text=True, check=True).stdout
    fields = {k: re.findall(r"\.%s: +(\S+)" % k, notes) for k in ("private_segment_fixed_size", "vgpr_spill_count")}
    names = re.findall(r"\.symbol: +(\S+)", notes)
    assert len(names) > 50 and all(len(v) == len(names) for v in fields.values())
    bad = [(n, s, v) for n, s, v in zip(names, *fields.values()) if s != "0" or v != "0"]
    assert not bad, bad
