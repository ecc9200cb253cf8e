"""What the compiler gave the kernels of the built library, from the code
objects' own metadata (no device needed): private memory of a kernel is
mapped by the runtime at its launch, on a card that the program may have
filled, so no kernel of the library's has any."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1708_09707_amd", "libhmx.so")
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _device_objects(blob):
    """The gfx950 code objects of the offload bundles in the library."""
    at = blob.find(MAGIC)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, tl = struct.unpack_from("<QQQ", blob, p)
            triple = blob[p + 24:p + 24 + tl].decode()
            p += 24 + tl
            if "gfx950" in triple and size:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + 1)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    d = tmp_path_factory.mktemp("objects")
    out = {}
    for i, obj in enumerate(_device_objects(open(LIB, "rb").read())):
        f = d / ("%d.co" % i)
        f.write_bytes(obj)
        notes = subprocess.check_output([READELF, "--notes", str(f)], text=True)
        for entry in re.split(r"\n  - ", notes)[1:]:
            v = dict(re.findall(r"^\s*\.(\w+):\s+'?([\w.]+)'?\s*$", entry, re.M))
            if "private_segment_fixed_size" in v:
                out[v["name"]] = int(v["private_segment_fixed_size"])
    assert len(out) > 100
    names = subprocess.check_output(["c++filt"] + list(out), text=True).splitlines()
    return dict(zip(names, out.values()))


@pytest.mark.parametrize("kernel", ["p1_tile_kernel", "rowtile_kernel", "aca_kernel",
                                    "aca_lds_kernel", ""])
def test_no_private_memory(kernels, kernel):
    """By family, and ("") every kernel of the library."""
    found = {k: v for k, v in kernels.items() if kernel in k}
    assert found
    bad = {k: v for k, v in found.items() if v}
    assert not bad
