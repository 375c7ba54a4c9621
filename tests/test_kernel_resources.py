"""What the compiler gave the built kernels, read from the library's own code
object (no GPU needed): the plain search kernels spill nothing, and those
without the parent cache leave its 4 KiB of LDS."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_1811_03374_amd import build_lib

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(path):
    """The gfx950 code objects bundled in the shared library."""
    data = open(path, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + idlen]
            p += 24 + idlen
            if b"gfx950" in name and size:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + 1)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Kernel symbol -> its integer metadata fields."""
    if not os.path.exists(build_lib.LIB):
        build_lib.build()
    d, out = tmp_path_factory.mktemp("co"), {}
    for i, co in enumerate(code_objects(build_lib.LIB)):
        f = d / f"{i}.co"
        f.write_bytes(co)
        text = subprocess.run([READELF, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
        for part in re.split(r"\n\s+- (?=\.a)", text):
            name = re.search(r"\.symbol:\s+'?(\S+?)'?\s", part)
            if name:
                out[name.group(1)] = {k: int(v) for k, v in re.findall(r"\.(\w+):\s+(\d+)\s", part)}
    return out


def fused(kernels):
    """(mode, batched, candidates, quadratic, parent cache) -> fields of each
    instance of the search kernel (mode 0 plain, 1 counting, 2 refining)."""
    found = {}
    for name, x in kernels.items():
        m = re.search(r"k_fusedILi(\d)ELb(\d)ELb(\d)ELb(\d)ELb(\d)E", name)
        if m:
            found[tuple(int(v) for v in m.groups())] = x
    assert len(found) == 12
    return found


def test_plain_kernels_spill_nothing(kernels):
    for key, x in fused(kernels).items():
        assert x["vgpr_count"] <= 128, key                   # four waves a SIMD
        if key[0] != 2:
            assert x["private_segment_fixed_size"] == 0 and x["vgpr_spill_count"] == 0, key


@pytest.mark.parametrize("mode", [0, 2])
def test_no_parent_cache_no_lds_for_it(kernels, mode):
    f = fused(kernels)
    cached, replayed = (f[mode, 1, 0, 0, pc]["group_segment_fixed_size"] for pc in (1, 0))
    assert replayed == cached - 16 * 64 * 4
