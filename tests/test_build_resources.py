"""Registers of the built kernels (CPU; reads this repository's own library).

Two kinds of kernel rest on what the compiler does with their registers:
- those whose waits count copies into LDS (gemm_big_kernel,
  gemm_big_int4_kernel, gemm_mid_kernel): a spill's loads would be counted
  with them and the waits would end too early, so nothing may be spilled;
- those that read matrix-core results after a branch (big_fix_kernel, and
  dec_main_kernel, whose expand branches by row block): this compiler reads
  accumulation registers too early there, so they may use none.
The kernel descriptors in the library say both."""
import os
import re
import shutil
import struct
import subprocess

import pytest

import paper_2510_23346_amd as bd

ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
READELF = next((p for p in (os.path.join(ROCM, "llvm", "bin", "llvm-readelf"), shutil.which("llvm-readelf") or "")
                if p and os.path.exists(p)), None)
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(data: bytes):
    """The gfx950 code objects of the offload bundles in a host library."""
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(min(n, 16)):
            off, size, k = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + k]
            p += 24 + k
            if b"gfx950" in name and size:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + 1)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if READELF is None:
        pytest.skip("needs llvm-readelf")
    if not os.path.exists(bd.lib_path()):
        from paper_2510_23346_amd.build import build
        build()
    with open(bd.lib_path(), "rb") as f:
        data = f.read()
    out = {}
    tmp = str(tmp_path_factory.mktemp("co") / "a.co")
    for co in _code_objects(data):
        with open(tmp, "wb") as f:
            f.write(co)
        notes = subprocess.run([READELF, "--notes", tmp], capture_output=True, text=True).stdout
        for part in re.split(r"\n\s*- \.agpr_count:", "\n" + notes)[1:]:
            part = ".agpr_count:" + part
            get = lambda key: int(re.search(rf"\.{key}:\s*(\d+)", part)[1])  # noqa: E731
            out[re.search(r"\n\s*\.name:\s*(_Z\S+)", part)[1]] = {
                k: get(k) for k in ("agpr_count", "vgpr_spill_count", "private_segment_fixed_size", "vgpr_count")}
    return out


@pytest.mark.parametrize("name,count", [("gemm_big_kernel", 2), ("gemm_big_int4_kernel", 1), ("gemm_mid_kernel", 4),
                                        ("big_fix_kernel", 2), ("dec_main_kernel", 24)])
def test_kernel_registers(kernels, name, count):
    mine = {k: v for k, v in kernels.items() if re.match(rf"_ZN3bdl\d+{name}[IE]", k)}
    assert len(mine) == count, sorted(mine)
    for k, v in mine.items():
        assert v["vgpr_spill_count"] == 0 and v["private_segment_fixed_size"] == 0, (k, v)
        if name in ("big_fix_kernel", "dec_main_kernel"):
            assert v["agpr_count"] == 0, (k, v)
