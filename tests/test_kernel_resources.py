"""Registers of the built kernels whose workgroups share a compute unit by design (CPU only: read from the library's own
kernel descriptions)."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2603_18636_amd import svoo

READELF = shutil.which("llvm-readelf", path="/opt/rocm/llvm/bin:" + os.environ.get("PATH", ""))
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Mangled kernel name -> (vector registers, scratch bytes)."""
    if READELF is None:
        pytest.skip("llvm-readelf is not installed")
    if not os.path.exists(svoo.LIB_PATH):
        from paper_2603_18636_amd import build
        build.build(verbose=False)
    data = open(svoo.LIB_PATH, "rb").read()
    found = {}
    for start in (m.start() for m in re.finditer(MAGIC, data)):
        at = start + len(MAGIC) + 8
        for _ in range(struct.unpack_from("<Q", data, at - 8)[0]):
            offset, size, chars = struct.unpack_from("<QQQ", data, at)
            target = data[at + 24:at + 24 + chars]
            at += 24 + chars
            if b"gfx950" not in target:
                continue
            path = tmp_path_factory.mktemp("code") / "object"
            path.write_bytes(data[start + offset:start + offset + size])
            notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
            for part in re.split(r"\n\s+- \.agpr_count", notes)[1:]:
                number = lambda key: int(re.search(r"\.%s:\s+(\d+)" % key, part).group(1))
                found[re.search(r"\.name:\s+(\S+)", part).group(1)] = (number("vgpr_count"),
                                                                       number("private_segment_fixed_size"))
    return found


@pytest.mark.parametrize("name,registers", [
    ("assign_small_kernel", {"t": 128, "f": 128}),                          # two workgroups of eight waves
    ("assign_kernelI[tf]Li64E", {"t": 168, "f": 168}),                      # three workgroups of four waves
    ("assign_kernelI[tf]Li128E", {"t": 168, "f": 256}),                     # float32 tokens: two
    ("sparse_attn_bf16_kernel", {"": 256}),                                 # eight waves, two a SIMD
    ("sparse_attn_f32_kernelILi64E", {"": 168}),                            # three workgroups of four waves
    ("sparse_attn_f32_kernelILi128E", {"": 256}),                           # two
    ("sparse_attn_f32_few_kernelILi64E", {"": 256}),                        # two
])
def test_registers_leave_room_for_the_workgroups_of_a_unit(kernels, name, registers):
    mine = {k: v for k, v in kernels.items() if re.search(r"^_Z\d+%s" % name, k)}
    assert mine
    for kernel, (vgprs, scratch) in mine.items():
        token = re.search(r"kernelI([tf]?)L", kernel).group(1)
        assert vgprs <= registers[token] and scratch == 0, (kernel, vgprs, scratch)
