"""What the compiler made of kernels whose speed depends on it, from the metadata of the built library."""
import os
import re
import struct
import subprocess

import pytest

from paper_1905_10830_amd import binding as fmtc

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def scratch_bytes(tmp_path_factory):
    """{kernel name: bytes of scratch memory per lane}"""
    if not os.path.exists(fmtc.LIB_PATH):
        from paper_1905_10830_amd import build

        build.build()
    tmp = tmp_path_factory.mktemp("code")
    fat = str(tmp / "fatbin")
    subprocess.run([f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", fmtc.LIB_PATH, str(tmp / "copy.so")], check=True)
    data, out = open(fat, "rb").read(), {}
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        n, at = struct.unpack_from("<Q", data, m.end())[0], m.end() + 8
        for _ in range(n):
            offset, size, id_len = struct.unpack_from("<QQQ", data, at)
            target, at = data[at + 24:at + 24 + id_len], at + 24 + id_len
            if b"gfx950" not in target or not size:
                continue
            obj = str(tmp / "code.o")
            open(obj, "wb").write(data[m.start() + offset:m.start() + offset + size])
            notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", obj], check=True, capture_output=True, text=True).stdout
            names = re.findall(r"\.name:\s+(_Z\S+)", notes)
            scratch = re.findall(r"\.private_segment_fixed_size:\s*(\d+)", notes)
            assert len(names) == len(scratch)
            out.update(zip(names, map(int, scratch)))
    return out


def test_packer_of_large_tensors_keeps_nothing_on_the_stack(scratch_bytes):
    """(A copy of the container's header on the stack, filled by every lane, was 9.4 MB of writes per launch.)"""
    packers = {k: v for k, v in scratch_bytes.items() if "k_pack_stream" in k}
    assert len(packers) == 4 and not any(packers.values()), packers


def test_projection_of_planar_tensors_keeps_no_addresses_on_the_stack(scratch_bytes):
    """(Channel counts that are no multiple of 16: reloaded for every tile, they took a third of the kernel's time.)"""
    rows = {k: v for k, v in scratch_bytes.items() if re.search(r"rowsILi[124]ELi0ELb0E", k)}  # coefficient tiles, planar, masked loads
    assert len(rows) == 3 and not any(rows.values()), rows
