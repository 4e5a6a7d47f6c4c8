"""Registers of the built kernels, from the code objects' own metadata.

A SIMD lane has 512 vector registers, handed out by eights, so w wavefronts per
SIMD leave each 512 / w.
"""
import os
import re
import struct
import subprocess

import pytest

import paper_1812_06545_amd as L

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects():
    """The gfx950 code objects bundled in the library, one per translation unit."""
    data = open(os.path.join(os.path.dirname(L.__file__), "libldpc.so"), "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        (entries,) = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(entries):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            triple = data[p + 24:p + 24 + length].decode()
            p += 24 + length
            if "gfx950" in triple and size:
                yield data[at + offset:at + offset + size]
        at = data.find(MAGIC, at + 1)


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled name: (vector registers, spilled ones, spilled scalar registers)}"""
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    out = {}
    folder = tmp_path_factory.mktemp("co")
    for i, co in enumerate(_code_objects()):
        path = folder / f"{i}.co"
        path.write_bytes(co)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for part in re.split(r"\n  - \.agpr_count", notes)[1:]:
            name = re.search(r"\.name:\s+(\S+)", part).group(1)
            out[name] = (int(re.search(r"\.vgpr_count:\s+(\d+)", part).group(1)),
                         int(re.search(r"\.vgpr_spill_count:\s+(\d+)", part).group(1)),
                         int(re.search(r"\.sgpr_spill_count:\s+(\d+)", part).group(1)))
    assert len(out) > 40
    return out


@pytest.mark.parametrize("degree,waves", [(8, 6), (16, 6), (24, 6), (32, 5)])
def test_layered_frames_that_share_a_cu(kernels, degree, waves):
    """The layered FP32 instance whose frames share a CU: its registers allow
    `waves` wavefronts per SIMD, and nothing is spilled inside the layer loop (a
    pair of registers may be, once per frame)."""
    (got,) = [v for k, v in kernels.items() if f"k_fusedINS_8ArithF32ELi{degree}ELNS0_8InstanceE2ELb0E" in k]
    assert got[0] <= 512 // waves // 8 * 8 and got[1] <= 2, got


def test_check_kernel_of_rows_up_to_16(kernels):
    """Its registers allow 6 wavefronts per SIMD, with and without early stop."""
    got = [v for k, v in kernels.items() if "flood7k_checkINS_8ArithF32ELi16E" in k]
    assert len(got) == 4 and all(v <= 80 and spilled == 0 for v, spilled, _ in got), got


def test_check_kernel_of_long_rows(kernels):
    """Rows of 33 to 64 edges in FP32 (whose guards alone spill some 200 scalar
    registers): no sign masks beside them."""
    got = [v for k, v in kernels.items() if "flood7k_checkINS_8ArithF32ELi64E" in k]
    assert len(got) == 4 and all(scalars < 250 for _, _, scalars in got), got


def test_check_kernel_with_early_stop(kernels):
    """Rows of up to 32 edges: the sign masks stay in scalar registers."""
    got = [v for k, v in kernels.items() for d in (8, 16, 24, 32) if f"flood7k_checkINS_8ArithF32ELi{d}E" in k]
    assert len(got) == 16 and all(scalars < 10 for _, _, scalars in got), got
