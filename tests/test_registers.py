"""Registers of the compiled kernels where a rule of the host counts on them (no GPU needed): the metadata of the
kernels in the built libvq.so."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2402_15319_amd import build as vqbuild

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
pytestmark = pytest.mark.skipif(not os.path.exists(READELF), reason="needs llvm-readelf")


@pytest.fixture(scope="module")
def resources(tmp_path_factory):
    """{kernel: (vector registers, bytes of scratch per lane)}"""
    with open(vqbuild.LIB_PATH, "rb") as f:
        lib = f.read()
    magic, found = b"__CLANG_OFFLOAD_BUNDLE__", {}
    for m in re.finditer(re.escape(magic), lib):       # one bundle per source: count, then offset, size and name of each part
        at = m.end()
        count, = struct.unpack_from("<Q", lib, at)
        at += 8
        for _ in range(count):
            offset, size, name_len = struct.unpack_from("<QQQ", lib, at)
            name = lib[at + 24:at + 24 + name_len].decode()
            at += 24 + name_len
            if not name.endswith("gfx950"):
                continue
            part = tmp_path_factory.mktemp("code") / "part.elf"
            part.write_bytes(lib[m.start() + offset:m.start() + offset + size])
            res = subprocess.run([READELF, "--notes", str(part)], capture_output=True, text=True)
            assert res.returncode == 0, res.stderr[-2000:]
            for k in re.split(r"\n  - (?=\.)", res.stdout)[1:]:
                value = lambda key: re.search(rf"^ *\.{key}: +(\S+)", k, re.M)[1]
                found[value("symbol").removesuffix(".kd")] = (int(value("vgpr_count")), int(value("private_segment_fixed_size")))
    assert found
    return found


def test_wide_group_products(resources):
    """Kernels of the formats whose tables 64 or more rows share: none spills, and with four workgroups of 8 waves to 64 rows three
    of them fit a CU (6 waves per SIMD: 80 registers of 512), which the number of workgroups per 64 rows counts on up to
    192 items on 256 CUs.  With block scales and an adapter: two."""
    kernels = {n: r for n, r in resources.items() if "gemv_d4_kernel" in n or "gemv_k256i8_kernel" in n}
    assert {n: r for n, r in kernels.items() if r[1] != 0} == {}
    four = {n: r[0] for n, r in kernels.items() if re.search(r"Li4ELi4ELb0EE", n)}
    assert len(four) == 2 * 2 + 2 * 3
    both = re.compile(r"gemv_k256i8_kernelILb1ELb1E")
    assert {n: r for n, r in four.items() if r > (96 if both.search(n) else 80)} == {}


def test_m_step(resources):
    """The M-step of tall d = 4 groups spills nothing and leaves room for three workgroups of 8 waves on a CU; that of d = 1
    with many centroids for seven waves per SIMD (72 registers)."""
    counted = [r for n, r in resources.items() if "em_update_counted_kernel" in n]
    assert len(counted) == 1 and counted[0][0] <= 80 and counted[0][1] == 0
    small = [r for n, r in resources.items() if re.search(r"em_update_kernelILi(64|256)ELi1ELi1ELi1ELi1ELi0EE", n)]
    assert small == [(72, 0), (72, 0)]
