"""Registers of the compiled kernels where a rule of the host counts on them (no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2402_15319_amd import build as vqbuild

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not available")


@pytest.fixture(scope="module")
def resources(tmp_path_factory):
    """f(source) -> {kernel: (vector registers, bytes of scratch per lane)}"""
    def of(source):
        out = tmp_path_factory.mktemp("regs") / "kernels.s"
        cmd = [HIPCC, *[f for f in vqbuild.HIPCC_FLAGS if f != "-fPIC"], "-S", "--cuda-device-only", "-o", str(out), os.path.join(vqbuild.CSRC, source)]
        res = subprocess.run(cmd, capture_output=True, text=True)
        assert res.returncode == 0, res.stderr[-2000:]
        found = {}
        for m in re.finditer(r"\.amdhsa_kernel (\S+)\n(.*?)\.end_amdhsa_kernel", out.read_text(), re.S):
            value = lambda key: int(re.search(rf"\.amdhsa_{key} (\d+)", m[2])[1])
            found[m[1]] = (value("next_free_vgpr"), value("private_segment_fixed_size"))
        assert found
        return found
    return of


def test_wide_group_products(resources):
    """Kernels of the formats whose tables 64 or more rows share: none spills, and with four workgroups of 8 waves to 64 rows three
    of them fit a CU (6 waves per SIMD: 80 registers of 512), which the number of workgroups per 64 rows counts on up to
    192 items on 256 CUs.  With block scales and an adapter: two."""
    kernels = resources("vq_gemv_d4.hip")
    assert {n: r for n, r in kernels.items() if r[1] != 0} == {}
    four = {n: r[0] for n, r in kernels.items() if re.search(r"Li4ELi4EE", n)}
    assert len(four) == 2 * 2 + 2 * 3
    both = re.compile(r"gemv_k256i8_kernelILb1ELb1E")
    assert {n: r for n, r in four.items() if r > (96 if both.search(n) else 80)} == {}
