"""What the library launches, seen from a stand-in for the HIP runtime (tests/host/launch_recorder.cpp): which kernel,
over which grid, with which integer arguments.  No GPU needed; the built libvq.so is what is tested."""
import itertools
import os
import shutil
import subprocess

import pytest

import paper_2402_15319_amd as vq
from paper_2402_15319_amd import build as vqbuild

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BITS = {4: 2, 8: 3, 16: 4, 32: 5, 64: 6, 256: 8}
pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime_api.h"),
                                reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    """f([(op, out, in, group_rows, d, k, dtype, B, count, cus), ..]) -> [(status, [(kernel, (gx, gy, gz), threads,
    [integers]), ..]), ..]; out and in may be lists (gemv)."""
    vq.lib()   # builds nothing: fails if the library is missing
    exe = tmp_path_factory.mktemp("launch") / "launch_recorder"
    cmd = ["g++", "-std=c++17", "-O1", "-rdynamic", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           os.path.join(ROOT, "tests", "host", "launch_recorder.cpp"), vqbuild.LIB_PATH,
           "-Wl,-rpath," + os.path.dirname(vqbuild.LIB_PATH), "-Wl,-rpath,/opt/rocm/lib", "-L/opt/rocm/lib", "-lamdhip64", "-o", str(exe)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]

    def run(calls):
        def line(op, out, inp, gr, d, k, dtype, B=1, count=1, cus=256):
            outs, ins = ("+".join(str(v) for v in (t if isinstance(t, (list, tuple)) else [t])) for t in (out, inp))
            return f"{op} {outs} {ins} {gr} {d} {k} {BITS[k]} {dtype} {B} {count} {cus}"
        text = "\n".join(line(*c) for c in calls) + "\n"
        res = subprocess.run([str(exe)], input=text, capture_output=True, text=True, timeout=300)
        assert res.returncode == 0, res.stderr[-2000:]
        out = []
        for ln in res.stdout.splitlines():
            status, *ls = [p.strip() for p in ln.split(" ; ")]
            parsed = []
            for l in ls:
                name, gx, gy, gz, threads, *ints = l.split()
                parsed.append((name, (int(gx), int(gy), int(gz)), int(threads), [int(i) for i in ints]))
            out.append((int(status), parsed))
        assert len(out) == len(calls)
        return out
    return run


def _em_shapes():
    """Every (k, d, group_rows) the two EM steps accept, as their descriptor rules are documented."""
    return [(k, d, gr) for k, d, gr in itertools.product(BITS, (1, 2, 4), (1, 4, 8, 16, 32, 64, 128, 256))
            if not (gr == 1 and k * d > 64) and not (gr == 4 and d == 4)]


@pytest.mark.parametrize("op", ["assign", "update"])
def test_every_accepted_em_shape_launches_one_kernel(launches, op):
    """A step that reports success without a launch would leave the caller's buffer as it was."""
    shapes = _em_shapes()
    got = launches([(op, max(gr, 8) * 3, 512, gr, d, k, vq.VQ_F16) for k, d, gr in shapes])
    bad = [(s, st, len(ls)) for s, (st, ls) in zip(shapes, got) if st != 0 or len(ls) != 1]
    assert bad == []
