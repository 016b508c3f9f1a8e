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
        run.allocations = int(res.stderr.split()[-1])   # of the library in these calls
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


# (group_rows, d, k, dtype) of every representation the decode side takes
DECODE_FORMATS = [(8, 2, 16, vq.VQ_F16), (8, 2, 256, vq.VQ_F16), (4, 2, 16, vq.VQ_I8), (8, 2, 16, vq.VQ_I8), (8, 2, 32, vq.VQ_I8),
                  (8, 1, 16, vq.VQ_F16), (1, 1, 4, vq.VQ_I8), (8, 2, 16, vq.VQ_I8_BN)]
DECODE_FORMATS += [(gr, 2, 64, t) for gr in (8, 16, 32) for t in (vq.VQ_I8, vq.VQ_I8_BN)]
DECODE_FORMATS += [(gr, 1, 8, t) for gr in (8, 16, 32) for t in (vq.VQ_I8, vq.VQ_I8_BN)]
DECODE_FORMATS += [(gr, 2, 256, t) for gr in (64, 128, 256) for t in (vq.VQ_I8, vq.VQ_I8_BN)]
DECODE_FORMATS += [(gr, 4, 256, t) for gr in (64, 128, 256) for t in (vq.VQ_I8, vq.VQ_I8_BN, vq.VQ_F16)]


def test_batched_product_divides_by_no_zero(launches):
    """The batched kernels divide row-blocks by the number that share a codebook: at least 1 in every
    format, also where a codebook covers one or four rows only."""
    sizes = [(256, 512, 3), (256, 2560, 40), (4096, 1024, 96), (11008, 512, 2048)]
    calls = [("gemm", out // gr * gr, inp, gr, d, k, t, B) for gr, d, k, t in DECODE_FORMATS for out, inp, B in sizes]
    where = {"gemm_tiny_kernel": 2, "gemm_small_kernel": 3, "gemm_kernel": 3}
    seen = set()
    for call, (status, ls) in zip(calls, launches(calls)):
        assert status == 0 and ls, call
        for name, _, _, ints in ls:
            kernel = next(n for n in where if n in name)
            seen.add(kernel)
            assert ints[0] == call[1] // 8 and ints[1] == call[2] // 256, (call, name, ints)   # n_rb, n_cb: the right arguments
            assert ints[where[kernel]] == max(1, call[3] // 8), (call, name, ints)
    assert seen == set(where)


# (format, rows, columns, B, kernel): which tiles a batched product takes, on both sides of the rule (256 CUs); the
# times behind it are at the rule
K16, K64, K256 = (8, 2, 16, vq.VQ_F16), (32, 2, 64, vq.VQ_I8), (8, 2, 256, vq.VQ_F16)
K64_BN, K256_BN, D4, D4_F16 = (32, 2, 64, vq.VQ_I8_BN), (64, 2, 256, vq.VQ_I8_BN), (64, 4, 256, vq.VQ_I8), (64, 4, 256, vq.VQ_F16)
TILES = [
    (K64, 11008, 4096, 16, "tiny"), (K64, 4096, 4096, 32, "tiny"), (K64, 5120, 11008, 17, "tiny"), (K64, 6144, 4096, 32, "tiny"),
    (K64, 6176, 4096, 32, "small"), (K16, 5120, 4096, 24, "tiny"), (K256, 5120, 11008, 32, "small"), (K256, 4224, 2048, 17, "tiny"),
    (D4, 5120, 2048, 24, "small"), ((128, 4, 256, vq.VQ_I8), 4224, 11008, 17, "tiny"), (D4_F16, 4160, 4096, 32, "small"),
    (K64_BN, 4160, 1024, 32, "small"), (K64_BN, 4160, 4096, 17, "tiny"), (K256_BN, 6144, 2048, 32, "small"), (K256_BN, 4160, 11008, 17, "tiny"),
    (K64, 2048, 4096, 64, "tiny"), (K64, 2048, 4096, 96, "small"), (D4_F16, 1024, 1024, 64, "small"), (D4_F16, 512, 4096, 64, "tiny"),
    (D4_F16, 1024, 11008, 64, "tiny"), (K256, 2560, 4096, 48, "tiny"), (K256, 1024, 4096, 128, "small"),
    (K16, 256, 4096, 512, "small"), (K64_BN, 256, 4096, 512, "tiny"), (K16, 1024, 1024, 128, "small"), (K16, 1024, 1024, 80, "tiny"),
    (K64, 1024, 1024, 96, "tiny"), (K16, 2048, 1024, 48, "tiny"), (D4, 1024, 1024, 128, "tiny"),
]


def test_batched_product_takes_the_faster_tiles(launches):
    calls = [("gemm", out, inp, *fmt, B) for fmt, out, inp, B, _ in TILES]
    calls += [("gemm", out, inp, *fmt, B, 1, 128) for fmt, out, inp, B, _ in TILES[1:2]]     # half the CUs: twice the rounds
    got = [ls[0][0] for _, ls in launches(calls)]
    wrong = [(t, name) for t, name in zip(TILES, got) if "gemm_" + t[4] not in name]
    assert wrong == []
    assert "gemm_small" in got[-1]


# (format, rows of the products, columns, CUs, workgroups per 64 rows): on both sides of the lines of the rule
K256_I8, D4_BN = (64, 2, 256, vq.VQ_I8), (64, 4, 256, vq.VQ_I8_BN)
WIDE = [
    (D4, [4096], [8192], 256, 8), (D4, [4160], [8192], 256, 4), (D4_F16, [2048], [8192], 256, 8), (D4_F16, [4096], [8192], 256, 4),
    (D4_F16, [1024] * 3 + [64], [256] * 3 + [11008], 256, 8), (D4_F16, [11008, 1024], [256, 11008], 256, 4),
    (K256_I8, [28672], [2048], 256, 2), (K256_I8, [28672], [4096], 256, 1), (K256_I8, [4096], [8192], 256, 8), (K256_I8, [4160], [8192], 256, 4),
    (D4, [4096], [7680], 256, 4), (D4, [8192], [1024], 256, 2), (D4, [8256], [1024], 256, 1), (K256_I8, [12288], [1024], 256, 1), (K256_I8, [20480], [1024], 256, 2),
    (D4, [8192], [512], 256, 1), (D4, [64], [512], 256, 1), (D4, [64], [768], 256, 2), (D4, [8192], [2048], 256, 4),
    (D4, [12288], [4096], 256, 4), (D4_BN, [12288], [4096], 256, 4), (D4_F16, [12288], [4096], 256, 2), (K256_I8, [12288], [2048], 256, 4),
    (D4, [12288], [2048], 256, 1), (D4, [12352], [4096], 256, 2), (D4, [16384], [2048], 256, 1), (K256_I8, [12352], [4096], 256, 2),
    (D4, [16448], [2048], 256, 2), (D4, [20480], [1024], 256, 1), (D4_F16, [20480], [4096], 256, 1), (D4_F16, [20480], [8192], 256, 2),
    (D4, [24576], [4096], 256, 2), (D4, [24640], [4096], 256, 1), (K256_I8, [24640], [4096], 256, 1), (K256_I8, [32768], [8192], 256, 2),
    (K256_I8, [32832], [8192], 256, 1), (D4, [4096, 4096], [256, 8448], 256, 4), (D4, [1024] * 5, [4096] * 5, 256, 1),
    (D4, [24576], [4096], 128, 1), (D4, [4864], [8192], 304, 8),      # counted against the CUs of the device
]


def test_wide_gemv_splits(launches):
    calls = [("gemv", outs, ins, *fmt, 1, 1, cus) for fmt, outs, ins, cus, _ in WIDE]
    got = launches(calls)
    wrong = [(w, ls[0][1][0]) for w, (st, ls) in zip(WIDE, got)
             if st != 0 or len(ls) != 1 or ls[0][1][0] != sum(w[1]) // 64 * w[4] or f"Li{w[4]}E" not in ls[0][0]]
    assert wrong == []


def test_neighbouring_items_on_one_xcd(launches):
    """The order of workgroups that lets 64-row items share their tables in an L2: unsplit launches of d = 4 whose groups have 256
    rows, but for short launches of up to 2048 columns (times at the rule); no variant of any other kernel."""
    def d4(rows, dtype=vq.VQ_I8):
        return (rows, 4, 256, dtype)
    cases = [(d4(256), [32768], [2304], True), (d4(256), [32768], [2048], False), (d4(256), [33024], [2048], True),
             (d4(128), [32768], [4096], False), (d4(64), [32768], [4096], False), (d4(256), [4096], [4096], False),   # (the last is split)
             (d4(256), [1024] * 5, [4096] * 5, True), (d4(128), [1024] * 5, [4096] * 5, False), (d4(256), [1024] * 5, [1024] * 5, False),
             (d4(256, vq.VQ_F16), [32000], [4096], True), (d4(256, vq.VQ_I8_BN), [32000], [4096], True),
             ((256, 2, 256, vq.VQ_I8), [32000], [4096], False), ((256, 2, 256, vq.VQ_I8_BN), [11008] * 5, [4096] * 5, False)]
    for op in ("gemv", "lora"):
        got = launches([(op, outs, ins, *fmt) for fmt, outs, ins, _ in cases])
        assert [(st, ls[-1][0].split("EEEv")[0].endswith("Lb1")) for st, ls in got] == [(0, want) for *_, want in cases]


def test_no_call_allocates(launches):
    """Many products, of widths in any order (the tall-group formats start the widest first), with and without adapters."""
    widths = [256, 2304, 768, 2304, 512, 1280, 4096] * 30
    fmts = [K16, K64, K64_BN, K256, D4, D4_F16, D4_BN, K256_I8, K256_BN]
    calls = [(op, [1024] * len(w), w, *fmt) for fmt in fmts for op in ("gemv", "lora") for w in (widths, sorted(widths), sorted(widths)[::-1])]
    calls += [(op, 4096, 2304, *fmt, 40) for fmt in fmts for op in ("gemm", "pack")]
    calls += [(op, 4096, 2304, gr, d, k, vq.VQ_F16) for gr, d, k in ((8, 2, 16), (64, 4, 256), (256, 4, 256), (8, 1, 8)) for op in ("assign", "update")]
    assert all(st == 0 and ls for st, ls in launches(calls))
    assert launches.allocations == 0


@pytest.mark.parametrize("fmt", [K16, K64, (8, 2, 32, vq.VQ_I8), (1, 1, 4, vq.VQ_I8)], ids=str)
def test_gemv_argument_goes_by_the_number_of_products(launches, fmt):
    """A call of a few products is bound by the host, which copies the kernel's argument: one line of 64 bytes for a single
    product, over a grid of one dimension; four lines for up to four, a grid row each; the whole table beyond."""
    got = launches([("gemv", 1056, 2304, *fmt, 1, n) for n in (1, 2, 4, 5)] + [("gemv", [32, 1056], [512, 512], *fmt)])
    for n, (status, ls) in zip((1, 2, 4, 5, 2), got):
        assert status == 0 and len(ls) == 1
        name, grid = ls[0][:2]
        cap = 1 if n == 1 else 4 if n <= 4 else 256
        assert "gemv_split_kernel" in name and f"Li{cap}EE" in name, name
        assert grid[1:] == (n if cap == 4 else 1, 1)


@pytest.mark.parametrize("fmt", [K64, K64_BN, (8, 2, 64, vq.VQ_I8_BN), (8, 1, 8, vq.VQ_I8), (8, 1, 8, vq.VQ_I8_BN)], ids=str)
def test_re_layout_of_the_6_bit_formats_keeps_to_the_size_of_a_launch(launches, fmt):
    """A launch takes fewer than 2^32 threads; matrices that fit the memory (2^28 rows x 256 columns: 160 GB in all with
    block scales) are re-packed in several.  Workgroups: 4 (8-row block, quad)s of indices or of table records (256
    records with d = 1), 8 of block codes."""
    rows = 2 ** 28
    slots, tables = rows // 8, rows // fmt[0]
    want = slots // 4 + (tables // 256 if fmt[1] == 1 else tables // 4) + (slots // 8 if fmt[3] == vq.VQ_I8_BN else 0)
    (status, ls), (status1, ls1) = launches([("pack", rows, 256, *fmt), ("pack", 4096, 11008, *fmt)])
    assert status == 0 and sum(l[1][0] for l in ls) == want
    assert all(l[1][0] * l[2] < 2 ** 32 for l in ls)
    assert status1 == 0 and len(ls1) == 1


@pytest.mark.parametrize("shape", [(8, 2, 256), (16, 4, 64), (256, 4, 256)], ids=str)
def test_e_step_keeps_to_the_size_of_a_launch(launches, shape):
    """A launch takes fewer than 2^32 threads; larger matrices (fp32 weights up to the size of the memory) go in several."""
    gr, d, k = shape
    (status, ls), = launches([("assign", 2 ** 19 + 256, 65536, gr, d, k, vq.VQ_F16)])
    assert status == 0
    assert all(l[1][0] * l[2] < 2 ** 32 for l in ls)
    strip = min(gr, 32)
    assert sum(l[1][0] for l in ls) == (2 ** 19 + 256) // strip * 256


def test_e_step_strips(launches):
    """Rows of a workgroup of the filtered E-step, by the number of blocks of 8 x 256 weights and the height of the groups
    (256 CUs, and 128)."""
    table = [(2, 64, 32, 2032, 8), (2, 256, 128, 2048, 16), (2, 64, 16, 8192, 16), (2, 64, 32, 4080, 16), (2, 256, 32, 4096, 32), (2, 64, 8, 4096, 8),
             (4, 64, 16, 1008, 8), (4, 64, 16, 1024, 16), (4, 256, 256, 3040, 16), (4, 256, 64, 3072, 32), (4, 256, 8, 8192, 8), (4, 64, 16, 8192, 16)]
    calls = [("assign", blocks * 8, 256, gr, d, k, vq.VQ_F16) for d, k, gr, blocks, _ in table]
    calls += [("assign", blocks * 4, 256, gr, d, k, vq.VQ_F16, 1, 1, 128) for d, k, gr, blocks, _ in table if blocks * 4 % gr == 0]
    want = [8 * b // rows for _, _, _, b, rows in table] + [4 * b // rows for _, _, gr, b, rows in table if b * 4 % gr == 0]
    got = launches(calls)
    assert [(st, len(ls), ls[0][1]) for st, ls in got] == [(0, 1, (n, 1, 1)) for n in want]


def test_e_step_rows_of_a_wave(launches):
    """Without the filter a wave takes 2 rows in launches of few blocks (a workgroup to a block), else 8."""
    most = {(1, 4): 5, (1, 8): 6, (1, 16): 8, (1, 64): 8, (1, 256): 8, (2, 4): 5, (2, 8): 6, (2, 16): 6, (2, 32): 6, (4, 4): 5, (4, 16): 6, (4, 32): 6}
    calls, want = [], []
    for (d, k), per_cu in most.items():
        for cus in (256, 128):
            for blocks in (per_cu * cus, per_cu * cus + 4):
                calls.append(("assign", blocks * 8, 256, 8, d, k, vq.VQ_F16, 1, 1, cus))
                want.append(blocks if blocks == per_cu * cus else blocks // 4)
    got = launches(calls)
    assert [(st, len(ls), ls[0][1]) for st, ls in got] == [(0, 1, (n, 1, 1)) for n in want]
    for gr, d, k in ((4, 2, 16), (1, 1, 4)):          # several codebooks to a block: always 8
        (_, ls), = launches([("assign", 64, 256, gr, d, k, vq.VQ_F16)])
        assert ls[0][1][0] == 2


def test_m_step_workgroups_of_a_group(launches):
    """A workgroup per coordinate where there are few groups, else one per group (256 CUs, and 128)."""
    calls, want = [], []
    for (d, k, gr), per_cu in {(2, 256, 64): 1, (2, 64, 128): 1, (2, 256, 256): 1, (2, 64, 32): 2, (2, 256, 16): 2, (4, 64, 16): 2, (4, 256, 64): 2,
                               (4, 256, 256): 2}.items():
        for cus in (256, 128):
            most = per_cu * cus // d
            for groups in (most, most + 1):
                calls.append(("update", groups * gr, 256, gr, d, k, vq.VQ_F16, 1, 1, cus))
                want.append(groups * (d if groups == most else 1))
    got = launches(calls)
    assert [(st, len(ls), ls[0][1]) for st, ls in got] == [(0, 1, (n, 1, 1)) for n in want]


# The kernel of each size of the GPU test of the tiles with k = 256 and fp16 tables (256 CUs): 16 x 16 tiles of so many waves, 32 x 32
# tiles of so many groups of waves, 32 x 128 tiles, then (32-row steps a wave, columns, wave rows) of the large tiles
TILE_KERNELS = ["ring", "small 1", "1 256 2", "2 128 1", "2 512 2", "2 512 2", "1 256 2", "1 256 2", "2 256 2", "2 128 1", "2 256 2", "2 256 1",
                "tiny 16", "tiny 16", "small 2", "small 2", "small 1", "small 1", "ring", "2 512 2 + 2 256 2",
                "2 128 1", "1 256 2", "2 512 2 + 2 256 2"]


def _kernel_of(name):
    import re
    kind, k, rest = re.search(r"(ring_gemm|gemm_tiny|gemm_small|gemm)_kernelILi(\d+)E((?:Li\d+E)*)", name).groups()
    return " ".join({"ring_gemm": ["ring"], "gemm_tiny": ["tiny"], "gemm_small": ["small"], "gemm": []}[kind] + re.findall(r"Li(\d+)E", rest))


def test_tiles_of_the_gpu_test(launches):
    """What the sizes of test_gpu_gemm_tiles.py are there for."""
    from test_gpu_gemm_tiles import SIZES
    got = launches([("gemm", out, inp, *K256, B) for out, inp, B in SIZES])
    assert [(st, " + ".join(_kernel_of(l[0]) for l in ls)) for st, ls in got] == [(0, t) for t in TILE_KERNELS]
    assert set(sum((t.split(" + ") for t in TILE_KERNELS), [])) == {"ring", "small 1", "small 2", "tiny 16", "2 128 1", "2 256 1", "1 256 2", "2 256 2", "2 512 2"}
    wide = [(out, inp, B) for (out, inp, B), t in zip(SIZES, TILE_KERNELS) if "512" in t.split()[1:2]]
    for fmt in (K64_BN, K256_BN):       # block scales: no 512-column tiles; 16 x 16 tiles of 8 waves
        for out, inp, B in wide + [(1088, 2304, 16)]:
            (_, ls), = launches([("gemm", out, inp, *fmt, B)])
            assert all(_kernel_of(l[0]).split()[:2] != ["2", "512"] and _kernel_of(l[0]) != "tiny 16" for l in ls)


# (format, rows, columns, B, kernels): the large tiles on both sides of a round of workgroups; the times are at the rule
LARGE = [
    (K256, 4096, 4096, 512, "2 128 1"), (K256, 4160, 4096, 512, "1 256 2"), (K256, 8192, 4096, 256, "2 128 1"), (K256, 8256, 4096, 256, "1 256 2"),
    (K256, 11008, 4096, 203, "1 256 2"), (K256, 11008, 4096, 400, "2 256 2"), ((16, 1, 8, vq.VQ_I8), 11424, 8192, 350, "2 256 2"),
    ((8, 2, 32, vq.VQ_I8), 8192, 5120, 1513, "2 512 2"), (K256, 11008, 4096, 2048, "2 512 2 + 2 256 2"), (K64, 16384, 4096, 256, "1 256 2"),
    (K64, 16416, 4096, 256, "2 256 2"), (K64_BN, 8192, 8192, 1350, "2 256 1"), (K64_BN, 4928, 7424, 787, "2 256 2"), (K64_BN, 8096, 1536, 1131, "2 256 1"),
    (D4_F16, 13824, 1024, 140, "2 128 1"), (D4_F16, 13824, 2048, 140, "2 128 1"), (D4_F16, 13824, 11008, 140, "1 256 2"), (D4_F16, 4864, 1536, 2197, "2 512 2"),
]


def test_batched_product_takes_the_faster_large_tiles(launches):
    got = launches([("gemm", out, inp, *fmt, B) for fmt, out, inp, B, _ in LARGE])
    wrong = [(t, ls) for t, (st, ls) in zip(LARGE, got) if st != 0 or " + ".join(_kernel_of(l[0]) for l in ls) != t[4]]
    assert wrong == []
    (_, ls), = launches([("gemm", 4128, 4096, *K256, 256, 1, 128)])     # half the CUs: half the rows
    assert _kernel_of(ls[0][0]) == "1 256 2"


def test_tiles_of_an_xcd(launches):
    """With more columns than rows an XCD takes whole column tiles, else whole tile rows."""
    sizes = [(1024, 512, 1024, 0), (1024, 512, 1025, 1), (576, 768, 4601, 1), (11072, 256, 203, 0), (800, 512, 1000, 1), (15424, 2048, 1090, 0)]
    got = launches([("gemm", out, inp, *K256, B) for out, inp, B, _ in sizes])
    assert [f"Lb{by}E" in ls[0][0] for (_, _, _, by), (_, ls) in zip(sizes, got)] == [True] * len(sizes)


def test_waves_of_the_16_x_16_tiles(launches):
    """16 from nine col-blocks on in the formats that have the registers, but not where the 6-bit layouts would have two
    col-blocks to nearly every wave; 8 else, and 4 beyond a workgroup per CU or up to four col-blocks."""
    d1_k8, k16_i8 = (32, 1, 8, vq.VQ_I8), (8, 2, 16, vq.VQ_I8)
    table = [(K64, 9, 16), (K64, 8, 8), (K64, 24, 16), (K64, 25, 8), (K64, 34, 8), (K64, 35, 16), (K64, 43, 16), (K64, 4, 4), (d1_k8, 32, 8), (d1_k8, 36, 16),
             (K256, 32, 16), (K16, 32, 16), (k16_i8, 28, 16), (K64_BN, 32, 8), (K64_BN, 8, 4), (K64_BN, 9, 8), (K256_BN, 16, 8), (D4, 16, 8)]
    got = launches([("gemm", 2048, n_cb * 256, *fmt, 16) for fmt, n_cb, _ in table] + [("gemm", 4160, 2560, *K64, 16)])
    want = [waves for _, _, waves in table] + [4]
    assert [_kernel_of(ls[0][0]) for _, ls in got] == [f"tiny {w}" for w in want]


def test_groups_of_waves_of_the_32_x_32_tiles(launches):
    """Two where a CU has one workgroup and the steps rounded up to four a group are at most a fifth more (a tenth: k = 256)."""
    table = [(K64, 8, 2), (K64, 9, 1), (K64, 12, 1), (K64, 13, 2), (K64, 17, 2), (K64, 28, 2), (K64, 7, 1), (K256, 8, 2), (K256, 9, 1), (K256, 16, 2),
             (K256, 17, 1), (K256, 20, 1), (K256, 21, 2), (K256, 28, 1), (K256, 32, 2), (K256, 36, 1), (K256, 43, 2), (D4_F16, 16, 1)]
    got = launches([("gemm", 2048, n_cb * 256, *fmt, 100) for fmt, n_cb, _ in table] + [("gemm", 2048, 4096, *K64, 130)])
    assert [_kernel_of(ls[0][0]) for _, ls in got] == [f"small {g}" for _, _, g in table] + ["small 1"]
