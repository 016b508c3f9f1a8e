"""GPU parity of the quantiser kernels (E- and M-step of the Hessian-weighted EM) against the
CPU oracle, through the C ABI.  Assignments are compared bit for bit (both sides take the
decision in binary32 with the same operation order); centroids within the bound derived from
binary32 summation of at most 1,024 terms."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2402_15319_amd as vq
    from paper_2402_15319_amd import device as vqdev
    assert torch.cuda.is_available()
    vq.lib()
    return torch, vq, vqdev


def _inputs(out_f, in_f, k, seed, from_data=False):
    """Seeded synthetic quantiser inputs: N(0, 0.02) weights, column weights 1/[H^-1]_cc spread
    over a factor of 25, and a starting codebook (random, or k vectors drawn from the group)."""
    rng = np.random.default_rng(seed)
    W = rng.normal(0, 0.02, (out_f, in_f)).astype(np.float32)
    h = rng.uniform(0.2, 5.0, in_f).astype(np.float32)
    n_groups = (out_f // 8) * (in_f // 256)
    if from_data:
        cb = np.zeros((n_groups, k, 2), dtype=np.float32)
        n_cb = in_f // 256
        for g in range(n_groups):
            rb, c = divmod(g, n_cb)
            X = W[rb * 8:(rb + 1) * 8, c * 256:(c + 1) * 256].reshape(-1, 2)
            cb[g] = X[rng.choice(X.shape[0], size=k, replace=False)]
    else:
        cb = rng.normal(0, 0.02, (n_groups, k, 2)).astype(np.float32)
    return W, h, cb


def _fmt(out_f, in_f, k):
    return oracle.VQFormat(out_f, in_f, k, {16: 4, 64: 6, 256: 8}[k])


def _desc(vq, out_f, in_f, k):
    return vq.make_desc(out_f, in_f, k, {16: 4, 64: 6, 256: 8}[k])


def _gpu_assign(env, desc, W, h, cb):
    torch, vq, vqdev = env
    a = torch.full((desc.out_features, desc.in_features // 2), 255, dtype=torch.uint8, device="cuda:0")
    vq.vq_em_assign(desc, vqdev.to_device_bytes(W), vqdev.to_device_bytes(h), vqdev.to_device_bytes(cb), a)
    torch.cuda.synchronize()
    return a.cpu().numpy()


def _gpu_update(env, desc, W, h, assign, k):
    torch, vq, vqdev = env
    n_groups = (desc.out_features // 8) * (desc.in_features // 256)
    out = torch.full((n_groups, k, 2), 777.0, dtype=torch.float32, device="cuda:0")
    vq.vq_em_update(desc, vqdev.to_device_bytes(W), vqdev.to_device_bytes(h),
                    vqdev.to_device_bytes(assign.astype(np.uint8)), out)
    torch.cuda.synchronize()
    return out.cpu().numpy()


# several groups, group counts that are not a multiple of the waves of a workgroup (4 for the
# E-step, 2 for the M-step), every codebook size
SHAPES = [(8, 256, 16), (16, 512, 16), (40, 768, 16), (24, 1280, 64), (8, 768, 256), (24, 256, 256)]


@pytest.mark.parametrize("from_data", [False, True], ids=["random_cb", "cb_from_data"])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_e_step_bit_exact(env, shape, from_data):
    out_f, in_f, k = shape
    W, h, cb = _inputs(out_f, in_f, k, 900 + out_f + k, from_data)
    got = _gpu_assign(env, _desc(env[1], out_f, in_f, k), W, h, cb)
    np.testing.assert_array_equal(got, oracle.em_assign(_fmt(out_f, in_f, k), W, h, cb))


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_m_step_within_summation_bound(env, shape):
    """fp32 sequential summation of n <= 1,024 terms is off by at most n * 2^-24 relative to the
    sum of magnitudes, for numerator and denominator each: |error| <= 1.3e-4 * max|W| of the
    group; the test uses 1.5e-4.  Clusters nobody chose must come out as exact zeros."""
    out_f, in_f, k = shape
    # k = 256 starts from random centroids, so that some clusters stay empty
    W, h, cb = _inputs(out_f, in_f, k, 950 + out_f + k, from_data=(k != 256))
    f = _fmt(out_f, in_f, k)
    a = oracle.em_assign(f, W, h, cb)
    got = _gpu_update(env, _desc(env[1], out_f, in_f, k), W, h, a, k)
    want = oracle.em_update(f, W, h, a)
    assert np.abs(got - want).max() <= 1.5e-4 * np.abs(W).max()
    counts = np.zeros((f.n_groups, k), dtype=np.int64)
    n_cb = in_f // 256
    for g in range(f.n_groups):
        rb, c = divmod(g, n_cb)
        counts[g] = np.bincount(a[rb * 8:(rb + 1) * 8, c * 128:(c + 1) * 128].reshape(-1), minlength=k)
    assert np.all(got[counts == 0] == 0.0)
    if k == 256:
        assert (counts == 0).any()        # 1,024 vectors over 256 centroids: the case occurs


def test_tie_and_zero_weight_cases(env):
    """Two centroids at the same weighted distance -> the lower index, on the GPU as in the
    oracle; a column whose weight is zero contributes nothing and gives a zero coordinate."""
    torch, vq, vqdev = env
    out_f, in_f, k = 8, 256, 16
    W = np.ones((out_f, in_f), dtype=np.float32)
    h = np.ones(in_f, dtype=np.float32)
    h[1::2] = 0.0                                    # second coordinate of every vector has no weight
    cb = np.zeros((1, k, 2), dtype=np.float32)
    cb[0, :, 0] = np.array([5, 3, 0, 2, 2, 9, 9, 9, 9, 9, 9, 9, 9, 9, 9, 9], dtype=np.float32)
    cb[0, :, 1] = np.arange(k, dtype=np.float32)     # ignored: weight 0
    desc = _desc(vq, out_f, in_f, k)
    a = _gpu_assign(env, desc, W, h, cb)
    assert np.all(a == 2)                            # |1-0| = |1-2| = 1: index 2 comes before 3 and 4
    np.testing.assert_array_equal(a, oracle.em_assign(_fmt(out_f, in_f, k), W, h, cb))
    new = _gpu_update(env, desc, W, h, a, k)
    np.testing.assert_array_equal(new[0, 2], [1.0, 0.0])
    assert np.all(new[0, np.arange(k) != 2] == 0.0)


def test_em_iterations_track_the_oracle_and_lower_the_objective(env):
    """Five E/M rounds on the GPU: every E-step equals the oracle's on the GPU's own centroids,
    and the objective (evaluated by the oracle in fp64) never increases."""
    out_f, in_f, k = 32, 1024, 16
    W, h, cb = _inputs(out_f, in_f, k, 977, True)
    f = _fmt(out_f, in_f, k)
    desc = _desc(env[1], out_f, in_f, k)
    last = np.inf
    for _ in range(5):
        a = _gpu_assign(env, desc, W, h, cb)
        np.testing.assert_array_equal(a, oracle.em_assign(f, W, h, cb))
        obj_e = oracle.em_objective(f, W, h, cb, a)
        assert obj_e <= last * (1 + 1e-6)
        cb = _gpu_update(env, desc, W, h, a, k)
        last = oracle.em_objective(f, W, h, cb, a)
        assert last <= obj_e * (1 + 1e-6)


def test_full_size_layer(env):
    """4096 x 4096, k = 16 (8,192 groups), in the launch configuration the bench times: the
    E-step compared in full, the M-step on 64 sampled groups."""
    out_f, in_f, k = 4096, 4096, 16
    W, h, cb = _inputs(out_f, in_f, k, 990)
    f = _fmt(out_f, in_f, k)
    desc = _desc(env[1], out_f, in_f, k)
    a = _gpu_assign(env, desc, W, h, cb)
    np.testing.assert_array_equal(a, oracle.em_assign(f, W, h, cb))
    new = _gpu_update(env, desc, W, h, a, k)
    rng = np.random.default_rng(3)
    for g in rng.choice(f.n_groups, size=64, replace=False):
        rb, c = divmod(int(g), in_f // 256)
        sub = oracle.VQFormat(8, 256, k, 4)
        want = oracle.em_update(sub, W[rb * 8:(rb + 1) * 8, c * 256:(c + 1) * 256], h[c * 256:(c + 1) * 256],
                                a[rb * 8:(rb + 1) * 8, c * 128:(c + 1) * 128])
        assert np.abs(new[g] - want[0]).max() <= 1.5e-4 * np.abs(W).max()


# ---------------------------------------------------------------- other dimensionalities and group heights
def _inputs_any(out_f, in_f, k, d, group_rows, seed, from_data=True):
    rng = np.random.default_rng(seed)
    W = rng.normal(0, 0.02, (out_f, in_f)).astype(np.float32)
    h = rng.uniform(0.2, 5.0, in_f).astype(np.float32)
    n_cb = in_f // 256
    n_groups = (out_f // group_rows) * n_cb
    if from_data:
        cb = np.zeros((n_groups, k, d), dtype=np.float32)
        for g in range(n_groups):
            gr, c = divmod(g, n_cb)
            X = W[gr * group_rows:(gr + 1) * group_rows, c * 256:(c + 1) * 256].reshape(-1, d)
            cb[g] = X[rng.choice(X.shape[0], size=k, replace=X.shape[0] < k)]
    else:
        cb = rng.normal(0, 0.02, (n_groups, k, d)).astype(np.float32)
    return W, h, cb


# (out, in, k, d, group_rows): the group shapes of the decode formats, with block counts that are not
# multiples of the waves of a workgroup
ANY_SHAPES = [
    (8, 256, 16, 1, 8), (40, 768, 16, 1, 8),          # scalar codebooks, 4-bit
    (64, 512, 8, 1, 32), (96, 256, 8, 1, 16),         # 3-bit, 32- and 16-row groups
    (8, 512, 4, 1, 1), (24, 768, 4, 1, 1),            # 2-bit, a codebook per row
    (64, 512, 64, 2, 32), (48, 256, 64, 2, 16),       # d = 2 with taller groups
    (256, 512, 256, 2, 128), (64, 256, 256, 2, 64),
    (128, 512, 256, 4, 64), (256, 256, 256, 4, 256), (256, 768, 256, 4, 128),   # four-dimensional vectors
    (8, 256, 16, 2, 4), (40, 768, 16, 2, 4), (24, 512, 16, 1, 4),   # groups of 4 rows: two codebooks per 8-row block
    (8, 256, 32, 2, 8), (40, 768, 32, 2, 8),          # k = 32 (5-bit indices)
    (16, 256, 16, 4, 8), (8, 256, 4, 2, 1),           # combinations no decode format uses, same kernels
    (8, 256, 32, 2, 1), (24, 512, 64, 1, 1), (16, 256, 16, 4, 1),   # the largest codebooks of one-row groups
]


def _gpu_em_any(env, shape, W, h, cb):
    torch, vq, vqdev = env
    out_f, in_f, k, d, gr = shape
    bits = {4: 2, 8: 3, 16: 4, 32: 5, 64: 6, 256: 8}[k]
    desc = vq.make_desc(out_f, in_f, k, bits, group_rows=gr, d=d)
    a = torch.full((out_f, in_f // d), 255, dtype=torch.uint8, device="cuda:0")
    W_d, h_d = vqdev.to_device_bytes(W), vqdev.to_device_bytes(h)
    vq.vq_em_assign(desc, W_d, h_d, vqdev.to_device_bytes(cb), a)
    new = torch.full(cb.shape, 777.0, dtype=torch.float32, device="cuda:0")
    vq.vq_em_update(desc, W_d, h_d, a, new)
    torch.cuda.synchronize()
    return a.cpu().numpy(), new.cpu().numpy()


@pytest.mark.parametrize("shape", ANY_SHAPES, ids=str)
def test_e_and_m_step_any_dimensionality_and_group_height(env, shape):
    """E-step bit for bit; M-step (on the E-step's own assignments) within the binary32 summation
    bound: a lane sums at most n / 64 terms one after the other, then 64 lane totals are added, so the
    error is at most (n / 64 + 64) * 2^-24 relative to the sum of magnitudes, for numerator and
    denominator each; with weights within a factor 25 of each other that is below
    (n / 64 + 64) * 2^-24 * 2 * 25 * max|W| -- the test uses that bound, which is 1.5e-4 max|W| for the
    8 x 256 groups."""
    out_f, in_f, k, d, gr = shape
    # big codebooks start from random centroids, so that some clusters stay empty
    W, h, cb = _inputs_any(out_f, in_f, k, d, gr, 1200 + out_f + k + d, from_data=(k < 256))
    f = oracle.VQFormat(out_f, in_f, k, 8, gr, 256, d)
    want_a = oracle.em_assign(f, W, h, cb)
    a, new = _gpu_em_any(env, shape, W, h, cb)
    np.testing.assert_array_equal(a, want_a)
    want = oracle.em_update(f, W, h, want_a)
    n = gr * 256 // d
    bound = max(1.5e-4, (n / 64 + 64) * 2.0 ** -24 * 50) * np.abs(W).max()
    assert np.abs(new - want).max() <= bound
    n_cb = in_f // 256
    counts = np.zeros((f.n_groups, k), dtype=np.int64)
    for g in range(f.n_groups):
        gi, c = divmod(g, n_cb)
        counts[g] = np.bincount(want_a[gi * gr:(gi + 1) * gr, c * (256 // d):(c + 1) * (256 // d)].reshape(-1), minlength=k)
    assert np.all(new[counts == 0] == 0.0)


def test_em_rounds_on_a_deployed_group_shape(env):
    """Four E/M rounds with k = 64, 32 x 256 groups (the deployed representation's groups): each
    E-step equals the oracle's on the GPU's own centroids, the objective never rises."""
    shape = (64, 512, 64, 2, 32)
    out_f, in_f, k, d, gr = shape
    W, h, cb = _inputs_any(out_f, in_f, k, d, gr, 1300)
    f = oracle.VQFormat(out_f, in_f, k, 6, gr, 256, d)
    last = np.inf
    for _ in range(4):
        a, new = _gpu_em_any(env, shape, W, h, cb)
        np.testing.assert_array_equal(a, oracle.em_assign(f, W, h, cb))
        obj_e = oracle.em_objective(f, W, h, cb, a)
        assert obj_e <= last * (1 + 1e-6)
        cb = new
        last = oracle.em_objective(f, W, h, cb, a)
        assert last <= obj_e * (1 + 1e-6)


# (out, in, k, d, group_rows): tables per lane (small k * d) and per wave, one wave and several per group, group
# counts that are not multiples of a workgroup's
M_SHAPES = [
    (8, 256, 4, 1, 1), (40, 768, 16, 1, 4), (24, 768, 16, 2, 8), (64, 256, 8, 1, 32),        # a table per lane
    (8, 256, 64, 1, 1), (8, 256, 32, 2, 1), (24, 768, 16, 2, 4), (40, 768, 32, 2, 8), (96, 512, 64, 2, 16),      # a table per wave
    (96, 768, 64, 2, 32), (192, 256, 4, 4, 64), (128, 512, 256, 1, 128), (512, 768, 256, 4, 256),
]


@pytest.mark.parametrize("shape", M_SHAPES, ids=str)
def test_m_step_against_64_bit_sums_and_repeated(env, shape):
    """Bytes beyond the codebook count nowhere, the result is the same on every run, and it is as near
    to 64-bit sums as the kernels' arithmetic allows.  A table per group holds sums in fixed point, n * 2^-46 or
    better of their largest term: numerator, denominator and quotient are rounded once each, 3 * 2^-24 of
    the centroid (3.1 with second-order terms) beside gr * 256 * 2^-53 of the summed magnitudes (an entry of these inputs
    has fewer than 1,000 vectors).  A table per lane adds binary32 products: at most n_lane + 8 roundings of
    2^-24 of the magnitudes, numerator and denominator alike."""
    torch, vq, vqdev = env
    out_f, in_f, k, d, gr = shape
    W, h, cb = _inputs_any(out_f, in_f, k, d, gr, 1400 + out_f + k + d, from_data=False)
    rng = np.random.default_rng(out_f + k)
    assign = rng.integers(0, min(k + k // 4, 256), (out_f, in_f // d)).astype(np.uint8)   # a fifth beyond the codebook
    bits = {4: 2, 8: 3, 16: 4, 32: 5, 64: 6, 256: 8}[k]
    desc = vq.make_desc(out_f, in_f, k, bits, group_rows=gr, d=d)
    W_d, h_d, a_d = (vqdev.to_device_bytes(t) for t in (W, h, assign))
    runs = []
    for _ in range(5):
        new = torch.full(cb.shape, 777.0, dtype=torch.float32, device="cuda:0")
        vq.vq_em_update(desc, W_d, h_d, a_d, new)
        torch.cuda.synchronize()
        runs.append(new.cpu().numpy())
    for r in runs[1:]:
        np.testing.assert_array_equal(r, runs[0])
    n_cb = in_f // 256
    small = {1: 8, 4: 2}.get(gr, 1) * k * d <= 32 and gr <= 32
    for g in range(cb.shape[0]):
        gi, c = divmod(g, n_cb)
        x = W[gi * gr:(gi + 1) * gr, c * 256:(c + 1) * 256].astype(np.float64).reshape(-1, d)
        hv = np.broadcast_to(h[c * 256:(c + 1) * 256].astype(np.float64), (gr, 256)).reshape(-1, d)
        a = assign[gi * gr:(gi + 1) * gr, c * (256 // d):(c + 1) * (256 // d)].reshape(-1)
        for t in range(d):
            num = np.bincount(a, hv[:, t] * x[:, t], 256)[:k]
            mag = np.bincount(a, hv[:, t] * np.abs(x[:, t]), 256)[:k]
            den = np.bincount(a, hv[:, t], 256)[:k]
            safe = np.where(den != 0, den, 1)
            want = np.where(den != 0, num / safe, 0)
            per_lane = (gr * 4 // d + 8) * 2.0 ** -24 if small else gr * 256 * 2.0 ** -53
            bound = 3.1 * 2.0 ** -24 * np.abs(want) + 2.1 * per_lane * mag / safe
            assert np.all(np.abs(runs[0][g, :, t] - want) <= bound)


@pytest.mark.parametrize("rows", [128, 256])
def test_m_step_by_counts_at_full_positions_and_infinite_weights(env, rows):
    """Tall groups with d = 4, k = 256: every row's vector of a position in one centroid (counts up to the
    number of rows, both halves of a counter), and weights that are infinite or NaN count for the
    centroids that use them alone.  Powers of two and small integers: every sum is exact, so is the quotient
    of equal weights."""
    torch, vq, vqdev = env
    out_f, in_f, k, d = rows, 512, 256, 4
    W = np.broadcast_to(np.arange(in_f, dtype=np.float32) - 200, (out_f, in_f)).copy()
    h = np.ones(in_f, np.float32)
    h[4:8], h[132:136], h[300] = np.inf, np.nan, np.inf
    assign = np.broadcast_to(np.arange(in_f // d, dtype=np.uint8) % 64, (out_f, in_f // d)).copy()
    assign[:, 20] = 19                             # lower half: two positions in one centroid
    assign[:, 50] = 19                             # and one of the upper half
    desc = vq.make_desc(out_f, in_f, k, 8, group_rows=rows, d=d)
    new = torch.full((2, k, d), 777.0, dtype=torch.float32, device="cuda:0")
    vq.vq_em_update(desc, vqdev.to_device_bytes(W), vqdev.to_device_bytes(h), vqdev.to_device_bytes(assign), new)
    got = new.cpu().numpy()
    hw = np.broadcast_to(h, W.shape).astype(np.float64)
    with np.errstate(invalid="ignore"):
        for c in range(2):
            for m in range(k):
                used = assign[:, 64 * c:64 * (c + 1)] == m
                for t in range(d):
                    x, hv = (z[:, 256 * c + t:256 * (c + 1):4][used].astype(np.float64) for z in (W, hw))
                    num, den = (hv * x).sum(), hv.sum()
                    want = np.float32(num) / np.float32(den) if den != 0 else np.float32(0)
                    np.testing.assert_equal(got[c, m, t], want)


# tables per group (without copies, which lanes would share by their number): four groups to a workgroup, one with waves
# of 8 rows, and one with waves of 16 (twice with 256 rows)
ORDER_SHAPES = [(32, 512, 64, 2, 8), (16, 256, 32, 2, 4), (16, 256, 32, 1, 1), (64, 512, 256, 2, 32), (128, 256, 64, 1, 128),
                (256, 512, 256, 4, 256)]


@pytest.mark.parametrize("uneven", [False, True], ids=["even weights", "uneven weights"])
@pytest.mark.parametrize("shape", ORDER_SHAPES, ids=str)
def test_m_step_does_not_depend_on_the_order_of_the_vectors(env, shape, uneven):
    """The vectors of a group in another order, as the lanes of a wave might reach an entry in another order: sums that
    cancel down to 2^-40 of their terms come out the same to the bit."""
    torch, vq, vqdev = env
    out_f, in_f, k, d, gr = shape
    n_cb, rng = in_f // 256, np.random.default_rng(out_f + k + d)
    groups, n = out_f // gr * n_cb, gr * 256 // d
    x = rng.normal(0, 1, (groups, n, d)) * 2.0 ** rng.integers(0, 40, (groups, n, 1))
    x[:, 1::2] = -x[:, ::2] + rng.normal(0, 1e-3, (groups, n // 2, d))       # pairs that nearly cancel
    a = rng.integers(0, k, (groups, n // 2)).repeat(2, axis=1).astype(np.uint8)
    h = np.ones(in_f, np.float32) * (2.0 ** rng.integers(-15, 16) if uneven else 1)
    if uneven:
        h[0::256] = np.float32(2.0 ** -30)              # far from the others, the same for every order (x = 0 there)

    def matrix(v, width):
        return np.ascontiguousarray(v.reshape(out_f // gr, n_cb, gr, 256 // d, width).transpose(0, 2, 1, 3, 4)
                                    .reshape(out_f, -1))

    desc = vq.make_desc(out_f, in_f, k, {16: 4, 32: 5, 64: 6, 256: 8}[k], group_rows=gr, d=d)
    h_d, results = vqdev.to_device_bytes(h), []
    for order in range(3):
        p = rng.permutation(n) if order else np.arange(n)
        W = matrix(x[:, p].astype(np.float32), d)
        if uneven:
            W[:, 0::256] = 0
            if order:
                continue
        new = torch.full((groups, k, d), 777.0, dtype=torch.float32, device="cuda:0")
        vq.vq_em_update(desc, vqdev.to_device_bytes(W), h_d, vqdev.to_device_bytes(matrix(a[:, p][:, :, None], 1)), new)
        results.append(new.cpu().numpy())
        if uneven:                                      # the rows in another order instead: columns keep their weights
            for _ in range(2):
                rows = np.concatenate([g * gr + rng.permutation(gr) for g in range(out_f // gr)])
                new = torch.full((groups, k, d), 777.0, dtype=torch.float32, device="cuda:0")
                vq.vq_em_update(desc, vqdev.to_device_bytes(W[rows]), h_d,
                                vqdev.to_device_bytes(matrix(a[:, :, None], 1)[rows]), new)
                results.append(new.cpu().numpy())
    for r in results[1:]:
        np.testing.assert_array_equal(r.view(np.uint32), results[0].view(np.uint32))


@pytest.mark.parametrize("uneven", [False, True], ids=["even weights", "uneven weights"])
@pytest.mark.parametrize("shape", [(32, 512, 64, 2, 8), (16, 256, 32, 2, 4), (64, 512, 256, 2, 32), (64, 256, 16, 1, 64),
                                   (256, 256, 256, 4, 256)], ids=str)
def test_m_step_of_infinities_and_tiny_values(env, shape, uneven):
    """Infinite and NaN values of W show in the centroids they are assigned to, as in a floating-point sum, and in no
    other; subnormal and zero values count; a centroid for most vectors (kept in registers) beside the rest."""
    torch, vq, vqdev = env
    out_f, in_f, k, d, gr = shape
    W, h, cb = _inputs_any(out_f, in_f, k, d, gr, 1700 + out_f + k, from_data=False)
    rng = np.random.default_rng(out_f + 2 * k + d)
    if uneven:
        h = (h * 10.0 ** rng.uniform(-4, 4, in_f)).astype(np.float32)
    kind = rng.random(W.shape)
    W[kind < 0.004], W[(kind > 0.01) & (kind < 0.014)], W[(kind > 0.02) & (kind < 0.022)] = np.inf, -np.inf, np.nan
    W[(kind > 0.1) & (kind < 0.3)] *= np.float32(1e-37)
    W[kind > 0.8] = 0
    assign = rng.integers(0, k, (out_f, in_f // d)).astype(np.uint8)
    assign[rng.random(assign.shape) < 0.5] = 3
    desc = vq.make_desc(out_f, in_f, k, {16: 4, 32: 5, 64: 6, 256: 8}[k], group_rows=gr, d=d)
    new = torch.full(cb.shape, 777.0, dtype=torch.float32, device="cuda:0")
    vq.vq_em_update(desc, vqdev.to_device_bytes(W), vqdev.to_device_bytes(h), vqdev.to_device_bytes(assign), new)
    got, n_cb = new.cpu().numpy(), in_f // 256
    for g in range(cb.shape[0]):
        gi, c = divmod(g, n_cb)
        x = W[gi * gr:(gi + 1) * gr, c * 256:(c + 1) * 256].astype(np.float64).reshape(-1, d)
        hv = np.broadcast_to(h[c * 256:(c + 1) * 256].astype(np.float64), (gr, 256)).reshape(-1, d)
        a = assign[gi * gr:(gi + 1) * gr, c * (256 // d):(c + 1) * (256 // d)].reshape(-1)
        for t in range(d):
            with np.errstate(invalid="ignore"):
                num = np.bincount(a, hv[:, t] * x[:, t], 256)[:k]
                mag = np.bincount(a, hv[:, t] * np.abs(x[:, t]), 256)[:k]
                den = np.bincount(a, hv[:, t], 256)[:k]
                want = np.where(den != 0, num / np.where(den != 0, den, 1), 0)
            finite = np.isfinite(want)
            np.testing.assert_array_equal(got[g, ~finite, t], want[~finite].astype(np.float32))
            # three roundings to binary32, n * 2^-36 of the magnitudes at most, and what the rounding of a subnormal
            # numerator (2^-150) or quotient leaves
            safe = np.where(den != 0, den, 1)
            bound = 3.1 * 2.0 ** -24 * np.abs(want) + (2.1 * (gr * 256 // d) * 2.0 ** -36 * mag + 2.0 ** -149) / safe + 2.0 ** -149
            assert np.all(np.abs(got[g, finite, t] - want[finite]) <= bound[finite])


@pytest.mark.parametrize("shape", [(64, 2, 32), (256, 2, 8), (32, 2, 8), (64, 4, 16), (256, 4, 64)], ids=str)
def test_m_step_with_one_centroid_for_all_costs_no_more(env, shape):
    """Assignments that meet in one entry of the table, as zeroed weights leave them, against uniform ones: 0.5 .. 1.0 of
    the time (three to six times it while every lane added to that entry)."""
    torch, vq, vqdev = env
    k, d, gr = shape
    n = 4096
    g = torch.Generator("cuda").manual_seed(6)
    W = torch.randn((n, n), device="cuda", generator=g) * 0.02
    h = 0.2 + 4.8 * torch.rand(n, device="cuda", generator=g)
    uniform = torch.randint(0, k, (n, n // d), dtype=torch.uint8, device="cuda", generator=g)
    half = torch.where(torch.rand(uniform.shape, device="cuda", generator=g) < 0.5, torch.ones_like(uniform), uniform)
    new = torch.empty((n // gr * 16, k, d), device="cuda")
    desc = vq.make_desc(n, n, k, {32: 5, 64: 6, 256: 8}[k], group_rows=gr, d=d)

    def us(assign):
        best = 1e9
        for _ in range(6):
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            t0.record()
            for _ in range(20):
                vq.vq_em_update(desc, W, h, assign, new)
            t1.record()
            torch.cuda.synchronize()
            best = min(best, t0.elapsed_time(t1) * 50)
        return best

    base = us(uniform)
    assert us(torch.ones_like(uniform)) < 1.4 * base
    assert us(half) < 1.6 * base


# the codebooks that the matrix cores filter: one tile and several, one group and several per strip of rows
FILTERED = [(2, 256, 8, 24, 512), (2, 256, 128, 128, 256), (4, 64, 16, 48, 512), (4, 256, 8, 8, 768), (4, 256, 64, 64, 512),
            (2, 64, 8, 24, 512), (2, 64, 32, 64, 512)]


def _filter_margin(d):
    """The share of a vector's norm sum h x^2 by which the second block of 8 centroids has to lie above the first, as the
    kernel has it (the rest of its margin is a share of the distance itself, 1e-4 at most)."""
    import os
    import re
    path = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2402_15319_amd", "csrc", "vq_em.hip")
    text = open(path).read()
    a, b = re.search(r"kScoreError = ([\d.]+)f \+ ([\d.]+)f \* D;", text).groups()
    m = re.search(r"kX = ([\d.]+)f \* \(([\d.]+)f \* kScoreError \+ ([\d.]+)f\) / 1048576\.f;", text)
    assert m, "the constant is not where this test looks for it"
    return float(m[1]) * (float(m[2]) * (float(a) + float(b) * d) + float(m[3])) / 2.0 ** 20


def _undecided(W, h, cb, d, k, gr):
    """Which vectors of W [rows, in / d] the filter can not tell from the second block of 8 centroids, and which it can with
    ten times the margin to spare.  For codebooks without equal centroids, which lie in blocks as they come."""
    out_f, in_f = W.shape
    margin, unsure, sure = _filter_margin(d), np.zeros((out_f, in_f // d), bool), np.zeros((out_f, in_f // d), bool)
    for g in range(cb.shape[0]):
        gi, c = divmod(g, in_f // 256)
        assert len(np.unique(cb[g], axis=0)) == k
        rows, cols = slice(gi * gr, (gi + 1) * gr), slice(c * (256 // d), (c + 1) * (256 // d))
        x = W[rows, c * 256:(c + 1) * 256].astype(np.float64).reshape(gr, 256 // d, 1, d)
        hv = h[c * 256:(c + 1) * 256].astype(np.float64).reshape(1, 256 // d, 1, d)
        dist = (hv * (x - cb[g].astype(np.float64)) ** 2).sum(3).reshape(gr, 256 // d, k // 8, 8).min(3)
        two = np.partition(dist, 1, axis=2)
        gap, norm = two[..., 1] - two[..., 0], (hv * x ** 2).sum(3)[..., 0]
        unsure[rows, cols] = gap < 0.9 * margin * norm
        sure[rows, cols] = gap > 10 * (margin * norm + 1e-4 * two[..., 0])
    return unsure, sure


def _in_steps(a, d):
    """[rows, vectors of a row] -> [row, place of 32 vectors], the share of them"""
    return a.reshape(a.shape[0], -1, 32).mean(2)


@pytest.mark.parametrize("case", ["plain", "centroids twice", "zero centroids and weights", "all zero", "rounded to a grid",
                                  "far from zero", "uneven weights", "zero weights", "negative weights", "huge", "tiny",
                                  "nan and inf", "zero weights in one set", "equal centroids for the later rows",
                                  "near centroids for the later rows", "far from zero in the later rows"])
@pytest.mark.parametrize("shape", FILTERED, ids=str)
def test_filtered_e_step_is_the_defined_one(env, shape, case):
    """The scores that pick the candidates are approximate, the result is not: ties, vectors that the
    filter cannot decide and values outside its ranges, all bit for bit."""
    d, k, gr, out_f, in_f = shape
    W, h, cb = _inputs_any(out_f, in_f, k, d, gr, 1500 + out_f + k + d, from_data=False)
    rng = np.random.default_rng(out_f + d)
    if case == "centroids twice":
        cb[:, k // 2:] = cb[:, :k // 2]
    elif case == "zero centroids and weights":
        cb[:, ::3] = 0
        W[rng.random(W.shape) < 0.5] = 0
    elif case == "all zero":
        W[:] = 0
        cb[:, 1::2] = 0
    elif case == "rounded to a grid":
        W, cb, h = np.round(W * 100) / np.float32(100), np.round(cb * 100) / np.float32(100), np.ones_like(h)
    elif case == "far from zero":
        W, cb = W + np.float32(1), cb + np.float32(1)
    elif case == "uneven weights":
        h = (10.0 ** rng.uniform(-6, 6, in_f)).astype(np.float32)
    elif case == "zero weights":
        h[::2] = 0
    elif case == "negative weights":
        h[::7] *= -1
    elif case == "huge":
        W = W * np.float32(1e30)
    elif case == "tiny":
        W, cb = W * np.float32(1e-25), cb * np.float32(1e-25)
    elif case == "nan and inf":
        W[rng.random(W.shape) < 0.01] = np.nan
        W[rng.random(W.shape) < 0.01] = np.inf
    elif case == "zero weights in one set":        # the second 32 vectors of a col-block
        h[32 * d:64 * d] = 0
    elif case == "equal centroids for the later rows":   # one of the equal ones is left: all rows are decided
        cb[:, ::2] = 0
        W.reshape(-1, 8, in_f)[:, 4:] = 0
    elif case == "near centroids for the later rows":    # decided at first, undecided in rows 4 .. 7 of every 8
        cb[:, ::2] = (0.5 + rng.integers(0, 256, cb[:, ::2].shape) * 2.0 ** -23).astype(np.float32)
        cb[:, ::2, 0] = (0.5 + rng.permuted(np.tile(np.arange(k // 2), (cb.shape[0], 1)), axis=1) * 2.0 ** -23).astype(np.float32)
        W.reshape(-1, 8, in_f)[:, 4:] = 0.5
        unsure, sure = _undecided(W, h, cb, d, k, gr)
        in_step = np.arange(out_f) % 8 < 4
        assert _in_steps(sure, d)[in_step].mean() > 0.8 and unsure[in_step].mean() < 0.02
        assert _in_steps(unsure, d)[~in_step].min() > 0.9
    elif case == "far from zero in the later rows":      # ... and there beyond what the filter tries
        cb[:, 1::2] += 5
        W.reshape(-1, 8, in_f)[:, 4:] += 5
    f = oracle.VQFormat(out_f, in_f, k, 8, gr, 256, d)
    with np.errstate(all="ignore"):
        want = oracle.em_assign(f, W, h, cb)
    a, _ = _gpu_em_any(env, (out_f, in_f, k, d, gr), W, h, cb)
    np.testing.assert_array_equal(a, want)


@pytest.mark.parametrize("shape", [(2, 256, 8), (4, 64, 16), (4, 256, 64), (2, 64, 8), (2, 64, 32)], ids=str)
def test_undecided_vectors_cost_no_more_than_a_loop_over_the_codebook(env, shape):
    """Codebooks of one value, weights that the filter does not take and vectors too far from zero for it: they meet the whole
    codebook, and that must not take longer than the kernels without a filter do (by the one for d = 2, k = 32, per
    coordinate and centroid: 0.72 to 0.98 of its time; 1.4 and more when a read of a centroid served one vector, up to 1.16 when
    far ones were tried first).  Vectors that only the scores show to be undecided, in the second half of the rows, cost half
    of the filter on top: 0.8 to 1.2 (1.41 when the first half was taken again with them)."""
    torch, vq, vqdev = env
    d, k, gr = shape
    n = 4096
    g = torch.Generator("cuda").manual_seed(5)
    W = torch.randn((n, n), device="cuda", generator=g) * 0.02
    h = 0.2 + 4.8 * torch.rand(n, device="cuda", generator=g)

    def us(desc, h, cb, W=W):
        a = torch.empty((n, n // desc.d), dtype=torch.uint8, device="cuda")
        best = 1e9
        for _ in range(6):
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            t0.record()
            for _ in range(5):
                vq.vq_em_assign(desc, W, h, cb, a)
            t1.record()
            torch.cuda.synchronize()
            best = min(best, t0.elapsed_time(t1) * 200)
        return best

    loop = us(vq.make_desc(n, n, 32, 5), h, torch.randn((n // 8 * 16, 32, 2), device="cuda", generator=g) * 0.02)
    per_coordinate = loop / (32 * n * n)                     # d coordinates a vector, n * n / d vectors
    cb = torch.randn((n // gr * 16, k, d), device="cuda", generator=g) * 0.02
    tied = cb[:, :1].expand(-1, k, -1).contiguous()
    desc = vq.make_desc(n, n, k, {64: 6, 256: 8}[k], group_rows=gr, d=d)
    zeros = h.clone()
    zeros[::2] = 0
    whole = per_coordinate * k * n * n
    ratio = [us(desc, h, tied) / whole, us(desc, zeros, cb) / whole, us(desc, h, cb + 5, W + 5) / whole]
    assert max(ratio) < 1.1, ratio      # an eighth above the largest for boxes that differ
    later = W.clone()
    later.view(-1, 8, n)[:, 4:] += 5
    cb[:, 1::2] += 5
    ratio = us(desc, h, cb, later) / whole
    assert ratio < 1.35, ratio
