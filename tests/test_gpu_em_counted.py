"""The M-step of many tall groups (d = 4, k = 256, 128 or 256 rows, more than half a group per CU): one scale for a group,
taken from its first rows, centroids summed again where that leaves open what their numerators round to, and the general
path for infinities.  Against 64-bit sums, on every run the same, and, where no row has a centroid that many lanes share, in every
order of the rows: the numerator is the exact sum, rounded once."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KINDS = ["normal", "later rows larger", "odd rows larger", "one value larger", "small and cancelling", "zeros", "uneven weights",
         "infinities"]


def _inputs(rows, kind):
    rng = np.random.default_rng(rows + KINDS.index(kind))
    gr, gc = 26, 5                                  # 130 groups
    W = (rng.standard_normal((gr, rows, gc * 256)) * 0.02).astype(np.float32)
    h = rng.uniform(0.2, 5.0, gc * 256).astype(np.float32)
    a = rng.integers(0, 256, (gr, rows, gc * 64)).astype(np.uint8)
    if kind == "later rows larger":                 # by more than the first ones' scale allows
        W[::2, 8:] *= 300
    elif kind == "odd rows larger":
        W[1::2, 1::2] *= 2.0 ** 20
    elif kind == "one value larger":
        W[:, -1, 255::256] = -3e3
    elif kind == "small and cancelling":
        at = np.repeat(a, 4, axis=2)
        W[(at >= 5) & (at < 9)] *= np.float32(2.0 ** -60)     # four centroids far below the rest, subnormal ones too
        W[at == 5] *= np.float32(2.0 ** -70)
        W[:, 1] = -W[:, 0]                                    # pairs that cancel, each in the same centroid
        a[:, 1] = a[:, 0]
        W[:, 2:][np.repeat(a[:, 2:], 4, axis=2) == 9] = 0     # ... and nothing else in it
    elif kind == "zeros":
        W[::2] = 0
        W[1::2][np.repeat(a[1::2], 4, axis=2) < 200] = 0
    elif kind == "uneven weights":
        h[::7] *= np.float32(2.0 ** -20)
        h[3::256] = 0
    elif kind == "infinities":
        W[0, -1, 5], W[1, 3, 300], W[2, rows // 2, 7], W[3, 0, 0] = np.inf, -np.inf, np.nan, 1e37   # (h x below 2^128: the numerator is rounded to binary32)
    return W.reshape(gr * rows, gc * 256), h, a.reshape(gr * rows, gc * 64)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("rows", [128, 256])
def test_against_64_bit_sums_in_any_order(rows, kind):
    import torch
    import paper_2402_15319_amd as vq
    W, h, a = _inputs(rows, kind)
    gr, gc = W.shape[0] // rows, W.shape[1] // 256
    desc = vq.make_desc(W.shape[0], W.shape[1], 256, 8, rows, 256, 4)
    order = np.random.default_rng(1).permutation(rows)

    def update(W, a):
        new = torch.full((gr, gc, 256, 4), 777.0, dtype=torch.float32, device="cuda:0")
        vq.vq_em_update(desc, torch.from_numpy(W).cuda(), torch.from_numpy(h).cuda(), torch.from_numpy(a).cuda(), new)
        return new.cpu().numpy()

    got = update(W, a)
    np.testing.assert_array_equal(update(W, a), got)
    shuffled = [m.reshape(gr, rows, -1)[:, order].reshape(m.shape) for m in (W, a)]
    np.testing.assert_array_equal(update(*shuffled), got)
    with np.errstate(invalid="ignore"):
        for g in range(gr):
            for c in range(gc):
                x = W[g * rows:(g + 1) * rows, c * 256:(c + 1) * 256].astype(np.float64).reshape(-1, 4)
                hv = np.broadcast_to(h[c * 256:(c + 1) * 256].astype(np.float64), (rows, 256)).reshape(-1, 4)
                m = a[g * rows:(g + 1) * rows, c * 64:(c + 1) * 64].reshape(-1)
                n = np.bincount(m, minlength=256)
                for t in range(4):
                    num = np.bincount(m, hv[:, t] * x[:, t], 256)
                    den = np.bincount(m, hv[:, t], 256)
                    want = np.where(den != 0, num / np.where(den != 0, den, 1), 0)
                    top = np.zeros(256)
                    np.maximum.at(top, m, np.abs(hv[:, t] * x[:, t]))
                    # numerator, denominator and quotient rounded once each, the numerator's sum good to 2^-28 of itself or,
                    # with even weights, to n * 2^-36 of its largest term (n * 2^-34 with the roundings of these sums)
                    with np.errstate(over="ignore"):
                        bound = 3.2 * 2.0 ** -24 * np.abs(want) + n * 2.0 ** -34 * top / np.where(den != 0, den, 1) + 2.0 ** -149
                    ok = (np.abs(got[g, c, :, t] - want) <= bound) | (np.isnan(want) & np.isnan(got[g, c, :, t])) | (want == got[g, c, :, t])
                    assert ok.all(), (g, c, t, np.flatnonzero(~ok)[:4], got[g, c, ~ok, t][:4], want[~ok][:4])


@pytest.mark.parametrize("low", [0, 4, 6, 8, 40])
@pytest.mark.parametrize("rows", [128, 256])
def test_numerators_are_the_exact_sums_rounded_once(rows, low):
    """Most centroids' values 2^-low of the others': however few bits the group's scale leaves their sums, and in whatever order
    the rows come, the quotient is that of the exact sums, each rounded to binary32.  (The weights' sums are exact in
    binary64; the reference's numerators are off by 2^-57 of the largest term at most.)"""
    import torch
    import paper_2402_15319_amd as vq
    W, h, a = _inputs(rows, "normal")
    W[np.repeat(a, 4, axis=1) >= 10] *= np.float32(2.0 ** -low)
    gr, gc = W.shape[0] // rows, W.shape[1] // 256
    desc = vq.make_desc(W.shape[0], W.shape[1], 256, 8, rows, 256, 4)
    for order in (np.arange(rows), np.random.default_rng(2).permutation(rows)):
        Wo, ao = (m.reshape(gr, rows, -1)[:, order].reshape(m.shape) for m in (W, a))
        new = torch.full((gr, gc, 256, 4), 777.0, dtype=torch.float32, device="cuda:0")
        vq.vq_em_update(desc, torch.from_numpy(Wo).cuda(), torch.from_numpy(h).cuda(), torch.from_numpy(ao).cuda(), new)
        got = new.cpu().numpy()
        for g in range(gr):
            for c in range(gc):
                x = W[g * rows:(g + 1) * rows, c * 256:(c + 1) * 256].astype(np.longdouble).reshape(-1, 4)
                hv = np.broadcast_to(h[c * 256:(c + 1) * 256].astype(np.longdouble), (rows, 256)).reshape(-1, 4)
                m = a[g * rows:(g + 1) * rows, c * 64:(c + 1) * 64].reshape(-1)
                by = np.argsort(m, kind="stable")
                start = np.searchsorted(m[by], np.arange(256))
                assert np.all(np.diff(start) > 0)       # no centroid is empty
                num, den = (np.add.reduceat(v[by], start, axis=0).astype(np.float32) for v in (hv * x, hv))
                np.testing.assert_array_equal(got[g, c], num / den)


def _update_and_compare(W, h, a, rows):
    """One call and a second one, which gives the same, against 64-bit sums: numerator, denominator and quotient rounded once
    each, and sums of n terms that are off by n * 2^-34 of the largest (n * 2^-52 in the kernel, more in the reference)."""
    import torch
    import paper_2402_15319_amd as vq
    gr, gc = W.shape[0] // rows, W.shape[1] // 256
    desc = vq.make_desc(W.shape[0], W.shape[1], 256, 8, rows, 256, 4)
    args = [torch.from_numpy(v).cuda() for v in (W, h, a)]
    runs = []
    for _ in range(2):
        new = torch.full((gr, gc, 256, 4), 777.0, dtype=torch.float32, device="cuda:0")
        vq.vq_em_update(desc, *args, new)
        runs.append(new.cpu().numpy())
    got = runs[0]
    np.testing.assert_array_equal(runs[1], got)
    with np.errstate(invalid="ignore", over="ignore", divide="ignore"):
        for g in range(gr):
            for c in range(gc):
                x = W[g * rows:(g + 1) * rows, c * 256:(c + 1) * 256].astype(np.float64).reshape(-1, 4)
                hv = np.broadcast_to(h[c * 256:(c + 1) * 256].astype(np.float64), (rows, 256)).reshape(-1, 4)
                m = a[g * rows:(g + 1) * rows, c * 64:(c + 1) * 64].reshape(-1)
                n = np.bincount(m, minlength=256)
                for t in range(4):
                    num, den = np.bincount(m, hv[:, t] * x[:, t], 256), np.bincount(m, hv[:, t], 256)
                    want = np.where(den != 0, num.astype(np.float32) / den.astype(np.float32), np.float32(0))
                    top = np.zeros(256)
                    np.maximum.at(top, m, np.abs(hv[:, t] * x[:, t]))
                    bound = 3.2 * 2.0 ** -24 * np.abs(want) + n * 2.0 ** -34 * top / np.where(den != 0, den, 1) + 2.0 ** -149
                    ok = (np.abs(got[g, c, :, t] - want) <= bound) | (np.isnan(want) & np.isnan(got[g, c, :, t])) | (want == got[g, c, :, t])
                    assert ok.all(), (g, c, t, np.flatnonzero(~ok)[:4], got[g, c, ~ok, t][:4], want[~ok][:4])
    return got


@pytest.mark.parametrize("kind", ["few", "few, first rows too", "lanes at the line", "group", "group and infinities", "beyond 2^127"])
@pytest.mark.parametrize("rows", [128, 256])
def test_values_beyond_the_scale(rows, kind):
    """Values that the scale from the first rows leaves no room for: a few, whose centroids are formed again; so many (17 lanes
    of a wave) that the group is taken once more; some that no scale takes."""
    W, h, a = _inputs(rows, "normal")
    group = W.reshape(-1, rows, W.shape[1])
    if kind == "few":
        group[:, rows // 2::7, 5::301] *= 60
        group[::3, rows - 1, 9] = 1e30
    elif kind == "few, first rows too":              # infinities in the sample: the others give the scale
        group[::2, 0, 7], group[::2, 2, 300], group[1::2, 4, 1000] = np.inf, np.nan, 1e30
        group[:, 1, 5::301] *= 60
    elif kind == "lanes at the line":
        group[::2, 9, :4 * 16:4] = 5                 # 16 lanes of one wave: formed again; 17: the group once more
        group[1::2, 9, :4 * 17:4] = 5
    elif kind == "group":
        group[:, rows // 2:] *= 50
    elif kind == "group and infinities":
        group[:, rows // 2:] *= 50
        group[::2, rows // 2 + 3, 5], group[::3, 3, 9], group[::5, rows - 1, 700] = np.inf, -np.inf, np.nan
    elif kind == "beyond 2^127":
        h[:] = np.minimum(h, 0.5)
        group[:, 2, 4], group[::2, 64, 300] = 2e38, -3e38
    got = _update_and_compare(W, h, a, rows)
    # where the scale comes from the same rows or not: the same in another order
    order = np.random.default_rng(3).permutation(rows)
    W2, a2 = (v.reshape(-1, rows, v.shape[1])[:, order].reshape(v.shape) for v in (W, a))
    np.testing.assert_array_equal(_update_and_compare(W2, h, a2, rows), got)


@pytest.mark.parametrize("kind", ["one centroid", "half of the lanes", "half of the lanes, cancelling", "kept by some waves",
                                  "kept by some waves, cancelling", "more than an entry holds", "infinite weights", "no weights"])
@pytest.mark.parametrize("rows", [128, 256])
def test_skewed_assignments_and_weights(rows, kind):
    """Centroids that many lanes of a row share, whose sums a wave keeps in registers: all waves, or those whose first rows
    have it; entries with more vectors than their bits take; weights that are infinite, NaN or zero."""
    W, h, a = _inputs(rows, "normal")
    group, ga = W.reshape(-1, rows, W.shape[1]), a.reshape(-1, rows, a.shape[1])
    first = np.arange(rows) % 64 < 32                # rows of waves 0 to 3
    if kind == "one centroid":
        a[:] = 200
    elif kind.startswith("half of the lanes"):
        a[:, 1::2] = 3
        if "cancelling" in kind:
            group[:, 1::2] = -group[:, ::2]
            ga[:, 1::2] = ga[:, ::2]
    elif kind.startswith("kept by some waves"):      # and in the table by the others
        ga[:, first, ::3] = 77
        ga[:, ~first, 5::9] = 77
        if "cancelling" in kind:
            group[:, 1::2] = -group[:, ::2]
            ga[:, 1::2] = ga[:, ::2]
    elif kind == "more than an entry holds":         # not in the rows that the waves look at first: 3 / 4 of the group's vectors
        group[:] = np.abs(group) / 64 + np.float32(0.49)
        group[:, 64:] *= 4                           # as far as the scale reaches, all of one sign
        ga[:, 64:] = 9
        h[:] = 1.96875
    elif kind == "infinite weights":
        h[4:8], h[132:136], h[300], h[700] = np.inf, np.nan, np.inf, -np.inf
        W[:, 700] = 1
    elif kind == "no weights":
        h[:300] = 0
        h[512:520] = 0
    _update_and_compare(W, h, a, rows)
