"""The quantiser's steps divide their work by the size of a launch: strips of 8 to 32 rows, waves of 8 or 2 rows, a group's
coordinates to one workgroup or to several.  A launch over many rows against launches over a few rows each; and codebooks
with any number of equal centroids against the oracle."""
import numpy as np
import pytest

import oracle
from test_gpu_em import _gpu_em_any, _inputs_any, env  # noqa: F401

pytestmark = pytest.mark.gpu

BITS = {8: 3, 16: 4, 32: 5, 64: 6, 256: 8}


# (k, d, group rows): filtered with strips of 8, 16 and 32 rows, loops; groups that a wave, a workgroup or several take
@pytest.mark.parametrize("shape", [(64, 2, 8), (64, 2, 32), (256, 2, 128), (64, 4, 16), (256, 4, 64), (256, 4, 256), (16, 1, 8),
                                   (32, 2, 32), (16, 2, 256)], ids=str)
def test_one_launch_and_many(env, shape):  # noqa: F811
    torch, vq, _ = env
    k, d, gr = shape
    out_f, in_f, part = 5120, 2048, 512                       # 5120 blocks of 8 x 256; 512
    g = torch.Generator("cuda").manual_seed(k + d + gr)
    W = torch.randn((out_f, in_f), device="cuda", generator=g) * 0.02
    h = 0.2 + 4.8 * torch.rand(in_f, device="cuda", generator=g)
    cb = torch.randn((out_f // gr, in_f // 256, k, d), device="cuda", generator=g) * 0.02
    cb[::2, :, k // 2:] = cb[::2, :, :k - k // 2]             # equal centroids in every other row of groups
    cb[:, :, 1] = 0
    cb[:, :, k - 1] = -0.0

    def both(rows):
        a = torch.full((out_f, in_f // d), 255, dtype=torch.uint8, device="cuda")
        new = torch.full_like(cb, 777.0)
        for r in range(0, out_f, rows):
            desc = vq.make_desc(rows, in_f, k, BITS[k], gr, 256, d)
            at = slice(r // gr, (r + rows) // gr)
            vq.vq_em_assign(desc, W[r:r + rows], h, cb[at].contiguous(), a[r:r + rows])
            out = torch.full_like(cb[at], 777.0).contiguous()
            vq.vq_em_update(desc, W[r:r + rows], h, a[r:r + rows], out)
            new[at] = out
        torch.cuda.synchronize()
        return a, new

    (a, new), (a_parts, new_parts) = both(out_f), both(part)
    assert torch.equal(a, a_parts)
    # each sum is off by n * 2^-36 of its largest term at most (n vectors of a group), the quotient by three roundings
    # to binary32 more; sums of both signs cancel, so the bound is taken on the magnitudes: all |x| <= 0.02 * 6
    assert (new - new_parts).abs().max().item() <= 0.12 * (gr * 256 / d * 2.0 ** -36 * 25 + 2.0 ** -22)
    assert not (new == 777.0).any()


# the filter works on the distinct centroids, spread over the blocks of 8: fewer than blocks, as many, one more, all but one
@pytest.mark.parametrize("distinct", ["blocks - 1", "blocks", "blocks + 1", "blocks + 7", "half", "all but one", "all"])
@pytest.mark.parametrize("shape", [(2, 64, 8, 16, 512), (2, 64, 32, 64, 256), (2, 256, 8, 16, 256), (4, 64, 16, 32, 512),
                                   (4, 256, 64, 64, 256)], ids=str)
def test_equal_centroids(env, shape, distinct):  # noqa: F811
    d, k, gr, out_f, in_f = shape
    W, h, cb = _inputs_any(out_f, in_f, k, d, gr, 70 + k + d, from_data=False)
    rng = np.random.default_rng(k + d)
    n = {"half": k // 2, "all but one": k - 1, "all": k}.get(distinct)
    if n is None:
        n = k // 8 + int(distinct[6:].replace(" ", "") or 0)
    for g in range(cb.shape[0]):
        values = cb[g, :n].copy()
        values[0] = 0
        order = np.concatenate([np.arange(n), rng.integers(0, n, k - n)])
        rng.shuffle(order)
        cb[g] = values[order]
        cb[g][(order == 0) & (rng.random(k) < 0.5)] = -0.0    # equal to the other zeros
    f = oracle.VQFormat(out_f, in_f, k, 8, gr, 256, d)
    a, _ = _gpu_em_any(env, (out_f, in_f, k, d, gr), W, h, cb)
    np.testing.assert_array_equal(a, oracle.em_assign(f, W, h, cb))


# rows and columns of the large launch: strips of 16 (d = 4: 4 to 12 blocks per CU, d = 2: 8 to 16) and of 32 rows
@pytest.mark.parametrize("case", ["far in later runs", "near ties in later runs", "zero weights in one place", "nan and inf"])
@pytest.mark.parametrize("shape", [(64, 2, 16, 2560), (64, 2, 32, 5120), (256, 2, 128, 2560), (256, 2, 32, 5120), (64, 4, 16, 2560), (64, 4, 64, 5120),
                                   (256, 4, 64, 2560), (256, 4, 256, 5120)], ids=str)
def test_strips_of_undecided_vectors(env, shape, case):  # noqa: F811
    """Waves that give up the filter after some rows, or in some places only, in strips of every height: against launches of
    few rows, which take strips of 8."""
    torch, vq, _ = env
    k, d, gr, out_f = shape
    in_f, part = 2048, 512
    g = torch.Generator("cuda").manual_seed(k + d + gr)
    W = torch.randn((out_f, in_f), device="cuda", generator=g) * 0.02
    h = 0.2 + 4.8 * torch.rand(in_f, device="cuda", generator=g)
    cb = torch.randn((out_f // gr, in_f // 256, k, d), device="cuda", generator=g) * 0.02
    row = torch.arange(out_f, device="cuda")
    if case == "far in later runs":           # from a row of each 32 on that differs from strip to strip
        far = row % 32 >= 4 * (row // 32 % 8)
        W[far] += 5
        cb[:, :, 1::2] += 5
    elif case == "near ties in later runs":   # distinct centroids that the scores cannot tell apart
        ulps = torch.argsort(torch.rand((*cb.shape[:2], k // 2), device="cuda", generator=g), dim=2)
        cb[:, :, ::2] = 0.5
        cb[:, :, ::2, 0] += ulps * 2.0 ** -23
        W[row % 32 >= 4 * (row // 32 % 8)] = 0.5
    elif case == "zero weights in one place":
        h[32 * d:64 * d] = 0
        h[1024::256] = 0
    elif case == "nan and inf":
        noise = torch.rand(W.shape, device="cuda", generator=g)
        W[noise < 0.001] = float("nan")
        W[noise > 0.999] = float("inf")

    def assign(rows):
        a = torch.full((out_f, in_f // d), 255, dtype=torch.uint8, device="cuda")
        for r in range(0, out_f, rows):
            vq.vq_em_assign(vq.make_desc(rows, in_f, k, BITS[k], gr, 256, d), W[r:r + rows], h,
                            cb[r // gr:(r + rows) // gr].contiguous(), a[r:r + rows])
        torch.cuda.synchronize()
        return a

    large = assign(out_f)
    assert torch.equal(large, assign(part))
    # and the defined arithmetic itself, on the first group
    x, c, hv = W[:gr].view(gr, -1, 256 // d, 1, d), cb[0][:, None], h.view(1, -1, 256 // d, 1, d)
    dist = None
    for t in range(d):
        e = x[..., t] - c[..., t]
        term = hv[..., t] * (e * e)
        dist = term if dist is None else dist + term
    dist = torch.where(torch.isnan(dist), torch.full_like(dist, float("inf")), dist)
    best = dist.min(dim=-1, keepdim=True).values
    first = torch.where(torch.isinf(best[..., 0]), 0, (dist == best).int().argmax(dim=-1))
    assert torch.equal(large[:gr], first.reshape(gr, -1).to(torch.uint8))


@pytest.mark.parametrize("shape", [(64, 2, 16), (256, 2, 64), (256, 2, 128), (64, 2, 256), (64, 4, 16), (256, 4, 64), (64, 4, 128), (256, 4, 256)], ids=str)
def test_sums_of_shared_groups_keep_their_bits(env, shape):  # noqa: F811
    """A group's sums are integers of 62 bits less the logarithm of its vectors, from the largest term down (at most 51), also
    where its coordinates go to different workgroups: two values that cancel leave a third of the last of those bits."""
    torch, vq, _ = env
    k, d, gr = shape
    bits = min(51, 62 - (max(14, int(np.log2(gr * 256))) - int(np.log2(d))))
    tiny = 4 * 2.0 ** -bits               # terms below 2 (h) * 2 (x)
    rng = np.random.default_rng(k + gr)
    W = rng.normal(0, 1, (gr, 256)).astype(np.float32)
    a = rng.integers(1, k, (gr, 256 // d)).astype(np.uint8)
    where = rng.permutation(gr * 256 // d)[:3]
    for at, v in zip(where, (1.0, -1.0, tiny)):
        a.reshape(-1)[at] = 0
        W.reshape(-1, d)[at] = v
    new = torch.full((1, k, d), 777.0, device="cuda")
    dev = [torch.from_numpy(t).cuda() for t in (W, np.ones(256, np.float32), a)]
    vq.vq_em_update(vq.make_desc(gr, 256, k, BITS[k], gr, 256, d), *dev, new)
    np.testing.assert_array_equal(new[0, 0].cpu().numpy(), np.full(d, np.float32(tiny) / np.float32(3)))
