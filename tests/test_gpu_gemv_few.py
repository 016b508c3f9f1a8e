"""Launches of up to four products take their argument from one line per product and a grid row each; launches of more
search a table.  Products of unlike heights in one launch (workgroups beyond the shorter ones), an odd number of
row-blocks, against the same products in a longer launch, bit for bit, and nothing written beyond a result."""
import pytest

import workloads

pytestmark = pytest.mark.gpu

FORMATS = {
    "k16": dict(k=16, index_bits=4, group_rows=8), "k256": dict(k=256, index_bits=8, group_rows=8),
    "k64_i8": dict(k=64, index_bits=6, group_rows=16, int8_tables=True),
    "k64_bn": dict(k=64, index_bits=6, group_rows=8, int8_tables=True, block_norm=True),
}


@pytest.mark.parametrize("heights", [(16,), (272, 16), (16, 528, 48), (16, 48, 16, 1040)], ids=str)
@pytest.mark.parametrize("in_f", [256, 1024, 2304])      # one chunk by one wave, several waves, several chunks
@pytest.mark.parametrize("fmt", sorted(FORMATS))
def test_few_products(fmt, in_f, heights):
    import torch
    import paper_2402_15319_amd as vq
    from paper_2402_15319_amd import device as vqdev
    descs, idx_d, cb_d, xs = [], [], [], []
    for i, out_f in enumerate(heights):
        s = workloads.VQShape(out_f, in_f, **FORMATS[fmt])
        if s.block_norm:
            idx, *tables = workloads.make_weights_bn(s, i)
            cb = workloads.tables_bn_bytes(s, *tables)
        elif s.int8_tables:
            idx, q, scale = workloads.make_weights_i8(s, i)
            cb = workloads.tables_i8_bytes(s, q, scale)
        else:
            idx, cb = workloads.make_weights(s, i)
        descs.append(vqdev.desc_from_shape(s))
        a, b = vqdev.upload_and_pack(descs[-1], idx, cb)
        idx_d.append(a), cb_d.append(b), xs.append(torch.from_numpy(workloads.make_x(in_f, i)).cuda())

    def run(n):
        ids = [i % len(heights) for i in range(n)]
        ys = [torch.full((heights[i] + 64,), 777.0, dtype=torch.float32, device="cuda:0") for i in ids]
        vq.vq_gemv_multi(*([t[i] for i in ids] for t in (descs, idx_d, cb_d, xs)), ys, y_dtype=vq.VQ_F32)
        torch.cuda.synchronize()
        return ys

    few, many = run(len(heights)), run(5)
    for i, out_f in enumerate(heights):
        assert torch.equal(few[i], many[i])
        assert (few[i][out_f:] == 777.0).all() and not (few[i][:out_f] == 777.0).any()


@pytest.mark.parametrize("heights", [(272, 64), (64, 528, 1088), (64, 1088, 128, 256)], ids=str)
@pytest.mark.parametrize("ranks", [(16, 16, 16, 16), (8, 0, 64, 16), (0, 64, 0, 0)], ids=str)
@pytest.mark.parametrize("fmt", sorted(FORMATS) + ["d4"])
def test_few_products_with_adapters(fmt, ranks, heights):
    """The same with an adapter next to each product, or to some of them: t = A x has a grid row per adapter, whose ranks
    differ, and the product a line for each.  Against five products in a launch, and the sums in 64 bits."""
    import torch
    import paper_2402_15319_amd as vq
    from paper_2402_15319_amd import device as vqdev
    in_f, n = 1280, len(heights)
    if fmt == "d4":
        heights = tuple(h // 64 * 64 for h in heights)
    descs, idx_d, cb_d, xs, As, Bs, refs = [], [], [], [], [], [], []
    gen = torch.Generator("cuda").manual_seed(sum(heights) + sum(ranks))
    for i, out_f in enumerate(heights):
        s = workloads.VQShape(out_f, in_f, **FORMATS[fmt]) if fmt != "d4" else workloads.VQShape(out_f, in_f, 256, 8, 64, 256, 4)
        if s.block_norm:
            idx, *tables = workloads.make_weights_bn(s, i)
            cb = workloads.tables_bn_bytes(s, *tables)
        elif s.int8_tables:
            idx, q, scale = workloads.make_weights_i8(s, i)
            cb = workloads.tables_i8_bytes(s, q, scale)
        else:
            idx, cb = workloads.make_weights(s, i)
        descs.append(vqdev.desc_from_shape(s))
        a, b = vqdev.upload_and_pack(descs[-1], idx, cb)
        idx_d.append(a), cb_d.append(b), xs.append(torch.from_numpy(workloads.make_x(in_f, i)).cuda())
        As.append((torch.randn((max(ranks[i], 8), in_f), device="cuda", generator=gen) / in_f ** 0.5).half())
        Bs.append((torch.randn((out_f, max(ranks[i], 8)), device="cuda", generator=gen) * 0.3).half())
        W = torch.empty((out_f, in_f), dtype=torch.float16, device="cuda:0")
        vq.vq_decode_dense(descs[-1], a, b, W)
        x = xs[-1].view(torch.float16).double().flatten()
        y, size = W.double() @ x, W.double().abs() @ x.abs()
        if ranks[i]:
            t = As[-1].double() @ x
            y += Bs[-1].double() @ t
            size += Bs[-1].double().abs() @ (As[-1].double().abs() @ x.abs())
        refs.append((y, size))

    def run(count):
        ids = [i % n for i in range(count)]
        ys = [torch.full((heights[i] + 64,), 777.0, dtype=torch.float32, device="cuda:0") for i in ids]
        args = vq.GemvMultiArgs(*([t[i] for i in ids] for t in (descs, idx_d, cb_d, xs)), ys)
        vq.vq_gemv_lora_multi_static(args, *([t[i] for i in ids] for t in (As, Bs, ranks)), y_dtype=vq.VQ_F32)
        torch.cuda.synchronize()
        return ys

    few, many = run(n), run(5)
    for i, out_f in enumerate(heights):
        if fmt != "d4":        # few d = 4 products share their rows among workgroups: another order of the sums
            assert torch.equal(few[i], many[i])
        assert (few[i][out_f:] == 777.0).all() and (many[i][out_f:] == 777.0).all()
        y, size = refs[i]      # exact products, at most in_f + 64 + 2 additions in binary32 and t rounded to it
        assert ((few[i][:out_f].double() - y).abs() <= (2 * in_f + 70) * 2.0 ** -24 * size).all()
