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
