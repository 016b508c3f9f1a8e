"""The batched product where few workgroups cover it: 16 x 16 tiles with four and with eight waves that
split k, on both sides of the rules that choose them, against products of the decoded matrix in 64 bits."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

FORMATS = {
    "k16": dict(k=16, index_bits=4),
    "k64_i8": dict(k=64, index_bits=6, group_rows=32, int8_tables=True),
    "k64_bn": dict(k=64, index_bits=6, group_rows=8, int8_tables=True, block_norm=True),
    "d4": dict(k=256, index_bits=8, group_rows=64, d=4, int8_tables=True),
}
# (rows in multiples of the group height's, columns, batch): one col-block a wave (4 and 5 of them: four and
# eight waves), more col-blocks than waves, an odd number of row-blocks, batches that are not multiples of 16;
# then more than one 16 x 16 tile per CU and at most two (33 groups of 8 rows, 323 tiles with four waves that walk
# nine col-blocks; the same columns with the taller groups pass the line), and up to three for 17..32 columns
SIZES = [(1, 1024, 3), (1, 1280, 16), (3, 2304, 17), (5, 2816, 40), (2, 4352, 130), (33, 1280, 200),
         (33, 2304, 300), (9, 2304, 250), (129, 2304, 32)]


@pytest.mark.parametrize("size", SIZES, ids=str)
@pytest.mark.parametrize("fmt", sorted(FORMATS))
def test_small_grids(fmt, size):
    import torch
    import paper_2402_15319_amd as vq
    from paper_2402_15319_amd import device as vqdev
    groups, in_f, B = size
    opts = FORMATS[fmt]
    s = workloads.VQShape(groups * max(opts.get("group_rows", 8), 8), in_f, **opts)
    seed = 40 + in_f + B
    if s.block_norm:
        idx, *tables = workloads.make_weights_bn(s, seed)
        cb = workloads.tables_bn_bytes(s, *tables)
    elif s.int8_tables:
        idx, q, scale = workloads.make_weights_i8(s, seed)
        cb = workloads.tables_i8_bytes(s, q, scale)
    else:
        idx, cb = workloads.make_weights(s, seed)
    desc = vqdev.desc_from_shape(s)
    idx_d, cb_d = vqdev.upload_and_pack(desc, idx, cb)
    W = torch.empty((s.out_features, in_f), dtype=torch.float16, device="cuda:0")
    vq.vq_decode_dense(desc, idx_d, cb_d, W)
    ld = (B + 7) // 8 * 8
    X = workloads.make_X(in_f, ld, seed)
    Y = torch.full((s.out_features, ld), 777.0, dtype=torch.float32, device="cuda:0")
    vq.vq_gemm_batched(desc, idx_d, cb_d, torch.from_numpy(X).cuda(), B, ld, Y, ld, vq.VQ_F32)
    torch.cuda.synchronize()
    Wd, Xd = W.cpu().numpy().astype(np.float64), X.astype(np.float64)[:, :B]
    got = Y.cpu().numpy()
    # exact products of fp16 values; at most in_f additions in binary32, 2^-24 of the magnitudes each
    assert np.all(np.abs(got[:, :B] - Wd @ Xd) <= in_f * 2.0 ** -24 * (np.abs(Wd) @ np.abs(Xd)))
    assert np.all(got[:, B:] == 777.0)
