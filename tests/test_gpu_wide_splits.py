"""The GEMV kernels of the formats whose tables are shared by 64 or more rows, at every number of workgroups
and waves that share 64 rows (8, 4, 2 or 1), against the decoded matrix in 64 bits, with and without an
adapter."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

FORMATS = {
    "d4": dict(d=4, int8_tables=True), "d4_f16": dict(d=4), "d4_bn": dict(d=4, int8_tables=True, block_norm=True),
    "k256_i8": dict(int8_tables=True), "k256_bn": dict(int8_tables=True, block_norm=True),
}
# (rows, columns, products); columns may differ between products: a narrow one beside a wide one has empty splits.
# Workgroups per 64 rows on 256 CUs behind each (d = 2; d = 4; d = 4 with fp16 tables, or one figure for all).
SIZES = [
    (64, 256, 1), (128, 768, 2), (192, 1280, 3), (64, 4352, 1), (64, 8448, 1), (128, 8960, 2),   # 1, 2, 2, 4, 8, 8
    (64, 768, 5), (4160, 1024, 2), (4288, 2048, 3), (4288, 512, 3), (8512, 2048, 2),             # 1; 1; 2, 1, 1; 1; 2
    (12352, 1024, 2), (16448, 1024, 2),                                                          # 1, 1
    (64, (256, 8448), 2), (192, (8448, 256, 768, 512), 4), (2048, (256, 2304), 2),               # 8, 8, 4
    (4160, (256, 4352), 2), (4288, (512, 4352, 256), 3),                                         # 4, 4, 2; 2
]


@pytest.mark.parametrize("size", SIZES, ids=str)
@pytest.mark.parametrize("fmt", sorted(FORMATS))
def test_splits(fmt, size, group_rows=64):
    import torch
    import paper_2402_15319_amd as vq
    from paper_2402_15319_amd import device as vqdev
    out_f, widths, count = size
    widths = widths if isinstance(widths, tuple) else (widths,) * count
    rank = 16
    descs, mats, xs, ys, zs, As, Bs, want, want_lora, bound = [], [], [], [], [], [], [], [], [], []
    for i, in_f in enumerate(widths):
        s = workloads.VQShape(out_f, in_f, 256, 8, group_rows, **FORMATS[fmt])
        desc = vqdev.desc_from_shape(s)
        descs.append(desc)
        seed = 60 + in_f + i
        if s.block_norm:
            idx, *tables = workloads.make_weights_bn(s, seed)
            cb = workloads.tables_bn_bytes(s, *tables)
        elif s.int8_tables:
            idx, q, scale = workloads.make_weights_i8(s, seed)
            cb = workloads.tables_i8_bytes(s, q, scale)
        else:
            idx, cb = workloads.make_weights(s, seed)
        mats.append(vqdev.upload_and_pack(desc, idx, cb))
        W = torch.empty((out_f, in_f), dtype=torch.float16, device="cuda:0")
        vq.vq_decode_dense(desc, *mats[-1], W)
        x = workloads.make_x(in_f, seed)
        rng = np.random.default_rng(seed)
        A = (rng.standard_normal((rank, in_f)) / 64).astype(np.float16)
        B = (rng.standard_normal((out_f, rank)) / 64).astype(np.float16)
        xs.append(torch.from_numpy(x).cuda())
        As.append(torch.from_numpy(A).cuda())
        Bs.append(torch.from_numpy(B).cuda())
        ys.append(torch.full((out_f,), 777.0, dtype=torch.float32, device="cuda:0"))
        zs.append(torch.full((out_f,), 777.0, dtype=torch.float32, device="cuda:0"))
        Wd, xd = W.double().cpu().numpy(), x.astype(np.float64)
        want.append(Wd @ xd)
        want_lora.append(want[-1] + B.astype(np.float64) @ (A.astype(np.float64) @ xd))
        mag = np.abs(Wd) @ np.abs(xd) + np.abs(B).astype(np.float64) @ (np.abs(A).astype(np.float64) @ np.abs(xd))
        # exact products; at most in_f additions in binary32 (and in_f + rank with the adapter)
        bound.append((in_f + rank + 2) * 2.0 ** -24 * mag)
    idx_d, cb_d = [m[0] for m in mats], [m[1] for m in mats]
    args = vq.GemvMultiArgs(descs, idx_d, cb_d, xs, ys)
    vq.vq_gemv_multi(args, y_dtype=vq.VQ_F32)
    ws = torch.zeros(vq.vq_lora_workspace_bytes(count), dtype=torch.uint8, device="cuda:0")
    vq.vq_gemv_lora_multi(vq.GemvMultiArgs(descs, idx_d, cb_d, xs, zs), As, Bs, [rank] * count, ws, vq.VQ_F32)
    torch.cuda.synchronize()
    for i in range(count):
        assert np.all(np.abs(ys[i].cpu().numpy() - want[i]) <= bound[i])
        assert np.all(np.abs(zs[i].cpu().numpy() - want_lora[i]) <= bound[i])
