"""The batched product's larger tiles: every kernel that launch_gemm chooses from, with rows and columns that do not fill the
last tile, one to several col-blocks, numbers of tile rows on both sides of a multiple of eight, and a padded X."""
import pytest

import workloads

pytestmark = pytest.mark.gpu

FORMATS = {
    "k16": dict(k=16, index_bits=4), "k256": dict(k=256, index_bits=8),
    "k64_i8": dict(k=64, index_bits=6, group_rows=16, int8_tables=True),
    "k256_bn": dict(k=256, index_bits=8, group_rows=64, int8_tables=True, block_norm=True),
    "d4_f16": dict(k=256, index_bits=8, group_rows=64, d=4),
}
# (rows, columns, B); which kernel each takes on 256 CUs is at the test of that without a GPU (test_launches.py)
SIZES = [(3904, 256, 200), (3904, 1280, 161), (8256, 256, 130), (8256, 768, 66), (25664, 512, 400), (8256, 512, 1090), (11072, 256, 203),
         (8384, 512, 256), (11072, 512, 410), (21568, 256, 384), (11072, 256, 2040), (11072, 768, 1281), (1088, 2304, 16), (64, 8448, 21),
         (1088, 2048, 161), (1088, 3328, 170), (1088, 5120, 130), (1088, 2304, 161), (4032, 768, 250), (15424, 2048, 1090),
         (576, 512, 1793), (576, 768, 4601), (2112, 2048, 10100)]     # more columns than rows


@pytest.mark.parametrize("size", SIZES, ids=str)
@pytest.mark.parametrize("fmt", sorted(FORMATS))
def test_tiles(fmt, size):
    import torch
    import paper_2402_15319_amd as vq
    from paper_2402_15319_amd import device as vqdev
    out_f, in_f, B = size
    s = workloads.VQShape(out_f, in_f, **FORMATS[fmt])
    if s.block_norm:
        idx, *tables = workloads.make_weights_bn(s, 3)
        cb = workloads.tables_bn_bytes(s, *tables)
    elif s.int8_tables:
        idx, q, scale = workloads.make_weights_i8(s, 3)
        cb = workloads.tables_i8_bytes(s, q, scale)
    else:
        idx, cb = workloads.make_weights(s, 3)
    desc = vqdev.desc_from_shape(s)
    idx_d, cb_d = vqdev.upload_and_pack(desc, idx, cb)
    W = torch.empty((out_f, in_f), dtype=torch.float16, device="cuda:0")
    vq.vq_decode_dense(desc, idx_d, cb_d, W)
    ld = (B + 7) // 8 * 8 + 8
    g = torch.Generator("cuda").manual_seed(B)
    X = torch.randn((in_f, ld), device="cuda", generator=g).half()
    X[:, B:] = float("inf")                           # columns beyond the batch reach no result
    Y = torch.full((out_f, ld), 777.0, dtype=torch.float32, device="cuda:0")
    vq.vq_gemm_batched(desc, idx_d, cb_d, X, B, ld, Y, ld, vq.VQ_F32)
    torch.cuda.synchronize()
    Xd, Wd = X[:, :B].double(), W.double()
    # exact products, at most in_f additions in binary32
    bound = (in_f + 2) * 2.0 ** -24 * (Wd.abs() @ Xd.abs())
    assert ((Y[:, :B].double() - Wd @ Xd).abs() <= bound).all()
    assert (Y[:, B:] == 777.0).all()
