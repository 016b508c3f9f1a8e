"""Launches of more than four products of the formats whose tables are shared by 64 or more rows: the widest product's
workgroups start first, whatever the order of the call.  With d = 4 and groups of 256 rows, neighbouring 64-row items go to one XCD
in aligned sets of 32, also in long launches of one product.  Every result, with and without an adapter, goes to its own y: less than 32
items, one set and a remainder, several."""
import pytest

import test_gpu_wide_splits as splits

pytestmark = pytest.mark.gpu

SIZES = [(64, (256, 2304, 768, 2304, 512, 1280), 6), (704, (512, 2304, 768, 256, 1280), 5), (2048, (768, 256, 1280, 256, 512), 5)]


@pytest.mark.parametrize("size", SIZES, ids=str)
@pytest.mark.parametrize("fmt", sorted(splits.FORMATS))
def test_unlike_widths(fmt, size):
    splits.test_splits(fmt, size)


@pytest.mark.parametrize("size", [(256, (256, 2304, 768, 2304, 512, 1280), 6), (768, (512, 2304, 768, 256, 1280), 5), (33024, 256, 1)], ids=str)
@pytest.mark.parametrize("fmt", ["d4", "d4_bn", "d4_f16"])
def test_groups_of_256_rows(fmt, size):
    splits.test_splits(fmt, size, group_rows=256)
