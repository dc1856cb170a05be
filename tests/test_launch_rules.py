"""The rules by which a call's launches are shaped, asked on the host: what they choose by the lengths of a call's tensors
where that is more than a matter of speed by a percent.  Lengths in chunks of 1024 elements."""
import pytest

import paper_2605_01708_amd as sz


def compress_plan(dtype, chunks):
    return sz.internal_compress_plan([c * 1024 for c in chunks], dtype)


def decompress_plan(dtype, chunks):
    return sz.internal_decompress_plan([c * 1024 for c in chunks], dtype)


FORMATS = [sz.BF16, sz.FP8_E5M2]


@pytest.mark.parametrize("dtype", FORMATS)
def test_tiles_that_are_not_there_do_not_make_a_launch_long(dtype):
    """xcd_order is for launches of many tiles; a row of workgroups per tensor, as long as the longest, is not that."""
    for chunks in ([13000] + [2] * 63, [32768] + [2] * 63, [8192] + [100] * 63, [8192] * 4 + [200] * 60):
        assert not compress_plan(dtype, chunks)["by_xcd"], chunks
        assert not decompress_plan(dtype, chunks)["by_xcd"], chunks
    for chunks in ([32768] * 64, [32768] * 63 + [5]):
        assert compress_plan(dtype, chunks)["by_xcd"] and decompress_plan(dtype, chunks)["by_xcd"]
