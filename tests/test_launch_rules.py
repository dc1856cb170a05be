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


def test_short_launches_keep_the_order_of_the_tiles():
    """Under 2048 tiles, and where a wave has one chunk of BF16."""
    assert [compress_plan(sz.BF16, [c])["by_xcd"] for c in (8192, 9983, 20480, 20481, 32768)] == [0, 0, 0, 1, 1]
    assert [compress_plan(sz.BF16, [c] * k)["by_xcd"] for c, k in ((5000, 2), (1000, 10), (300, 64), (330, 64))] == [0, 0, 0, 1]
    assert [compress_plan(sz.FP8_E5M2, [c])["by_xcd"] for c in (6144, 16376, 16384, 32768)] == [0, 0, 1, 1]


@pytest.mark.parametrize("dtype", FORMATS)
def test_a_third_launch_only_where_the_counts_are_many(dtype):
    """The finishing pass sums the tile counts itself, with no launch in between, until its workgroups would together read
    128 MB of them: 23 169 tiles, 8 chunks each, whatever smaller tiles a shorter tensor has."""
    assert compress_plan(dtype, [40 if dtype == sz.BF16 else 48])["launches"] == 1
    for chunks in (49, 6144, 6145, 16384, 16385, 18000, 20480, 20481, 32768, 32769, 40000, 49152, 65536, 65537, 131072, 185344):
        assert compress_plan(dtype, [chunks])["launches"] == 2, chunks
    for chunks in (185345, 200000, 400000):
        assert compress_plan(dtype, [chunks])["launches"] == 3, chunks
    assert compress_plan(dtype, [32768] * 64)["launches"] == 2


@pytest.mark.parametrize("dtype,most", [(sz.BF16, 2), (sz.FP8_E5M2, 4)])
def test_tiles_where_the_tensors_differ_in_length(dtype, most):
    """Workgroups without a tile cost a launch, too: batches with many of them take the largest tiles, whatever the tiles
    that a launch of their chunks would take; a few do not matter."""
    for chunks in ([13000] + [2] * 63, [32768] + [2] * 63, [8192] + [100] * 63, [8192] * 4 + [200] * 60, [3000] + [2] * 63,
                   [20000] + [2] * 7, [4096] * 32 + [512] * 32, [2] * 63 + [13000] + [5] * 100):
        assert compress_plan(dtype, chunks)["cpt"] == most, chunks
    for chunks in ([600] + [5] * 63, [100] * 40 + [60] * 24, [2048], [49]):
        assert compress_plan(dtype, chunks)["cpt"] == 1, chunks
    # and so do batches to decode
    large = {sz.BF16: 2, sz.FP8_E5M2: 4}[dtype]
    for chunks in ([13000] + [2] * 63, [32768] + [2] * 63, [8192] + [100] * 63, [8192] * 4 + [200] * 60, [3000] + [2] * 63, [20000] + [2] * 7):
        assert decompress_plan(dtype, chunks)["cpw"] >= large, chunks
    for chunks in ([40] * 40 + [20] * 24, [2048], [49]):
        assert decompress_plan(dtype, chunks)["cpw"] == 1, chunks


def test_chunks_per_wave_of_several_streams():
    """A long BF16 stream takes two chunks per wave from 114 688 on, several in a launch from 32 768 on."""
    for chunks in ([512] * 64, [1024] * 64, [8192] * 8, [32768] * 2, [1700] * 64):
        assert decompress_plan(sz.BF16, chunks)["cpw"] == 2, chunks
    for chunks in ([32768], [65536], [100000], [300] * 64, [3000], [40] * 64):
        assert decompress_plan(sz.BF16, chunks)["cpw"] == 1, chunks
    # and a stream that just fills the chip from 5120 on
    assert [decompress_plan(sz.BF16, [c])["cpw"] for c in (4096, 5119, 5120, 16384, 16385)] == [1, 1, 2, 2, 1]


def test_chunks_per_wave_of_streams_with_many_escapes():
    """Above one escape in 16 elements, as the streams' lengths tell, launches that just fill the chip keep to fewer chunks
    per wave; the rule for few escapes holds up to there."""
    def cpw(dtype, chunks, share):
        n = [c * 1024 for c in chunks]
        return sz.internal_decompress_plan(n, dtype, [sz.total_bytes(v, v // share, dtype) for v in n])["cpw"]
    for share in (1, 4, 14):
        assert [cpw(sz.BF16, [c], share) for c in (4096, 6144, 8192, 12288, 16384, 65536)] == [1, 1, 1, 2, 2, 1]
        assert cpw(sz.BF16, [2048] * 4, share) == 1
        assert [cpw(sz.FP8_E5M2, [c], share) for c in (4096, 8192, 12288, 16384, 24576, 65536)] == [1, 1, 2, 2, 4, 4]
    for share in (17, 50, 1000):
        assert [cpw(sz.BF16, [c], share) for c in (4096, 6144, 8192, 12288, 16384, 65536)] == [1, 2, 2, 2, 2, 1]
        assert [cpw(sz.FP8_E5M2, [c], share) for c in (4096, 8192, 12288, 16384, 24576, 65536)] == [1, 2, 2, 4, 4, 4]


def test_occupancy_of_long_launches_with_many_escapes():
    """Long launches have fewer workgroups per CU only where a wave's records fit the run that it asks for ahead."""
    def padded(dtype, chunks, per_chunk):
        n = [c * 1024 for c in chunks]
        p = sz.internal_decompress_plan(n, dtype, [sz.total_bytes(v, v // 1024 * per_chunk, dtype) for v in n])
        return p["lds_pad"] > 0
    for chunks in ([200000], [8192] * 32, [32768] * 64):
        assert [padded(sz.BF16, chunks, q) for q in (0, 1, 32, 63, 65, 200, 1024)] == [True] * 4 + [False] * 3
    for chunks in ([1 << 20], [32768] * 64):
        assert [padded(sz.FP8_E5M2, chunks, q) for q in (0, 1, 16, 27, 29, 100, 1024)] == [True] * 4 + [False] * 3
    for dtype in FORMATS:
        assert not padded(dtype, [2048], 0) and not padded(dtype, [32768], 0)


def test_no_more_chunks_per_wave_than_the_rules_may_choose():
    """Kernels are built for what the rules may choose: single streams up to two (BF16) and four, batches twice that."""
    try:
        for cpw in (1, 2, 4, 8):
            sz.internal_test_launch(cpw=cpw)
            for dtype, most in ((sz.BF16, 2), (sz.FP8_E5M2, 4)):
                assert decompress_plan(dtype, [5000])["cpw"] == min(cpw, most)
                assert decompress_plan(dtype, [5000, 3])["cpw"] == min(cpw, 2 * most)
    finally:
        sz.internal_test_launch()
    for chunks in ([1 << 22], [1 << 22, 1], [1 << 20] + [1] * 63):
        assert decompress_plan(sz.BF16, chunks)["cpw"] <= (4 if len(chunks) > 1 else 2)
        assert decompress_plan(sz.FP8_E5M2, chunks)["cpw"] <= (8 if len(chunks) > 1 else 4)


@pytest.mark.parametrize("dtype", FORMATS)
def test_short_launches_leave_others_the_chip(dtype):
    """A compress launch whose workgroups wait for one another: chunks per wave (0: no such launch) by the tensors' lengths.  Four
    of them, on streams side by side, are resident together, where a tensor has long rows of workgroups, and a stream's own CUs
    are what counts."""
    def short(chunks, cus=256):
        return sz.internal_compress_plan([c * 1024 for c in chunks], dtype, cus)["short"]
    assert [short([c]) for c in (16, 17, 1023, 1024, 1025, 2047, 2048, 2049, 2816, 4096)] == [0, 1, 1, 1, 2, 2, 2, 0, 0, 0]
    assert short([1024] * 2) == 2 and short([1000] * 4) == 0 and short([2000] * 2) == 0
    assert [short([512] * k) for k in (1, 2, 4, 5)] == [1, 1, 1, 0]
    assert [short([32] * k) for k in (2, 64, 65)] == [1, 1, 0] and short([60] * 64) == 0 and short([100] * 16) == 1
    assert [short([c], 32) for c in (100, 128, 129, 256, 257, 1000)] == [1, 1, 2, 2, 0, 0]
    assert [short([c], 128) for c in (512, 513, 1024, 1025)] == [1, 2, 2, 0]
    for cus in (256, 128, 32):
        for chunks in [[c] for c in range(17, 3000, 13)] + [[c] * k for k in (2, 5, 16, 64) for c in range(17, 1500, 37)]:
            cpt = short(chunks, cus)
            if cpt:
                tiles = [-(-c // (4 * cpt)) for c in chunks]
                assert max(tiles) <= min(cus, 256) and sum(tiles) <= (cus if cpt > 1 else 2 * cus), (cus, chunks)
                assert max(tiles) <= cus // 2 or 4 * sum(tiles) <= 5 * cus, (cus, chunks)


@pytest.mark.parametrize("dtype", FORMATS)
def test_short_launches_of_tensors_that_differ_in_length(dtype):
    """Workgroups without a tile: no more than 5000 of them, 3000 where they are larger."""
    def short(chunks):
        return sz.internal_compress_plan([c * 1024 for c in chunks], dtype)["short"]
    assert short([500] + [12] * 40) == 1 and short([1000] + [4] * 20) == 1 and short([1024] + [8] * 10) == 1 and short([1500] + [8] * 10) == 2
    assert short([500] + [12] * 63) == 0 and short([512] + [4] * 159) == 0 and short([1000] + [4] * 40) == 0
    assert [short([1024] + [8] * k) for k in (20, 30, 50)] == [2, 0, 0] and [short([1500] + [8] * k) for k in (15, 20)] == [2, 0]
    assert short([2000] + [12] * 63) == 0 and short([1024] + [40] * 63) == 0


@pytest.mark.parametrize("dtype", FORMATS)
def test_launches_of_more_than_64_tensors(dtype):
    """There are no kernels for so many with more chunks per wave than they take at once, and none of the short ones with two."""
    try:
        for cpt, count in ((1, 70), (2, 70), (4, 64 if dtype == sz.BF16 else 70), (8, 64)):
            sz.internal_test_launch(cpt=cpt)
            assert compress_plan(dtype, [100] * 70)["tensors"] == count, cpt
    finally:
        sz.internal_test_launch()
    for chunks in ([c] + [1] * k for c in range(17, 2049, 11) for k in (64, 65, 80, 100, 159)):
        plan = compress_plan(dtype, chunks)
        assert plan["tensors"] <= 64 or plan["short"] < 2, chunks
