"""The decoder takes the escape records of a wave's chunks as one run, the first 128 of it in registers: streams whose runs
and chunks begin and end around those limits, at every number of chunks per wave, and tables that are not in order."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_01708_amd as sz

FORMATS = [(sz.BF16, np.uint16, 0x3f80, 0x0080), (sz.FP8_E5M2, np.uint8, 0x3c, 0x04)]   # words of a member and of another exponent


def _words(counts, last, dtype, np_dt, member, escape, seed):
    """counts[c] escapes in chunk c, the last chunk `last` words long; every word has sign and mantissa bits of its own"""
    rng = np.random.default_rng(seed)
    low = 0x7f if dtype == sz.BF16 else 0x3
    sign = 0x8000 if dtype == sz.BF16 else 0x80
    n = (len(counts) - 1) * 1024 + last
    x = (member | rng.integers(0, low + 1, n)).astype(np_dt)
    for c, k in enumerate(counts):
        size = last if c == len(counts) - 1 else 1024
        at = c * 1024 + rng.choice(size, min(k, size), replace=False)
        x[at] = (x[at] & low) | (escape * rng.integers(0, 2, at.size).astype(np_dt))   # exponents 0 and 1
    return (x | np.where(rng.integers(0, 2, n), sign, 0).astype(np_dt)).astype(np_dt)


def _codebook(dtype):
    # 16 exponents around the member's, neither 0 nor 1
    return sz.codebook_from_dec(range(120, 136) if dtype == sz.BF16 else range(8, 24), dtype)


COUNTS = {
    "around_64": [63, 1, 0, 64, 0, 65, 1, 2, 62, 1, 1, 64, 64, 0, 0, 66, 5],
    "around_128": [127, 1, 128, 0, 129, 3, 64, 64, 64, 1, 126, 2, 1, 127, 0, 128, 130],
    "few_then_many": [1, 1, 1, 125, 1, 1, 1, 126, 0, 3, 0, 1024, 1, 0, 0, 2, 3],
    "many": [1024, 1023, 385, 384, 383, 257, 256, 255, 641, 128, 1024, 1024, 5, 1024, 0, 700, 800],
    "none": [0] * 9,
}


@pytest.mark.gpu
@pytest.mark.parametrize("cpw", [1, 2, 4, 8])
@pytest.mark.parametrize("case", sorted(COUNTS))
@pytest.mark.parametrize("dtype,np_dt,member,escape", FORMATS)
def test_runs_of_records(dtype, np_dt, member, escape, case, cpw):
    cb = _codebook(dtype)
    for last in (1024, 1023, 682, 681, 9, 1):
        x = _words(COUNTS[case], last, dtype, np_dt, member, escape, 7 * cpw + last)
        ref, _ = oracle.compress(x, oracle.Codebook(cb.dec, cb.enc, cb.member, dtype))
        xd = torch.from_numpy(x.view(np.int16) if dtype == sz.BF16 else x).cuda()
        out = torch.zeros(sz.compress_bound(x.size, dtype), dtype=torch.uint8, device="cuda")
        rec, drec = sz.new_sizes(), sz.new_sizes()
        sz.compress(xd, cb, out, sz.Workspace(x.size, dtype), rec)
        total, m, status = sz.read_sizes(rec)
        assert status == 0 and np.array_equal(out[:total].cpu().numpy(), ref)
        try:
            sz.internal_test_launch(cpw=cpw)
            for batch in (False, True):
                y = torch.full((x.size + 64,), 0x55, dtype=xd.dtype, device="cuda")
                drec.zero_()
                if batch:
                    sz.DecompressBatch([out, out], [total, total], [x.size] * 2, [cb] * 2, [y, torch.empty_like(y)]).launch(drec)
                else:
                    sz.decompress(out, total, x.size, cb, y, drec)
                torch.cuda.synchronize()
                assert sz.read_sizes(drec) == (total, m, 0)
                assert torch.equal(y[:x.size], xd) and (y[x.size:] == 0x55).all()
        finally:
            sz.internal_test_launch()


@pytest.mark.gpu
@pytest.mark.parametrize("cpw", [1, 2, 4])
@pytest.mark.parametrize("dtype,np_dt,member,escape", FORMATS)
def test_tables_that_are_not_in_order(dtype, np_dt, member, escape, cpw):
    """Chunks with inconsistent entries are decoded without their records and flagged; the others are right."""
    cb = _codebook(dtype)
    counts = [3, 70, 2, 130, 0, 4, 1, 90, 2, 2]
    x = _words(counts, 1000, dtype, np_dt, member, escape, 3)
    xd = torch.from_numpy(x.view(np.int16) if dtype == sz.BF16 else x).cuda()
    out = torch.zeros(sz.compress_bound(x.size, dtype), dtype=torch.uint8, device="cuda")
    rec, drec = sz.new_sizes(), sz.new_sizes()
    sz.compress(xd, cb, out, sz.Workspace(x.size, dtype), rec)
    total, m, _ = sz.read_sizes(rec)
    start = np.concatenate([[0], np.cumsum(counts)]).astype(np.uint32)
    assert m == start[-1] and np.array_equal(out[64:64 + 4 * start.size].cpu().numpy().view(np.uint32), start)
    for entry, value in ((0, 5), (1, 0), (2, 1), (3, 0xffffffff), (4, m + 1), (5, 0), (8, 2 ** 31), (9, 7), (len(counts), 3), (len(counts), 0xffffffff)):
        bad = start.copy()
        bad[entry] = value
        s = out.clone()
        s[64:64 + 4 * bad.size] = torch.from_numpy(bad.view(np.uint8)).cuda()
        y = torch.zeros_like(xd)
        drec.zero_()
        try:
            sz.internal_test_launch(cpw=cpw)
            sz.decompress(s, total, x.size, cb, y, drec)
            torch.cuda.synchronize()
        finally:
            sz.internal_test_launch()
        assert sz.read_sizes(drec)[2] & sz.STATUS_BAD_STREAM
        got, all_m = y.cpu().numpy().view(np_dt), int(bad[-1]) if bad[-1] <= m else 0
        for c in range(len(counts)):
            lo, hi = int(bad[c]), int(bad[c + 1])
            size = 1000 if c == len(counts) - 1 else 1024
            # right where a chunk's entries are its own, and where it has no records and its entries cannot be followed (with
            # another M the values lie elsewhere)
            refused = hi < lo or hi - lo > size or hi > all_m
            own = (lo, hi) == (start[c], start[c + 1]) and not refused and (entry < len(counts) or lo == hi)
            if own or refused and counts[c] == 0:
                assert np.array_equal(got[c * 1024:c * 1024 + size], x[c * 1024:c * 1024 + size]), (entry, c)


@pytest.mark.parametrize("dtype", [sz.BF16, sz.FP8_E5M2])
def test_room_for_records_by_the_length_of_a_stream(dtype):
    """The most records that a stream of a length holds, worked out in closed form on the host: the largest m whose total fits."""
    for n in (0, 1, 5, 1000, 5000, 123456, 2 ** 32 - 1):
        fixed, m = sz.fixed_bytes(n, dtype), 0
        for more in range(2000):
            while m < n and sz.total_bytes(n, m + 1, dtype) <= fixed + more:
                m += 1
            assert sz.internal_stream_room(fixed + more, n, dtype) == m
        for m in (n // 7, n // 2, n - 129, n - 128, n - 1, n):
            if m > 0:
                total = sz.total_bytes(n, m, dtype)
                assert sz.internal_stream_room(total, n, dtype) == m
                assert sz.internal_stream_room(total - 1, n, dtype) < m
        assert sz.internal_stream_room(sz.compress_bound(n, dtype) + 10 ** 12, n, dtype) == n


@pytest.mark.gpu
@pytest.mark.parametrize("m", [1, 126, 127, 128, 129, 130, 255, 256, 257, 1024])
@pytest.mark.parametrize("dtype,np_dt,member,escape", FORMATS)
def test_streams_that_are_cut_short(dtype, np_dt, member, escape, m):
    """A stream decoded by its own length is right; one byte less than it takes, and it is flagged and its records, whose
    sections reach over the end, are left alone: the words come out as the planes have them."""
    cb = _codebook(dtype)
    x = _words([m // 2, m - m // 2, 0], 77, dtype, np_dt, member, escape, m)
    xd = torch.from_numpy(x.view(np.int16) if dtype == sz.BF16 else x).cuda()
    out = torch.full((sz.compress_bound(x.size, dtype) + 4096,), 0xff, dtype=torch.uint8, device="cuda")   # allocated beyond the stream's end
    rec, drec = sz.new_sizes(), sz.new_sizes()
    sz.compress(xd, cb, out, sz.Workspace(x.size, dtype), rec, capacity=sz.compress_bound(x.size, dtype))
    total, got_m, status = sz.read_sizes(rec)
    assert (got_m, status) == (m, 0) and total == sz.total_bytes(x.size, m, dtype)
    # escapes have the dummy code, that of the codebook's first exponent
    low, shift = (0x807f, 7) if dtype == sz.BF16 else (0x83, 2)
    exps = (x.astype(np.uint32) >> shift) & (0xff if dtype == sz.BF16 else 0x1f)
    planes = np.where(exps < 2, (x & low) | (cb.dec[0] << shift), x).astype(np_dt)
    for cut, want in ((0, x), (1, planes)):
        for batch in (False, True):
            y = torch.full((x.size + 64,), 0x55, dtype=xd.dtype, device="cuda")
            drec.zero_()
            if batch:
                sz.DecompressBatch([out, out], [total, total - cut], [x.size] * 2, [cb] * 2, [torch.empty_like(y), y]).launch(drec)
            else:
                sz.decompress(out, total - cut, x.size, cb, y, drec)
            torch.cuda.synchronize()
            assert sz.read_sizes(drec) == (total, m, sz.STATUS_BAD_STREAM if cut else 0)
            assert np.array_equal(y[:x.size].cpu().numpy().view(np_dt), want) and (y[x.size:] == 0x55).all()
