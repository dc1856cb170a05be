"""The variants' decoder asks for a chunk's first 64 or 128 escape records before it knows how many there are and for the others
256 at a time, narrow values as two bytes each: blocks with counts around those limits and ragged ends, against the oracle."""
import numpy as np
import pytest
import torch

import paper_2605_01708_amd as sz
from oracle import variants as ov

pytestmark = pytest.mark.gpu

COUNTS = [0, 1, 63, 64, 65, 127, 128, 129, 191, 192, 193, 1024, 0, 5]
MORE = [319, 320, 321, 383, 384, 385, 447, 448, 449, 639, 640, 641, 0, 895, 896, 897, 1023, 900]   # the rest comes 256 at a time
# dtype, words of a member and of another exponent, mask of sign and mantissa
FORMATS = {sz.BF16: (np.uint16, 0x3f80, 0x0080, 0x807f), sz.FP8_E5M2: (np.uint8, 0x3c, 0x04, 0x83), sz.FP8_E4M3: (np.uint8, 0x38, 0x08, 0x87)}
DEC = {sz.BF16: range(120, 135), sz.FP8_E5M2: range(8, 23), sz.FP8_E4M3: [5, 6, 7, 8, 9, 10, 11, 12]}
CASES = [(sz.BF16, 3, 8, sz.ESC_POS, 1024, 8), (sz.BF16, 4, 15, sz.ESC_POS, 256, 8), (sz.BF16, 4, 15, sz.ESC_SENTINEL, 1024, 8),
         (sz.FP8_E5M2, 3, 8, sz.ESC_POS, 1024, 5), (sz.FP8_E5M2, 3, 7, sz.ESC_SENTINEL, 256, 5), (sz.FP8_E5M2, 4, 15, sz.ESC_POS, 256, 8),
         (sz.FP8_E4M3, 3, 8, sz.ESC_POS, 1024, 4), (sz.FP8_E4M3, 3, 7, sz.ESC_SENTINEL, 1024, 4), (sz.FP8_E4M3, 3, 8, sz.ESC_ABS32, 1024, 8)]


@pytest.mark.parametrize("counts", [COUNTS, MORE], ids=["few", "many"])
@pytest.mark.parametrize("dt,bits,k,mode,chunk,vb", CASES)
def test_blocks_with_few_and_many_records(dt, bits, k, mode, chunk, vb, counts):
    v = sz.variant(dt, bits, k, mode, chunk, 0 if vb == 8 else vb)
    o = ov.variant(dt, bits, k, mode, chunk, 0 if vb == 8 else vb)
    np_dt, member, escape, low = FORMATS[dt]
    dec = np.zeros(16, np.uint8)
    dec[:k] = list(DEC[dt])[:k]
    cb = sz.variant_codebook_from_dec(dec[:k], v)
    for last in (1024, 1023, 770, 256, 9, 1):
        rng = np.random.default_rng(last)
        n = (len(counts) - 1) * 1024 + last
        x = rng.integers(0, low + 1, n).astype(np_dt) & np_dt(low) | np_dt(member)
        for c, m in enumerate(counts):
            size = last if c == len(counts) - 1 else 1024
            at = c * 1024 + rng.choice(size, min(m, size), replace=False)
            x[at] = x[at] & np_dt(low) | (np_dt(escape) * rng.integers(0, 2, at.size).astype(np_dt))
        ref, m = ov.compress(x, o, dec)
        out = torch.full((sz.variant_compress_bound(n, v),), 0xA5, dtype=torch.uint8, device="cuda")
        ws = torch.empty(sz.variant_workspace_bytes(n, v), dtype=torch.uint8, device="cuda")
        rec, st = sz.new_sizes(), sz.new_sizes()
        xd = torch.from_numpy(x.view(np.int16) if dt == sz.BF16 else x).cuda()
        sz.variant_compress(xd, v, cb, out, ws, rec)
        assert sz.read_sizes(rec) == (ref.size, m, 0) and np.array_equal(out[:ref.size].cpu().numpy(), ref)
        y = torch.full((n + 64,), 0x55, dtype=xd.dtype, device="cuda")
        sz.variant_decompress(out, ref.size, n, v, cb, y, st)
        assert sz.read_sizes(st) == (ref.size, m, 0)
        assert torch.equal(y[:n], xd) and (y[n:] == 0x55).all()


@pytest.mark.parametrize("dt", [sz.BF16, sz.FP8_E5M2, sz.FP8_E4M3])
def test_positions_out_of_order_in_every_round(dt):
    """Two records of a chunk the wrong way round, at the edges of the rounds that records are taken in: the one that does not
    ascend is left out and flagged, the others are applied."""
    v = sz.variant(dt, 3, 8, sz.ESC_POS, 1024, 0)
    np_dt, member, escape, low = FORMATS[dt]
    cb = sz.variant_codebook_from_dec(list(DEC[dt])[:8], v)
    n, m = 2 * 1024, 900
    rng = np.random.default_rng(3)
    x = rng.integers(0, low + 1, n).astype(np_dt) & np_dt(low) | np_dt(member)
    at = 1024 + np.sort(rng.choice(1024, m, replace=False))
    unit = {sz.BF16: 0x80, sz.FP8_E5M2: 4, sz.FP8_E4M3: 8}[dt]   # an exponent's lowest bit
    x[at] = x[at] & np_dt(low) | np_dt(unit) * rng.integers(0, 3, m).astype(np_dt)   # exponents 0 to 2
    xd = torch.from_numpy(x.view(np.int16) if dt == sz.BF16 else x).cuda()
    out = torch.zeros(sz.variant_compress_bound(n, v), dtype=torch.uint8, device="cuda")
    ws = torch.empty(sz.variant_workspace_bytes(n, v), dtype=torch.uint8, device="cuda")
    rec, st = sz.new_sizes(), sz.new_sizes()
    sz.variant_compress(xd, v, cb, out, ws, rec)
    total, got_m, status = sz.read_sizes(rec)
    assert (got_m, status) == (m, 0)
    pos_at = sz.variant_total_bytes(n, 0, v)   # the positions follow the fixed part
    stream = out[:total].cpu().numpy().copy()
    pos = stream[pos_at:pos_at + 2 * m].view(np.uint16)
    assert np.array_equal(pos, at - 1024)
    for i in (1, 63, 64, 65, 127, 128, 129, 191, 192, 193, 319, 320, 383, 384, 385, 448, 639, 640, 641, 899):
        bad = stream.copy()
        p = bad[pos_at:pos_at + 2 * m].view(np.uint16)
        p[i - 1], p[i] = pos[i], pos[i - 1]
        want = x.copy()
        want[at[i]] = x[at[i]] & np_dt(low) | x[at[i - 1]] & np_dt(~low & (0x7fff if dt == sz.BF16 else 0x7f))
        want[at[i - 1]] = x[at[i - 1]] & np_dt(low) | np_dt(unit) * np_dt(DEC[dt][0])
        y = torch.zeros_like(xd)
        st.zero_()
        sz.variant_decompress(torch.from_numpy(bad).cuda(), total, n, v, cb, y, st)
        assert sz.read_sizes(st) == (total, m, sz.STATUS_BAD_STREAM)
        assert np.array_equal(y.cpu().numpy().view(np_dt), want), i
