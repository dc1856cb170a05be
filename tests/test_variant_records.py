"""The variants' decoder asks for a chunk's first 64 or 128 escape records before it knows how many there are, narrow values
as two bytes each: blocks with counts around those limits and ragged ends, against the oracle."""
import numpy as np
import pytest
import torch

import paper_2605_01708_amd as sz
from oracle import variants as ov

pytestmark = pytest.mark.gpu

COUNTS = [0, 1, 63, 64, 65, 127, 128, 129, 191, 192, 193, 1024, 0, 5]
# dtype, words of a member and of another exponent, mask of sign and mantissa
FORMATS = {sz.BF16: (np.uint16, 0x3f80, 0x0080, 0x807f), sz.FP8_E5M2: (np.uint8, 0x3c, 0x04, 0x83), sz.FP8_E4M3: (np.uint8, 0x38, 0x08, 0x87)}
DEC = {sz.BF16: range(120, 135), sz.FP8_E5M2: range(8, 23), sz.FP8_E4M3: [5, 6, 7, 8, 9, 10, 11, 12]}
CASES = [(sz.BF16, 3, 8, sz.ESC_POS, 1024, 8), (sz.BF16, 4, 15, sz.ESC_POS, 256, 8), (sz.BF16, 4, 15, sz.ESC_SENTINEL, 1024, 8),
         (sz.FP8_E5M2, 3, 8, sz.ESC_POS, 1024, 5), (sz.FP8_E5M2, 3, 7, sz.ESC_SENTINEL, 256, 5), (sz.FP8_E5M2, 4, 15, sz.ESC_POS, 256, 8),
         (sz.FP8_E4M3, 3, 8, sz.ESC_POS, 1024, 4), (sz.FP8_E4M3, 3, 7, sz.ESC_SENTINEL, 1024, 4), (sz.FP8_E4M3, 3, 8, sz.ESC_ABS32, 1024, 8)]


@pytest.mark.parametrize("dt,bits,k,mode,chunk,vb", CASES)
def test_blocks_with_few_and_many_records(dt, bits, k, mode, chunk, vb):
    v = sz.variant(dt, bits, k, mode, chunk, 0 if vb == 8 else vb)
    o = ov.variant(dt, bits, k, mode, chunk, 0 if vb == 8 else vb)
    np_dt, member, escape, low = FORMATS[dt]
    dec = np.zeros(16, np.uint8)
    dec[:k] = list(DEC[dt])[:k]
    cb = sz.variant_codebook_from_dec(dec[:k], v)
    for last in (1024, 1023, 770, 256, 9, 1):
        rng = np.random.default_rng(last)
        n = (len(COUNTS) - 1) * 1024 + last
        x = rng.integers(0, low + 1, n).astype(np_dt) & np_dt(low) | np_dt(member)
        for c, m in enumerate(COUNTS):
            size = last if c == len(COUNTS) - 1 else 1024
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
