"""Calibration on the device where its work is cut: counts on both sides of 2^31 (32-bit and 64-bit compares), ties,
and batches whose samples share the workgroups of a launch by their lengths."""
import numpy as np
import pytest
import torch

import kv_synth
import paper_2605_01708_amd as sz

pytestmark = pytest.mark.gpu


def same_tables(dcb, ref):
    h = dcb.to_host()
    return (h.dec, h.enc, h.member, h.dtype) == (ref.dec, ref.enc, ref.member, ref.dtype)


@pytest.mark.parametrize("dtype,n", [(sz.BF16, 256), (sz.FP8_E5M2, 32)])
def test_ranking_of_counts(dtype, n):
    rng = np.random.default_rng(1)
    cases = [np.zeros(n, np.int64), np.full(n, 7), np.arange(n), np.arange(n)[::-1].copy(), rng.integers(0, 3, n),
             rng.integers(0, 1 << 31, n), rng.integers((1 << 31) - 3, (1 << 31) + 3, n), rng.integers(0, 1 << 62, n),
             (1 << 31) - 1 - rng.integers(0, 2, n), (1 << 32) + rng.integers(0, 2, n), rng.permutation(n) << 40]
    for k, c in enumerate(cases):
        hist = torch.zeros(256, dtype=torch.int64)
        hist[:n] = torch.from_numpy(np.asarray(c, np.int64))
        ref = sz.codebook_from_hist(hist, dtype)
        assert same_tables(sz.codebook_device(hist.cuda(), dtype), ref), f"case {k}"


@pytest.mark.parametrize("dtype", [sz.BF16, sz.FP8_E5M2])
@pytest.mark.parametrize("sizes", [[0], [1], [0, 0, 5], [3000000, 1, 0, 17, 4096], [70000 * k + 13 for k in range(64)],
                                   [8191, 8192, 8193] * 30, [16 * 1024 * 4 * 3 + 5, 12],
                                   [1 << 18] * 9 + [(1 << 18) + 13] * 8, [65535, 65536, 65537, 32767, 32769] * 4])
def test_batches_count_every_word_once(dtype, sizes):
    gen = kv_synth.kv_bf16 if dtype == sz.BF16 else kv_synth.kv_e5m2
    pool = gen(max(sizes) // 1024 + 2, 9, device="cuda")
    xs = [pool[:s].clone() for s in sizes]
    dcbs = sz.DeviceCodebooks(len(xs), dtype)
    dcbs.hists.fill_(-1)                      # the call clears them
    sz.CalibrateBatchDevice(xs, dcbs).launch()
    torch.cuda.synchronize()
    shift, mask = (7, 255) if dtype == sz.BF16 else (2, 31)
    for k, x in enumerate(xs):
        e = (x.to(torch.int32) >> shift) & mask
        want = torch.bincount(e.long(), minlength=256)
        assert torch.equal(dcbs.hists[k], want), k
        host = dcbs.to_host(k)
        assert host.dec == sz.codebook_from_hist(want.cpu(), dtype).dec
        assert torch.equal(sz.histogram(x, dtype), want)
