"""The variant kernels where their work is cut: escape counts around what the finishing pass fetches of a block's slot
at a time (16 or 64 records ahead, 64 more behind the counts, 128 in the slot, more: encoded once more), and tensors
of more workgroups than it sums up itself."""
import numpy as np
import pytest
import torch

import kv_synth
from oracle import variants as ov
import paper_2605_01708_amd as sz
from test_variants import Run, check, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt,cb,k,mode,chunk,vb", [
    (sz.BF16, 4, 16, sz.ESC_POS, 1024, 0), (sz.BF16, 3, 8, sz.ESC_POS, 256, 0), (sz.BF16, 4, 15, sz.ESC_SENTINEL, 256, 0),
    (sz.BF16, 3, 8, sz.ESC_ABS32, 0, 0), (sz.FP8_E5M2, 3, 7, sz.ESC_SENTINEL, 1024, 0), (sz.FP8_E4M3, 3, 8, sz.ESC_POS, 1024, 4)])
def test_escape_counts_at_the_edges_of_a_slot(dt, cb, k, mode, chunk, vb):
    v = sz.variant(dt, cb, k, mode, chunk, vb)
    o = ov.variant(dt, cb, k, mode, chunk, vb)
    counts = [0, 1, 2, 15, 16, 17, 31, 32, 63, 64, 65, 79, 80, 81, 127, 128, 129, 255, 256, 257, 1023, 1024]
    rng = np.random.default_rng(5)
    shift, nexp = {sz.BF16: (7, 256), sz.FP8_E5M2: (2, 32), sz.FP8_E4M3: (3, 16)}[dt]
    dec = np.zeros(16, np.uint8)
    dec[:k] = rng.permutation(nexp)[:k]
    others = np.setdiff1d(np.arange(nexp), dec[:k])
    blocks = []
    for c in counts + counts[::-1]:                      # 44 blocks: two workgroups of the finishing pass, one not full
        e = dec[rng.integers(0, k, 1024)].astype(np.uint32)
        at = np.sort(rng.permutation(1024)[:c])
        if c > 1:
            at[0], at[-1] = 0, 1023                      # the ends of the block among them
        e[at] = others[rng.integers(0, others.size, c)]
        word = (e << shift) | rng.integers(0, 1 << shift, 1024, dtype=np.uint32)
        sign = rng.integers(0, 2, 1024, dtype=np.uint32) << (15 if dt == sz.BF16 else 7)
        blocks.append((word | sign).astype(np.uint16 if dt == sz.BF16 else np.uint8))
    x = np.concatenate(blocks)
    run = Run(x.size, v)
    check(run, o, x, dec, "edges")
    check(run, o, x[:-1021].copy(), dec, "edges, ragged")


@pytest.mark.parametrize("chunk", [1024, 256])
def test_tensors_of_many_workgroups(chunk):
    """Above 64 Mi elements the counts are summed by a launch of their own.  The bytes behind the header are those of
    the main format's calls (for 256-element chunks: the planes, and every fourth entry of the table)."""
    n = 16384 * 4096 + 5003
    x = kv_synth.kv_e5m2(n // 1024 + 1, 3, device="cuda")[:n].contiguous()
    v = sz.variant(sz.FP8_E5M2, 4, 16, sz.ESC_POS, chunk)
    cb = sz.calibrate(kv_synth.kv_e5m2(64, 1), sz.FP8_E5M2)
    cbv = sz.variant_codebook_from_dec(cb.dec, v)
    most = n // 50
    main = torch.zeros(sz.total_bytes(n, most, sz.FP8_E5M2), dtype=torch.uint8, device="cuda")
    ws, rec = sz.Workspace(n, sz.FP8_E5M2), sz.new_sizes()
    sz.compress(x, cb, main, ws, rec)
    total, m, status = sz.read_sizes(rec)
    assert status == 0 and m > 0
    out = torch.zeros(sz.variant_total_bytes(n, most, v), dtype=torch.uint8, device="cuda")
    wsv = torch.full((sz.variant_workspace_bytes(n, v),), 0x3C, dtype=torch.uint8, device="cuda")
    sz.variant_compress(x, v, cbv, out, wsv, rec)
    vt, vm, status = sz.read_sizes(rec)
    assert (vt, vm, status) == (sz.variant_total_bytes(n, m, v), m, 0)
    a256 = lambda b: (b + 255) // 256 * 256  # noqa: E731
    chunks = -(-n // 1024)
    off_main = a256(64 + 4 * (chunks + 1))
    if chunk == 1024:
        assert vt == total and torch.equal(out[64:vt], main[64:total])
    else:
        off = a256(64 + 4 * (-(-n // 256) + 1))
        planes = a256((3 * n + 7) // 8) + a256((n + 1) // 2)
        assert torch.equal(out[off:off + planes], main[off_main:off_main + planes])
        tab = out[64:64 + 4 * (-(-n // 256) + 1)].view(torch.int32)
        tab_main = main[64:64 + 4 * (chunks + 1)].view(torch.int32)
        assert torch.equal(tab[::4][:chunks], tab_main[:chunks]) and int(tab[-1]) == m
        assert torch.equal(out[vt - m:vt], main[total - m:total])       # the values
    y, st = torch.empty_like(x), sz.new_sizes()
    sz.variant_decompress(out, vt, n, v, cbv, y, st)
    assert sz.read_sizes(st)[2] == 0 and torch.equal(y, x)


@pytest.mark.parametrize("dt,cb,k,chunk,vb", [(sz.BF16, 4, 15, 1024, 0), (sz.BF16, 4, 10, 256, 0), (sz.BF16, 3, 7, 1024, 0), (sz.FP8_E5M2, 4, 15, 256, 0),
                                              (sz.FP8_E5M2, 3, 7, 1024, 5), (sz.FP8_E5M2, 3, 5, 256, 5), (sz.FP8_E4M3, 4, 12, 1024, 4), (sz.FP8_E4M3, 3, 7, 256, 0)])
def test_both_ways_to_put_sentinels_right(dt, cb, k, chunk, vb):
    """A stream longer than a quarter or half of its elements escaped would make it is decoded by another kernel; the
    length given decides, so any stream can be sent both ways: the same words, and the same verdict on what is wrong."""
    v, o = sz.variant(dt, cb, k, sz.ESC_SENTINEL, chunk, vb), ov.variant(dt, cb, k, ov.ESC_SENTINEL, chunk, vb)
    rng = np.random.default_rng(11)
    bits, raw = (16, np.uint16) if dt == sz.BF16 else (8, np.uint8)
    random = rng.integers(0, 1 << bits, 9 * 1024, dtype=np.uint32).astype(raw)
    gen = {sz.BF16: kv_synth.kv_bf16, sz.FP8_E5M2: kv_synth.kv_e5m2, sz.FP8_E4M3: kv_synth.kv_e4m3}[dt]
    usual = kv_synth.to_numpy_words(gen(9, 4)).copy()
    dec, _ = ov.calibrate(usual, o.dtype, k)
    mixed = np.where((np.arange(usual.size) // 64) % 3 == 0, random, usual).astype(raw)
    for name, x in (("usual", usual), ("random", random), ("mixed", mixed)):
        for n in (x.size, x.size - 1021, 7, 1024):
            blob, m = ov.compress(x[:n].copy(), o, dec)
            cbv = sz.variant_codebook_from_dec(list(dec), v)
            bound = sz.variant_compress_bound(n, v)
            buf = torch.zeros(bound, dtype=torch.uint8, device="cuda")
            buf[:blob.size] = dev(blob)

            def decode(stream, length):
                y, st = torch.full((n + 64,), 0x5A, dtype=torch.int16 if dt == sz.BF16 else torch.uint8, device="cuda"), sz.new_sizes()
                sz.variant_decompress(stream, length, n, v, cbv, y, st)
                return y, sz.read_sizes(st)

            for length in (blob.size, bound):
                y, (total, got_m, status) = decode(buf, length)
                print(f"case {name} n={n} m={m} length={length}", flush=True)
                assert (total, got_m, status) == (blob.size, m, 0)
                assert np.array_equal(y[:n].cpu().numpy().view(raw), x[:n]) and bool((y[n:] == 0x5A).all())
            # wrong streams: an offset moved, codes turned into sentinels without a value
            off_sm = (64 + 4 * (-(-n // chunk) + 1) + 255) // 256 * 256
            sm_bytes = (n * {sz.BF16: 8, sz.FP8_E5M2: 3, sz.FP8_E4M3: 4}[dt] + 7) // 8
            off_code = off_sm + (sm_bytes + 255) // 256 * 256
            for at, byte in ((64, 1), (67, 0x80), (off_code, 0xFF), (off_code + n * cb // 16, 0xFF)):
                bad = buf.clone()
                bad[at] = byte
                assert decode(bad, blob.size)[1] == decode(bad, bound)[1], (name, n, at)


@pytest.mark.parametrize("chunks,share", [(65532, 0.0), (65533, 0.0), (65533, 0.05), (65533, 0.2), (98304, 0.0)])
def test_long_streams_of_4_bit_codes(chunks, share):
    """BF16 streams of 16 384 workgroups and more, with few escapes, are decoded with fewer workgroups per CU."""
    n = chunks * 1024 - 7
    x = kv_synth.kv_bf16(chunks, 1, device="cuda").view(-1)[:n].view(torch.int16)
    if share:
        x = torch.where(torch.rand(n, device="cuda") < share, torch.randint(-32768, 32767, (n,), dtype=torch.int16, device="cuda"), x)
    x = x.contiguous()
    v = sz.variant(sz.BF16, 4, 16, sz.ESC_POS, 1024)
    cb = sz.variant_codebook_from_dec(sz.calibrate(kv_synth.kv_bf16(64, 1), sz.BF16).dec, v)
    out = torch.zeros(sz.variant_total_bytes(n, n // 4, v), dtype=torch.uint8, device="cuda")
    ws = torch.empty(sz.variant_workspace_bytes(n, v), dtype=torch.uint8, device="cuda")
    rec, st = sz.new_sizes(), sz.new_sizes()
    sz.variant_compress(x, v, cb, out, ws, rec)
    total, m, status = sz.read_sizes(rec)
    assert status == 0 and (m > n // 16) == (share > 0.1)
    for comp_bytes in (total, out.numel()):
        y = torch.full((n + 64,), 0x55, dtype=torch.int16, device="cuda")
        st.zero_()
        sz.variant_decompress(out, comp_bytes, n, v, cb, y, st)
        assert sz.read_sizes(st) == (total, m, 0)
        assert torch.equal(y[:n], x) and (y[n:] == 0x55).all()
