"""Compress calls of one launch whose workgroups tell one another their counts: the oracle's streams at the edges of its
range and of its tiles of four chunks, in workspaces that hold anything, where workgroups leave their tiles to others, and
byte for byte what the two launches leave where the stream does not fit."""
import numpy as np
import pytest
import torch

import kv_synth
import oracle
import paper_2605_01708_amd as sz
from conftest import LEAVE

pytestmark = pytest.mark.gpu
FORMATS = [(sz.BF16, oracle.BF16), (sz.FP8_E5M2, oracle.E5M2)]


def words(dtype, n, seed, escapes="few"):
    gen = kv_synth.kv_bf16 if dtype == sz.BF16 else kv_synth.kv_e5m2
    x = gen(n // 1024 + 1, seed)[:n].contiguous()
    if escapes == "few":
        return x
    rng = np.random.default_rng(seed)   # random patterns: nearly all escape; "many": in every third chunk
    r = torch.from_numpy(rng.integers(0, 1 << (16 if dtype == sz.BF16 else 8), n).astype(np.uint16 if dtype == sz.BF16 else np.uint8).view(np.int16 if dtype == sz.BF16 else np.uint8))
    return r if escapes == "all" else torch.where((torch.arange(n) // 1024) % 3 == 0, r, x)


def books(dtype, odt):
    sample = words(dtype, 64 * 1024, 1)
    return sz.calibrate(sample, dtype), oracle.calibrate(kv_synth.to_numpy_words(sample), odt)


def compress(x, cb, cap=None, ws=None):
    cap = sz.compress_bound(x.numel(), cb.dtype) if cap is None else cap
    out = torch.full((cap + 512,), 0xA5, dtype=torch.uint8, device="cuda")
    ws, rec = sz.Workspace(x.numel(), cb.dtype) if ws is None else ws, sz.new_sizes()
    sz.compress(x.cuda(), cb, out, ws, rec, capacity=cap)
    return out, sz.read_sizes(rec)


def check(x, cb, ocb, ws=None):
    blob, m = oracle.compress(kv_synth.to_numpy_words(x), ocb)
    out, got = compress(x, cb, ws=ws)
    assert got == (blob.size, m, 0)
    assert np.array_equal(out[:blob.size].cpu().numpy(), blob) and bool((out[blob.size:] == 0xA5).all())


@pytest.mark.parametrize("dtype,odt", FORMATS)
@pytest.mark.parametrize("chunks", [16, 17, 49, 52, 255, 257, 1023, 1024, 1025, 2047, 2048, 2049])
def test_streams_at_the_edges(dtype, odt, chunks, looks):
    """Lengths around a whole tile, around where a wave has two chunks and around the range's end, with few, many and all words
    escaping; each also with workgroups that leave their tiles to others, and in two launches."""
    cb, ocb = books(dtype, odt)
    for n in (chunks * 1024, chunks * 1024 - 3):
        for escapes in ("few", "many", "all") if chunks < 1000 else ("few", "many"):
            x = words(dtype, n, 3, escapes)
            for limit in (0, LEAVE, sz.INTERNAL_NO_SHORT):
                print(f"case {dtype} n={n} {escapes} looks={limit}", flush=True)
                with looks(limit):
                    check(x, cb, ocb)


@pytest.mark.parametrize("dtype,odt", FORMATS)
def test_two_chunks_a_wave(dtype, odt, looks):
    """Tensors of more than 256 tiles of four chunks have half as many of eight: odd ends, the range's end and one word beyond it,
    every way for a wave's records, alone and with short ones."""
    cb, ocb = books(dtype, odt)
    for n in (1024 * 1024 + 1, 1031 * 1024, 1500 * 1024 - 1025, 2048 * 1024, 2048 * 1024 + 1):
        for escapes in ("many", "all"):
            for limit in (0, 1, LEAVE):
                print(f"case {dtype} n={n} {escapes} looks={limit}", flush=True)
                with looks(limit):
                    check(words(dtype, n, 3, escapes), cb, ocb)
    sizes = [1500 * 1024 - 7, 0, 300 * 1024, 16 * 1024, 9 * 1024 + 1]
    xs = [words(dtype, n, 11 + k) for k, n in enumerate(sizes)]
    assert sz.internal_compress_plan(sizes, dtype)["short"] == 2
    for limit in (0, LEAVE):
        outs = [torch.full((sz.compress_bound(n, dtype) + 256,), 0xA5, dtype=torch.uint8, device="cuda") for n in sizes]
        ws, rec = sz.Workspace(max(sizes), dtype), sz.new_sizes_array(len(xs))
        with looks(limit):
            sz.compress_batch([x.cuda() for x in xs], [cb] * len(xs), outs, ws, rec)
        for x, out, got in zip(xs, outs, sz.read_sizes_array(rec)):
            blob, m = oracle.compress(kv_synth.to_numpy_words(x), ocb)
            assert got == (blob.size, m, 0) and np.array_equal(out[:blob.size].cpu().numpy(), blob) and bool((out[blob.size:] == 0xA5).all())


@pytest.mark.parametrize("dtype,odt", FORMATS)
@pytest.mark.parametrize("chunks", [300, 1024, 1100, 2048])
def test_tiles_left_and_taken(dtype, odt, chunks, looks):
    """Workgroups leave their tiles to those that come after them, which encode them again: out of pages, under a
    codebook in device memory.  The words in the workspace tell of every tile whether it was left and, if so, taken."""
    n, page = chunks * 1024 - 5, 4096
    pages, es = -(-n // page), 2 if dtype == sz.BF16 else 1
    table = torch.randperm(pages, generator=torch.Generator().manual_seed(4)).to(torch.int32)
    pool = words(dtype, pages * page, 3, "many").cuda()
    x = pool.view(pages, page)[table.long().cuda()].reshape(-1)[:n].contiguous()
    d = sz.DeviceCodebooks(1, dtype)
    sz.CalibrateBatchDevice([x], d).launch()
    cb, ocb = d.to_host(0), oracle.calibrate(kv_synth.to_numpy_words(x.cpu()), odt)
    blob, m = oracle.compress(kv_synth.to_numpy_words(x.cpu()), ocb)
    ws, tiles = sz.Workspace(n, dtype), -(-chunks // (4 if chunks <= 1024 else 8))
    for limit in (0, 1, LEAVE):
        for how in ("pages", "device codebook"):
            out, rec = torch.full((blob.size + 512,), 0xA5, dtype=torch.uint8, device="cuda"), sz.new_sizes()
            paged = sz.Paged(pool, table.cuda(), page, page * es)
            with looks(limit):
                if how == "pages":
                    sz.compress_paged(paged, n, cb, out, ws, rec)
                else:
                    sz.CompressBatchDcb([x], d, [out]).launch(ws, rec.view(1, 3))
            assert sz.read_sizes(rec) == (blob.size, m, 0), (limit, how)
            assert np.array_equal(out[:blob.size].cpu().numpy(), blob) and bool((out[blob.size:] == 0xA5).all())
            told = ws.buf[512:512 + 8 * tiles].view(torch.int64).cpu()
            was_left, was_taken = (told & 0x8000) != 0, (told & 0x10000) != 0
            assert torch.equal(was_left, was_taken)
            left = int(was_left.sum())
            print(f"case {dtype} chunks={chunks} {how}: {left} of {tiles} tiles left", flush=True)
            assert limit != LEAVE or left > 0


@pytest.mark.parametrize("dtype,odt", FORMATS)
def test_streams_side_by_side(dtype, odt):
    """Several streams, each with a workspace of its own, keep short launches in flight together."""
    cb, ocb = books(dtype, odt)
    for n in (100 * 1024, 1024 * 1024, 2048 * 1024 - 5):
        x = words(dtype, n, 3)
        blob, m = oracle.compress(kv_synth.to_numpy_words(x), ocb)
        xd, want = x.cuda(), torch.from_numpy(blob).cuda()
        lanes = [(torch.cuda.Stream(), sz.Workspace(n, dtype), [torch.zeros(blob.size, dtype=torch.uint8, device="cuda") for _ in range(6)],
                  [sz.new_sizes() for _ in range(6)]) for _ in range(6)]
        torch.cuda.synchronize()
        for k in range(6):
            for stream, ws, outs, recs in lanes:
                sz.compress(xd, cb, outs[k], ws, recs[k], stream=stream)
        torch.cuda.synchronize()
        for _, _, outs, recs in lanes:
            for out, rec in zip(outs, recs):
                assert sz.read_sizes(rec) == (blob.size, m, 0) and torch.equal(out, want)


def test_a_stream_of_few_compute_units(few_cus):
    """A stream with a mask, by the rules: calls whose workgroups its CUs hold, and calls that take two launches there."""
    cb, ocb = books(sz.BF16, oracle.BF16)
    for n in (30 * 1024 - 1, 100 * 1024 - 1, 400 * 1024, 2048 * 1024 - 3):
        x = words(sz.BF16, n, 3)
        blob, m = oracle.compress(kv_synth.to_numpy_words(x), ocb)
        xd, ws, want = x.cuda(), sz.Workspace(n, sz.BF16), torch.from_numpy(blob).cuda()
        out, rec = torch.zeros(blob.size, dtype=torch.uint8, device="cuda"), sz.new_sizes()
        torch.cuda.synchronize()
        for _ in range(3):
            sz.compress(xd, cb, out, ws, rec, stream=few_cus)
        torch.cuda.synchronize()
        assert sz.read_sizes(rec) == (blob.size, m, 0) and torch.equal(out, want)


@pytest.mark.parametrize("dtype,odt", FORMATS)
def test_what_the_workspace_holds(dtype, odt, looks):
    """One workspace for calls of different lengths, and words of it overwritten in between: no value in it means anything."""
    cb, ocb = books(dtype, odt)
    ws = sz.Workspace(1 << 20, dtype)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    for k, n in enumerate((900 * 1024, 100 * 1024, 1024 * 1024, 60 * 1024 - 1, 1000 * 1024, 500 * 1024)):
        if k == 2:
            ws.buf.fill_(0xFF)
        elif k == 3:
            ws.buf.zero_()
        elif k > 3:
            ws.buf.random_(0, 256, generator=gen)
        with looks(LEAVE if k % 2 else 0):
            check(words(dtype, n, k), cb, ocb, ws)


@pytest.mark.parametrize("dtype,odt", FORMATS)
@pytest.mark.parametrize("limit", [0, 1, LEAVE])
def test_batches(dtype, odt, limit, looks):
    """Tensors of a launch have their own counts: unequal lengths, none at all, a batch of 64."""
    cb, ocb = books(dtype, odt)
    for sizes in ([0, 50 * 1024 + 1, 3, 0, 300 * 1024, 4096, 1024 * 257 - 5], [63 * 1024 + 7 * k for k in range(64)], [31 * 1024 + 7 * k for k in range(64)], [0, 60 * 1024],
                  [500 * 1024 - 1] * 4, [1024 * 1024 - 1] * 4, [1025 * 1024, 1000 * 1024 - 1]):
        xs = [words(dtype, n, 7 + k, "many" if k % 5 == 4 else "few") for k, n in enumerate(sizes)]
        blobs = [oracle.compress(kv_synth.to_numpy_words(x), ocb) for x in xs]
        outs = [torch.full((sz.compress_bound(n, dtype) + 256,), 0xA5, dtype=torch.uint8, device="cuda") for n in sizes]
        ws, rec = sz.Workspace(max(sizes), dtype), sz.new_sizes_array(len(xs))
        print(f"case {dtype} batch of {len(sizes)} looks={limit}", flush=True)
        with looks(limit):
            sz.compress_batch([x.cuda() for x in xs], [cb] * len(xs), outs, ws, rec)
        for (blob, m), out, got in zip(blobs, outs, sz.read_sizes_array(rec)):
            assert got == (blob.size, m, 0) and np.array_equal(out[:blob.size].cpu().numpy(), blob) and bool((out[blob.size:] == 0xA5).all())


@pytest.mark.parametrize("dtype", [sz.BF16, sz.FP8_E5M2])
@pytest.mark.parametrize("limit", [0, LEAVE])
def test_what_does_not_fit(dtype, limit, looks):
    cb = sz.codebook_from_dec(list(range(16)), dtype)          # hardly anything is in this codebook
    for n in (70 * 1024 - 9, 200 * 1024, 1100 * 1024 - 5):
        x = words(dtype, n, 5)
        fixed, total = sz.fixed_bytes(n, dtype), compress(x, cb)[1][0]
        for cap in (fixed, fixed + (total - fixed) // 3, total - 1, total):
            with looks(limit):
                out, got = compress(x, cb, cap)
            with looks(sz.INTERNAL_NO_SHORT):
                ref, want = compress(x, cb, cap)
            assert got == want and torch.equal(out, ref)


def test_beside_other_work_on_the_device():
    """Another stream keeps the device busy: workgroups of a launch get onto it one after the other."""
    cb, ocb = books(sz.BF16, oracle.BF16)
    x = words(sz.BF16, 2048 * 1024 - 1, 3)
    blob, m = oracle.compress(kv_synth.to_numpy_words(x), ocb)
    xd, ws = x.cuda(), sz.Workspace(x.numel(), sz.BF16)
    recs, outs = [sz.new_sizes() for _ in range(20)], [torch.zeros(blob.size, dtype=torch.uint8, device="cuda") for _ in range(20)]
    busy, side = torch.ones(1 << 28, device="cuda"), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(20):
            busy.mul_(1.0001)
    for out, rec in zip(outs, recs):
        sz.compress(xd, cb, out, ws, rec)
    torch.cuda.synchronize()
    want = torch.from_numpy(blob).cuda()
    for out, rec in zip(outs, recs):
        assert sz.read_sizes(rec) == (blob.size, m, 0) and torch.equal(out, want)


def test_captured_calls_are_replayed():
    """A captured call takes the two launches: its replays see new words and other calls on the workspace in between."""
    cb, ocb = books(sz.BF16, oracle.BF16)
    n = 100 * 1024 - 37
    x, ws, rec = words(sz.BF16, n, 1).cuda(), sz.Workspace(4096 * 1024, sz.BF16), sz.new_sizes()
    out = torch.zeros(sz.compress_bound(n, sz.BF16), dtype=torch.uint8, device="cuda")
    sz.compress(x, cb, out, ws, rec)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sz.compress(x, cb, out, ws, rec)
    for k in range(4):
        y = words(sz.BF16, n, 20 + k)
        x.copy_(y)
        graph.replay()
        torch.cuda.synchronize()
        blob, m = oracle.compress(kv_synth.to_numpy_words(y), ocb)
        assert sz.read_sizes(rec) == (blob.size, m, 0) and np.array_equal(out[:blob.size].cpu().numpy(), blob)
        check(words(sz.BF16, (50 + 900 * (k % 2)) * 1024, k), cb, ocb, ws)
