"""Batches around what a launch takes, 64 and 160 tensors: the oracle's streams and the words back, through the launches of short
calls and of others, of equal and of unequal lengths."""
import numpy as np
import pytest
import torch

import kv_synth
import oracle
import paper_2605_01708_amd as sz

FORMATS = [(sz.BF16, oracle.BF16), (sz.FP8_E5M2, oracle.E5M2)]


@pytest.mark.gpu
@pytest.mark.parametrize("short", [True, False])
@pytest.mark.parametrize("dtype,odt", FORMATS)
@pytest.mark.parametrize("count", [64, 65, 160, 161])
def test_streams_and_words(dtype, odt, count, short):
    gen = kv_synth.kv_bf16 if dtype == sz.BF16 else kv_synth.kv_e5m2
    sample = gen(64, 1)
    cb, ocb = sz.calibrate(sample, dtype), oracle.calibrate(kv_synth.to_numpy_words(sample), odt)
    sizes = [(1, 17, 5, 23)[k % 4] * 1024 - 3 * (k % 7) if k % 9 else 0 for k in range(count)]
    if not short:
        sizes[3] = 300 * 1024 - 1
    xs = [gen(s // 1024 + 1, k)[:s].contiguous() for k, s in enumerate(sizes)]
    dx = [x.cuda() for x in xs]
    blobs = [oracle.compress(kv_synth.to_numpy_words(x), ocb) for x in xs]
    outs = [torch.full((-(-sz.compress_bound(s, dtype) // 256) * 256,), 0xA5, dtype=torch.uint8, device="cuda") for s in sizes]
    ws, rec = sz.Workspace(max(sizes), dtype), sz.new_sizes_array(count)
    try:
        sz.internal_test_short(0 if short else sz.INTERNAL_NO_SHORT)
        sz.compress_batch(dx, [cb] * count, outs, ws, rec)
    finally:
        sz.internal_test_short()
    got = sz.read_sizes_array(rec)
    for (blob, m), out, g in zip(blobs, outs, got):
        assert g == (blob.size, m, 0) and np.array_equal(out[:blob.size].cpu().numpy(), blob) and bool((out[blob.size:] == 0xA5).all())
    ys, drec = [torch.zeros_like(x) for x in dx], sz.new_sizes()
    sz.DecompressBatch(outs, [g[0] for g in got], sizes, [cb] * count, ys).launch(drec)
    assert sz.read_sizes(drec)[2] == 0 and all(torch.equal(x, y) for x, y in zip(dx, ys))


def batch(dtype, sizes, seed):
    """Words of these lengths, in every third tensor mostly random ones (more records than a wave stages or a slot holds), on the device,
    their codebook, their streams"""
    gen = kv_synth.kv_bf16 if dtype == sz.BF16 else kv_synth.kv_e5m2
    sample = gen(64, 1)
    cb, ocb = sz.calibrate(sample, dtype), oracle.calibrate(kv_synth.to_numpy_words(sample), dict(FORMATS)[dtype])
    pool = gen(max(sizes) // 1024 + len(sizes) + 1, seed)
    r = torch.randint(0, 256, (pool.numel() * pool.element_size(),), dtype=torch.uint8, generator=torch.Generator().manual_seed(seed)).view(pool.dtype)
    xs = [torch.where(torch.arange(n) // 512 % 4 < 3, r[1024 * k:1024 * k + n], pool[1024 * k:1024 * k + n]) if k % 3 == 1 else pool[1024 * k:1024 * k + n].contiguous()
          for k, n in enumerate(sizes)]
    return xs, cb, [oracle.compress(kv_synth.to_numpy_words(x), ocb) for x in xs]


def buffers(dtype, sizes):
    return [torch.full((sz.compress_bound(n, dtype) + 256,), 0xA5, dtype=torch.uint8, device="cuda") for n in sizes], sz.Workspace(max(sizes), dtype), sz.new_sizes_array(len(sizes))


def check(blobs, outs, rec):
    for k, ((blob, m), out, got) in enumerate(zip(blobs, outs, sz.read_sizes_array(rec))):
        assert got == (blob.size, m, 0) and np.array_equal(out[:blob.size].cpu().numpy(), blob) and bool((out[blob.size:] == 0xA5).all()), k


@pytest.mark.gpu
@pytest.mark.parametrize("cpt,groups,direct,xcd", [(1, 1, 0, 1), (2, 2, 0, 2), (2, 4, 1, 1), (4, 1, 1, 2), (4, 4, 0, 1)])
@pytest.mark.parametrize("dtype", [sz.BF16, sz.FP8_E5M2])
def test_every_kernel_of_more_than_64_tensors(dtype, cpt, groups, direct, xcd):
    """Tiles of all sizes, all numbers of groups in the finishing pass and its sums of counts, with tiles that are encoded again."""
    if dtype == sz.BF16 and cpt == 4:
        cpt = 2   # what a wave of it takes at once
    sizes = [((1, 70, 33, 0, 150)[k % 5] * 1024 - (3 * (k % 7) if k % 5 != 3 else 0)) for k in range(90)]
    xs, cb, blobs = batch(dtype, sizes, 5)
    outs, ws, rec = buffers(dtype, sizes)
    try:
        sz.internal_test_launch(cpt=cpt, xcd=xcd)
        sz.internal_test_hooks(0, 0, groups, direct)
        plan = sz.internal_compress_plan(sizes, dtype)
        assert (plan["tensors"], plan["cpt"], plan["finish_groups"], plan["group_sums"], plan["small"], plan["short"]) == (90, cpt, groups, direct, 0, 0)
        sz.compress_batch([x.cuda() for x in xs], [cb] * len(xs), outs, ws, rec)
        torch.cuda.synchronize()
    finally:
        sz.internal_test_hooks()
        sz.internal_test_launch()
    check(blobs, outs, rec)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [sz.BF16, sz.FP8_E5M2])
def test_long_launch_of_more_than_64_tensors(dtype):
    """By the rules, two chunks per wave and enough tiles that memory alone bounds the launch."""
    sizes = [500 * 1024 - 5 * (k % 3) for k in range(100)]
    xs, cb, blobs = batch(dtype, sizes, 6)
    plan = sz.internal_compress_plan(sizes, dtype)
    assert plan["tensors"] == 100 and plan["cpt"] == 2 and 100 * plan["tiles_max"] >= 6144 and plan["by_xcd"]
    outs, ws, rec = buffers(dtype, sizes)
    sz.compress_batch([x.cuda() for x in xs], [cb] * len(xs), outs, ws, rec)
    check(blobs, outs, rec)


@pytest.mark.gpu
@pytest.mark.parametrize("short", [True, False])
@pytest.mark.parametrize("dtype", [sz.BF16, sz.FP8_E5M2])
def test_pages_of_more_than_64_tensors(dtype, short):
    """166 tensors in pools behind one table, two launches of them."""
    page, count = 2048, 166
    sizes = [(3 if short else 49) * 1024 - 11 * (k % 4) for k in range(count)]
    if short:
        sizes[70] = 30 * 1024 - 1
    xs, cb, blobs = batch(dtype, sizes, 7)
    pages = -(-max(sizes) // page)
    table = torch.randperm(pages, generator=torch.Generator().manual_seed(4)).to(torch.int32)
    pools = []
    for x in xs:
        pool = torch.zeros(pages, page, dtype=x.dtype)
        whole = torch.zeros(pages * page, dtype=x.dtype)
        whole[:x.numel()] = x
        pool[table.long()] = whole.view(pages, page)
        pools.append(pool.cuda())
    geometry = sz.Paged(pools[0], table.cuda(), page, page * xs[0].element_size(), 0, pages)
    outs, ws, rec = buffers(dtype, sizes)
    try:
        sz.internal_test_short(0 if short else sz.INTERNAL_NO_SHORT)
        sz.CompressBatchPaged(pools, sizes, [cb] * count, outs, geometry).launch(ws, rec)
        torch.cuda.synchronize()
    finally:
        sz.internal_test_short()
    check(blobs, outs, rec)
    back = [torch.zeros_like(p) for p in pools]
    st = sz.new_sizes()
    sz.DecompressBatchPaged(outs, [b.size for b, _ in blobs], sizes, [cb] * count, back, geometry).launch(st)
    assert sz.read_sizes(st)[2] == 0 and all(torch.equal(a, b) for a, b in zip(pools, back))


@pytest.mark.parametrize("dtype", [sz.BF16, sz.FP8_E5M2])
def test_tensors_of_a_launch(dtype):
    """More than 64 go into a launch where hardly any workgroup has no tile."""
    def tensors(chunks):
        return sz.internal_compress_plan([c * 1024 for c in chunks], dtype)["tensors"]
    assert [tensors([100] * n) for n in (64, 65, 160, 161, 400)] == [64, 65, 160, 160, 160]
    assert tensors([8192] * 64 + [2] * 96) == 68 and tensors([2] * 64 + [8192] * 96) == 64 and tensors([2000, 1900] * 80) == 160
    assert tensors([0] * 200) == 160


@pytest.mark.parametrize("dtype", [sz.BF16, sz.FP8_E5M2])
def test_room_for_records(dtype):
    """A launch takes more than 64 only where that leaves a chunk four records of the workspace, which one tensor sizes; what does
    not go into one launch goes into equal ones."""
    def tensors(chunks):
        return sz.internal_compress_plan([c * 1024 for c in chunks], dtype)["tensors"]
    for chunks in (2000, 2700, 4096, 8192, 16384, 32768, 100000):
        for n in (65, 100, 160, 300):
            count, room = tensors([chunks] * n), sz.workspace_bytes(chunks * 1024, dtype) // 16
            assert count <= 64 or count * chunks <= room, (chunks, n)
            assert count == min(n, 160) or -(-min(n, 160) // count) * max(64, room // chunks) >= min(n, 160) > (-(-min(n, 160) // count) - 1) * max(64, room // chunks), (chunks, n)
    assert [tensors([c] * 160) for c in (2000, 4096, 8192, 16384, 32768)] == [160, 80, 80, 80, 54]
    assert [tensors([32768] * n) for n in (64, 65, 72, 73, 100)] == [64, 65, 72, 37, 50]
    assert tensors([32768] * 70 + [100] * 90) == 71 and tensors([8192] * 64 + [2] * 96) == 68
