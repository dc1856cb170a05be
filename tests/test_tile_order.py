"""Launches that take their tiles in the order of the XCDs (launches of many tiles): the same streams and words as one
call per tensor, which takes the tiles in their own order.  The rules would ask for tensors of many gigabytes, so the
order, and the chunks per wave that go with it, are forced."""
import pytest
import torch

import kv_synth
import paper_2605_01708_amd as sz


@pytest.mark.parametrize("n", [0, 1, 25, 64, 127, 128, 129, 200, 255, 256, 1000, 4096, 4099])
def test_every_tensor_is_spread_over_all_xcds(n):
    """A row of a launch has as many workgroups as its longest tensor has tiles.  Whatever the row, the first n workgroups
    take the n tiles, the others none, and the hardware's 8 XCDs (workgroups dealt out in turn) get equal shares."""
    order = [sz.internal_xcd_tile(b, n) for b in range(max(2 * n, 4200))]
    assert sorted(order[:n]) == list(range(n)) and all(t >= n for t in order[n:])
    share = [sum(1 for t in order[x::8] if t < n) for x in range(8)]
    assert max(share) - min(share) <= 1
    whole = n // 128 * 128   # runs of 16 tiles to an XCD in the whole windows
    assert all(order.index(t) % 8 == (t // 16) % 8 for t in range(whole))


@pytest.fixture
def launch():
    """forces what the launch rules choose; by the rules again afterwards"""
    yield sz.internal_test_launch
    sz.internal_test_launch()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [sz.BF16, sz.FP8_E5M2])
def test_batches_in_xcd_order_equal_single_calls(launch, dtype):
    gen = kv_synth.kv_bf16 if dtype == sz.BF16 else kv_synth.kv_e5m2
    # the long tensor: whole groups of 128 tiles, a part of one, a ragged last chunk
    sizes = [(12288 + 4 * 131) * 1024 + 517] + [(37 * k) % 3001 for k in range(63)]
    x = gen(sum(sizes) // 1024 + 64, 7, device="cuda")
    xs, at = [], 0
    for n in sizes:
        xs.append(x[at:at + n].clone())
        at += n
    cb = sz.calibrate(gen(64, 1), dtype)
    caps = [sz.total_bytes(n, min(n, n // 50 + 4096), dtype) for n in sizes]
    outs = [torch.full((c,), 0xA5, dtype=torch.uint8, device="cuda") for c in caps]
    ws, rec = sz.Workspace(max(sizes), dtype), sz.new_sizes_array(len(xs))
    launch(xcd=2)
    sz.compress_batch(xs, [cb] * len(xs), outs, ws, rec)
    got = sz.read_sizes_array(rec)
    launch()
    one = sz.new_sizes()
    for x1, out, (total, m, status), cap in zip(xs, outs, got, caps):
        ref = torch.full((cap,), 0xA5, dtype=torch.uint8, device="cuda")
        sz.compress(x1, cb, ref, ws, one)
        assert sz.read_sizes(one) == (total, m, status) and status == 0
        assert torch.equal(out, ref)
    ys = [torch.full_like(x1, 0x5A) for x1 in xs]
    st = sz.new_sizes()
    launch(xcd=2)
    sz.decompress_batch(outs, [g[0] for g in got], sizes, [cb] * len(xs), ys, st)
    assert sz.read_sizes(st)[2] == 0
    assert all(torch.equal(a, b) for a, b in zip(xs, ys))


@pytest.mark.gpu
@pytest.mark.parametrize("how", ["host codebooks", "device codebooks", "paged"])
@pytest.mark.parametrize("xcd", [1, 2])
@pytest.mark.parametrize("per_wave", [1, 2, 4, 8])
@pytest.mark.parametrize("dtype", [sz.BF16, sz.FP8_E5M2])
def test_every_choice_of_the_rules(launch, dtype, per_wave, xcd, how):
    """All sizes of tile and both orders, on tensors that end inside a window of 128 tiles, at its edges and before its
    first XCD has had its run, in every form of a batch call."""
    gen = kv_synth.kv_bf16 if dtype == sz.BF16 else kv_synth.kv_e5m2
    tile = 4 * per_wave * 1024
    sizes = [261 * tile - 517, 128 * tile, 25 * tile + 1, 0, 1, 127 * tile + tile // 2 + 3, 129 * tile - 1024, 5000]
    page = 16 * 1024
    pages = -(-max(sizes) // page)
    pool = gen((pages * page * 2) // 1024 + 64, 7, device="cuda")   # two tensors per page of a pool for the paged form
    table = torch.randperm(pages, generator=torch.Generator().manual_seed(3)).to(torch.int32)
    es = pool.element_size()
    if how == "paged":
        # tensor k lies in half k % 2 of every page of a pool that all share, the logical page p at table[p]
        src = pool[:pages * 2 * page].view(pages, 2, page)
        xs = [src[table.long(), k % 2].reshape(-1)[:n].clone() for k, n in enumerate(sizes)]
        views = [src.reshape(-1)[(k % 2) * page:] for k in range(len(sizes))]
    else:
        xs = [pool[16 * k:16 * k + n].clone() for k, n in enumerate(sizes)]
    caps = [sz.total_bytes(n, min(n, n // 50 + 4096), dtype) for n in sizes]
    outs = [torch.full((c,), 0xA5, dtype=torch.uint8, device="cuda") for c in caps]
    ws, rec, one, st = sz.Workspace(max(sizes), dtype), sz.new_sizes_array(len(xs)), sz.new_sizes(), sz.new_sizes()
    cb = sz.calibrate(gen(64, 1), dtype)
    cbs = [cb] * len(xs)
    if how == "device codebooks":
        dcbs = sz.DeviceCodebooks(len(xs), dtype)
        sz.CalibrateBatchDevice(xs, dcbs).launch()
        cbs = [dcbs.to_host(k) for k in range(len(xs))]
    launch(per_wave, per_wave, xcd)
    if how == "host codebooks":
        sz.compress_batch(xs, cbs, outs, ws, rec)
    elif how == "device codebooks":
        sz.CompressBatchDcb(xs, dcbs, outs).launch(ws, rec)
    else:
        geometry = sz.Paged(pool, table.cuda(), page, 2 * page * es, 0, pages)
        sz.CompressBatchPaged(views, sizes, cbs, outs, geometry).launch(ws, rec)
    got = sz.read_sizes_array(rec)
    ys = [torch.full_like(x, 0x5A) for x in xs]
    lengths = [g[0] for g in got]
    if how == "host codebooks":
        sz.decompress_batch(outs, lengths, sizes, cbs, ys, st)
    elif how == "device codebooks":
        sz.DecompressBatchDcb(outs, lengths, sizes, dcbs, ys).launch(st)
    else:
        back = torch.full((len(sizes), pages, 2, page), 0x5A, dtype=pool.dtype, device="cuda")   # a pool for each
        sz.DecompressBatchPaged(outs, lengths, sizes, cbs, [b.reshape(-1)[(k % 2) * page:] for k, b in enumerate(back)], geometry).launch(st)
        ys = [b[table.long(), k % 2].reshape(-1)[:n] for k, (b, n) in enumerate(zip(back, sizes))]
        assert all(bool((b[:, 1 - k % 2] == 0x5A).all()) for k, b in enumerate(back))
    assert sz.read_sizes(st)[2] == 0
    launch()
    for k, (x, out, g, cap) in enumerate(zip(xs, outs, got, caps)):
        ref = torch.full((cap,), 0xA5, dtype=torch.uint8, device="cuda")
        sz.compress(x, cbs[k], ref, ws, one)
        assert sz.read_sizes(one) == g and g[2] == 0, k
        assert torch.equal(out, ref), k
        assert torch.equal(ys[k], x), k
