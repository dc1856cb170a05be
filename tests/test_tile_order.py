"""Launches that take their tiles in the order of the XCDs (many tiles in a launch row): the same streams and words as
one call per tensor, which takes the tiles in their own order.  The launch rule looks at the longest tensor times the
number of tensors, so one long tensor among short ones gets there."""
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


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [sz.BF16, sz.FP8_E5M2])
def test_batches_in_xcd_order_equal_single_calls(dtype):
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
    sz.compress_batch(xs, [cb] * len(xs), outs, ws, rec)
    got = sz.read_sizes_array(rec)
    one = sz.new_sizes()
    for x1, out, (total, m, status), cap in zip(xs, outs, got, caps):
        ref = torch.full((cap,), 0xA5, dtype=torch.uint8, device="cuda")
        sz.compress(x1, cb, ref, ws, one)
        assert sz.read_sizes(one) == (total, m, status) and status == 0
        assert torch.equal(out, ref)
    ys = [torch.full_like(x1, 0x5A) for x1 in xs]
    st = sz.new_sizes()
    sz.decompress_batch(outs, [g[0] for g in got], sizes, [cb] * len(xs), ys, st)
    assert sz.read_sizes(st)[2] == 0
    assert all(torch.equal(a, b) for a, b in zip(xs, ys))
