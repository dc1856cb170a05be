"""Tiles of one, two and four chunks per wave: which one a launch takes depends on its chunks in all, and the streams
must not.  A long batch call against single calls on its tensors, which take smaller tiles."""
import pytest
import torch

import kv_synth
import paper_2605_01708_amd as sz


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,chunks", [
    (sz.BF16, [8191, 6500, 5790, 0, 17]),            # 20 498 chunks: two per wave; alone: one
    (sz.FP8_E5M2, [3000, 3133, 12, 1]),              # 6146: two; alone: one
    (sz.FP8_E5M2, [12290] * 63 + [12201, 3]),        # a launch of 786 471: four; alone: two
])
def test_streams_do_not_depend_on_the_tile(dtype, chunks):
    gen = kv_synth.kv_bf16 if dtype == sz.BF16 else kv_synth.kv_e5m2
    cb = sz.calibrate(gen(64, 1), dtype)
    pool = gen(max(chunks) + 70, 11, device="cuda")
    if dtype == sz.BF16:
        pool = kv_synth.kv_bf16_outliers(max(chunks) + 70, 11, device="cuda")
    sizes = [max(0, 1024 * c - (37 * k) % 1024) for k, c in enumerate(chunks)]
    xs = [pool[16 * k:16 * k + n] for k, n in enumerate(sizes)]
    caps = [(sz.total_bytes(n, n // 40 + min(n, 2000), dtype) + 255) // 256 * 256 for n in sizes]
    out = torch.full((sum(caps),), 0xA5, dtype=torch.uint8, device="cuda")
    outs, at = [], 0
    for c in caps:
        outs.append(out[at:at + c])
        at += c
    ws, rec, one = sz.Workspace(max(sizes), dtype), sz.new_sizes_array(len(xs)), sz.new_sizes()
    sz.compress_batch(xs, [cb] * len(xs), outs, ws, rec)
    got = sz.read_sizes_array(rec)
    ref = torch.empty(max(caps), dtype=torch.uint8, device="cuda")
    for x, o, g, cap in zip(xs, outs, got, caps):
        ref.fill_(0xA5)
        sz.compress(x, cb, ref, ws, one, capacity=cap)
        assert sz.read_sizes(one) == g and g[2] == 0
        assert torch.equal(o, ref[:cap])
    y = torch.empty(max(sizes), dtype=pool.dtype, device="cuda")
    for x, o, g in zip(xs[:3], outs, got):
        sz.decompress(o, g[0], x.numel(), cb, y, one)
        assert torch.equal(y[:x.numel()], x)
