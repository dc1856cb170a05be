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
