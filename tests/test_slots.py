"""Escape records in batches of many tensors, whose tiles share the workspace: the oracle's streams where the records of a tile
fit its slot, where they do not, and with what the tiles' counts leave of the status area at its smallest."""
import numpy as np
import pytest
import torch

import kv_synth
import oracle
import paper_2605_01708_amd as sz

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("status", [0, 64 * 256])   # bytes of the status area, 0: all of it; 64 x 256: no more than the counts take
@pytest.mark.parametrize("dtype,odt", [(sz.BF16, oracle.BF16), (sz.FP8_E5M2, oracle.E5M2)])
def test_many_tensors_with_escapes(dtype, odt, status):
    gen = kv_synth.kv_bf16 if dtype == sz.BF16 else kv_synth.kv_e5m2
    sample = gen(64, 1)
    cb, ocb = sz.calibrate(sample, dtype), oracle.calibrate(kv_synth.to_numpy_words(sample), odt)
    xs = []
    for k in range(64):
        x = gen(70 + k % 3, k).reshape(-1)[: (70 + k % 3) * 1024 - k].contiguous()
        if dtype == sz.BF16 and k % 2 == 0:
            x = kv_synth.kv_bf16_outliers(70, k).reshape(-1).contiguous()
        if k % 4 == 1:    # every twentieth word at random: dozens of escapes per chunk
            r = torch.randint(0, 256, (x.numel() * x.element_size(),), dtype=torch.uint8, generator=torch.Generator().manual_seed(k)).view(x.dtype)
            x = torch.where(torch.arange(x.numel()) % 20 == 0, r, x)
        xs.append(x)
    blobs = [oracle.compress(kv_synth.to_numpy_words(x), ocb) for x in xs]
    outs = [torch.full((sz.compress_bound(x.numel(), dtype) + 256,), 0xA5, dtype=torch.uint8, device="cuda") for x in xs]
    ws, rec = sz.Workspace(max(x.numel() for x in xs), dtype), sz.new_sizes_array(len(xs))
    try:
        sz.internal_test_short(sz.INTERNAL_NO_SHORT)
        sz.internal_test_hooks(0, status, 0, 0)
        sz.compress_batch([x.cuda() for x in xs], [cb] * len(xs), outs, ws, rec)
    finally:
        sz.internal_test_hooks()
        sz.internal_test_short()
    for (blob, m), out, got in zip(blobs, outs, sz.read_sizes_array(rec)):
        assert got == (blob.size, m, 0) and np.array_equal(out[:blob.size].cpu().numpy(), blob) and bool((out[blob.size:] == 0xA5).all())
