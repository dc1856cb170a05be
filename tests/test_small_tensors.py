"""Tensors that one workgroup compresses in one launch (up to 40 chunks of BF16, 48 of E5M2; by the rules in captured calls and in batches
too long for the short launch, here wherever that is switched off): the oracle's streams on both sides of the limit and beyond what a
wave stages of its escapes, and, where the stream does not fit, byte for byte what the two-launch path leaves (the test hook for its
groups asks for that path).  Each also by the rules."""
import numpy as np
import pytest
import torch

import kv_synth
import oracle
import paper_2605_01708_amd as sz

pytestmark = pytest.mark.gpu
FORMATS = [(sz.BF16, oracle.BF16, 40), (sz.FP8_E5M2, oracle.E5M2, 48)]


@pytest.fixture(params=[0, sz.INTERNAL_NO_SHORT], ids=["by the rules", "no short launch"])
def no_short(request):
    sz.internal_test_short(request.param)
    yield request.param
    sz.internal_test_short()


def words(dtype, n, seed):
    gen = kv_synth.kv_bf16 if dtype == sz.BF16 else kv_synth.kv_e5m2
    return gen(n // 1024 + 1, seed)[:n].contiguous()


def gpu_stream(x, cb, cap):
    out = torch.full((cap + 512,), 0xA5, dtype=torch.uint8, device="cuda")
    ws, rec = sz.Workspace(x.numel(), cb.dtype), sz.new_sizes()
    sz.compress(x.cuda(), cb, out, ws, rec, capacity=cap)
    return out, sz.read_sizes(rec)


@pytest.mark.parametrize("dtype,odt,limit", FORMATS)
def test_streams_at_the_edges(dtype, odt, limit, no_short):
    sample = words(dtype, 64 * 1024, 1)
    cb = sz.calibrate(sample, dtype)
    ocb = oracle.calibrate(kv_synth.to_numpy_words(sample), odt)
    rng = np.random.default_rng(2)
    for n in (1, 1023, 16 * 1024, 16 * 1024 + 1, 17 * 1024 - 3, limit * 1024 - 1, limit * 1024, limit * 1024 + 1, (limit + 1) * 1024):
        assert sz.internal_compress_plan([n], dtype)["small"] == (n <= limit * 1024)   # the kernel at hand, where there is no short launch
        for escapes in ("few", "many", "all"):
            x = words(dtype, n, 3)
            if escapes != "few":      # random patterns: nearly all escape; "many": in every third chunk
                r = torch.from_numpy(rng.integers(0, 1 << (16 if dtype == sz.BF16 else 8), n).astype(np.uint16 if dtype == sz.BF16 else np.uint8).view(np.int16 if dtype == sz.BF16 else np.uint8))
                x = r if escapes == "all" else torch.where((torch.arange(n) // 1024) % 3 == 0, r, x)
            print(f"case {dtype} n={n} {escapes}", flush=True)
            blob, m = oracle.compress(kv_synth.to_numpy_words(x), ocb)
            cap = sz.compress_bound(n, dtype)
            out, got = gpu_stream(x, cb, cap)
            assert got == (blob.size, m, 0)
            assert np.array_equal(out[:blob.size].cpu().numpy(), blob)
            assert bool((out[blob.size:] == 0xA5).all())


@pytest.mark.parametrize("dtype,odt,limit", FORMATS)
def test_what_does_not_fit_and_batches(dtype, odt, limit, no_short):
    cb = sz.codebook_from_dec(list(range(16)), dtype)          # hardly anything is in this codebook
    sizes = [0, 5, 1024, 5000, 16 * 1024 + 7, limit * 1024]
    xs = [words(dtype, n, 5) for n in sizes]
    caps = []
    for x in xs:
        total = gpu_stream(x, cb, sz.compress_bound(x.numel(), dtype))[1][0]
        fixed = sz.fixed_bytes(x.numel(), dtype)
        for cap in (fixed, fixed + (total - fixed) // 3, total - 1):
            cap = max(cap, fixed)
            caps.append((x, cap, gpu_stream(x, cb, cap)))
    ws, rec = sz.Workspace(max(sizes), dtype), sz.new_sizes_array(len(xs))
    outs = [torch.full((sz.compress_bound(n, dtype),), 0xA5, dtype=torch.uint8, device="cuda") for n in sizes]
    sz.compress_batch([x.cuda() for x in xs], [cb] * len(xs), outs, ws, rec)
    got = sz.read_sizes_array(rec)
    try:
        sz.internal_test_hooks(0, 0, 1, 0)
        for x, cap, (out, sizes_) in caps:
            ref, ref_sizes = gpu_stream(x, cb, cap)
            assert sizes_ == ref_sizes and torch.equal(out, ref)
        for x, out, g in zip(xs, outs, got):
            ref, ref_sizes = gpu_stream(x, cb, out.numel())
            assert g == ref_sizes and torch.equal(out, ref[:out.numel()])
    finally:
        sz.internal_test_hooks()


@pytest.mark.parametrize("dtype,odt,limit", FORMATS)
def test_batches_too_long_for_the_short_launch(dtype, odt, limit):
    """By the rules a launch of 160 workgroups, whose waves have several chunks each, and one of five."""
    sample = words(dtype, 64 * 1024, 1)
    cb, ocb = sz.calibrate(sample, dtype), oracle.calibrate(kv_synth.to_numpy_words(sample), odt)
    sizes = [limit * 1024 - 7 * (k % 5) for k in range(165)]
    plan = sz.internal_compress_plan(sizes, dtype)
    assert plan["small"] and not plan["short"] and plan["tensors"] == 160
    pool = words(dtype, (limit + 165) * 1024, 3)
    pool[::701] = 0
    xs = [pool[1024 * k:1024 * k + n].contiguous() for k, n in enumerate(sizes)]
    outs = [torch.full((sz.compress_bound(n, dtype) + 256,), 0xA5, dtype=torch.uint8, device="cuda") for n in sizes]
    ws, rec = sz.Workspace(max(sizes), dtype), sz.new_sizes_array(len(xs))
    sz.compress_batch([x.cuda() for x in xs], [cb] * len(xs), outs, ws, rec)
    for x, out, got in zip(xs, outs, sz.read_sizes_array(rec)):
        blob, m = oracle.compress(kv_synth.to_numpy_words(x), ocb)
        assert got == (blob.size, m, 0) and np.array_equal(out[:blob.size].cpu().numpy(), blob) and bool((out[blob.size:] == 0xA5).all())
