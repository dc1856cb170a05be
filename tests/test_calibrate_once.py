"""Calibration of a batch in one launch, whose workgroups settle among themselves who clears and who ranks: around the numbers of
workgroups and of samples where it takes several launches instead, into buffers that hold anything, again and captured."""
import pytest
import torch

import kv_synth
import paper_2605_01708_amd as sz



def check(xs, dcbs, dtype):
    shift, values = (7, 256) if dtype == sz.BF16 else (2, 32)
    hists = dcbs.hists.cpu()
    for k, x in enumerate(xs):
        want = torch.zeros(256, dtype=torch.int64)
        want[:values] = torch.bincount(((x.to(torch.int32) >> shift) & (values - 1)).long(), minlength=values).cpu()
        assert torch.equal(hists.view(-1, 256)[k], want), k
        ref, got = sz.codebook_from_hist(want, dtype), dcbs.to_host(k)
        assert (got.dec, got.enc, got.member, got.dtype) == (ref.dec, ref.enc, ref.member, ref.dtype), k


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [sz.BF16, sz.FP8_E5M2])
@pytest.mark.parametrize("per", [[63], [64], [65], [72], [73], [256], [72, 72, 0], [73, 5] + [1] * 70, [3, 0, 1], [60, 61], [1] * 65, [1] * 161, [2] * 64, [2] * 130, [5] * 70])
def test_numbers_of_workgroups_and_samples(dtype, per):
    """per: a sample's workgroups at most, four vectors of 16 bytes per thread each"""
    each = 16 * 4096 // (2 if dtype == sz.BF16 else 1)
    pool = (kv_synth.kv_bf16 if dtype == sz.BF16 else kv_synth.kv_e5m2)(max(per) * each // 1024 + 8, 3, device="cuda")
    xs = [pool[16 * (k % 5): 16 * (k % 5) + max(0, w * each - 5 * (k % 3))].clone() for k, w in enumerate(per)]
    dcbs = sz.DeviceCodebooks(len(xs), dtype)
    cal = sz.CalibrateBatchDevice(xs, dcbs)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    for k in range(4):
        if k == 1:
            dcbs.buf.fill_(-1 if dcbs.buf.dtype.is_signed else 255)
            dcbs.hists.fill_(-1)
        elif k == 2:
            dcbs.buf.view(torch.uint8).random_(0, 256, generator=gen)
            dcbs.hists.view(torch.uint8).random_(0, 256, generator=gen)
        cal.launch()
        torch.cuda.synchronize()
        check(xs, dcbs, dtype)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [sz.BF16, sz.FP8_E5M2])
def test_captured(dtype):
    gen = kv_synth.kv_bf16 if dtype == sz.BF16 else kv_synth.kv_e5m2
    xs = [gen(200 + 30 * k, k, device="cuda") for k in range(3)]
    dcbs = sz.DeviceCodebooks(3, dtype)
    cal = sz.CalibrateBatchDevice(xs, dcbs)
    cal.launch()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cal.launch()
    for k in range(4):
        for q, x in enumerate(xs):
            x.copy_(gen(200 + 30 * q, 10 * k + q, device="cuda"))
        graph.replay()
        torch.cuda.synchronize()
        check(xs, dcbs, dtype)
        cal.launch()
        torch.cuda.synchronize()
        check(xs, dcbs, dtype)


def test_who_waits():
    """At a word that bears the call's tag and not yet the mark, and at no other: another call's, with the mark or without, a
    codebook's flags, anything."""
    tag, ready = 1 << 63 | 0x1234567 << 17, 1 << 16
    assert all(sz.internal_calibrate_waits(tag | added, tag) for added in (0, 1, 255))
    assert not any(sz.internal_calibrate_waits(tag | ready | added, tag) for added in (0, 1, 255))
    for other in (tag + (1 << 17), tag - (1 << 17), tag ^ 1 << 63, tag ^ 1 << 62):
        assert not sz.internal_calibrate_waits(other, tag) and not sz.internal_calibrate_waits(other | ready, tag)
    for flags in (0, 0x0101010101010101, 0x0100010001000100, 0x0001000000000000, (1 << 64) - 1):
        assert not sz.internal_calibrate_waits(flags, tag)


@pytest.mark.gpu
def test_calls_that_overlap_on_the_same_outputs_end():
    """What they leave is nobody's to use; the next call on those outputs has them to itself and is right."""
    xs = [kv_synth.kv_bf16(300 + 500 * k, k, device="cuda") for k in range(4)]
    dcbs = sz.DeviceCodebooks(4, sz.BF16)
    cal, streams = sz.CalibrateBatchDevice(xs, dcbs), [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for _ in range(20):
        for s in streams:
            cal.launch(stream=s)
    torch.cuda.synchronize()
    cal.launch()
    torch.cuda.synchronize()
    check(xs, dcbs, sz.BF16)


@pytest.mark.parametrize("dtype", [sz.BF16, sz.FP8_E5M2])
def test_launches(dtype):
    """One where no sample has more than 72 workgroups, else one that clears, one that ranks and one per 64 samples between them;
    samples with as many workgroups as they can have, and samples that share 256."""
    each = 16 * 4096 // (2 if dtype == sz.BF16 else 1)
    def launches(per):
        return sz.internal_calibrate_launches([w * each for w in per], dtype)
    assert [launches([w]) for w in (0, 1, 63, 72, 73, 128, 256, 257, 4096)] == [1] * 4 + [3] * 5
    assert [launches([w, w]) for w in (1, 72, 73, 128, 300)] == [1, 1, 3, 3, 3]
    assert launches([72, 72, 72, 0, 1]) == 1 and launches([72, 73, 5]) == 3
    assert [launches([300] * k) for k in (1, 2, 3, 4, 64, 65)] == [3, 3, 3, 1, 1, 4]
    assert [launches([1] * k) for k in (64, 65, 160, 161, 256, 257)] == [1, 1, 1, 2, 2, 7]
    assert launches([73] + [1] * 100) == 4 and launches([72] + [1] * 100) == 1
