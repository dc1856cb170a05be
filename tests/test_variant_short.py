"""Variant compress calls in one launch, whose workgroups tell one another their counts: lengths at the edges of its tiles of four
blocks and of its range, every way through it (all wait, most leave, two launches), what does not fit."""
import numpy as np
import pytest
import torch

import kv_synth
import test_variant_edges as edges
from oracle import variants as ov
import paper_2605_01708_amd as sz
from conftest import LEAVE
from test_variants import Run, check, dev

pytestmark = pytest.mark.gpu
FORMS = [(sz.BF16, 4, 16, sz.ESC_POS, 1024, 0), (sz.BF16, 3, 8, sz.ESC_POS, 256, 0), (sz.BF16, 4, 15, sz.ESC_SENTINEL, 256, 0),
         (sz.BF16, 3, 8, sz.ESC_ABS32, 0, 0), (sz.FP8_E5M2, 3, 8, sz.ESC_POS, 1024, 5), (sz.FP8_E5M2, 3, 7, sz.ESC_SENTINEL, 1024, 0),
         (sz.FP8_E4M3, 3, 8, sz.ESC_POS, 1024, 4), (sz.FP8_E4M3, 4, 16, sz.ESC_ABS32, 0, 4)]
GEN = {sz.BF16: kv_synth.kv_bf16, sz.FP8_E5M2: kv_synth.kv_e5m2, sz.FP8_E4M3: kv_synth.kv_e4m3}


def words(dt, n, seed):
    return GEN[dt](n // 1024 + 1, seed)[:n].numpy().view(np.uint16 if dt == sz.BF16 else np.uint8).copy()


@pytest.mark.parametrize("form", FORMS)
def test_lengths_at_the_edges(form, looks):
    v, o = sz.variant(*form), ov.variant(*form)
    dec = np.zeros(16, np.uint8)
    dec[:v.k] = sz.variant_calibrate(GEN[form[0]](64, 1), v).dec[:v.k]
    for blocks in (1, 4, 5, 8, 33 * 4, 257, 1025, 2048, 2049):
        for n in (blocks * 1024, blocks * 1024 - 5):
            x = words(form[0], n, blocks)
            run = Run(n, v)
            for limit in (0, LEAVE, sz.INTERNAL_NO_SHORT) if blocks < 1100 else (0, LEAVE):
                with looks(limit):
                    check(run, o, x, dec, f"looks {limit}")


@pytest.mark.parametrize("form", FORMS)
def test_two_blocks_a_wave(form, looks):
    """Tensors of more than 256 tiles of four blocks have half as many of eight: the first, odd ends, the last, and one word beyond."""
    v, o = sz.variant(*form), ov.variant(*form)
    dec = np.zeros(16, np.uint8)
    dec[:v.k] = sz.variant_calibrate(GEN[form[0]](64, 1), v).dec[:v.k]
    for n in (1024 * 1024, 1024 * 1024 + 1, 1531 * 1024 - 5, 2045 * 1024 + 3, 2048 * 1024, 2048 * 1024 + 1):
        x, run = words(form[0], n, 5), Run(n, v)
        for limit in (0, 1, LEAVE):
            with looks(limit):
                check(run, o, x, dec, f"looks {limit}")


@pytest.mark.parametrize("limit", [1, LEAVE, sz.INTERNAL_NO_SHORT])
@pytest.mark.parametrize("form", FORMS)
def test_escape_counts(form, limit, looks):
    if form[1] == 4 and form[0] == sz.FP8_E4M3:
        return   # all exponents have a code: there are no escapes to count
    with looks(limit):
        edges.test_escape_counts_at_the_edges_of_a_slot(*form)


@pytest.mark.parametrize("form", FORMS[:5])
def test_what_does_not_fit(form, looks):
    v = sz.variant(*form)
    cb = sz.variant_codebook_from_dec(list(range(v.k)), v)     # hardly anything is in this codebook
    n = 37 * 1024 - 9
    x, run = dev(words(form[0], n, 2)), Run(n, v)
    total = run.compress(x, cb)[0]
    fixed = sz.variant_total_bytes(n, 0, v)
    for cap in (fixed, fixed + (total - fixed) // 3, total - 1):
        with looks(0):
            got = run.compress(x, cb, cap)
            out = run.out.clone()
        with looks(sz.INTERNAL_NO_SHORT):
            assert run.compress(x, cb, cap) == got and torch.equal(run.out, out)


def test_captured_calls_are_replayed():
    v, o = sz.variant(*FORMS[1]), ov.variant(*FORMS[1])
    cb = sz.variant_calibrate(GEN[sz.BF16](64, 1), v)
    dec = np.zeros(16, np.uint8)
    dec[:8] = cb.dec[:8]
    n = 100 * 1024 - 37
    x, run = dev(words(sz.BF16, n, 1)), Run(n, v)
    run.compress(x, cb)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sz.variant_compress(x, v, cb, run.out, run.ws, run.sizes)
    for k in range(3):
        y = words(sz.BF16, n, 20 + k)
        x.copy_(dev(y))
        graph.replay()
        torch.cuda.synchronize()
        blob, m = ov.compress(y, o, dec)
        assert sz.read_sizes(run.sizes) == (blob.size, m, 0) and np.array_equal(run.out[:blob.size].cpu().numpy(), blob)
        check(run, o, words(sz.BF16, n, k), dec, "between replays")
