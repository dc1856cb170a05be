"""The binding's short way (lib().fast) against its general way: what it takes gives the same streams, words and records,
what it does not take is left to the general way, errors included."""
import os
import shutil
import subprocess
import sys
import timeit

import numpy as np
import pytest
import torch

import kv_synth
import paper_2605_01708_amd as sz
from paper_2605_01708_amd import binding


class Sub(torch.Tensor):
    pass


def _general(monkeypatch):
    """every function of lib().fast answers that it has done nothing"""
    L = sz.lib()
    for name in vars(L.fast):
        monkeypatch.setattr(L.fast, name, lambda *a: binding._NOT_TAKEN)


def test_other_forms_are_not_taken():
    cb = sz.codebook_from_dec(range(100, 116), sz.BF16)
    x, out, rec = torch.zeros(64, dtype=torch.int16), torch.zeros(4096, dtype=torch.uint8), torch.zeros(3, dtype=torch.int64)
    f = sz.lib().fast
    assert f.splitzip_compress(x, cb.c, out, None, out, 1 << 24, rec, 0) == 1                     # host tensors
    assert f.splitzip_compress(x.as_subclass(Sub), cb.c, out, None, out, 1 << 24, rec, 0) == 1    # another class
    assert f.splitzip_compress(None, None, None) == 1 and f.splitzip_compress() == 1              # not enough of them
    assert f.splitzip_decompress(out, 2.0, 64, cb.c, x, None, 0) == 1                             # not an integer
    with pytest.raises(AttributeError):
        sz.decompress(None, 4096, 64, cb, x, None, stream=torch.zeros(1))
    with pytest.raises(ValueError):
        sz.compress(x.view(torch.uint8), cb, out, type("W", (), {"buf": out, "nbytes": 4096}), rec)
    with pytest.raises(ValueError):
        sz.decompress(out, 4096, 65, cb, x)


def test_a_form_that_is_not_taken_costs_next_to_nothing():
    """less than the general way's own call into the library, which follows (best of many: 0.1 us against 0.7)"""
    L, items, rec = sz.lib(), (binding._CDItem * 1)(), torch.zeros(3, dtype=torch.int64)
    cb = sz.codebook_from_dec(range(100, 116), sz.BF16)
    x, out = torch.zeros(64, dtype=torch.int16), torch.zeros(4096, dtype=torch.uint8)
    assert L.fast.splitzip_compress(x, cb.c, out, None, out, 1 << 24, rec, 0) == 1
    refused = min(timeit.repeat(lambda: L.fast.splitzip_compress(x, cb.c, out, None, out, 1 << 24, rec, 0), number=500, repeat=20))
    general = min(timeit.repeat(lambda: L.splitzip_decompress_batch(items, 0, sz.BF16, None, 0), number=500, repeat=20))
    assert refused < general


def test_every_function_has_its_library_function():
    for name in vars(sz.lib().fast):
        assert hasattr(sz.lib(), name)


def test_codebooks_of_a_batch_are_all_looked_at():
    """a bad codebook is refused wherever it stands among good ones"""
    good = [sz.codebook_from_dec(range(100 + q, 116 + q), sz.BF16) for q in range(3)]
    bad = sz.codebook_from_dec(range(100, 116), sz.BF16)
    bad.c.member[100] = 0
    x, out = torch.zeros(64, dtype=torch.int16), torch.zeros(8192, dtype=torch.uint8)
    base = (out.data_ptr() + 15) & ~15
    # three by turns: none of the two looked at last comes again; K's and V's by turns and runs of one: it does, before the
    # bad one and behind it
    for order, at in ((order, at) for order in ((0, 1, 2), (0, 1), (0,), (0, 0, 1, 1)) for at in range(6)):
        cbs = [good[order[q % len(order)]] for q in range(6)]
        cbs[at] = bad
        items = (binding._CItem * 6)()
        ditems = (binding._CDItem * 6)()
        for q, cb in enumerate(cbs):
            items[q] = binding._CItem(base, 64, base, 4096, binding.C.pointer(cb.c))
            ditems[q] = binding._CDItem(base, 4096, 64, base, binding.C.pointer(cb.c))
        assert sz.lib().splitzip_compress_batch(items, 6, sz.BF16, base, 1 << 30, base, None) == -1
        assert sz.lib().splitzip_decompress_batch(ditems, 6, sz.BF16, base, None) == -1
    del x


def test_batches_are_decoded_without_a_record():
    """the record of a batch decompress call may be left out: no reason to refuse it (no streams: nothing is launched)"""
    f, items = sz.lib().fast, (binding._CDItem * 1)()
    assert f.splitzip_decompress_batch(items, 0, sz.BF16, None, 0) == 0
    assert f.splitzip_decompress_batch_own(items, 0, sz.BF16, None, 0) == 0


def test_a_record_in_host_memory_is_taken():
    """a record may lie in pinned host memory (here: any host memory, no streams, nothing is launched)"""
    f, items, rec = sz.lib().fast, (binding._CDItem * 1)(), torch.zeros(3, dtype=torch.int64)
    assert f.splitzip_decompress_batch(items, 0, sz.BF16, rec, 0) == 0
    assert f.splitzip_decompress_batch_own(items, 0, sz.BF16, rec, 0) == 0


def _elsewhere(tmp_path, code, with_module=False, **env):
    """code run on a copy of the package; what it prints"""
    here, there = os.path.dirname(os.path.abspath(binding.__file__)), tmp_path / "paper_2605_01708_amd"
    there.mkdir()
    for name in os.listdir(here):
        if name.endswith(".py") or name == "libsplitzip.so" or (with_module and name.startswith("_fastcall")):
            shutil.copy(os.path.join(here, name), there)
    run = subprocess.run([sys.executable, "-c", code], cwd=tmp_path, env={**os.environ, "PYTHONPATH": str(tmp_path), **env}, capture_output=True,
                         text=True, timeout=120)
    assert run.returncode == 0, run.stderr
    return run.stdout


CALLS = """
import warnings
import torch
{before}
with warnings.catch_warnings(record=True) as told:
    warnings.simplefilter("always")
    import paper_2605_01708_amd as sz
    from paper_2605_01708_amd import binding
    L = sz.lib()
assert binding.__file__.startswith({at!r})
items = (binding._CDItem * 1)()
assert L.splitzip_decompress_batch(items, 0, sz.BF16, None, 0) == 0
assert L.fast.splitzip_decompress_batch(items, 0, sz.BF16, None, 0) == {answer}
assert sz.calibrate(torch.zeros(64, dtype=torch.int16), sz.BF16).dec[0] == 0
print([str(w.message) for w in told])
"""


def test_the_library_alone_serves_every_call(tmp_path):
    told = _elsewhere(tmp_path, CALLS.format(before="", at=str(tmp_path), answer=1))
    assert "paper_2605_01708_amd.build" in told


def test_a_module_for_another_torch_is_not_used(tmp_path):
    told = _elsewhere(tmp_path, CALLS.format(before="torch.__version__ = '0.0'", at=str(tmp_path), answer=1), with_module=True)
    assert "built for torch " + torch.__version__ in told


def test_the_module_of_this_torch_is_used(tmp_path):
    assert _elsewhere(tmp_path, CALLS.format(before="", at=str(tmp_path), answer=0), with_module=True) == "[]\n"


def test_the_library_is_built_where_the_module_cannot_be(tmp_path):
    code = "from paper_2605_01708_amd import build as b; import os; print(b.build() == b.LIB, [n for n in os.listdir(b.HERE) if n.startswith('_fastcall')])"
    assert _elsewhere(tmp_path, code, with_module=True, HIPCC="true", CXX="no-such-compiler") == "True []\n"


def _in_a_child(what) -> int:
    pid = os.fork()
    if pid == 0:
        code = 99
        try:
            code = what()
        finally:
            os._exit(code)
    return os.waitstatus_to_exitcode(os.waitpid(pid, 0)[1])


def test_nothing_is_taken_in_a_fork_that_must_not_use_the_gpu(monkeypatch):
    items = (binding._CDItem * 1)()

    def taken():
        return sz.lib().fast.splitzip_decompress_batch(items, 0, sz.BF16, None, 0)   # no streams: nothing is launched

    assert taken() == 0 and _in_a_child(taken) == 0
    monkeypatch.setattr(torch._C, "_cuda_isInBadFork", lambda: True)
    assert _in_a_child(taken) == 1

    def loaded_there():
        binding._lib = None
        return taken()
    assert _in_a_child(loaded_there) == 1
    monkeypatch.undo()
    assert taken() == 0


@pytest.mark.gpu
def test_a_child_of_a_process_on_the_gpu_is_refused():
    x = kv_synth.kv_bf16(8, 0).cuda()
    cb = sz.calibrate(kv_synth.kv_bf16(8, 1), sz.BF16)
    ws, rec = sz.Workspace(x.numel(), sz.BF16), sz.new_sizes()
    out = torch.zeros(sz.compress_bound(x.numel(), sz.BF16), dtype=torch.uint8, device="cuda")
    sz.compress(x, cb, out, ws, rec)
    torch.cuda.synchronize()

    def child():
        if not torch._C._cuda_isInBadFork():
            return 3   # nothing would refuse it: go no further
        try:
            sz.compress(x, cb, out, ws, rec)
        except RuntimeError as e:
            return 0 if "fork" in str(e) else 4
        return 5
    assert _in_a_child(child) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [sz.BF16, sz.FP8_E5M2])
@pytest.mark.parametrize("form", ["plain", "capacity", "stream", "parameter", "subclass", "shaped", "mode"])
def test_both_ways_give_the_same(dtype, form, monkeypatch):
    gen = kv_synth.kv_bf16 if dtype == sz.BF16 else kv_synth.kv_e5m2
    x = gen(70, 5)[:-11].contiguous()
    cb = sz.calibrate(gen(64, 1), dtype)
    v = sz.variant(dtype, 3, 8)
    vcb = sz.variant_calibrate(gen(64, 1), v)
    n = x.numel()
    xd = x.cuda()
    shaped = xd.view(1, n) if form == "shaped" else xd
    if form == "subclass":
        shaped = xd.as_subclass(Sub)
    if form == "parameter":
        shaped = torch.nn.Parameter(xd, requires_grad=False)
    stream = torch.cuda.Stream() if form == "stream" else None
    bound = sz.compress_bound(n, dtype)
    answers = {}   # entry point -> what its short way answered, call by call

    def all_calls():
        torch.cuda.synchronize()
        ws = sz.Workspace(n, dtype)
        vws = torch.empty(sz.variant_workspace_bytes(n, v), dtype=torch.uint8, device="cuda")
        outs = [torch.zeros(max(bound, sz.variant_compress_bound(n, v)) + 64, dtype=torch.uint8, device="cuda") for _ in range(5)]
        recs = [sz.new_sizes() for _ in range(5)]
        brec, drec = sz.new_sizes_array(2), sz.new_sizes()
        ys = [torch.zeros_like(xd) for _ in range(4)]
        d_cbs, d_cb = sz.DeviceCodebooks(2, dtype), sz.DeviceCodebook(dtype)
        d_cb.buf.copy_(torch.from_numpy(np.frombuffer(bytes(cb.c) + bytes(-len(bytes(cb.c)) % 8), np.int64).copy()))
        # the words in pages of 2048, in reverse, and such a pool to decode into
        table = torch.arange(-(-n // 2048) - 1, -1, -1, dtype=torch.int32, device="cuda")
        pool = torch.zeros(table.numel() * 2048, dtype=xd.dtype, device="cuda")
        pool[:n] = xd.view(-1)
        pools = [pool.view(-1, 2048).flip(0).contiguous(), torch.zeros_like(pool), torch.zeros_like(pool), torch.zeros_like(pool)]
        paged = [sz.Paged(p, table, 2048, 2048 * xd.element_size()) for p in pools]
        outs2 = [torch.zeros(bound + 64, dtype=torch.uint8, device="cuda") for _ in range(5)]
        rec2, brec2 = [sz.new_sizes() for _ in range(2)], [sz.new_sizes_array(2), sz.new_sizes_array(1)]
        ys2, spare = [torch.zeros_like(xd) for _ in range(8)], torch.zeros_like(xd)
        cap = bound if form == "capacity" else None
        torch.cuda.synchronize()
        sz.compress(shaped, cb, outs[0], ws, recs[0], stream, cap)
        sz.compress_noalloc(shaped, cb, outs[1], recs[1], stream, cap)
        sz.variant_compress(shaped, v, vcb, outs[2], vws, recs[2], stream)
        sz.CalibrateBatchDevice([xd, xd], d_cbs).launch(stream)
        sz.CompressBatchDcb([xd, xd], d_cbs, outs[3:5]).launch(ws, brec, stream)
        sz.compress_dcb(shaped, d_cb, outs2[0], ws, rec2[0], stream, cap)
        sz.compress_paged(paged[0], n, cb, outs2[1], ws, rec2[1], stream, cap)
        sz.CompressBatch([xd, xd], [cb, cb], outs2[2:4]).launch(ws, brec2[0], stream)
        sz.CompressBatchPaged([pools[0]], [n], [cb], outs2[4:5], paged[0]).launch(ws, brec2[1], stream)
        torch.cuda.synchronize()
        sizes = [sz.read_sizes(r)[0] for r in recs[:3]] + [r[0] for r in sz.read_sizes_array(brec)]
        sizes2 = [sz.read_sizes(r)[0] for r in rec2] + [r[0] for b in brec2 for r in sz.read_sizes_array(b)]
        assert sizes2 == sizes[:1] * 5 and all(torch.equal(o[:sizes[0]], outs[0][:sizes[0]]) for o in outs2)
        sz.decompress(outs[0], sizes[0], n, cb, ys[0], drec, stream)
        sz.decompress_own(outs[1], sizes[1], n, dtype, ys[1], None, stream)
        sz.variant_decompress(outs[2], sizes[2], n, v, vcb, ys[2], None, stream)
        sz.DecompressBatchOwn(outs[3:4], sizes[3:4], [n], dtype, ys[3:4]).launch(drec, stream)
        for q, r in enumerate((drec, None)):   # with a record and without one
            sz.decompress_dcb(outs2[0], sizes[0], n, d_cb, ys2[4 * q], r, stream)
            sz.decompress_paged(outs2[1], sizes[0], n, cb, paged[1 + q], r, stream)
            sz.DecompressBatch(outs2[2:4], sizes[:1] * 2, [n] * 2, [cb] * 2, ys2[4 * q + 1:4 * q + 3]).launch(r, stream)
            sz.DecompressBatchDcb(outs[3:5], sizes[3:5], [n] * 2, d_cbs, [ys2[4 * q + 3], spare]).launch(r, stream)
            sz.DecompressBatchPaged(outs2[4:5], sizes[:1], [n], [cb], pools[3:4], paged[3]).launch(r, stream)
        sz.decompress(outs[0], sizes[0], n, cb, ys[0], None, stream)
        sz.decompress_own(outs[1], sizes[1], n, dtype, ys[1], drec, stream)
        sz.variant_decompress(outs[2], sizes[2], n, v, vcb, ys[2], drec, stream)
        sz.DecompressBatchOwn(outs[3:4], sizes[3:4], [n], dtype, ys[3:4]).launch(None, stream)
        torch.cuda.synchronize()
        for y in ys2:
            assert torch.equal(y, xd)
        for p in pools[1:]:
            assert torch.equal(p.view(-1, 2048).flip(0).reshape(-1)[:n], xd.view(-1))
        assert drec[2] == 0
        return [t.cpu() for t in outs + recs + [brec, d_cbs.buf, d_cbs.hists, drec[2:]] + ys] + sizes

    L = sz.lib()
    entries = sorted(vars(L.fast))
    for name in entries:
        def asked(*a, name=name, real=getattr(L.fast, name)):
            answers.setdefault(name, []).append(real(*a))
            return answers[name][-1]
        monkeypatch.setattr(L.fast, name, asked)
    if form == "mode":
        class Watch(torch.overrides.TorchFunctionMode):
            def __torch_function__(self, func, types, args=(), kwargs=None):
                return func(*args, **(kwargs or {}))
        with Watch():
            fast = all_calls()
    else:
        fast = all_calls()
    # every entry point was called, and taken wherever all of its arguments had the plain form
    assert sorted(answers) == entries and len(entries) == 18
    of_x = ("splitzip_compress", "splitzip_compress_noalloc", "splitzip_compress_dcb", "splitzip_variant_compress")
    for name, got in answers.items():
        assert set(got) == {1 if form == "mode" or (form == "subclass" and name in of_x) else 0}, name
    _general(monkeypatch)
    general = all_calls()
    for a, b in zip(fast, general):
        assert torch.equal(a, b) if torch.is_tensor(a) else a == b
    for y in fast[-9:-5]:
        assert np.array_equal(kv_synth.to_numpy_words(y), kv_synth.to_numpy_words(x))


@pytest.mark.gpu
def test_refusals_are_those_of_the_general_way(monkeypatch):
    x = kv_synth.kv_bf16(8, 0).cuda()
    n = x.numel()
    cb = sz.calibrate(kv_synth.kv_bf16(8, 1), sz.BF16)
    ws = sz.Workspace(n, sz.BF16)
    out, rec = torch.zeros(sz.compress_bound(n, sz.BF16), dtype=torch.uint8, device="cuda"), sz.new_sizes()
    calls = [
        lambda: sz.compress(x.view(-1)[::2], cb, out, ws, rec),                     # not contiguous
        lambda: sz.compress(x.view(torch.uint8), cb, out, ws, rec),                 # another word size
        lambda: sz.compress(x, cb, out, ws, rec, capacity=100),                     # too small
        lambda: sz.compress(x.view(-1)[1:], cb, out, ws, rec),                      # not aligned
        lambda: sz.decompress(out, sz.fixed_bytes(n, sz.BF16), n, cb, x.view(-1)[:-1], rec),   # too short
        lambda: sz.decompress(out, 10, n, cb, x, rec),
        lambda: sz.decompress(out, 4096, -1, cb, x, rec),
        lambda: sz.compress(x, cb, out, ws, None),
    ]

    def answers():
        got = []
        for call in calls:
            with pytest.raises(Exception) as e:
                call()
            got.append((type(e.value), getattr(e.value, "code", None)))
        return got

    fast = answers()
    _general(monkeypatch)
    assert fast == answers()
