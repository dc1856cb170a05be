"""The dense pass has a kernel for each number of chunks per wave, one for launches that memory alone bounds and one with a
loop over the chunks: around the limits of each, the stream of every one is the one of one chunk per wave, which other tests
compare with the oracle."""
import pytest
import torch

import kv_synth
import paper_2605_01708_amd as sz

pytestmark = pytest.mark.gpu

LONG_TILES = 6144   # of eight chunks


def _gen(dtype):
    return kv_synth.kv_bf16 if dtype == sz.BF16 else kv_synth.kv_e5m2


@pytest.fixture
def launch():
    yield sz.internal_test_launch
    sz.internal_test_launch()


@pytest.mark.parametrize("dtype", [sz.BF16, sz.FP8_E5M2])
@pytest.mark.parametrize("tensors", [1, 3])
def test_kernels_for_long_launches_and_loops(launch, dtype, tensors):
    cb = sz.calibrate(_gen(dtype)(64, 1), dtype)
    pool = _gen(dtype)(LONG_TILES * 8 + 16, 5, device="cuda").reshape(-1)
    at = torch.randint(0, pool.numel(), (pool.numel() // 500,), device="cuda")
    pool[at] = 0   # more escapes than the codebook's own
    for total in (LONG_TILES * 8 * 1024, (LONG_TILES - 1) * 8 * 1024, LONG_TILES * 8 * 1024 + 8191, (LONG_TILES - 1) * 8 * 1024 + 1):
        sizes = [total] if tensors == 1 else [total // 2 // 8192 * 8192, 8192 * 5 + 77]
        if tensors == 3:
            sizes.append(total - sum(sizes))
        xs, a = [], 0
        for n in sizes:
            xs.append(pool[a:a + n] if a % 64 == 0 else pool[a:a + n].clone())
            a += n
        caps = [sz.total_bytes(n, n // 50 + 4096, dtype) for n in sizes]
        ws, ref = sz.Workspace(max(sizes), dtype), None
        for cpt in (1, 0, 4, 8):   # 0: as the rules have it
            outs = [torch.full((c,), 0xA5, dtype=torch.uint8, device="cuda") for c in caps]
            rec = sz.new_sizes_array(len(xs))
            launch(cpt=cpt)
            if tensors == 1:
                sz.compress(xs[0], cb, outs[0], ws, rec)
            else:
                sz.CompressBatch(xs, [cb] * len(xs), outs).launch(ws, rec)
            got = outs, sz.read_sizes_array(rec)
            assert all(r[2] == 0 for r in got[1])
            if ref is None:
                ref = got
            assert got[1] == ref[1] and all(torch.equal(o, r) for o, r in zip(outs, ref[0])), (total, cpt)
        launch()
        for x, out, (nbytes, _, _) in zip(xs, ref[0], ref[1]):
            y, st = torch.zeros_like(x), sz.new_sizes()
            sz.decompress(out, nbytes, x.numel(), cb, y, st)
            assert sz.read_sizes(st)[2] == 0 and torch.equal(x, y)


@pytest.mark.parametrize("dtype", [sz.BF16, sz.FP8_E5M2])
def test_long_launch_from_a_paged_pool(launch, dtype):
    """blocks in any order, further apart than they are long"""
    block, blocks = 4096, LONG_TILES * 2 + 3
    cb = sz.calibrate(_gen(dtype)(64, 1), dtype)
    pool = _gen(dtype)((block + 1024) * blocks // 1024, 9, device="cuda").reshape(blocks, block + 1024)
    table = torch.randperm(blocks, generator=torch.Generator().manual_seed(4)).to("cuda", torch.int32)
    n = blocks * block - 1000
    x = pool[:, :block][table.long()].reshape(-1)[:n].contiguous()
    cap, ws, res = sz.total_bytes(n, n // 50 + 4096, dtype), sz.Workspace(n, dtype), []
    for paged in (False, True):
        out, rec = torch.full((cap,), 0xA5, dtype=torch.uint8, device="cuda"), sz.new_sizes()
        if paged:
            sz.compress_paged(sz.Paged(pool, table, block, (block + 1024) * pool.element_size()), n, cb, out, ws, rec)
        else:
            launch(cpt=1)
            sz.compress(x, cb, out, ws, rec)
            launch()
        res.append((out, sz.read_sizes(rec)))
    assert res[0][1] == res[1][1] and res[0][1][2] == 0 and torch.equal(res[0][0], res[1][0])
