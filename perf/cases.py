"""The codec's work as its users have it done: the cases that its speed is judged by.

Every case goes through the public calls of paper_2605_01708_amd, with the buffers, workspaces, codebooks and
marshalled item lists that a serving program keeps from call to call.  Sizes are those of the repository's workloads:
KV tensors of [tokens, 8 heads, 128], i.e. 1024 elements (one escape chunk) per token; "trim" cuts elements off the
end, so that the last chunk is ragged.

Fields of a case
  api      "single"   one call per tensor (splitzip_compress / splitzip_decompress)
           "batch"    one call for a list of tensors
           "paged"    one call for a list of tensors in paged pools behind one block table (16-token pages, K and V of
                      a layer side by side in a page)
           "dynamic"  codebooks counted per tensor on the device, compression under them, and decoding under the
                      codebook in each stream's own header
           "variant"  one of the ablation formats (code_bits, k, mode, chunk, value_bits)
  op       "compress", "decompress" or "roundtrip" (compress, then decompress what it wrote)
  dtype    "bf16", "e5m2" or (variants only) "e4m3"
  tokens, trim, tensors
  law      "kv" (normal times a log-normal scale per channel: about 0.12 % escapes under a calibrated codebook) or
           "outliers" (the same with 0.5 % outliers and 0.1 % zeros and subnormals)
"""
import math

import torch

import paper_2605_01708_amd as sz

CHANNELS = 8 * 128
PAGE_TOKENS = 16
DTYPES = {"bf16": sz.BF16, "e5m2": sz.FP8_E5M2, "e4m3": sz.FP8_E4M3}
FLOATS = {"bf16": torch.bfloat16, "e5m2": torch.float8_e5m2, "e4m3": torch.float8_e4m3fn}
MODES = {"pos": sz.ESC_POS, "sentinel": sz.ESC_SENTINEL, "abs32": sz.ESC_ABS32}
LARGEST = 64 * 32768 * CHANNELS      # elements of the largest listed case, compressed or decompressed once


def _case(name, api, op, dtype, tokens, tensors=1, trim=0, law="kv", code_bits=4, k=16, mode="pos", chunk=1024, value_bits=0):
    c = {"api": api, "op": op, "dtype": dtype, "tokens": tokens, "tensors": tensors, "trim": trim, "law": law}
    if api == "variant":
        c.update(code_bits=code_bits, k=k, mode=mode, chunk=chunk, value_bits=value_bits)
    return {"name": name, **c} if name else c


def listed():
    return [
        # the end of a prompt handed over by itself: a ragged tensor of 100 tokens, launches and host work count
        _case("tail_roundtrip", "single", "roundtrip", "bf16", 100, trim=37),
        # one layer's K of a 2048-token prefill chunk (4 MiB), compressed as soon as it is there and decoded on arrival
        _case("chunk_roundtrip", "single", "roundtrip", "bf16", 2048),
        # one layer's K of a 32768-token sequence (64 MiB), one call per tensor
        _case("tensor_compress", "single", "compress", "bf16", 32768),
        _case("tensor_decompress", "single", "decompress", "bf16", 32768),
        # the whole 4 GiB cache of that sequence, 32 layers x {K, V}, in one call
        _case("cache_compress", "batch", "compress", "bf16", 32768, 64),
        _case("cache_decompress", "batch", "decompress", "bf16", 32768, 64),
        # the same cache kept in FP8
        _case("cache_compress_e5m2", "batch", "compress", "e5m2", 32768, 64),
        _case("cache_decompress_e5m2", "batch", "decompress", "e5m2", 32768, 64),
        # a cache with outliers under a codebook that was calibrated without them: about seven escapes per chunk
        _case("outliers_roundtrip", "batch", "roundtrip", "bf16", 16384, 8, law="outliers"),
        # a sequence of 1999 tokens out of, and into, the paged pools of a serving stack
        _case("paged_roundtrip", "paged", "roundtrip", "bf16", 1999, 64),
        # codebooks per tensor, counted on the device at the time of the call
        _case("dynamic_roundtrip", "dynamic", "roundtrip", "bf16", 4096, 64),
        # an ablation format: 3-bit codes over a top-8 codebook, about 6 % escapes
        _case("top8_roundtrip", "variant", "roundtrip", "bf16", 32768, code_bits=3, k=8),
    ]


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    api = rng.choice(("single", "single", "batch", "batch", "paged", "dynamic", "variant"))
    op = rng.choice(("compress", "decompress", "roundtrip"))
    law = "outliers" if api in ("single", "batch") and rng.random() < 0.2 else "kv"
    dtype = "bf16" if law == "outliers" else rng.choice(("bf16", "bf16", "e5m2"))
    tokens = _spread(rng, 16, 32768)
    trim = 0 if rng.random() < 0.4 else rng.randrange(1, CHANNELS)
    if api == "variant":
        form = rng.choice((("bf16", 4, 16, "pos", 1024, 0), ("bf16", 4, 15, "sentinel", 1024, 0), ("bf16", 3, 8, "pos", 1024, 0),
                           ("bf16", 4, 16, "pos", 256, 0), ("bf16", 4, 16, "abs32", 1024, 0), ("e5m2", 4, 16, "pos", 1024, 0),
                           ("e5m2", 3, 8, "pos", 1024, 5), ("e4m3", 3, 8, "pos", 1024, 4)))
        return _case(None, api, op, form[0], tokens, 1, trim, "kv", *form[1:])
    tensors = 1
    if api != "single":
        tensors = min(_spread(rng, 2, 160), max(2, LARGEST // (4 * tokens * CHANNELS)))
    return _case(None, api, op, dtype, tokens, tensors, trim, law)


def _elems(case):
    return case["tokens"] * CHANNELS - case["trim"]


def _variant(case):
    return sz.variant(DTYPES[case["dtype"]], case["code_bits"], case["k"], MODES[case["mode"]], case["chunk"], case["value_bits"])


def _total(case, escapes):
    if case["api"] == "variant":
        return sz.variant_total_bytes(_elems(case), escapes, _variant(case))
    return sz.total_bytes(_elems(case), escapes, DTYPES[case["dtype"]])


def _values(tokens, scale, gen):
    return torch.randn(tokens, CHANNELS, generator=gen, device="cuda") * scale


def _outliers(x, gen):
    """0.5 % of the elements scaled up by 2^6 .. 2^14, 0.1 % zeros and subnormals; BF16 words"""
    u = torch.rand(x.shape, generator=gen, device="cuda")
    up = torch.exp2(torch.randint(6, 15, x.shape, generator=gen, device="cuda", dtype=torch.int32).float())
    w = torch.where(u < 0.005, x * up, x).to(torch.bfloat16).view(torch.int16)
    low = torch.randint(0, 128, x.shape, generator=gen, device="cuda", dtype=torch.int16)
    low = torch.where(low < 64, torch.zeros_like(low), low)
    return torch.where(u > 0.999, low | (w & -32768), w)


def prepare(case, seed):
    api, op, n, nt = case["api"], case["op"], _elems(case), case["tensors"]
    dtype, fl = DTYPES[case["dtype"]], FLOATS[case["dtype"]]
    raw = torch.int16 if dtype == sz.BF16 else torch.uint8
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    # the tensors: K and V of one layer after the other, all in one allocation, each 256-byte aligned
    step = -(-n // 256) * 256
    words = torch.zeros(nt * step, dtype=raw, device="cuda")
    xs = [words[k * step:k * step + n] for k in range(nt)]
    sample = {0: [], 1: []}
    for k, x in enumerate(xs):
        scale = torch.exp(torch.randn(CHANNELS, generator=gen, device="cuda")) * (0.5 if k & 1 else 1.0)
        v = _values(case["tokens"], scale, gen)
        w = _outliers(v, gen) if case["law"] == "outliers" else v.to(fl).view(raw)
        x.copy_(w.reshape(-1)[:n])
        if k < 32:
            sample[k & 1].append(_values(max(8, 512 // min(nt, 32)), scale, gen).to(fl).view(raw).reshape(-1).cpu())
    s = {"case": case, "n": n, "xs": xs}
    # a stream's buffer: room for 3 % escapes (12 % under a top-8 codebook); small tensors: room for many more
    most = max(n * (12 if case.get("k", 16) <= 8 else 3) // 100, min(n, 65536))
    cap = -(-_total(case, most) // 256) * 256
    streams = torch.zeros(nt * cap, dtype=torch.uint8, device="cuda")
    s["streams"], s["outs"] = streams, [streams[k * cap:(k + 1) * cap] for k in range(nt)]
    s["rec"] = sz.new_sizes_array(nt)
    s["drec"] = sz.new_sizes()
    s["words"] = torch.zeros(nt * step, dtype=raw, device="cuda")
    ys = [s["words"][k * step:k * step + n] for k in range(nt)]
    s["ys"] = ys

    if api == "variant":
        s["v"] = _variant(case)
        s["cb"] = sz.variant_calibrate(torch.cat(sample[0]), s["v"])
        s["ws"] = torch.empty(sz.variant_workspace_bytes(n, s["v"]), dtype=torch.uint8, device="cuda")
    else:
        s["ws"] = sz.Workspace(n, dtype)
    if api in ("single", "batch", "paged"):
        books = [sz.calibrate(torch.cat(sample[q]), dtype) if sample[q] else None for q in (0, 1)]
        cbs = [books[k & 1] for k in range(nt)]
        s["cb"] = books[0]
    if api == "batch":
        s["enc"] = sz.CompressBatch(xs, cbs, s["outs"])
        make_dec = lambda sizes: sz.DecompressBatch(s["outs"], sizes, [n] * nt, cbs, ys)  # noqa: E731
    elif api == "dynamic":
        s["dcbs"] = sz.DeviceCodebooks(nt, dtype)
        s["cal"] = sz.CalibrateBatchDevice(xs, s["dcbs"])
        s["enc"] = sz.CompressBatchDcb(xs, s["dcbs"], s["outs"])
        make_dec = lambda sizes: sz.DecompressBatchOwn(s["outs"], sizes, [n] * nt, dtype, ys)  # noqa: E731
    elif api == "paged":
        # a pool per layer: [pages, {K, V}, 16 tokens]; the sequence's pages lie anywhere in it
        pe, es = PAGE_TOKENS * CHANNELS, words.element_size()
        blocks, layers = -(-n // pe), -(-nt // 2)
        pages = blocks + blocks // 4 + 1
        table = torch.randperm(pages, generator=gen, device="cuda")[:blocks]
        src = torch.zeros(layers, pages, 2, pe, dtype=raw, device="cuda")
        for k, x in enumerate(xs):
            full = torch.zeros(blocks * pe, dtype=raw, device="cuda")
            full[:n] = x
            src[k // 2, table, k % 2] = full.view(blocks, pe)
        s["words"] = torch.zeros_like(src)
        s["src"], s["table"] = src, table.to(torch.int32)
        views = [[p[k // 2].reshape(-1)[(k % 2) * pe:] for k in range(nt)] for p in (src, s["words"])]
        geometry = sz.Paged(src, s["table"], pe, 2 * pe * es, 0, pages)
        s["enc"] = sz.CompressBatchPaged(views[0], [n] * nt, cbs, s["outs"], geometry)
        make_dec = lambda sizes: sz.DecompressBatchPaged(s["outs"], sizes, [n] * nt, cbs, views[1], geometry)  # noqa: E731
    # a receiver knows the length of every stream: the streams of these tensors are made once here
    _compress(s)
    torch.cuda.synchronize()
    s["sizes"] = [r[0] for r in sz.read_sizes_array(s["rec"])]
    if api not in ("single", "variant"):
        s["dec"] = make_dec(s["sizes"])
    if op != "decompress":
        streams.zero_()
    return s


def _compress(s):
    api = s["case"]["api"]
    if api == "single":
        sz.compress(s["xs"][0], s["cb"], s["outs"][0], s["ws"], s["rec"])
    elif api == "variant":
        sz.variant_compress(s["xs"][0], s["v"], s["cb"], s["outs"][0], s["ws"], s["rec"])
    else:
        if api == "dynamic":
            s["cal"].launch()
        s["enc"].launch(s["ws"], s["rec"])


def _decompress(s):
    api = s["case"]["api"]
    if api == "single":
        sz.decompress(s["outs"][0], s["sizes"][0], s["n"], s["cb"], s["ys"][0], s["drec"])
    elif api == "variant":
        sz.variant_decompress(s["outs"][0], s["sizes"][0], s["n"], s["v"], s["cb"], s["ys"][0], s["drec"])
    else:
        s["dec"].launch(s["drec"])


def run(s):
    case = s["case"]
    got = {}
    if case["op"] != "decompress":
        _compress(s)
        got["streams"], got["sizes"] = s["streams"], s["rec"]
        if case["api"] == "dynamic":
            got["codebooks"], got["counts"] = s["dcbs"].buf, s["dcbs"].hists
    if case["op"] != "compress":
        _decompress(s)
        got["words"] = s["words"]
        # total_bytes and n_escapes of a batch's one record are those of whichever stream wrote last: its status alone
        got["status"] = s["drec"][2:]
    return got


def work(case):
    n, nt = _elems(case), case["tensors"]
    raw = n * (2 if case["dtype"] == "bf16" else 1)
    rate = 0.0066 if case["law"] == "outliers" else 0.058 if case.get("k", 16) <= 8 else 0.0012
    stream = _total(case, int(n * rate))
    return {"bytes": nt * (raw + stream) * (2 if case["op"] == "roundtrip" else 1), "flops": 0}


def tolerance(case):
    return "exact"   # bytes and words: a stream is a pure function of the words and the codebook
