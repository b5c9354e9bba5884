"""The calls that a serving engine makes of this library, as timed cases.

A case names an operation, the cache it runs on and how much of it moves:

  op       gather / scatter            one request's blocks <-> packed chunks (device memory)
           gather_list / scatter_list  many requests' chunks in one launch
           restore / offload           host chunk images <-> blocks through the pinned ring
  layers, heads, dim, block, dtype, layout, pool   the paged cache (pool: GPU blocks)
  first, last                          the call's layer range
  blocks                               blocks moved (all requests together)
  chunk                                tokens per transfer chunk
  requests                             requests of a list call; their lengths are uneven

Every operation moves words unchanged, so results are compared exactly.
"""
import torch

import paper_2609_11744_amd as kvx

DEVICE = "cuda:0"
# KV words: bf16; 8-bit floats, which engines keep in byte tensors; float32.
DTYPES = {"bf16": torch.bfloat16, "fp8": torch.uint8, "f32": torch.float32}
LAYOUTS = {"nhd": kvx.KVX_LAYOUT_NHD, "hnd": kvx.KVX_LAYOUT_HND,
           "paged": kvx.KVX_LAYOUT_PAGED_ATTN}
RING_SLOTS, RING_SLOT_BYTES, RING_THREADS = 4, 64 << 20, 8


def _case(name, op, **over):
    # The 8B shape in bf16 unless said otherwise.
    c = {"name": name, "op": op, "layers": 32, "heads": 8, "dim": 128, "block": 16,
         "dtype": "bf16", "layout": "nhd", "pool": 8192, "first": 0, "last": 32,
         "blocks": 512, "chunk": 256, "requests": 1}
    c.update(over)
    return c


def listed():
    return [
        # The smallest store: a 256-token prefix of a two-layer model. Launch latency.
        _case("tiny gather", "gather", layers=2, last=2, heads=2, dim=64, pool=64, blocks=16),
        # Layer-by-layer loading: one layer of a 32k-token prefix, so that the
        # layer's attention can start before the next layer's load.
        _case("one layer scatter 32k", "scatter", first=7, last=8, blocks=2048),
        # The long document of the benchmark: an 80k-token prefix stored.
        _case("8b gather 80k", "gather", pool=20000, blocks=5000),
        # A 32k-token prefix loaded.
        _case("8b scatter 32k", "scatter", blocks=2048),
        # One rank of an 80-layer model over eight GPUs: one KV head each.
        _case("tp8 shard scatter 32k", "scatter", layers=80, last=80, heads=1, pool=20000,
              blocks=2048),
        # The same rank with an 8-bit cache, a prefix of no whole number of chunks.
        _case("tp8 fp8 shard gather", "gather", layers=80, last=80, heads=1, dtype="fp8",
              pool=20000, blocks=2041),
        # The paged-attention kernels' cache layout: a store of an 8k-token
        # prefix, and a load of a longer one into an 8-bit cache.
        _case("paged gather 8k", "gather", layout="paged", pool=4096),
        _case("paged fp8 scatter", "scatter", layout="paged", dtype="fp8", blocks=1999),
        # Head-major blocks of 64 tokens, two KV heads of eight (tensor parallel
        # over four GPUs), 1,024-token chunks.
        _case("hnd block 64 gather", "gather", layout="hnd", heads=2, block=64, pool=4096,
              blocks=1000, chunk=1024),
        # A decode step's stores: the new blocks of 64 requests in one launch,
        # most of their last chunks short.
        _case("batch store", "gather_list", blocks=2560, requests=64),
        # A batched step's loads on the 80-layer shape: the missing chunks of 16 requests.
        _case("batch load 80 layers", "scatter_list", layers=80, last=80, pool=4096,
              blocks=1120, requests=16),
        # A 2k-token prefix from host memory through the staging ring.
        _case("restore 2k", "restore", pool=2048, blocks=128),
    ]


def draw(rng):
    """One more call of the same kinds: any layout and word size, models of one
    to eighty layers, blocks of 8 to 128 tokens, 256 KiB to 4 GiB moved."""
    op = rng.choice(["gather", "scatter", "gather", "scatter", "gather_list", "scatter_list",
                     "restore", "offload"])
    layout = rng.choice(["nhd", "nhd", "hnd", "paged"])
    dtype = rng.choice(["bf16", "bf16", "fp8", "f32"])
    layers = rng.choice([2, 16, 28, 32, 48, 80])
    heads = rng.choice([1, 1, 2, 3, 4, 5, 8])
    dim = rng.choice([64, 80, 96, 128, 128, 256])
    block = rng.choice([8, 16, 16, 32, 64, 128])
    word = torch.empty((), dtype=DTYPES[dtype]).element_size()
    while block * heads * dim * word > 48 * 1024:  # the largest slab of the reordering layouts
        if block > 8:
            block //= 2
        else:
            heads = (heads + 1) // 2
    slab = block * heads * dim * word
    first, last = 0, layers
    if rng.random() < 0.25:  # part of the layers
        first = rng.randrange(layers)
        last = rng.randrange(first + 1, layers + 1)
    most = 27 if op in ("restore", "offload") else 32
    moved = 2.0 ** rng.uniform(18, most)
    blocks = max(1, min(16000, int(moved / (2 * (last - first) * slab))))
    requests = 1
    if op.endswith("_list"):
        requests = rng.randrange(1, min(64, blocks) + 1)
    # a pool of two to six times the call, up to 24 GB
    pool = int(blocks * rng.uniform(2, 6)) + 8
    pool = max(blocks, min(pool, 24_000_000_000 // (2 * layers * slab)))
    chunk = block * rng.choice([1, 3, 4, 16, 16, 16, 64])
    while (last - first) * 2 * slab * (chunk // block) > 2 ** 31 or \
            2 * slab * (chunk // block) > RING_SLOT_BYTES:
        chunk = block * max(1, chunk // block // 2)
    return {"op": op, "layers": layers, "heads": heads, "dim": dim, "block": block,
            "dtype": dtype, "layout": layout, "pool": pool, "first": first, "last": last,
            "blocks": blocks, "chunk": chunk, "requests": requests}


# ---- inputs ----------------------------------------------------------------------------


def _word(case):
    return torch.empty((), dtype=DTYPES[case["dtype"]]).element_size()


def _slab(case):
    return case["block"] * case["heads"] * case["dim"] * _word(case)


def _image_bytes(case):
    return case["blocks"] * (case["last"] - case["first"]) * 2 * _slab(case)


def _fill(t, gen):
    """N(0, 1) in the tensor's words, a few hundred MB at a time."""
    flat = t.view(-1)
    for part in flat.split(1 << 28):
        if t.dtype == torch.uint8:
            v = torch.empty(part.shape, dtype=torch.bfloat16, device=t.device).normal_(generator=gen)
            part.copy_(v.to(torch.float8_e4m3fn).view(torch.uint8))
        else:
            part.normal_(generator=gen)
    return t


def _lengths(case):
    """Blocks of each request: uneven, from a third of the mean to five thirds of it."""
    n, r = case["blocks"], case["requests"]
    weights = [1 + (i * 37 % r) * 4 / max(1, r - 1) for i in range(r)]
    total, got = sum(weights), []
    for i, w in enumerate(weights):
        left = n - sum(got) - (r - 1 - i)  # one block at least for each later request
        got.append(max(1, min(left, int(n * w / total))))
    got[-1] += n - sum(got)
    return got


def _chunks(case):
    """(first table entry, blocks) of every chunk, request by request."""
    bpc = case["chunk"] // case["block"]
    out, at = [], 0
    for n in _lengths(case):
        for k in range(0, n, bpc):
            out.append((at + k, min(bpc, n - k)))
        at += n
    return out


def _to_packed(op):
    return op in ("gather", "gather_list", "offload")


def _inputs(case, seed):
    """Cache tensors (K and V of each layer), block table and packed image."""
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    ks, vs = kvx.layer_shapes(case["pool"], case["block"], case["heads"], case["dim"],
                              _word(case), LAYOUTS[case["layout"]])
    dtype = DTYPES[case["dtype"]]
    # a tensor of its own for each K and V; more than 64 of them share allocations
    per = -(-2 * case["layers"] // 64)
    elems = case["pool"] * _slab(case) // _word(case)
    bases = [_fill(torch.empty((min(per, 2 * case["layers"] - i), elems), dtype=dtype,
                               device=DEVICE), gen)
             for i in range(0, 2 * case["layers"], per)]
    flat = [t for b in bases for t in b]
    k = [t.view(ks) for t in flat[0::2]]
    v = [t.view(vs) for t in flat[1::2]]
    table = torch.randperm(case["pool"], generator=gen, device=DEVICE)[:case["blocks"]]
    words = _image_bytes(case) // _word(case)
    image = torch.empty(words, dtype=dtype, device=DEVICE)
    if _to_packed(case["op"]):
        image.zero_()
    else:
        _fill(image, gen)
    return bases, k, v, table.to(torch.int32), image


def prepare(case, seed):
    bases, k, v, table, image = _inputs(case, seed)
    cache = kvx.PagedKVCache(k, v, LAYOUTS[case["layout"]])
    st = {"case": case, "cache": cache, "bases": bases, "table": table, "image": image}
    chunks = _chunks(case)
    per_block = (case["last"] - case["first"]) * 2 * _slab(case)
    if case["op"].endswith("_list"):
        st["refs"] = kvx.chunk_refs([(at * per_block, at, n) for at, n in chunks], DEVICE)
        st["n_chunks"] = len(chunks)
    if case["op"] in ("restore", "offload"):
        host = image.view(torch.uint8).cpu().numpy()
        st["host"], st["image"] = host, None
        ring = st["ring"] = kvx.StagingRing(DEVICE, RING_SLOTS, RING_SLOT_BYTES)
        if case["op"] == "restore":
            ring.bind(cache, case["first"], case["last"], case["blocks"], case["chunk"], host,
                      fill_threads=RING_THREADS)
        else:
            ring.bind_offload(cache, case["first"], case["last"], case["chunk"],
                              [(host[at * per_block:(at + n) * per_block], at, n)
                               for at, n in chunks], drain_threads=RING_THREADS)
    return st


def run(st):
    c, op = st["case"], st["case"]["op"]
    cache, table, first, last = st["cache"], st["table"], c["first"], c["last"]
    if op == "gather":
        kvx.kvx_gather_blocks(cache, first, last, table, c["blocks"], c["chunk"], st["image"])
        return st["image"]
    if op == "gather_list":
        kvx.kvx_gather_chunks(cache, first, last, table, c["blocks"], st["refs"], st["n_chunks"],
                              c["chunk"], st["image"])
        return st["image"]
    if op == "offload":
        kvx.kvx_offload_to_staging(st["ring"], table)
        return st["host"]
    if op == "scatter":
        kvx.kvx_scatter_blocks(cache, first, last, table, c["blocks"], c["chunk"], st["image"])
    elif op == "scatter_list":
        kvx.kvx_scatter_chunks(cache, first, last, table, c["blocks"], st["refs"], st["n_chunks"],
                               c["chunk"], st["image"])
    else:
        kvx.kvx_restore_from_staging(st["ring"], table)
    return st["bases"]


def work(case):
    # the image read once and written once, and a block id for each block
    return {"bytes": 2 * _image_bytes(case) + 4 * case["blocks"], "flops": 0}


def tolerance(case):
    return "exact"


def exact(case, seed):
    """The same moves in plain torch indexing. Words are moved, not computed, so
    the results keep their type. None for an image of very many pieces (a copy each)."""
    if len(_chunks(case)) * (case["last"] - case["first"]) > 80_000:
        return None
    bases, k, v, table, image = _inputs(case, seed)
    ids = table.long()
    bs, h, d = case["block"], case["heads"], case["dim"]
    at, pos = 0, 0
    for start, n in _chunks(case):
        for l in range(case["first"], case["last"]):
            for kv, t in ((0, k[l]), (1, v[l])):
                part = image[pos:pos + n * bs * h * d]
                pos += part.numel()
                some = ids[start:start + n]
                # the cache's block as [token][head][dim] and back
                if case["layout"] == "nhd":
                    to, back = (lambda x: x), (lambda x: x)
                elif case["layout"] == "hnd":
                    to = back = lambda x: x.transpose(1, 2)
                elif kv == 0:  # [head][dim / x][token][x]
                    x16 = t.shape[-1]
                    to = lambda x: x.permute(0, 3, 1, 2, 4)  # noqa: E731
                    back = lambda x: x.reshape(-1, bs, h, d // x16, x16).permute(0, 2, 3, 1, 4)  # noqa: E731
                else:  # [head][dim][token]
                    to = lambda x: x.permute(0, 3, 1, 2)  # noqa: E731
                    back = lambda x: x.permute(0, 2, 3, 1)  # noqa: E731
                if _to_packed(case["op"]):
                    part.copy_(to(t[some]).reshape(-1))
                else:
                    t[some] = back(part.view(n, bs, h, d))
    if case["op"] == "offload":
        return image.view(torch.uint8).cpu().numpy()
    return image if _to_packed(case["op"]) else bases
