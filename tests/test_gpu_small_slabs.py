"""Slabs of at most 2 KiB, several of which one workgroup moves: the grouped
kernels at the sizes where they can go wrong (one vector; groups that fill a
workgroup and that leave lanes over; whole waves per slab; the largest grouped
slab and the first one that is not), in image order, on the linear walk and, for
the first that is not grouped, in destination order, as chunk lists with short
chunks, with bad block ids and bad references. Everything is compared whole with the oracle."""
import numpy as np
import pytest

import kvsynth
import oracle
from kvtest_util import (cache_and_mirror, check_cache_equals, device_table, first_mismatch,
                         seeded_ids, to_host)

torch = pytest.importorskip("torch")
import paper_2609_11744_amd as kvx  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
NHD, HND = oracle.LAYOUT_NHD, oracle.LAYOUT_HND
CANARY = 0xA5

SHAPES = [
    # (layout, block, heads, dim, elem): vectors per slab
    (NHD, 1, 1, 8, 2),      # 1
    (NHD, 3, 1, 8, 2),      # 3
    (NHD, 5, 1, 80, 1),     # 25: ten slabs, six lanes over
    (NHD, 8, 1, 64, 1),     # 32: half a wave
    (NHD, 8, 1, 64, 2),     # 64: one wave
    (NHD, 5, 3, 48, 2),     # 90: two slabs, 76 lanes over
    (NHD, 1, 1, 1016, 2),   # 127
    (NHD, 16, 1, 128, 1),   # 128: two waves, the largest
    (NHD, 1, 1, 1032, 2),   # 129: not grouped
    (HND, 2, 3, 32, 1),     # 12
    (HND, 8, 2, 64, 1),     # 64
    (HND, 16, 2, 64, 1),    # 128
    (HND, 3, 5, 128, 1),    # 120
    (HND, 16, 1, 64, 2),    # 128, one head
    (HND, 1, 4, 64, 2),     # 32, one token
    (HND, 43, 3, 16, 1),    # 129: not grouped
]


def _bt(ids):
    return device_table(ids, DEV)


def _setup(shape, L, NB, seed):
    layout, bs, h, d, e = shape
    s = oracle.Shape(L, NB, bs, h, d, e, layout)
    return (s, *cache_and_mirror(s, seed, DEV))


@pytest.mark.parametrize("shape", SHAPES, ids=[f"s{i}" for i in range(len(SHAPES))])
@pytest.mark.parametrize("n,bpc", [(1, 1), (37, 5), (1031, 16)])
def test_small_slabs_bit_exact(shape, n, bpc):
    L, l0, l1 = 5, 1, 4
    bs = shape[1]
    NB = 2 * n + 5
    s, cache, mirror = _setup(shape, L, NB, 400 + n)
    src, dst_ids = seeded_ids(400 + n, NB, n, n)
    expect = oracle.gather(s, *mirror, l0, l1, src, bpc * bs)
    out = torch.full((expect.size + 4096,), CANARY, dtype=torch.uint8, device=DEV)
    kvx.kvx_gather_blocks(cache, l0, l1, _bt(src), n, bpc * bs, out)
    torch.cuda.synchronize()
    kvx.kvx_check()
    got = to_host(out)
    assert first_mismatch(got[:expect.size], expect) is None
    assert (got[expect.size:] == CANARY).all()
    kvx.kvx_scatter_blocks(cache, l0, l1, _bt(dst_ids), n, bpc * bs, out)
    kvx.kvx_check()
    oracle.scatter(s, *mirror, l0, l1, dst_ids, bpc * bs, expect)
    check_cache_equals(cache, mirror, L)
    walk = kvx.kvx_copy_walk(cache, l0, l1, n, bpc * bs, False)
    slab = int(np.prod(shape[1:]))
    assert walk["ordered"] == (n >= 1024 and shape[0] == HND and slab > 2048)
    assert walk["linear"] == (n >= 1024 and 4096 % slab == 0)


@pytest.mark.parametrize("shape", SHAPES, ids=[f"s{i}" for i in range(len(SHAPES))])
def test_small_slab_chunk_lists_bit_exact(shape):
    L, bpc = 3, 7
    bs = shape[1]
    sizes = [7, 1, 3, 7, 2, 6, 7, 5]
    n = sum(sizes)
    NB = 2 * n + 3
    s, cache, mirror = _setup(shape, L, NB, 500)
    src, dst_ids = seeded_ids(500, NB, n, n)
    per_block = oracle.packed_bytes(s, 0, L, 1)
    refs, at, off = [], 0, 32
    for m in sizes:
        refs.append((off, at, m))
        at, off = at + m, off + m * per_block + 16
    rd = kvx.chunk_refs(refs, DEV)
    out = torch.full((off,), CANARY, dtype=torch.uint8, device=DEV)
    kvx.kvx_gather_chunks(cache, 0, L, _bt(src), n, rd, len(refs), bpc * bs, out)
    kvx.kvx_check()
    want = np.full(off, CANARY, np.uint8)
    images = [oracle.gather(s, *mirror, 0, L, src[a:a + m], m * bs) for _, a, m in refs]
    for (o, _, _), img in zip(refs, images):
        want[o:o + img.size] = img
    assert first_mismatch(to_host(out), want) is None
    kvx.kvx_scatter_chunks(cache, 0, L, _bt(dst_ids), n, rd, len(refs), bpc * bs, out)
    kvx.kvx_check()
    for (_, a, m), img in zip(refs, images):
        oracle.scatter(s, *mirror, 0, L, dst_ids[a:a + m], m * bs, img)
    check_cache_equals(cache, mirror, L)


@pytest.mark.parametrize("shape", [SHAPES[3], SHAPES[4], SHAPES[12]], ids=["lane", "wave", "hnd"])
def test_small_slabs_skip_and_report_bad_ids_and_refs(shape):
    L, n, bpc = 2, 20, 4
    bs = shape[1]
    NB = 50
    s, cache, mirror = _setup(shape, L, NB, 600)
    (ids,) = seeded_ids(600, NB, n)
    bad = ids.copy()
    bad[3], bad[11] = NB, -1
    good = np.array([i for i in range(n) if i not in (3, 11)])
    per_block = oracle.packed_bytes(s, 0, L, 1)
    img = kvsynth.host_bytes(n * per_block, 600, 77, mode=kvsynth.MODE_RAW)
    src = torch.from_numpy(img).to(DEV)
    # scatter in one-block chunks: block i's image is one run
    kvx.kvx_scatter_blocks(cache, 0, L, _bt(bad), n, bs, src)
    with pytest.raises(kvx.KvxError) as e:
        kvx.kvx_check()
    assert e.value.status == kvx.KVX_EBADBLOCK
    for i in good:
        oracle.scatter(s, *mirror, 0, L, ids[i:i + 1], bs,
                       img[i * per_block:(i + 1) * per_block])
    check_cache_equals(cache, mirror, L)
    # a chunk list with one reference past the table: the others still move
    refs = [(c * bpc * per_block, c * bpc, bpc) for c in range(n // bpc)]
    refs[2] = (refs[2][0], n - 1, bpc)
    out = torch.full((n * per_block,), CANARY, dtype=torch.uint8, device=DEV)
    kvx.kvx_gather_chunks(cache, 0, L, _bt(ids), n, kvx.chunk_refs(refs, DEV), len(refs), bpc * bs,
                          out)
    with pytest.raises(kvx.KvxError) as e:
        kvx.kvx_check()
    assert e.value.status == kvx.KVX_EINVAL
    want = np.full(n * per_block, CANARY, np.uint8)
    for c, (o, a, m) in enumerate(refs):
        if c != 2:
            want[o:o + m * per_block] = oracle.gather(s, *mirror, 0, L, ids[a:a + m], m * bs)
    assert first_mismatch(to_host(out), want) is None
