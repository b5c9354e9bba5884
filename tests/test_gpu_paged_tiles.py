"""Paged-attention tiles: several small heads per workgroup (with and without
heads left over), one head, a head cut along its rows, tiles of one, two, four and
twelve vectors a thread, a head that no piece of whole lines divides, and 8-bit
transposes with blocks that are and are not a multiple of 16 tokens; gather and
scatter in image and in destination order, and chunk lists. Everything is
compared whole with the oracle."""
import numpy as np
import pytest

import oracle
from kvtest_util import (cache_and_mirror, check_cache_equals, device_table, first_mismatch,
                         seeded_ids, to_host)

torch = pytest.importorskip("torch")
import paper_2609_11744_amd as kvx  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
PA = oracle.LAYOUT_PAGED_ATTN

SHAPES = [
    # (block, heads, dim, elem): tile
    (16, 8, 128, 1),    # two heads of 128 vectors
    (16, 5, 128, 1),    # the same, one head left over
    (16, 3, 96, 1),     # three heads of 96 (all the slab), two a thread
    (16, 4, 64, 1),     # four heads of 64
    (16, 7, 64, 2),     # two heads of 128, one left over
    (8, 3, 80, 2),      # three heads of 80
    (8, 5, 64, 1),      # five heads of 32 (all the slab)
    (16, 1, 128, 1),    # one head of 128
    (8, 1, 64, 1),      # one head of 32: a 512-byte slab
    (1, 3, 48, 2),      # one token a block
    (16, 2, 256, 2),    # 512 vectors a head: rows cut in halves
    (32, 4, 128, 2),    # the same with 32 tokens
    (32, 2, 96, 2),     # two heads of 384: no even line piece, four a thread
    (64, 2, 128, 2),    # a head of 1,024, four a thread
    (128, 1, 128, 2),   # 2,048, twelve a thread
    (160, 1, 128, 2),   # 2,560, the same
    (64, 3, 128, 1),    # 512 vectors, two a thread
    (32, 3, 128, 1),    # 256 vectors
    (48, 2, 80, 1),     # two heads of 240, two a thread
    (24, 2, 128, 1),    # 8-bit, 24 tokens a block
    (20, 2, 64, 1),     # 8-bit, 20 tokens
    (16, 3, 80, 4),     # 4-byte words: three heads of 320, four a thread
    (8, 2, 256, 4),     # 512 vectors, halves
    (4, 3, 32, 8),      # 8-byte words
]


def _bt(ids):
    return device_table(ids, DEV)


def _setup(shape, L, NB, seed):
    bs, h, d, e = shape
    s = oracle.Shape(L, NB, bs, h, d, e, PA)
    return (s, *cache_and_mirror(s, seed, DEV))


def _gather_and_scatter(shape, L, l0, l1, n, bpc):
    """Both directions compared whole; the scatter's walk."""
    bs = shape[0]
    NB = 2 * n + 5
    s, cache, mirror = _setup(shape, L, NB, 700 + n)
    src, dst_ids = seeded_ids(700 + n, NB, n, n)
    expect = oracle.gather(s, *mirror, l0, l1, src, bpc * bs)
    out = torch.full((expect.size + 4096,), 0xA5, dtype=torch.uint8, device=DEV)
    kvx.kvx_gather_blocks(cache, l0, l1, _bt(src), n, bpc * bs, out)
    kvx.kvx_check()
    got = to_host(out)
    assert first_mismatch(got[:expect.size], expect) is None
    assert (got[expect.size:] == 0xA5).all()
    kvx.kvx_scatter_blocks(cache, l0, l1, _bt(dst_ids), n, bpc * bs, out)
    kvx.kvx_check()
    oracle.scatter(s, *mirror, l0, l1, dst_ids, bpc * bs, expect)
    check_cache_equals(cache, mirror, L)
    return kvx.kvx_copy_walk(cache, l0, l1, n, bpc * bs, False)


@pytest.mark.parametrize("shape", SHAPES, ids=[f"p{i}" for i in range(len(SHAPES))])
@pytest.mark.parametrize("n,bpc", [(11, 4), (1027, 16)])
def test_paged_tiles_bit_exact(shape, n, bpc):
    walk = _gather_and_scatter(shape, *((3, 1, 3) if n < 100 else (2, 0, 2)), n, bpc)
    slab = int(np.prod(shape))
    small = slab <= 2048 or (shape[1] == 1 and slab <= 8192)
    assert walk["ordered"] == (n >= 1024 and not small)


@pytest.mark.parametrize("shape", [(16, 8, 128, 1), (16, 2, 256, 2), (64, 1, 128, 2)],
                         ids=["two heads", "half rows", "four vectors"])
def test_paged_tiles_in_pairs_of_slices_bit_exact(shape):
    """Eight layers, 16 KiB slabs: both directions move slices 2 MiB apart together."""
    walk = _gather_and_scatter(shape, 8, 0, 8, 1027, 16)
    assert walk["ordered"] == 1 and walk["fronts"] == 2 and walk["pair_slices"] == 8


@pytest.mark.parametrize("shape", SHAPES, ids=[f"p{i}" for i in range(len(SHAPES))])
def test_paged_tile_chunk_lists_bit_exact(shape):
    L, bpc = 2, 5
    bs = shape[0]
    sizes = [5, 1, 3, 5, 2, 4]
    n = sum(sizes)
    NB = 2 * n + 3
    s, cache, mirror = _setup(shape, L, NB, 800)
    src, dst_ids = seeded_ids(800, NB, n, n)
    per_block = oracle.packed_bytes(s, 0, L, 1)
    refs, at, off = [], 0, 48
    for m in sizes:
        refs.append((off, at, m))
        at, off = at + m, off + m * per_block + 32
    rd = kvx.chunk_refs(refs, DEV)
    out = torch.full((off,), 0xA5, dtype=torch.uint8, device=DEV)
    kvx.kvx_gather_chunks(cache, 0, L, _bt(src), n, rd, len(refs), bpc * bs, out)
    kvx.kvx_check()
    want = np.full(off, 0xA5, np.uint8)
    images = [oracle.gather(s, *mirror, 0, L, src[a:a + m], m * bs) for _, a, m in refs]
    for (o, _, _), img in zip(refs, images):
        want[o:o + img.size] = img
    assert first_mismatch(to_host(out), want) is None
    kvx.kvx_scatter_chunks(cache, 0, L, _bt(dst_ids), n, rd, len(refs), bpc * bs, out)
    kvx.kvx_check()
    for (_, a, m), img in zip(refs, images):
        oracle.scatter(s, *mirror, 0, L, dst_ids[a:a + m], m * bs, img)
    check_cache_equals(cache, mirror, L)


MIXED = [
    # 8-bit (block, heads, dim): vectors per slab, several slabs per workgroup
    (16, 1, 16),   # 16: a half-wave holds two slabs
    (16, 1, 48),   # 48: a slab ends inside a half-wave
    (16, 1, 80),   # 80
    (16, 1, 112),  # 112
    (16, 3, 16),   # 48, three heads
    (32, 1, 48),   # 96
    (16, 1, 64),   # 64: a slab a wave
    (16, 1, 32),   # 32: a slab a half-wave
]


@pytest.mark.parametrize("shape", MIXED, ids=[f"x{i}" for i in range(len(MIXED))])
def test_keys_and_values_in_one_wave(shape):
    """Slabs of 8-bit words so small that a wave, and half of one, holds keys of one
    slab and values of the next: only the values are turned. In one-block chunks
    every second slab is a value slab; in others the last key slab of a layer meets
    the first value slab."""
    bs, h, d = shape
    L, n = 3, 23
    NB = 2 * n + 3
    s, cache, mirror = _setup((bs, h, d, 1), L, NB, 850)
    src, dst_ids = seeded_ids(850, NB, n, n)
    for bpc in (1, 4):
        expect = oracle.gather(s, *mirror, 0, L, src, bpc * bs)
        out = torch.full((expect.size,), 0xA5, dtype=torch.uint8, device=DEV)
        kvx.kvx_gather_blocks(cache, 0, L, _bt(src), n, bpc * bs, out)
        kvx.kvx_check()
        assert first_mismatch(to_host(out), expect) is None, bpc
        kvx.kvx_scatter_blocks(cache, 0, L, _bt(dst_ids), n, bpc * bs, out)
        kvx.kvx_check()
        oracle.scatter(s, *mirror, 0, L, dst_ids, bpc * bs, expect)
        check_cache_equals(cache, mirror, L)
    per_block = oracle.packed_bytes(s, 0, L, 1)
    refs = [(i * per_block, i, 1) for i in range(n)]  # chunks of two blocks, half full
    out = torch.full((n * per_block,), 0xA5, dtype=torch.uint8, device=DEV)
    kvx.kvx_gather_chunks(cache, 0, L, _bt(src), n, kvx.chunk_refs(refs, DEV), n, 2 * bs, out)
    kvx.kvx_check()
    want = oracle.gather(s, *mirror, 0, L, src, bs)
    assert first_mismatch(to_host(out), want) is None
    kvx.kvx_scatter_chunks(cache, 0, L, _bt(dst_ids), n, kvx.chunk_refs(refs, DEV), n, 2 * bs, out)
    kvx.kvx_check()
    oracle.scatter(s, *mirror, 0, L, dst_ids, bs, want)
    check_cache_equals(cache, mirror, L)
