"""Chunk lists most of whose chunks are short, copied without padding: every
layout and grouping, more chunks than one listing workgroup takes, chunks whose
slices lie 2 MiB apart (the paired gather), chunks that share table entries (more
blocks than the table has: workgroups go round again), bad references and bad
block ids, the same list while a stream is capturing (the padded copy), list calls
that return before their stream has done anything, on more streams than there are
slots for their scratch, from several threads, and beside another stream's capture.
Everything is compared whole with the oracle."""
import threading

import numpy as np
import pytest

import oracle
from kvtest_util import (cache_and_mirror, check_cache_equals, device_table, first_mismatch,
                         seeded_ids, to_host)

torch = pytest.importorskip("torch")
import paper_2609_11744_amd as kvx  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
NHD, HND, PA = oracle.LAYOUT_NHD, oracle.LAYOUT_HND, oracle.LAYOUT_PAGED_ATTN

CASES = [
    # (layout, layers, block, heads, dim, elem, blocks per chunk, chunk lengths, slabs' workgroups)
    (NHD, 16, 16, 2, 128, 2, 64, [1, 64, 3, 32, 2, 64, 5, 1] + [2] * 40, 2),  # 8 KiB: D = 4, 8
    (NHD, 32, 16, 1, 64, 2, 64, [3, 1, 2] * 50, 1 / 2),                       # 2 KiB, 150 chunks
    (NHD, 32, 8, 1, 64, 1, 200, [7, 1, 4] * 90, 1 / 8),                       # 512 bytes
    (NHD, 17, 5, 3, 56, 2, 64, [1, 2, 64, 9] * 12, 1 / 2),                    # 1,680 bytes
    (NHD, 17, 16, 3, 80, 2, 64, [2, 5, 1] * 16, 2),                           # 7,680 bytes
    (HND, 16, 16, 2, 128, 2, 64, [1, 33, 2] * 5, 2),
    (HND, 32, 8, 2, 64, 1, 128, [5, 1, 17] * 23, 1 / 4),                      # 1 KiB
    (PA, 8, 16, 8, 128, 1, 64, [1, 4, 2] * 19, 4),                            # two heads a tile
    (PA, 16, 16, 1, 128, 2, 64, [1, 32, 3] * 8, 1),                           # one head a tile
    (PA, 32, 8, 1, 64, 2, 200, [3, 1, 11] * 35, 1 / 4),                       # 1 KiB
]


def _listed(case, table_len, n_chunks):
    """The list is copied without padding: enough work, and enough padding."""
    work = table_len * 2 * case[1] * case[8]
    padded = n_chunks * case[6] * 2 * case[1] * case[8]
    return work >= 1 << 13 and padded - work >= 1 << 15


def _bt(ids):
    return device_table(ids, DEV)


def _setup(case, NB, seed):
    layout, L, bs, h, d, e = case[:6]
    s = oracle.Shape(L, NB, bs, h, d, e, layout)
    return (s, *cache_and_mirror(s, seed, DEV))


def _refs(lengths, per_block, gap=16):
    refs, at, off = [], 0, 64
    for m in lengths:
        refs.append((off, at, m))
        at, off = at + m, off + m * per_block + gap
    return refs, at, off


def _want(s, mirror, L, ids, refs, size, bs):
    want = np.full(size, 0xA5, np.uint8)
    for o, a, m in refs:
        img = oracle.gather(s, *mirror, 0, L, ids[a:a + m], m * bs)
        want[o:o + img.size] = img
    return want


@pytest.mark.parametrize("case", CASES, ids=[f"r{i}" for i in range(len(CASES))])
def test_ragged_lists_bit_exact(case):
    _, L, bs, _, _, _, bpc, lengths, _ = case
    n = sum(lengths)
    assert _listed(case, n, len(lengths))
    s, cache, mirror = _setup(case, 2 * n + 3, 900)
    per_block = oracle.packed_bytes(s, 0, L, 1)
    refs, table_len, size = _refs(lengths, per_block)
    src, dst_ids = seeded_ids(900, 2 * n + 3, n, n)
    rd = kvx.chunk_refs(refs, DEV)
    out = torch.full((size,), 0xA5, dtype=torch.uint8, device=DEV)
    kvx.kvx_gather_chunks(cache, 0, L, _bt(src), table_len, rd, len(refs), bpc * bs, out)
    kvx.kvx_check()
    want = _want(s, mirror, L, src, refs, size, bs)
    assert first_mismatch(to_host(out), want) is None
    kvx.kvx_scatter_chunks(cache, 0, L, _bt(dst_ids), table_len, rd, len(refs), bpc * bs, out)
    kvx.kvx_check()
    for o, a, m in refs:
        oracle.scatter(s, *mirror, 0, L, dst_ids[a:a + m], m * bs, want[o:o + m * per_block])
    check_cache_equals(cache, mirror, L)


@pytest.mark.parametrize("case", [CASES[0], CASES[1], CASES[2], CASES[7], CASES[9]],
                         ids=["parts", "wave", "lane", "tile", "paged"])
def test_ragged_lists_sharing_entries_bad_refs_and_ids(case):
    _, L, bs, _, _, _, bpc, _, per_slab = case
    n = int(8192 / (2 * L * per_slab)) + 3
    NB = n + 9
    s, cache, mirror = _setup(case, NB, 910)
    per_block = oracle.packed_bytes(s, 0, L, 1)
    (ids,) = seeded_ids(910, NB, n)
    rng = np.random.default_rng(7)
    refs, off = [], 0
    for c in range(max(70, n // 2)):  # more blocks than the table has
        m = int(rng.integers(1, 8))
        refs.append((off, int(rng.integers(0, n - m + 1)), m))
        off += m * per_block
    assert _listed(case, n, len(refs)) and sum(r[2] for r in refs) > 1.2 * n
    bad = {5: (refs[5][0] + 8, refs[5][1], refs[5][2]), 64: (refs[64][0], n - 1, 4)}
    given = [bad.get(c, r) for c, r in enumerate(refs)]
    out = torch.full((off,), 0xA5, dtype=torch.uint8, device=DEV)
    kvx.kvx_gather_chunks(cache, 0, L, _bt(ids), n, kvx.chunk_refs(given, DEV), len(refs),
                          bpc * bs, out)
    with pytest.raises(kvx.KvxError) as e:
        kvx.kvx_check()
    assert e.value.status == kvx.KVX_EINVAL
    good = [r for c, r in enumerate(refs) if c not in bad]
    want = _want(s, mirror, L, ids, good, off, bs)
    assert first_mismatch(to_host(out), want) is None
    # a bad block id: its slabs alone are left as they are
    ids2 = ids.copy()
    ids2[4] = NB
    single, _, size = _refs([1] * n, per_block)
    out = torch.full((size,), 0xA5, dtype=torch.uint8, device=DEV)
    kvx.kvx_gather_chunks(cache, 0, L, _bt(ids2), n, kvx.chunk_refs(single, DEV), n, bpc * bs, out)
    with pytest.raises(kvx.KvxError) as e:
        kvx.kvx_check()
    assert e.value.status == kvx.KVX_EBADBLOCK
    want = _want(s, mirror, L, ids, [r for r in single if r[1] != 4], size, bs)
    assert first_mismatch(to_host(out), want) is None


def test_shared_entries_of_tiles_larger_than_the_second_launch():
    """2,560-vector tiles of a list with more blocks than its table: the second
    launch's 2,048 workgroups go round by their own number, not by the tile's
    vectors (which left 512 of every 2,560 slabs where they were)."""
    case = (PA, 64, 160, 1, 128, 2, 8, None, 1)
    _, L, bs, _, _, _, bpc, _, _ = case
    n, NB = 64, 70
    s, cache, mirror = _setup(case, NB, 930)
    per_block = oracle.packed_bytes(s, 0, L, 1)
    (ids,) = seeded_ids(930, NB, n)
    rng = np.random.default_rng(9)
    refs, off = [], 0
    for c in range(45):
        m = 1 + c % 4
        refs.append((off, int(rng.integers(0, n - m + 1)), m))
        off += m * per_block
    assert _listed(case, n, len(refs))
    # at least one whole round of the second launch, and more
    assert 2 * L * (sum(r[2] for r in refs) - n) > 2560
    out = torch.full((off,), 0xA5, dtype=torch.uint8, device=DEV)
    kvx.kvx_gather_chunks(cache, 0, L, _bt(ids), n, kvx.chunk_refs(refs, DEV), len(refs), bpc * bs,
                          out)
    kvx.kvx_check()
    want = _want(s, mirror, L, ids, refs, off, bs)
    assert first_mismatch(to_host(out), want) is None


@pytest.mark.parametrize("pad", [False, True], ids=["listed", "padded"])
def test_references_at_the_end_of_64_bits_are_refused(pad):
    """An offset to which the chunk's bytes cannot be added without wrapping."""
    case = CASES[0]
    _, L, bs, _, _, _, bpc, lengths, _ = case
    lengths = [4] * 4 if pad else lengths
    n = sum(lengths)
    assert _listed(case, n, len(lengths)) != pad
    s, cache, mirror = _setup(case, n, 970)
    per_block = oracle.packed_bytes(s, 0, L, 1)
    refs, table_len, size = _refs(lengths, per_block)
    (ids,) = seeded_ids(970, n, n)
    top = 2 ** 63 - 16
    given = [(top - 64 * per_block * (i == 3), a, m) if i in (1, 3) else (o, a, m)
             for i, (o, a, m) in enumerate(refs)]
    out = torch.full((size,), 0xA5, dtype=torch.uint8, device=DEV)
    kvx.kvx_gather_chunks(cache, 0, L, _bt(ids), table_len, kvx.chunk_refs(given, DEV), len(refs),
                          bpc * bs, out)
    with pytest.raises(kvx.KvxError) as e:
        kvx.kvx_check()
    assert e.value.status == kvx.KVX_EINVAL
    good = [r for i, r in enumerate(refs) if i not in (1, 3)]
    assert first_mismatch(to_host(out), _want(s, mirror, L, ids, good, size, bs)) is None


def test_ragged_list_under_capture_replays_bit_exact():
    case = CASES[0]
    _, L, bs, _, _, _, bpc, lengths, _ = case
    n = sum(lengths)
    s, cache, mirror = _setup(case, 2 * n + 3, 920)
    per_block = oracle.packed_bytes(s, 0, L, 1)
    refs, table_len, size = _refs(lengths, per_block)
    (src,) = seeded_ids(920, 2 * n + 3, n)
    rd, bt = kvx.chunk_refs(refs, DEV), _bt(src)
    out = torch.full((size,), 0xA5, dtype=torch.uint8, device=DEV)
    kvx.kvx_gather_chunks(cache, 0, L, bt, table_len, rd, len(refs), bpc * bs, out)
    kvx.kvx_check()
    want = _want(s, mirror, L, src, refs, size, bs)
    assert first_mismatch(to_host(out), want) is None
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        kvx.kvx_gather_chunks(cache, 0, L, bt, table_len, rd, len(refs), bpc * bs, out)
    for rep in range(3):
        out.fill_(0xA5)
        torch.cuda.synchronize()
        g.replay()
        kvx.kvx_check()
        assert first_mismatch(to_host(out), want) is None, f"replay {rep}"


def _streams_setup(n_streams, seed):
    """One cache, and per stream a list of its own, its output and what it must hold."""
    case = CASES[0]
    _, L, bs, _, _, _, bpc, lengths, _ = case
    NB = 2 * sum(lengths) + 3
    s, cache, mirror = _setup(case, NB, seed)
    per_block = oracle.packed_bytes(s, 0, L, 1)
    jobs = []
    for k in range(n_streams):
        some = lengths[k:] + lengths[:k]
        assert _listed(case, sum(some), len(some))
        refs, table_len, size = _refs(some, per_block, gap=16 * k)
        (ids,) = seeded_ids(seed + k, NB, table_len)
        args = (cache, 0, L, _bt(ids), table_len, kvx.chunk_refs(refs, DEV), len(refs), bpc * bs)
        out = torch.full((size,), 0xA5, dtype=torch.uint8, device=DEV)
        jobs.append((args, out, _want(s, mirror, L, ids, refs, size, bs)))
    torch.cuda.synchronize()
    return jobs


def test_ragged_lists_do_not_wait_on_the_host():
    """List calls behind a busy stream return while it is still busy, each of them
    (stream-ordered scratch made the second wait for the first)."""
    ((args, out, want),) = _streams_setup(1, 940)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        kvx.kvx_gather_chunks(*args, out)  # whatever a first call sets up
    torch.cuda.synchronize()
    out.fill_(0xA5)
    torch.cuda.synchronize()
    slept = torch.cuda.Event()
    with torch.cuda.stream(st):
        torch.cuda._sleep(500_000_000)  # some 0.2 s
        slept.record()
        for _ in range(4):
            kvx.kvx_gather_chunks(*args, out)
    assert not slept.query()
    torch.cuda.synchronize()
    kvx.kvx_check(st)
    assert first_mismatch(to_host(out), want) is None


def test_ragged_lists_on_many_streams_and_threads():
    """Seven streams, more than have scratch of their own, called in turn and then
    each by a thread of its own."""
    jobs = _streams_setup(7, 950)
    streams = [torch.cuda.Stream() for _ in jobs]

    def run(k, times):
        args, out, _ = jobs[k]
        for _ in range(times):
            kvx.kvx_gather_chunks(*args, out, stream=streams[k])

    def same():
        torch.cuda.synchronize()
        for k, (_, out, want) in enumerate(jobs):
            kvx.kvx_check(streams[k])
            assert first_mismatch(to_host(out), want) is None, f"stream {k}"
            out.fill_(0xA5)
        torch.cuda.synchronize()

    for _ in range(5):
        for k in range(len(jobs)):
            run(k, 1)
    same()
    threads = [threading.Thread(target=run, args=(k, 10)) for k in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    same()


def test_ragged_list_beside_another_streams_capture():
    (args, out, want), (args2, out2, want2) = _streams_setup(2, 960)
    side, own = torch.cuda.Stream(), torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        kvx.kvx_gather_chunks(*args, out)
        kvx.kvx_gather_chunks(*args2, out2, stream=own)  # runs at once
    torch.cuda.synchronize()
    kvx.kvx_check(own)
    assert first_mismatch(to_host(out2), want2) is None
    for rep in range(3):
        out.fill_(0xA5)
        torch.cuda.synchronize()
        g.replay()
        kvx.kvx_check()
        kvx.kvx_gather_chunks(*args2, out2)
        assert first_mismatch(to_host(out), want) is None, f"replay {rep}"
