"""The binding's own count of a call's packed bytes against the library's, over
valid and invalid ranges, sizes beyond 31 bits of pieces and invalid shapes, in
every integer type that the library call takes; and the buffer check that it feeds."""
import ctypes
import random

import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_2609_11744_amd as kvx  # noqa: E402

SHAPES = [
    # (layers, block, heads, dim, layout)
    (5, 16, 2, 64, kvx.KVX_LAYOUT_NHD),
    (3, 64, 8, 128, kvx.KVX_LAYOUT_NHD),
    (140, 1, 1, 8, kvx.KVX_LAYOUT_NHD),      # more layers than a call may cover
    (2, 1, 1, 2, kvx.KVX_LAYOUT_NHD),        # 4-byte slabs: invalid
    (2, 16, 3, 64, kvx.KVX_LAYOUT_HND),
    (2, 64, 8, 64, kvx.KVX_LAYOUT_HND),      # above the largest slab: invalid
    (2, 16, 12, 128, kvx.KVX_LAYOUT_PAGED_ATTN),
]


@pytest.mark.parametrize("shape", SHAPES, ids=[f"i{i}" for i in range(len(SHAPES))])
def test_image_bytes_is_the_librarys(shape):
    L, bs, h, d, layout = shape
    c = kvx.PagedKVCache.allocate(L, 3, bs, h, d, torch.bfloat16, "cpu", layout)
    r = random.Random(L)
    for _ in range(3000):
        l0, l1 = r.randint(-1, L + 2), r.randint(-1, L + 2)
        n = r.choice([-1, 0, 1, 7, 5000, 10 ** 6, 2 ** 24, 2 ** 31 - 1])
        assert kvx._image_bytes(c, l0, l1, n) == max(kvx.kvx_packed_bytes(c, l0, l1, n), 0), \
            (l0, l1, n)


SCALARS = [np.int16, np.uint16, np.int32, np.uint32, np.int64, np.array,
           lambda n: torch.tensor(n, dtype=torch.int16), lambda n: torch.tensor(n, dtype=torch.int32),
           torch.tensor, ctypes.c_int32]


@pytest.mark.parametrize("scalar", SCALARS, ids=[f"t{i}" for i in range(len(SCALARS))])
def test_a_short_buffer_is_refused_whatever_the_counts_type(scalar):
    """64 KiB a layer and block over 32 layers: in 16 or 32 bits 2,048 blocks wrap
    to 0 bytes, 1,024 to a negative count and 5,000 to less than they take. No call
    here reaches the library's copy, which would want a GPU."""
    L = 32
    c = kvx.PagedKVCache.allocate(L, 1, 16, 8, 128, torch.bfloat16, "cpu")
    table = torch.zeros(5000, dtype=torch.int32)
    short = torch.empty(128, dtype=torch.uint8)
    for n in (2048, 1024, 5000, 7):
        need = kvx.kvx_packed_bytes(c, 0, L, n)
        assert need == n * L * 65536
        assert kvx._image_bytes(c, scalar(0), scalar(L), scalar(n)) == need
        assert kvx._image_bytes(c, 0, L, scalar(n)) == need
        if scalar is ctypes.c_int32:  # no count that a table could be compared with
            continue
        for call in (kvx.kvx_gather_blocks, kvx.kvx_scatter_blocks,
                     kvx.kvx_scatter_blocks_noalloc):
            with pytest.raises(ValueError, match="packed buffer holds 128 bytes"):
                call(c, 0, L, table, scalar(n), 256, short)


def test_reversed_ranges_of_unsigned_counts_are_the_librarys():
    c = kvx.PagedKVCache.allocate(5, 3, 16, 2, 64, torch.bfloat16, "cpu")
    for t in (np.uint8, np.uint16, np.uint32):
        assert kvx._image_bytes(c, t(3), t(1), t(2)) == 0 > kvx.kvx_packed_bytes(c, t(3), t(1), t(2))


@pytest.mark.parametrize("count", [2.0, np.float32(2), "2", None], ids=["f", "f32", "s", "none"])
def test_what_the_library_call_refuses_is_refused(count):
    c = kvx.PagedKVCache.allocate(5, 3, 16, 2, 64, torch.bfloat16, "cpu")
    with pytest.raises(ctypes.ArgumentError):
        kvx._image_bytes(c, 0, 5, count)
