"""The binding's own count of a call's packed bytes against the library's, over
valid and invalid ranges, sizes beyond 31 bits of pieces and invalid shapes."""
import random

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
