"""The scatter walks of one-layer calls and of slabs that are not 4 KiB pieces
(kvx_copy_walk, host only): which run in destination order, which on the linear
walk and which in image order with XCD ranges, on both sides of each line."""
import pytest

pytest.importorskip("torch")
import paper_2609_11744_amd as kvx  # noqa: E402

NHD, HND, PA = kvx.KVX_LAYOUT_NHD, kvx.KVX_LAYOUT_HND, kvx.KVX_LAYOUT_PAGED_ATTN
RULES = [
    # (layers, block, heads, dim, elem, layout, n_blocks, blocks per chunk) -> (ordered, linear)
    ((1, 16, 8, 128, 2, NHD, 8192, 16), (0, 0)),   # one layer: image order
    ((2, 16, 8, 128, 2, NHD, 1024, 16), (1, 0)),   # two: destination order
    ((1, 16, 1, 128, 2, NHD, 2048, 16), (0, 1)),   # one layer of 4 KiB slabs: linear
    ((8, 16, 5, 64, 1, NHD, 2048, 16), (0, 0)),    # 5 KiB
    ((8, 16, 1, 240, 1, NHD, 2048, 16), (0, 0)),   # 3,840 bytes
    ((8, 16, 4, 128, 1, NHD, 2048, 16), (0, 1)),   # 8 KiB
    ((8, 16, 9, 64, 1, NHD, 2048, 16), (1, 0)),    # 9 KiB
    ((8, 16, 1, 64, 1, NHD, 2048, 16), (0, 1)),    # 1 KiB, grouped
    ((8, 16, 1, 80, 1, NHD, 2048, 16), (0, 0)),    # 1,280 bytes, grouped
    ((8, 16, 2, 64, 1, HND, 2048, 16), (0, 1)),    # 2 KiB of two heads, grouped
    ((8, 16, 2, 64, 1, PA, 2048, 16), (0, 1)),
    ((8, 16, 2, 80, 1, HND, 2048, 16), (1, 0)),    # 2,560 bytes of two heads
    ((8, 16, 1, 64, 1, NHD, 1023, 16), (0, 0)),    # below 1,024 blocks
]


@pytest.mark.parametrize("case,want", RULES, ids=[f"r{i}" for i in range(len(RULES))])
def test_scatter_walk(case, want):
    L, bs, h, d, e, layout, n, bpc = case
    c = kvx.shape_only_cache(L, n + 1, bs, h, d, e, layout)
    w = kvx.kvx_copy_walk(c, 0, L, n, bpc * bs, False)
    assert (w["ordered"], w["linear"]) == want
    assert kvx.kvx_copy_walk(c, 0, L, n, bpc * bs, True)["ordered"] == 0
