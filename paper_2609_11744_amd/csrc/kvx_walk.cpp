// Walk selection for the gather and scatter kernels (host code): how a call's
// work items are laid out over the chip's XCDs, whether a scatter visits its
// destinations in ascending order, and which slices move together. The launcher
// (kvx_kernels.hip) and kvx_copy_walk share it.
#include <algorithm>
#include <cstdint>

#include "kvx.h"
#include "kvx_internal.h"

namespace kvx {

uint32_t slab_pieces(int layout, uint32_t n16, uint32_t heads) {
  return layout == KVX_LAYOUT_NHD ? (n16 + kPartThreads - 1) / kPartThreads : heads;
}

int copy_layout(int layout, int32_t heads, int32_t block_size) {
  if (block_size == 1 || (layout == KVX_LAYOUT_HND && heads == 1)) return KVX_LAYOUT_NHD;
  return layout;
}

// The tile that keeps most lanes of its workgroups busy, of
//   - `g` whole neighbouring heads, up to 1,024 vectors, one, two or four a
//     thread (a single 8-bit head of 16 tokens x 128 dims would fill half of a
//     workgroup of one);
//   - for a head that large, an even piece of its rows, at least a 128-byte line
//     of the packed side wide, of at most 256 vectors.
// Two and four vectors a thread count a little less, and rows that are not
// whole lines much less unless the tile has all heads, so that its rows meet.
// With neither, gather / scatter, 0.9 to 1.6 GB, means of 5 allocation pairs,
// without -> with: 32-token blocks of 4 x 128 bf16 706 / 748 -> 710 / 736 us and of
// 2 x 96 bf16 548 / 591 -> 530 / 579; 16-token 8-bit blocks of 3 x 96 1048 / 830 ->
// 587 / 625, of 8 x 80 1003 / 643 -> 684 / 636 and of 5 x 80 990 / 735 -> 661 / 685.
TileShape paged_tile(uint32_t block_size, uint32_t heads, uint32_t v16) {
  constexpr uint32_t kLine = 8;  // vectors
  const uint32_t nh = block_size * v16;
  if (heads * nh <= kPartThreads) return {heads, v16};
  TileShape best = {1, v16};
  float score = 0;
  for (uint32_t g = 1; g <= heads && g * nh <= 4 * kPartThreads; ++g) {
    const uint32_t v = g * nh <= kPartThreads ? 1 : g * nh <= 2 * kPartThreads ? 2 : 4;
    const uint32_t tiles = (heads + g - 1) / g;
    float f = (float)(heads * nh) / (float)(tiles * v * kPartThreads);
    if (v > 1) f *= v == 2 ? 0.96f : 0.93f;
    if (g < heads && g * v16 % kLine != 0) f *= 0.5f;
    if (f > score) score = f, best = {g, v16};
  }
  for (uint32_t w = kLine; w < v16; w += kLine)
    if (v16 % w == 0 && block_size * w <= kPartThreads &&
        (float)(block_size * w) / kPartThreads > score)
      score = (float)(block_size * w) / kPartThreads, best = {1, w};
  return best;
}

void copy_parts(const kvx_cache* c, uint32_t n16, uint32_t* parts, uint32_t* shift) {
  *parts = (n16 + kPartThreads - 1) / kPartThreads;
  if (copy_layout(c->layout, c->num_kv_heads, c->block_size) == KVX_LAYOUT_PAGED_ATTN) {
    const uint32_t v16 = (uint32_t)((int64_t)c->head_dim * c->elem_bytes / 16);
    const TileShape t = paged_tile((uint32_t)c->block_size, (uint32_t)c->num_kv_heads, v16);
    *parts = ((uint32_t)c->num_kv_heads + t.heads - 1) / t.heads * (v16 / t.vectors);
  }
  *shift = (*parts & (*parts - 1)) == 0 ? (uint32_t)__builtin_ctz(*parts) : 32u;
}

uint32_t copy_group(uint32_t n16) {
  return n16 <= kGroupMaxVectors ? kPartThreads / n16 : 1;
}

namespace {

// Whether a large scatter of small slabs walks the image in order with no
// XCD ranges (workgroup b moves work item b: the whole chip reads the packed
// image front to back). Compared over 9-16 (cache, packed buffer) allocation
// pairs in one process at the tensor-parallel shard shapes of the 8B cache
// (80k prefix, 16-block chunks, default layout), against the destination-
// ordered walk: 4 KiB slabs 71.6-72.1 % of peak against 68.0-68.3 %, 8 KiB
// 70.8 against 69.3-69.8 %, 16 KiB level (73.7 / 73.6 %, a wider spread), and
// 32 KiB 71.1 against 75.3 % (image order with XCD ranges: 69.3 / 69.1 % at 4
// and 8 KiB). An HND cache with one KV head is the default layout byte for
// byte, and measured the same way (4 KiB slabs: 73.7 against 70.4 %); with
// two heads in 8 KiB it lost 1.8 points (1.4 on the current kernels, over 18
// pairs), so it keeps destination order. The paged-attention layout with one
// head takes the linear walk too, with its heads on 256 threads
// (kvx_kernels.hip): over 18 allocation pairs 73.2 % against 68.3 % for
// destination order on 128 threads, and about 1 point with either change
// alone; with two heads the linear walk lost 0.2 points. Slabs that neither
// divide 4 KiB nor are whole multiples of it straddle the pieces that
// consecutive workgroups of a linear walk write on different XCDs, so these
// walk the image with XCD ranges. 1 GiB, 32 layers, linear / destination order
// / image order with XCD ranges: 2,304 bytes 519 / 429 / 395 us, 2,560 bytes
// 474 / 409 / 393, 3,840 bytes 409 / 387 / 395, 5,120 bytes 483 / 392 / 383,
// 6 KiB 423 / 388 / 386, 7 KiB 398 / 388 / 386; 8 KiB 364 / 384 / 376. Grouped
// ones the same: 1,920 bytes 414 / 407 / 399 us, 1,280 bytes 407 / 412 / 400.
// Slabs of several heads in a reordering layout join them where they are grouped
// (2 KiB, two heads of 64 dims 8-bit, ordered / linear: HND 415 / 387 us, paged
// attention 400 / 370; 1,920 bytes ordered / image order 430 / 418, 543 / 450;
// eight-token blocks of two such heads lost 2 to 5 % in the latter). LDS reserved
// so that six workgroups of a linear walk run on a compute unit, not eight, is not
// taken: over 12 pairs, held / unheld, 4 KiB slabs 456 / 462 us (80 layers, 2,048
// blocks), 354 / 354 (32 layers, 4,096) and 94 / 91 (1,100), 8 KiB 637 / 632 and
// 344 / 340, 2 KiB 215 / 210 and 351 / 343, 1 KiB 176 / 167. Over 36 calls of 1 and
// 2 KiB slabs, 16 to 80 layers, six pairs each, unheld took 0.953 to 1.023 of the time
// held, 0.988 on the mean: where the buffers land decides, not the shape.
bool small_rows(int64_t slab, int layout, int32_t heads) {
  return slab <= 16 * (int64_t)kGroupMaxVectors ||
         (slab <= 8192 && (layout == KVX_LAYOUT_NHD || heads == 1));
}

bool scatter_linear(int64_t n_blocks, int64_t slab, int layout, int32_t heads) {
  return small_rows(slab, layout, heads) && n_blocks >= kOrderedScatterMinBlocks &&
         (4096 % slab == 0 || slab % 4096 == 0);
}

// Whether a scatter of n_blocks in chunks of bpc blocks runs in destination
// order. The rate of one walk over the same ids moves by up to 8 points of
// peak with where the cache and the packed buffer land in physical memory,
// so the walks were compared over 12 placements (4 caches x 3 packed buffers
// allocated in one process, each walk on each pair, alternated; 8B-shaped
// cache, 20,000-block pool, mean % of 8 TB/s). With one-block chunks image
// order averaged 76.8 against 73.6 in destination order at 2,048 blocks (at
// least as fast on 11 of the 12 pairs) and 76.3 against 76.1 at 5,000; with
// 4-block chunks the two were level (73.6 / 73.6), and destination order led
// with 16 and 64 (74.6 against 71.8 and 75.0 against 70.8 at 2,048 blocks,
// 76.9 against 71.9 at 5,000 with 16). A call over one layer keeps image
// order: bucketing its ids and the scratch for them take 10 us, more than the
// order gains there (32 KiB slabs in 16-block chunks, ordered / image order:
// 1,024 blocks 30.9 / 24.7 us, 2,048 55.5 / 51.3, 4,096 102.6 / 96.2, 8,192
// 194.5 / 188.6).
bool scatter_in_destination_order(int64_t n_blocks, int64_t bpc, int64_t slab, int layout,
                                  int32_t heads, int32_t layers) {
  return n_blocks >= kOrderedScatterMinBlocks && bpc > 1 && layers > 1 &&
         !small_rows(slab, layout, heads);
}

// Pairing for the ordered scatter of n_work work items (one launch) over
// n_slices layer|K|V slices: log2 of the distance D in slices between the two
// slices its fronts move together, or 32 for one front per XCD. Two fronts
// pay, as measured, where the paired slabs sit 2 MiB apart in the packed
// chunk (D chunk layers apart) and D <= 4: on the 80k scatter pattern
// (standalone probe, one allocation for the pool, two processes) pairs 2 MiB
// apart beat one front by 2.2-2.3 points with 16-block chunks (D = 4) and by
// 0.9-2.0 with 64-block chunks (D = 1), and lost 0.6-1.1 with 4-block chunks
// (D = 16); pairs at any other distance (32 KiB to 64 MiB) lost 0.5-2 points
// to one front in all but one process. In the library, alternated on three
// machines: the 80k scatter (D = 4) 75.1-75.6 % of peak against 72.7-72.9 %,
// 80.5-83.0 % against 78.9-80.5 % on two faster machines; the 32k scatter with
// 256-token chunks 72.6-72.8 % against 69.5-70.5 %. Why 2 MiB is the
// distance that pays is not established: it depends on how the chip maps
// physical addresses to memory channels, which these kernels do not see.
// log2 of D, the distance in slices at which two slices' runs in a packed
// chunk sit 2 MiB apart, where D is a power of two of at most 2^max_ds and
// the slice count a multiple of 2 D; else 32.
uint32_t pairing_2mib(uint32_t parts_shift, uint32_t n_slices, uint32_t bpc, uint64_t slab,
                      uint32_t max_ds) {
  constexpr uint64_t kPairBytes = 2u << 20;
  if (parts_shift >= 32) return 32;
  const uint64_t run = (uint64_t)bpc * slab;  // one slice's run in a chunk
  if (run == 0 || kPairBytes % run) return 32;
  const uint64_t d = kPairBytes / run;
  if ((d & (d - 1)) || d > (1ull << max_ds) || n_slices % (2 * d)) return 32;
  return (uint32_t)__builtin_ctzll(d);
}

// Farther apart (D = 8, 16) the fronts paid with slabs above 8 KiB, compared
// over 9-12 (cache, packed buffer) allocation pairs in one process: 32 KiB
// slabs in 8-block chunks (D = 8) 77.0 % of peak against 76.0 % for one front
// at 5,000 blocks and 74.6 against 73.8 % at 2,048, in 4-block chunks (D = 16)
// 76.6 against 76.0 % and 74.4 against 73.7 %; 16 KiB slabs in 16-block chunks
// (D = 8) 74.4 against 73.3 %. With 4 and 8 KiB slabs (D = 32, 16) they lost
// 1.3-1.4 points, so smaller slabs keep D <= 4.
uint32_t scatter_pairing(uint64_t n_work, uint32_t parts_shift, uint32_t n_slices, uint32_t bpc,
                         uint64_t slab) {
  if (n_work > kMaxWorkPerLaunch || n_slices % (2 * kXcds)) return 32;
  return pairing_2mib(parts_shift, n_slices, bpc, slab, slab > 8192 ? 4 : 2);
}

// Pairing for the gather: each chunk's slices walked in pairs 2 MiB apart in
// the chunk, D <= 32 slices (the packed-side writes then alternate between two
// runs 2 MiB apart). On the 80k gather pattern (standalone probe, two
// processes each) this measured 0.3-0.8 points above the plain walk with 16-
// and 64-block chunks (D = 4, 1); pairs at other distances (512 KiB to 32 MiB)
// were 0.5-4 points slower. Farther apart in slices, compared over 12 (cache,
// packed buffer) allocation pairs in one process (8B shape, 20,000-block
// pool; the rate of one walk moves by several points with where the
// allocations land): with 4- and 8-block chunks of 32 KiB slabs (D = 16, 8)
// 80.8 / 80.6 % of peak against 79.6 / 79.3 % for the plain walk at 2,048
// blocks, 81.2 / 81.1 against 80.7 / 80.5 at 5,000; at the tensor-parallel
// shard shapes (4 and 8 KiB slabs, 16-block chunks: D = 32, 16) 77.3 / 77.4
// against 75.5 / 75.6 over 16 pairs, faster on every pair.
uint32_t gather_pairing(uint32_t parts_shift, uint32_t n_slices, uint32_t bpc, uint64_t slab) {
  return pairing_2mib(parts_shift, n_slices, bpc, slab, 5);
}

}  // namespace

kvx_status choose_walk(bool to_packed, const kvx_cache* cache, const Geometry& g, Walk* w) {
  *w = Walk();
  if (g.n_units == 0) return KVX_OK;
  const uint32_t n16 = (uint32_t)(g.slab / 16), heads = (uint32_t)cache->num_kv_heads;
  w->pieces = slab_pieces(cache->layout, n16, heads);
  if ((uint64_t)g.n_units * w->pieces > 0x7FFFFFFF) return KVX_EINTERNAL;
  copy_parts(cache, n16, &w->parts, &w->parts_shift);
  const uint64_t n_work = (uint64_t)g.n_units * w->parts;
  // No pairs where slabs are grouped: they need none (gathers of 2 KiB slabs in
  // 64-block chunks, D = 16, 32 and 80 layers: 407 and 506 us paired with a slab per
  // workgroup, 356 and 440 grouped and unpaired).
  const uint32_t pair_parts = copy_group(n16) > 1 ? 32u : w->parts_shift;
  const uint32_t n_slices = (uint32_t)(2 * g.lr);
  if (to_packed) {
    w->gather_pair_shift = gather_pairing(pair_parts, n_slices, (uint32_t)g.bpc,
                                          (uint64_t)g.slab);
    return KVX_OK;
  }
  w->linear = scatter_linear(g.n_blocks, g.slab, cache->layout, cache->num_kv_heads);
  w->ordered = scatter_in_destination_order(g.n_blocks, g.bpc, g.slab, cache->layout,
                                            cache->num_kv_heads, g.lr);
  // One launch, counted in pieces where a slab has more of them than workgroups (HND):
  // pairs were measured only that far.
  if (w->ordered)
    w->pair_shift = scatter_pairing(std::max(n_work, (uint64_t)g.n_units * w->pieces), pair_parts,
                                    n_slices, (uint32_t)g.bpc, (uint64_t)g.slab);
  return KVX_OK;
}

}  // namespace kvx

// ---- the walk a copy takes -----------------------------------------------------

extern "C" kvx_status kvx_copy_walk(const kvx_cache* cache, int32_t l0, int32_t l1,
                                    int32_t n_blocks, int32_t chunk_tokens, int32_t to_packed,
                                    kvx_walk* out) {
  if (!out || (to_packed != 0 && to_packed != 1)) return KVX_EINVAL;
  try {
    *out = kvx_walk{};
    kvx::Geometry g;
    kvx_status st = kvx::validate(cache, l0, l1, n_blocks, chunk_tokens, false, &g);
    if (st != KVX_OK) return st;
    kvx::Walk w;
    st = kvx::choose_walk(to_packed == 1, cache, g, &w);
    if (st != KVX_OK || w.pieces == 0) return st;
    const uint32_t ps = to_packed ? w.gather_pair_shift : w.pair_shift;
    out->work_items = g.n_units * w.pieces;
    out->parts = (int32_t)w.pieces;
    out->ordered = w.ordered ? 1 : 0;
    out->linear = w.linear ? 1 : 0;
    out->pair_slices = ps < 32 ? (int32_t)(1u << ps) : 0;
    out->fronts = w.ordered && w.pair_shift < 32 ? 2 : 1;
    return KVX_OK;
  } catch (...) {
    return KVX_EINTERNAL;
  }
}
