// HIP kernels for gfx950: paged-KV gather (paged slabs -> packed image) and
// scatter (packed image -> paged slabs).
//
// The work is pure data movement, bound by HBM bandwidth, so the kernels use
// no MFMA. With the default cache layout every slab is contiguous and in the
// same order on both sides, so nothing is transposed and no LDS is used; of the
// other cache layouts only paged attention goes through LDS (see move_tile).
// A unit is a slab (layer, K|V, block) of `slab` bytes. With the default
// layout one workgroup moves one part of a unit: up to 256 threads, one 16-byte
// vector each, so a part is 4 KiB (a 32 KiB slab is 8 parts; the last part of
// a slab may be short, and slabs a little over 4 or 8 KiB are cut evenly:
// piece_vectors). On this chip a copy moves measurably more bytes per
// second with one load and one store per thread in many short workgroups than
// with several vectors per thread in fewer, longer ones (contiguous 4 GiB:
// 83 % of peak against 77.5 % at 1024 threads x 2 vectors; the 80k gather
// pattern 76.7 % against 73.6 %); persistent grids that loop over units
// measured lower still. HND moves the same pieces, paged attention tiles of about
// that size; slabs of at most 2 KiB share a workgroup (copy_unit_groups_kernel).
//   * the unit's decode (chunk, layer, K|V, block, part) and its block-table
//     read depend on blockIdx only, so they run on the scalar unit once per
//     workgroup;
//   * the slab moves as 16-byte vectors, consecutive lanes on consecutive
//     addresses, so every wave instruction reads or writes 1 KiB contiguous;
//   * both streams are touched once, so loads are non-temporal and stores
//     stream to memory at device scope (kvx_store.h);
//   * workgroups are dispatched round-robin over the 8 XCDs, so workgroup b
//     is mapped to a (unit, part) such that each XCD walks one contiguous
//     range of them. The packed side of an XCD's work is then one sequential
//     stream, which HBM serves measurably better than 8 interleaved ones (the
//     write side of a copy is what bounds it).
// The packed-side address of unit u is u * slab (see Geometry), so only the
// paged side goes through the block table.
//
// Large scatters write to caller-chosen (typically random) blocks. HBM takes
// writes faster when each XCD's write stream ascends through memory, so a
// large scatter first buckets the destination ids (order_kernel, into
// stream-ordered scratch) and then visits units layer by layer in ascending
// destination order; the packed side is then read out of order, which costs
// less than unordered writes. The exceptions measured faster in image order:
// a chunk of one block (each chunk is then one sequential read, and the
// writes go to one destination block of every layer in turn;
// scatter_in_destination_order in kvx_walk.cpp), a call over one layer, and
// slabs of at most 8 KiB, most of them walked with no XCD ranges so that the
// whole chip reads the packed image front to back (scatter_linear).
//
// Pairing at 2 MiB. Where a layer|K|V slice's run in a packed chunk (blocks
// per chunk x slab) times a power of two D is 2 MiB, both directions can move
// two slices D apart together: the gather walks each chunk's slices in such
// pairs (its packed-side writes alternate between two runs 2 MiB apart; D up
// to 32), and the ordered scatter walks each XCD's range as two fronts that
// move the same destination block of two such slices (D up to 16 for slabs
// above 8 KiB, else 4). Both
// measured faster than the plain walks on this chip, and pairs at other
// distances slower (scatter_pairing, gather_pairing in kvx_walk.cpp).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "kvx_internal.h"
#include "kvx_store.h"

namespace kvx {
namespace {

using kvx_dev::store_stream;
using kvx_dev::stream_dst;
using kvx_dev::v4u;

constexpr int kErrBadBlock = 1;
constexpr int kErrBadChunk = 2;
constexpr int kErrorWords = 1024;  // word 0: the null stream, and streams beyond the table

// One entry of a scatter's destination order: a block-table index and the
// block id found there (read once by the ordering kernel).
struct OrderEntry {
  uint32_t index;
  int32_t id;
};

// Device pointers of the call's layers, in image order: p[2 * (l - l0) + kv].
// Passed by value as a kernel argument (2 KiB for KVX_MAX_LAYERS = 128).
struct LayerPtrs {
  char* p[2 * KVX_MAX_LAYERS];
};

// Division by a divisor known only at run time, as a multiply: for d >= 2,
// m = ceil(2^32 / d) and n / d = umulhi(n, m) whenever n * d < 2^32 (the
// rounding error of m, below d, then moves n * m / 2^32 by less than 1/d);
// m = 0 stands for d = 1. A numerator here is a vector or element index inside a
// slab of a reordering layout (of at most 48 KiB) or of at most kGroupMaxVectors
// vectors, or a thread of a workgroup, and a divisor a dimension of that slab: both
// are below 2^16. Slabs of the default layout can be larger; their fields that do
// not keep to this (v16, outer, n16) are set but not divided by.
struct FastDiv {
  uint32_t d;
  uint32_t m;
};

__device__ __forceinline__ uint32_t fdiv(uint32_t n, FastDiv f) {
  return f.m ? __umulhi(n, f.m) : n;
}

// Shape of one head's part of a slab, for the reordering layouts.
struct SlabGeom {
  FastDiv bs;      // tokens per block
  FastDiv v16;     // 16-byte vectors per (token, head) row: head_dim * elem_bytes / 16
  uint32_t nh;     // vectors of one head: bs * v16
  uint32_t prow;   // packed row stride in vectors: heads * v16
  // Paged attention: a workgroup moves a tile of `gh` whole heads, or of `dw` of
  // v16 vectors of every token's row of one head (paged_tile).
  uint32_t heads;
  uint32_t gh;
  uint32_t dw;
  FastDiv dpieces;   // v16 / dw
  FastDiv row;       // gh * dw: vectors of a token in the tile
  FastDiv np;        // bs * dw: vectors of a head in the tile
  FastDiv dwd;       // dw
  // HND: destination vector w of a slab is (w / outer, rest / v16, rest % v16)
  // = (a, b, dv) and comes from source vector a * v16 + b * src_step + dv
  // (gather: a token, b head; scatter: a head, b token).
  FastDiv outer;
  uint32_t src_step;
  FastDiv n16;       // vectors per slab (used where slabs are grouped)
  uint32_t piece;    // default layout and HND: vectors per workgroup (piece_vectors)

  FastDiv pad;       // scatter: LDS pad period (see lds_slot)
  uint32_t v_pairs;  // paged-attention V of 2-byte words gathered as row pairs (v_pairs_gather)
  uint32_t v_bytes;  // paged-attention V of 1-byte words by transpose reads (v_bytes)
  FastDiv bs16;      // bs / 16, where v_bytes
  uint32_t swz;      // gather: LDS swizzle shift (see lds_slot)
  uint32_t image;    // vectors of a tile's LDS image: whole swizzle groups of 16, or with pads
};

// Division of any 32-bit numerator by a divisor fixed for the launch, as a
// multiply (Granlund and Montgomery, "Division by invariant integers using
// multiplication", 1994): with l = ceil(log2 d), m = floor(2^32 (2^l - d) / d)
// + 1 and t = umulhi(n, m), n / d = (t + ((n - t) >> 1)) >> (l - 1) for d >= 2;
// m = 0 stands for d = 1. The workgroup index decode divides unit indexes (up
// to 2^31) by slab and chunk counts, so the narrower FastDiv does not apply.
struct DivU32 {
  uint32_t d;
  uint32_t m;
  uint32_t s;
};

__device__ __forceinline__ uint32_t divu(uint32_t n, DivU32 f) {
  if (f.m == 0) return n;
  const uint32_t t = __umulhi(n, f.m);
  return (t + ((n - t) >> 1)) >> f.s;
}

struct UnitGeom {
  uint32_t units_per_chunk;  // (l1 - l0) * 2 * bpc
  uint32_t bpc;
  uint32_t n_blocks;
  uint32_t num_blocks;       // pool size
  uint32_t n_units;
  uint32_t n16;              // 16-byte vectors per slab
  uint32_t group;            // slabs per workgroup (copy_unit_groups_kernel; else 1)
  uint32_t parts;            // workgroups per slab (parts_shift: log2 of a power of two, else 32)
  uint32_t parts_shift;
  // Ordered scatter walked as two fronts per XCD (xcd_two_fronts) whose
  // slices are paired D = 2^pair_shift apart (paired_slice); pair_shift = 32
  // for one front per XCD. Gather: each chunk's slices walked in pairs
  // 2^gather_pair_shift apart (see the unit decode), or 32 for the plain walk.
  uint32_t pair_shift;
  uint32_t gather_pair_shift;
  uint32_t half_slices;      // slices per half of an XCD's range
  uint32_t linear_walk;      // 1: workgroup b moves work item b (no XCD ranges)
  DivU32 xcd_slices_div;     // by slices per XCD range
  DivU32 parts_div;
  DivU32 upc_div;            // by units_per_chunk
  DivU32 bpc_div;            // by bpc
  DivU32 last_div;           // by the last chunk's block count
  DivU32 nb_div;             // by n_blocks
  uint64_t slab;
  SlabGeom sg;
};

// Sticky error words, a table per device: each stream that launches copies
// gets a word of its own (stream_error_word), so that a check of one stream
// neither reports nor clears another stream's error. Host code reaches the
// table only through the address that hipGetSymbolAddress returns.
__device__ int g_error_words[kErrorWords];

// Workgroup b of a launch over n units -> unit index. XCD x = b % kXcds runs
// the workgroups b = x, x + kXcds, ...; they get the contiguous range
// [x*q + min(x, r), ...) of q or q + 1 units (q = n / kXcds, r = n % kXcds).
// A bijection on [0, n) for every n.
__device__ __forceinline__ uint32_t xcd_contiguous(uint32_t b, uint32_t n) {
  const uint32_t q = n / kXcds, r = n % kXcds, x = b % kXcds, k = b / kXcds;
  return x * q + (x < r ? x : r) + k;
}

// The same ranges for the destination-ordered scatter, walked as two fronts:
// XCD x's range is cut into halves (the first a whole number of slabs,
// `parts` work items each, parts a power of two, 2^shift) and its workgroups
// alternate between them, one work item at a time (items past twice the
// first half follow in order). A bijection on [0, n). The launcher uses it
// only where each XCD's range is a whole, even number of layer|K|V slices,
// so that the two fronts move the same destination block of two slices
// together (its writes in two cache tensors, its reads from one packed
// chunk), and paired_slice chooses which two (scatter_pairing, kvx_walk.cpp).
__device__ __forceinline__ uint32_t xcd_two_fronts(uint32_t b, uint32_t n, uint32_t shift) {
  const uint32_t q = n / kXcds, r = n % kXcds, x = b % kXcds, k = b / kXcds;
  const uint32_t len = q + (x < r ? 1u : 0u), start = x * q + (x < r ? x : r);
  const uint32_t half = ((len >> 1) >> shift) << shift;
  if (k >= 2 * half) return start + k;
  const uint32_t pair = k >> (shift + 1), i = k & ((2u << shift) - 1);
  return start + (i & 1) * half + (pair << shift) + (i >> 1);
}

// The layer|K|V slice moved at slice r of the ordered walk (XCD x's range is
// walk slices [x S, (x + 1) S), halves of H = S / 2): slice t of the first
// half of XCD x's range and slice t of its second half are pair j = H x + t,
// which moves slices a_j and a_j + D (a_j: the j-th slice whose index has bit
// log2 D clear, D = 2^ds). A bijection on the slices when their count is a
// multiple of 2 D.
__device__ __forceinline__ uint32_t paired_slice(uint32_t r, DivU32 sx, uint32_t half,
                                                 uint32_t ds) {
  const uint32_t x = divu(r, sx), rem = r - x * sx.d;
  const uint32_t h = rem >= half ? 1u : 0u, jj = half * x + rem - h * half;
  return ((jj >> ds) << (ds + 1)) + (jj & ((1u << ds) - 1)) + (h << ds);
}

// One vector per thread: n is at most the workgroup's threads.
__device__ __forceinline__ void move_piece(const v4u* __restrict__ s, v4u* __restrict__ d,
                                           uint32_t n) {
  const auto out = stream_dst(d, n * 16u);
  if (threadIdx.x < n)
    store_stream(out, threadIdx.x, __builtin_nontemporal_load(s + threadIdx.x));
}

// ---- cache layouts that reorder a slab ---------------------------------------
//
// The packed side is always [token][head][dim]. The cache side may be
//   KVX_LAYOUT_HND         [head][token][dim] rows (K and V);
//   KVX_LAYOUT_PAGED_ATTN  K [head][dim / x][token][x] (x = 16 / elem_bytes: the
//                          16-byte vectors of a row are re-strided), V
//                          [head][dim][token] (an element transpose).
// In every one of them a head's data is contiguous on the cache side (nh =
// bs * v16 vectors), and on the packed side it is one v16-vector row per token
// at stride prow = heads * v16.
//   * HND: vectors move directly (no LDS). A workgroup writes g.piece consecutive
//     vectors of the destination slab (at most 256: piece_vectors) and reads runs
//     of v16 vectors (or the parts of them that its piece covers).
//   * paged attention: a workgroup moves a tile of about 256 vectors: whole
//     neighbouring heads where they are small, and where a head is larger a
//     run of at least 128 bytes of each of its tokens' rows (tile_geom). Either
//     way the tile is contiguous on the cache side and a run per token on the
//     packed side.
//   * paged-attention K: a vector permutation. The tile is loaded in source
//     order into LDS, then written in destination order, each lane fetching
//     the source vector its output vector is. (Moving each vector straight
//     from its source to its destination, the packed side then in 64-byte
//     runs, measured 2.3 points slower both ways on the 80k workload: the
//     wave-contiguous runs on both sides are worth more than the LDS pass.)
//   * paged-attention V: an element transpose. The tile is loaded in source
//     order into LDS, then each output vector is assembled element by element
//     from it.
// Both global sides stay coalesced (consecutive lanes on consecutive 16-byte
// vectors, or whole runs) and only LDS sees the reordering; the LDS image is
// swizzled so that a wave's strided reads land on distinct banks. A thread
// holds V vectors of the tile, all of its loads issued before it waits for any
// of them: V = 1 for tiles of up to 256 vectors (the usual shapes: few
// registers, full occupancy), 2 or 4 for blocks of many tokens, else
// kVecPerThread, enough for the largest head (kMaxSlabVectors).
// Against one head per workgroup, with 12 vectors a thread for heads above 256
// vectors (1 GiB, 32 layers, gather / scatter, before -> now):
//   16-token blocks, 8 x 128 bf16    341 / 390 -> 342 / 391 us
//   8 x 128 8-bit                    534 / 412 -> 353 / 385 us
//   4 x 64 8-bit                     906 / 608 -> 353 / 397 us
//   32-token blocks, 4 x 128 bf16    464 / 374 -> 345 / 374 us
//   64-token blocks, 2 x 128 bf16    361 / 387 -> 356 / 379 us
//   5 x 80 bf16                      564 / 411 -> 409 / 395 us

constexpr int kTransposeThreads = 256;
constexpr uint32_t kMaxSlabVectors = 48 * 1024 / 16;
constexpr int kVecPerThread = (int)(kMaxSlabVectors / kTransposeThreads);  // 12

extern __shared__ __attribute__((aligned(16))) unsigned char kvx_lds[];

// LDS slot of vector v in the head's image; the layout differs by direction.
// Gather (kToPacked): inside each aligned group of 16 vectors (256 bytes, one
// pass over the 64 banks) the position is XORed with h(r), r = bits swz ..
// swz + 3 of v, which the XOR leaves alone, so the map is a permutation of
// every group. h(r) = r ^ (bit 3 of r moved to bit 1) is itself a permutation
// of 0 .. 15, so a wave walking the image at a stride of 2^swz vectors (the
// head's read stride, chosen on the host) meets 16 different positions per
// group, and consecutive vectors stay in one group; moving bit 3 to bit 1
// also keeps rows r and r + 8 apart modulo 8 positions (32 banks), where the
// 32-bit reads of a half-wave meet (see lane_perm). Scatter: one pad vector
// after every `pad` vectors (the read stride). Measured on gfx950 with the LDS
// bank-conflict counter, a 16 x 16 transposed read of 16-byte vectors costs
// no conflict cycles through an XOR swizzle, 4 per wave instruction with the
// pad and 28 with neither, and linear 16-byte writes cost none either way.
// The 80k paged-attention gather ran 1 to 2 points faster with the swizzle
// (no conflicts left) than with the pad; the scatter ran 2 points slower
// with it (also with no conflicts left): it is not bound by the LDS, and the
// swizzle's extra arithmetic in its element-by-element loop costs more than
// the conflicts it removes.
// 1-byte words take another h, r rotated by one bit: the transposing reads of a
// half-wave (v_bytes) cover 8 consecutive vectors of rows r and r + 1, which
// bit 0 of r then keeps in different halves of the group.
template <bool kToPacked, int kElem>
__device__ __forceinline__ uint32_t lds_slot(uint32_t v, const SlabGeom& g) {
  if (kToPacked) {
    const uint32_t r = (v >> g.swz) & 15u;
    if (kElem == 1) return v ^ (((r & 1u) << 3) | (r >> 1));
    return v ^ (r ^ ((r >> 2) & 2u));
  }
  return v + fdiv(v, g.pad);
}

// Quotient and remainder.
__device__ __forceinline__ uint32_t divmod(uint32_t n, FastDiv f, uint32_t& rem) {
  const uint32_t q = fdiv(n, f);
  rem = n - q * f.d;
  return q;
}

// HND: source vector of destination vector w of a slab.
__device__ __forceinline__ uint32_t hnd_source(uint32_t w, const SlabGeom& g) {
  uint32_t rest, dv;
  const uint32_t a = divmod(w, g.outer, rest);
  const uint32_t b = divmod(rest, g.v16, dv);
  return a * g.v16.d + b * g.src_step + dv;
}

// HND: move piece `part` of a slab: g.piece consecutive vectors of the destination,
// at most 256 (fewer in a slab's last piece).
__device__ __forceinline__ void move_rows(const v4u* __restrict__ src, v4u* __restrict__ dst,
                                          uint32_t n16, const SlabGeom& g, uint32_t part) {
  const uint32_t w = part * g.piece + threadIdx.x;
  const uint32_t end = (part + 1) * g.piece;
  const auto out = stream_dst(dst, n16 * 16u);
  if (w < (end < n16 ? end : n16))
    store_stream(out, w, __builtin_nontemporal_load(src + hnd_source(w, g)));
}

// A workgroup's tile of a paged-attention slab: its first vector on the cache
// side (contiguous from there) and on the packed side (a run of row.d vectors
// per token), and the vectors it has (the last tile of a slab may hold fewer
// heads than gh: the rest of its lanes idle).
struct Tile {
  uint32_t cache0, packed0;
  uint32_t heads;
};

// kOne, here and below: the tile is one whole head (the usual shapes), which
// spares each lane the split by head.
template <bool kOne>
__device__ __forceinline__ Tile tile_at(uint32_t part, const SlabGeom& g) {
  if (kOne) return Tile{part * g.nh, part * g.v16.d, 1};
  uint32_t piece;
  const uint32_t group = divmod(part, g.dpieces, piece), h0 = group * g.gh;
  const uint32_t left = g.heads - h0;
  return Tile{h0 * g.nh + piece * g.np.d, h0 * g.v16.d + piece * g.dw, left < g.gh ? left : g.gh};
}

// Vector w of the tile in packed order (token by token, then head, then
// vector): its packed-side offset from the tile's first vector; ok = false for
// a head the slab does not have.
template <bool kOne>
__device__ __forceinline__ uint32_t packed_at(uint32_t w, const SlabGeom& g, const Tile& tile,
                                              bool* ok) {
  uint32_t q;
  const uint32_t t = divmod(w, g.row, q);
  *ok = kOne ? w < g.nh : t < g.bs.d && q < tile.heads * g.dw;
  return t * g.prow + q;
}

// The same offset in the direction's destination or source order: the cache
// side is contiguous.
template <bool kPackedSide, bool kOne>
__device__ __forceinline__ uint32_t side_at(uint32_t w, const SlabGeom& g, const Tile& tile,
                                            bool* ok) {
  if (kPackedSide) return packed_at<kOne>(w, g, tile, ok);
  *ok = w < (kOne ? g.nh : tile.heads * g.np.d);
  return w;
}

// Load the tile's source vectors, in source order, into the LDS image. A gather
// reads the cache (contiguous), a scatter the packed rows.
template <bool kToPacked, int kElem, bool kOne, int T, int V>
__device__ __forceinline__ void stage_in(const v4u* __restrict__ src, const SlabGeom& g,
                                         const Tile& tile) {
  v4u* lds = reinterpret_cast<v4u*>(kvx_lds);
  v4u r[V];
  bool ok[V];
#pragma unroll
  for (int q = 0; q < V; ++q) {
    const uint32_t at = side_at<!kToPacked, kOne>(threadIdx.x + q * T, g, tile, &ok[q]);
    if (ok[q]) r[q] = __builtin_nontemporal_load(src + at);
  }
#pragma unroll
  for (int q = 0; q < V; ++q)
    if (ok[q]) lds[lds_slot<kToPacked, kElem>(threadIdx.x + q * T, g)] = r[q];
}

// The LDS serves 32-bit and narrower reads a half-wave (32 lanes) at a time
// over 32 banks (measured: two extra cycles per such read when a half-wave
// puts two words on one bank). The paired V gather below therefore lets lane
// L of a wave handle pair lane_perm(L) of the wave's 64 pairs, a permutation
// of the lane bits (b5 b4 b3 b2 b1 b0 -> b4 b3 b5 b2 b1 b0) that gives each
// half-wave 4 token pairs x 8 dim groups instead of 2 x 16; the 64 pairs of a
// wave, and so the bytes each store instruction writes, are the same as in
// lane order. (The scatter keeps lane order: permuting which lane stores
// which cache vector measured a point slower, the stores of a wave no longer
// running in address order; its reads are kept apart by the swizzle.)
__device__ __forceinline__ uint32_t lane_perm(uint32_t i) {
  const uint32_t l = i & 63u;
  return (i & ~63u) | (((l >> 3) & 3u) << 4) | (((l >> 5) & 1u) << 3) | (l & 7u);
}

// Bytes a tile's stores may reach from its first destination vector.
template <bool kToPacked>
__device__ __forceinline__ uint32_t tile_dst_bytes(const SlabGeom& g) {
  return (kToPacked ? (g.bs.d - 1) * g.prow + g.row.d : g.gh * g.np.d) * 16u;
}

// Write the tile's destination vectors, in destination order, each produced by
// f(w). A gather writes the packed rows, a scatter the cache.
template <bool kToPacked, bool kOne, int T, int V, typename F>
__device__ __forceinline__ void stage_out(v4u* __restrict__ dst, const SlabGeom& g,
                                          const Tile& tile, F f) {
  v4u r[V];
  uint32_t at[V];
  bool ok[V];
#pragma unroll
  for (int q = 0; q < V; ++q) {
    at[q] = side_at<kToPacked, kOne>(threadIdx.x + q * T, g, tile, &ok[q]);
    if (ok[q]) r[q] = f(threadIdx.x + q * T);
  }
  const auto out = stream_dst(dst, tile_dst_bytes<kToPacked>(g));
#pragma unroll
  for (int q = 0; q < V; ++q)
    if (ok[q]) store_stream(out, at[q], r[q]);
}

// Head and rest of a tile's vector: index in packed order -> (token, head of the
// tile, vector of the head's row); in cache order -> (head, vector of the head).
template <bool kOne>
__device__ __forceinline__ void packed_split(uint32_t w, const SlabGeom& g, uint32_t* t,
                                             uint32_t* h, uint32_t* dv) {
  *t = divmod(w, g.row, *dv);
  *h = 0;
  if (!kOne) *h = divmod(*dv, g.dwd, *dv);
}

template <bool kOne>
__device__ __forceinline__ uint32_t cache_split(uint32_t w, const SlabGeom& g, uint32_t* r) {
  *r = w;
  return kOne ? 0 : divmod(w, g.np, *r);
}

// Paged-attention K: source vector (in the LDS image) of destination vector w.
// Cache order inside a head is dv * bs + t, packed order (t, head, dv).
template <bool kToPacked, bool kOne>
__device__ __forceinline__ uint32_t k_source(uint32_t w, const SlabGeom& g) {
  uint32_t t, h, dv, r;
  if (kToPacked) {
    packed_split<kOne>(w, g, &t, &h, &dv);
    return h * g.np.d + dv * g.bs.d + t;
  }
  h = cache_split<kOne>(w, g, &r);
  dv = divmod(r, g.bs, t);
  return t * g.row.d + h * g.dw + dv;
}

template <typename E>
struct ElemRow {
  E e[16 / sizeof(E)];
};

// Paged-attention V: destination vector w assembled element by element from
// the LDS image of the source. Cache elements inside a head are (dim, t) at
// dim * bs + t; packed elements (t, head, dim).
template <bool kToPacked, bool kOne, typename E>
__device__ __forceinline__ v4u v_elements(uint32_t w, const SlabGeom& g,
                                          const unsigned char* image) {
  constexpr uint32_t kX = 16 / sizeof(E);
  ElemRow<E> out;
  if (kToPacked) {  // packed (t, dv * x + i) <- cache element (dv * x + i, t): stride bs
    uint32_t t, h, dv;
    packed_split<kOne>(w, g, &t, &h, &dv);
    const uint32_t e0 = (h * g.np.d + dv * g.bs.d) * kX + t;
#pragma unroll
    for (uint32_t i = 0; i < kX; ++i) {
      const uint32_t e = e0 + i * g.bs.d;
      out.e[i] = reinterpret_cast<const E*>(
          image + 16u * lds_slot<kToPacked, sizeof(E)>(e / kX, g))[e % kX];
    }
  } else {  // cache (dim, t .. t + x - 1) <- packed elements (t + i, dim); t wraps to dim + 1
    uint32_t r, t;
    const uint32_t h = cache_split<kOne>(w, g, &r);
    uint32_t dim = h * g.dw * kX + divmod(r * kX, g.bs, t);
#pragma unroll
    for (uint32_t i = 0; i < kX; ++i) {
      const uint32_t e = t * (g.row.d * kX) + dim;
      out.e[i] = reinterpret_cast<const E*>(
          image + 16u * lds_slot<kToPacked, sizeof(E)>(e / kX, g))[e % kX];
      if (++t == g.bs.d) {
        t = 0;
        ++dim;
      }
    }
  }
  return __builtin_bit_cast(v4u, out);
}

// Paged-attention V of 2-byte words in a gather, two packed rows per thread:
// the rows of tokens t and t + 1 (t even) at one group of dims, whose
// elements come from cache words (dim, t) and (dim, t + 1), adjacent in one
// dword. Each 32-bit LDS read yields one element of each vector, so no two
// lanes share a dword, and for the usual shapes (block size 16, 16 vectors
// per row) a wave's reads of one element land on 64 distinct banks; the two
// stores of a lane write whole token rows. A scatter does not pair its
// vectors this way: paired dims d, d + 1 would make each store instruction
// write every other 32-byte run of the cache lines (the 80k scatter ran at
// half speed that way). Pairs take half of a tile's threads, so a thread has
// (V + 1) / 2 of them.
template <bool kOne, int T, int V>
__device__ __forceinline__ void v_pairs_gather(v4u* __restrict__ dst, const SlabGeom& g,
                                               const Tile& tile) {
  typedef ElemRow<uint16_t> Row;
  constexpr int P = (V + 1) / 2;
  Row r0[P], r1[P];
  uint32_t at[P];
  bool ok[P];
#pragma unroll
  for (int q = 0; q < P; ++q) {
    // a half-wave takes 4 token pairs x 8 dim groups (16 vectors per row)
    const uint32_t p = lane_perm(threadIdx.x + q * T);
    uint32_t tp, h, dv;
    packed_split<kOne>(p, g, &tp, &h, &dv);  // tokens 2 tp, 2 tp + 1
    ok[q] = kOne ? 2 * p < g.nh : 2 * tp < g.bs.d && h < tile.heads;
    if (!ok[q]) continue;
    at[q] = 2 * tp * g.prow + h * g.dw + dv;
    const uint32_t e0 = (h * g.np.d + dv * g.bs.d) * 8 + 2 * tp;
#pragma unroll
    for (uint32_t i = 0; i < 8; ++i) {
      const uint32_t e = e0 + i * g.bs.d;
      const uint32_t w = *reinterpret_cast<const uint32_t*>(
          kvx_lds + 16u * lds_slot<true, 2>(e >> 3, g) + 2u * (e & 7u));
      r0[q].e[i] = (uint16_t)w;
      r1[q].e[i] = (uint16_t)(w >> 16);
    }
  }
  const auto out = stream_dst(dst, tile_dst_bytes<true>(g));
#pragma unroll
  for (int q = 0; q < P; ++q) {
    if (!ok[q]) continue;
    store_stream(out, at[q], __builtin_bit_cast(v4u, r0[q]));
    store_stream(out, at[q] + g.prow, __builtin_bit_cast(v4u, r1[q]));
  }
}

// Paged-attention V of 1-byte words in blocks of a multiple of 16 tokens, with
// the LDS transpose reads of gfx950: ds_read_b64_tr_b8 over 16 lanes, lane l
// giving the address of bytes 8 (l % 2) .. + 7 of row l / 2 of an 8 x 16 byte
// matrix, returns its column l to lane l. Two of them make one destination
// vector per lane, 16 rows of one column, where the element loop above takes
// sixteen byte reads. A gather transposes 16 dims x 16 tokens (rows: dims),
// a scatter 16 tokens x 16 dims. Vector w of the tile, in the order in which
// lanes take them: 16-lane group k = w / 16 of (head, 16 tokens, 16 dims); at:
// its destination offset. 8 x 128 dims, 16 tokens, 1 GiB: gather 365 -> 353 us,
// scatter 400 -> 385 us against element by element.
// Every lane of the wave must take part: a transposing read writes the result
// registers of all 64 lanes, also of those that are switched off, where the
// compiler may keep another value, such as what the other side of a branch
// computed. So lanes with nothing to turn give a vector that exists and drop the
// result.
typedef int v2i __attribute__((ext_vector_type(2)));

__device__ __forceinline__ v2i read_tr8(const unsigned char* p) {
  return __builtin_amdgcn_ds_read_tr8_b64_v2i32(
      (__attribute__((address_space(3))) v2i*)const_cast<unsigned char*>(p));
}

template <bool kToPacked>
__device__ __forceinline__ v4u v_bytes(uint32_t w, const SlabGeom& g, const unsigned char* image,
                                       uint32_t row, uint32_t* at) {
  const uint32_t k = w >> 4, l = w & 15u;
  uint32_t tg, dv, h, first, step;
  if (kToPacked) {  // rows: dims 16 dv + i; columns: tokens 16 tg ..
    h = divmod(divmod(k, g.dwd, dv), g.bs16, tg);
    first = h * g.np.d + dv * g.bs.d + (l >> 1) * g.bs16.d + tg;
    step = 8 * g.bs16.d;
    *at = (16 * tg + l) * row + h * g.dw + dv;
  } else {  // rows: tokens 16 tg + i; columns: dims 16 dv ..
    h = divmod(divmod(k, g.bs16, tg), g.dwd, dv);
    first = (16 * tg + (l >> 1)) * g.row.d + h * g.dw + dv;
    step = 8 * g.row.d;
    *at = h * g.np.d + (16 * dv + l) * g.bs16.d + tg;
  }
  // Odd groups read their rows 8 .. 15 first: a scatter's rows lie a vector
  // apart modulo the banks, and neighbouring groups' would meet there.
  const bool odd = !kToPacked && (k & 1u);
  const uint32_t a = odd ? first + step : first, b = odd ? first : first + step;
  const unsigned char* half = image + 8u * (l & 1u);
  const v2i x = read_tr8(half + 16u * lds_slot<kToPacked, 1>(a, g));
  const v2i y = read_tr8(half + 16u * lds_slot<kToPacked, 1>(b, g));
  const v2i lo = odd ? y : x, hi = odd ? x : y;
  return v4u{(uint32_t)lo.x, (uint32_t)lo.y, (uint32_t)hi.x, (uint32_t)hi.y};
}

template <bool kToPacked, int T, int V>
__device__ __forceinline__ void v_bytes_out(v4u* __restrict__ dst, const SlabGeom& g,
                                            const Tile& tile) {
  v4u r[V];
  uint32_t at[V];
  bool ok[V];
#pragma unroll
  for (int q = 0; q < V; ++q) {
    const uint32_t w = threadIdx.x + q * T;
    ok[q] = w < tile.heads * g.np.d;  // the same for the 16 lanes of a group
    r[q] = v_bytes<kToPacked>(ok[q] ? w : w & 15u, g, kvx_lds, g.prow, &at[q]);
  }
  const auto out = stream_dst(dst, tile_dst_bytes<kToPacked>(g));
#pragma unroll
  for (int q = 0; q < V; ++q)
    if (ok[q]) store_stream(out, at[q], r[q]);
}

// The same for a gather whose rows are not whole 64-byte runs of four lane
// groups: a group's 16 bytes of 16 tokens would be stored as parts of lines. The
// vectors go back to the LDS in packed order first and leave as whole rows.
// 3 heads of 80 dims, 1 GiB: 651 us stored directly, 388 by elements, 363
// this way; 5 heads of 96 dims 623, 375, 367 us.
template <int T, int V>
__device__ __forceinline__ void v_bytes_rows_out(v4u* __restrict__ dst, const SlabGeom& g,
                                                 const Tile& tile) {
  v4u* lds = reinterpret_cast<v4u*>(kvx_lds);
  v4u r[V];
  uint32_t at[V];
  bool ok[V];
#pragma unroll
  for (int q = 0; q < V; ++q) {
    const uint32_t w = threadIdx.x + q * T;
    ok[q] = w < tile.heads * g.np.d;
    r[q] = v_bytes<true>(ok[q] ? w : w & 15u, g, kvx_lds, g.row.d, &at[q]);
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < V; ++q)
    if (ok[q]) lds[at[q]] = r[q];
  __syncthreads();
  stage_out<true, false, T, V>(dst, g, tile, [&](uint32_t w) { return lds[w]; });
}

// One tile of a paged-attention slab (pv, pk: the slab's first vector on the
// cache and on the packed side).
template <bool kToPacked, int kElem, bool kOne, int T, int V>
__device__ __forceinline__ void move_tile(v4u* pv, v4u* pk, const SlabGeom& g, uint32_t kv,
                                          uint32_t part) {
  typedef typename std::conditional<
      kElem == 1, uint8_t,
      typename std::conditional<kElem == 2, uint16_t,
                                typename std::conditional<kElem == 4, uint32_t,
                                                          uint64_t>::type>::type>::type E;
  const Tile tile = tile_at<kOne>(part, g);
  const v4u* src = kToPacked ? pv + tile.cache0 : pk + tile.packed0;
  v4u* dst = kToPacked ? pk + tile.packed0 : pv + tile.cache0;
  stage_in<kToPacked, kElem, kOne, T, V>(src, g, tile);
  __syncthreads();
  const v4u* lds = reinterpret_cast<const v4u*>(kvx_lds);
  if (kv == 0)
    stage_out<kToPacked, kOne, T, V>(dst, g, tile, [&](uint32_t w) {
      return lds[lds_slot<kToPacked, kElem>(k_source<kToPacked, kOne>(w, g), g)];
    });
  else if (kElem == 1 && kToPacked && g.v_bytes == 2)
    v_bytes_rows_out<T, V>(dst, g, tile);
  else if (kElem == 1 && g.v_bytes)
    v_bytes_out<kToPacked, T, V>(dst, g, tile);
  else if (kToPacked && kElem == 2 && g.v_pairs)
    v_pairs_gather<kOne, T, V>(dst, g, tile);
  else
    stage_out<kToPacked, kOne, T, V>(dst, g, tile, [&](uint32_t w) {
      return v_elements<kToPacked, kOne, E>(w, g, kvx_lds);
    });
}

// Move part `part` of one slab in the direction and layout of the kernel: a piece of
// g.piece vectors (at most 256) with the default layout and HND, one tile with paged
// attention.
template <bool kToPacked, int kLayout, int kElem, bool kOne, int T, int V>
__device__ __forceinline__ void move_unit(char* paged, char* pk, uint32_t n16, const SlabGeom& g,
                                          uint32_t kv, uint32_t part) {
  v4u* pv = reinterpret_cast<v4u*>(paged);
  v4u* kv4 = reinterpret_cast<v4u*>(pk);
  if (kLayout == KVX_LAYOUT_NHD) {
    const uint32_t off = part * g.piece;  // < n16
    const uint32_t left = n16 - off;
    const uint32_t n = left < g.piece ? left : g.piece;
    if (kToPacked)
      move_piece(pv + off, kv4 + off, n);
    else
      move_piece(kv4 + off, pv + off, n);
  } else if (kLayout == KVX_LAYOUT_HND) {
    if (kToPacked)
      move_rows(pv, kv4, n16, g, part);
    else
      move_rows(kv4, pv, n16, g, part);
  } else {
    move_tile<kToPacked, kElem, kOne, T, V>(pv, kv4, g, kv, part);
  }
}

// Work item w of a launch -> (unit, part of the unit).
__device__ __forceinline__ uint32_t split_work(uint32_t w, uint32_t parts, uint32_t shift,
                                               DivU32 parts_div, uint32_t* part) {
  const uint32_t u = shift < 32 ? w >> shift : divu(w, parts_div);
  *part = w - u * parts;
  return u;
}

// Work item w = unit * parts + part.
// kOrdered = false: units in image order (u -> chunk, layer|K|V, block).
// kOrdered = true: unit v -> lk = v / n_blocks, k = v % n_blocks, (block index
// i, its block id) = order[k] (destinations ascending by bucket); the image
// position u of (chunk i / bpc, lk, block i % bpc) follows.
// A workgroup moves only 4 KiB, so the scalar loads before its first data
// load matter: the block id and the layer pointer (or, ordered, the order
// entry, which carries the id, and the layer pointer) are issued together
// and waited for once. The empty asm statements take the loaded values,
// which keeps the compiler from moving the layer pointer's load past the
// block-id check.
template <bool kToPacked, bool kOrdered, int kLayout, int kElem, bool kOne, int T, int V>
__global__ void __launch_bounds__(T)
    copy_units_kernel(LayerPtrs layers, const int32_t* __restrict__ block_table, UnitGeom g,
                      uint32_t unit_base, uint32_t part_base, uint32_t work_count,
                      const OrderEntry* __restrict__ order, char* __restrict__ packed,
                      int* __restrict__ err) {
  uint32_t part;
  const uint32_t w = g.linear_walk                  ? blockIdx.x
                     : kOrdered && g.pair_shift < 32 ? xcd_two_fronts(blockIdx.x, work_count,
                                                                      g.parts_shift)
                                                     : xcd_contiguous(blockIdx.x, work_count);
  uint32_t u =
      unit_base + split_work(part_base + w, g.parts, g.parts_shift, g.parts_div, &part);
  uint32_t c, first, nc, lk, j;
  int32_t id;
  char* layer;
  if (kOrdered) {
    const uint32_t walk = divu(u, g.nb_div);  // slice in walk order
    const OrderEntry e = order[u - walk * g.n_blocks];  // e.index < n_blocks (a permutation)
    lk = g.pair_shift < 32 ? paired_slice(walk, g.xcd_slices_div, g.half_slices, g.pair_shift)
                           : walk;
    layer = layers.p[lk];
    __asm__ volatile("" : : "s"(e.index), "s"(e.id), "s"(layer));
    const uint32_t i = e.index;
    id = e.id;
    c = divu(i, g.bpc_div);
    first = c * g.bpc;
    j = i - first;
    const uint32_t left = g.n_blocks - first;
    nc = left < g.bpc ? left : g.bpc;
    u = c * g.units_per_chunk + lk * nc + j;
  } else {
    c = divu(u, g.upc_div);
    const uint32_t r = u - c * g.units_per_chunk;
    first = c * g.bpc;
    const uint32_t left = g.n_blocks - first;
    nc = left < g.bpc ? left : g.bpc;  // blocks in this chunk
    const DivU32 ncd = nc == g.bpc ? g.bpc_div : g.last_div;
    if (g.gather_pair_shift < 32) {
      // Paired walk of the chunk: its work items in walk order are pair p of
      // slices (a_p, a_p + D) (a_p: the p-th slice whose index has bit log2 D
      // clear, D = 2^ds), then block j, then the two slices' part `part`
      // alternately. A bijection on the chunk's items.
      const uint32_t ps = g.parts_shift + 1, ds = g.gather_pair_shift;
      const uint32_t wi = (r << g.parts_shift) + part;  // walk position within the chunk
      const uint32_t p = divu(wi >> ps, ncd);            // 2 * nc * parts items per pair
      const uint32_t r2 = wi - ((p * nc) << ps);
      const uint32_t r3 = r2 & ((1u << ps) - 1);
      j = r2 >> ps;
      part = r3 >> 1;
      lk = ((p >> ds) << (ds + 1)) + (p & ((1u << ds) - 1)) + ((r3 & 1) << ds);
      u = c * g.units_per_chunk + lk * nc + j;  // image position of (lk, j)
    } else {
      lk = divu(r, ncd);  // 2 * (l - l0) + kv
      j = r - lk * nc;
    }
    id = block_table[first + j];
    layer = layers.p[lk];
    __asm__ volatile("" : : "s"(id), "s"(layer));
  }
  if ((uint32_t)id >= g.num_blocks) {
    if (threadIdx.x == 0) atomicOr(err, kErrBadBlock);
    return;
  }
  char* paged = layer + (uint64_t)(uint32_t)id * g.slab;
  char* pk = packed + (uint64_t)u * g.slab;
  move_unit<kToPacked, kLayout, kElem, kOne, T, V>(paged, pk, g.n16, g.sg, lk & 1, part);
}

// Chunk-list copy: a batch of chunks, each with its own block-table slice and
// its own place in the packed buffer (the fused block copy of several
// requests' chunks in one launch). Unit space is padded: chunk c owns units
// [c * upc, (c + 1) * upc) with upc = (l1 - l0) * 2 * bpc, unit r of a chunk
// is (lk = r / bpc, j = r % bpc), and units with j >= the chunk's n_blocks
// exit at once. So a workgroup finds its chunk by one division, with no
// search. Each reference is validated here (it lives in device memory): a bad
// one sets kErrBadChunk and its units are skipped.
struct ChunkGeom {
  uint32_t upc;          // (l1 - l0) * 2 * bpc
  uint32_t bpc;
  uint32_t lr2;          // (l1 - l0) * 2
  uint32_t n_chunks;
  uint32_t list_grid;    // workgroups of a copy without padding (copy_list_kernel)
  DivU32 lr2_div;
  uint32_t num_blocks;   // pool size
  uint32_t n_units;      // n_chunks * upc
  uint32_t n16;
  uint32_t group;        // slabs per workgroup, as in UnitGeom
  uint32_t parts;        // workgroups per slab, as in UnitGeom
  uint32_t parts_shift;
  DivU32 parts_div;
  DivU32 upc_div;
  DivU32 bpc_div;
  int32_t table_len;
  uint64_t slab;
  int64_t packed_bytes;
  SlabGeom sg;
};

__device__ __forceinline__ bool chunk_ref_ok(const kvx_chunk_ref& ref, const ChunkGeom& g) {
  return ref.n_blocks >= 1 && (uint32_t)ref.n_blocks <= g.bpc && ref.bt_offset >= 0 &&
         (int64_t)ref.bt_offset + ref.n_blocks <= (int64_t)g.table_len &&
         ref.packed_offset >= 0 && (ref.packed_offset & 15) == 0 &&
         ref.packed_offset <=  // a sum could wrap
             g.packed_bytes - (int64_t)g.lr2 * ref.n_blocks * (int64_t)g.slab;
}

template <bool kToPacked, int kLayout, int kElem, bool kOne, int T, int V>
__global__ void __launch_bounds__(T)
    copy_chunks_kernel(LayerPtrs layers, const int32_t* __restrict__ block_table,
                       const kvx_chunk_ref* __restrict__ refs, ChunkGeom g, uint32_t unit_base,
                       uint32_t part_base, uint32_t work_count, char* __restrict__ packed,
                       int* __restrict__ err) {
  uint32_t part;
  const uint32_t u =
      unit_base + split_work(part_base + xcd_contiguous(blockIdx.x, work_count), g.parts,
                             g.parts_shift, g.parts_div, &part);
  const uint32_t c = divu(u, g.upc_div);
  const uint32_t r = u - c * g.upc;
  const uint32_t lk = divu(r, g.bpc_div);
  const uint32_t j = r - lk * g.bpc;
  const kvx_chunk_ref ref = refs[c];
  if (!chunk_ref_ok(ref, g)) {
    if (r == 0 && part == 0 && threadIdx.x == 0) atomicOr(err, kErrBadChunk);
    return;
  }
  const uint32_t nc = (uint32_t)ref.n_blocks;
  if (j >= nc) return;  // padding unit
  const int32_t id = block_table[ref.bt_offset + j];
  if ((uint32_t)id >= g.num_blocks) {
    if (threadIdx.x == 0) atomicOr(err, kErrBadBlock);
    return;
  }
  char* paged = layers.p[lk] + (uint64_t)(uint32_t)id * g.slab;
  char* pk = packed + ref.packed_offset + (uint64_t)(lk * nc + j) * g.slab;
  move_unit<kToPacked, kLayout, kElem, kOne, T, V>(paged, pk, g.n16, g.sg, lk & 1, part);
}

// ---- chunk lists without padding ----------------------------------------------
//
// Where many of a list's chunks are short, the padded unit space above dispatches
// a workgroup for every piece that they do not have, and its equal ranges of
// units give the XCDs unequal bytes. list_kernel therefore writes one ListBlock
// per block that the list does have, in list order; the copy's units are then
// 0 .. lr2 * blocks - 1, chunk by chunk, and unit u belongs to the chunk of block
// u / lr2. (A search for the chunk in every 4 KiB workgroup, the other way to find
// it, would put several dependent loads before the data.) Decode and loads are as
// many as in the padded space. A gather moves slices 2 MiB apart in a chunk
// together, as in the unit walk (gather_pairing), where the chunk's own length
// puts them there. 1 GiB in chunks of 1 to 16 of 16 blocks, 32 layers, gather /
// scatter, padded -> listed: 32 KiB slabs 389 / 401 -> 354 / 378 us; of 64 blocks
// 487 / 498 -> 358 / 382; 80 layers of 4 KiB slabs 401 / 413 -> 359 / 388; 256 MiB
// of 32 KiB slabs 116 / 120 -> 94 / 100.

// What a unit's decode needs of the chunk that holds its block.
struct ListBlock {
  int64_t packed;   // the chunk's packed_offset
  uint32_t first;   // blocks of the list before the chunk
  uint32_t n;       // blocks of the chunk, and the multiplier and shift of DivU32 for n
  uint32_t m, s;
  int32_t bt;       // the chunk's bt_offset
  uint32_t pair;    // log2 of the distance of its paired slices, or 32
};
static_assert(sizeof(ListBlock) == 32, "one scalar load");

constexpr uint32_t kListThreads = 256;
constexpr uint32_t kListChunks = 64;    // chunks per workgroup of list_kernel
constexpr uint32_t kListMaxChunks = 4096;  // each workgroup sums the blocks of all chunks before its own
constexpr uint64_t kListMaxBlocks = 1u << 16;  // 2 MiB of entries

// Blocks of chunk c, or 0 for a bad reference.
__device__ __forceinline__ uint32_t list_blocks(const kvx_chunk_ref* refs, uint32_t c,
                                                const ChunkGeom& g) {
  const kvx_chunk_ref ref = refs[c];
  return chunk_ref_ok(ref, g) ? (uint32_t)ref.n_blocks : 0u;
}

// blocks[0 .. *count) for the list; bad references are reported and left out.
// pair: 1 if the slices of a chunk may be paired.
__global__ void __launch_bounds__(kListThreads)
    list_kernel(const kvx_chunk_ref* __restrict__ refs, ChunkGeom g, uint32_t pair,
                ListBlock* __restrict__ blocks, uint32_t* __restrict__ count,
                int* __restrict__ err) {
  __shared__ uint32_t before_wave[kListThreads / 64];
  __shared__ uint32_t end[kListChunks];  // blocks of this workgroup's chunks up to and with c
  const uint32_t t = threadIdx.x, c0 = blockIdx.x * kListChunks;
  const uint32_t nc = g.n_chunks - c0 < kListChunks ? g.n_chunks - c0 : kListChunks;
  uint32_t sum = 0;
  for (uint32_t c = t; c < c0; c += kListThreads) sum += list_blocks(refs, c, g);
  for (uint32_t off = 32; off; off >>= 1) sum += __shfl_down(sum, off, 64);
  if (t % 64 == 0) before_wave[t / 64] = sum;
  if (t < 64) {
    uint32_t n = t < nc ? list_blocks(refs, c0 + t, g) : 0u;
    if (t < nc && n == 0) atomicOr(err, kErrBadChunk);
    for (uint32_t off = 1; off < 64; off <<= 1) {
      const uint32_t y = __shfl_up(n, off, 64);
      if (t >= off) n += y;
    }
    end[t] = n;
  }
  __syncthreads();
  uint32_t before = 0;
  for (uint32_t w = 0; w < kListThreads / 64; ++w) before += before_wave[w];
  const uint32_t mine = end[nc - 1];
  if (t == 0 && c0 + nc == g.n_chunks) *count = before + mine;
  for (uint32_t k = t; k < mine; k += kListThreads) {
    uint32_t lo = 0, hi = nc - 1;  // the first chunk whose end is above k
    while (lo < hi) {
      const uint32_t mid = (lo + hi) / 2;
      if (end[mid] > k) hi = mid;
      else lo = mid + 1;
    }
    const kvx_chunk_ref ref = refs[c0 + lo];
    ListBlock b;
    b.packed = ref.packed_offset;
    b.first = before + (lo ? end[lo - 1] : 0u);
    b.n = (uint32_t)ref.n_blocks;
    uint32_t l = 0;  // ceil(log2 n), as div_u32
    while ((1ull << l) < b.n) ++l;
    b.m = b.n <= 1 ? 0u : (uint32_t)(((1ull << 32) * ((1ull << l) - b.n)) / b.n + 1);
    b.s = b.n <= 1 ? 0u : l - 1;
    b.bt = ref.bt_offset;
    b.pair = 32;
    const uint64_t run = (uint64_t)b.n * g.slab, two_mib = 2u << 20;
    if (pair && two_mib % run == 0) {
      const uint32_t d = (uint32_t)(two_mib / run);  // as gather_pairing
      if ((d & (d - 1)) == 0 && d <= 32 && g.lr2 % (2 * d) == 0) b.pair = 31 - __clz(d);
    }
    blocks[before + k] = b;
  }
}

// The copy over blocks[0 .. *count): as many workgroups as the table has entries
// for, which is as many as the list needs unless its chunks share entries. Then
// workgroups go round again, with paged attention (kLoop = false) those of a
// second launch from workgroup `first` on, which else end at once: around the
// LDS phases the loop cost 8 to 25 % (8 x 128 dims, 1 GiB, uneven lists, gather /
// scatter: bf16 389 / 398 us looped, 357 / 397 in two launches; 8-bit 423 / 510
// and 372 / 402), around plain moves nothing. A list that does share pays for the
// rounds, which the host cannot foresee (the lengths are in device memory): 16
// requests of four shared 16-block chunks and 3 blocks of their own, 2.25 GB gathered,
// padded / listed: 32 KiB slabs 763 / 845 us, paged attention 785 / 966; 32 such
// requests of 4 KiB slabs, 80 layers, 1.4 GB, 502 / 576. Decoding a round's part while
// the loads of the one before are in flight gained 1 to 5 % of that and lost 3 % with
// 8-bit tiles.
template <bool kToPacked, bool kLoop, int kLayout, int kElem, bool kOne, int T, int V>
__global__ void __launch_bounds__(T)
    copy_list_kernel(LayerPtrs layers, const int32_t* __restrict__ block_table,
                     const ListBlock* __restrict__ blocks, const uint32_t* __restrict__ count,
                     ChunkGeom g, uint32_t first, uint32_t stride, char* __restrict__ packed,
                     int* __restrict__ err) {
  constexpr bool kAgain = kLoop || kLayout != KVX_LAYOUT_PAGED_ATTN;
  const uint32_t total = *count * g.lr2 * g.parts;
  uint32_t b = first + blockIdx.x;
  if (b >= total) return;
  do {
    uint32_t part;
    const uint32_t u =
        split_work(xcd_contiguous(b, total), g.parts, g.parts_shift, g.parts_div, &part);
    const ListBlock e = blocks[divu(u, g.lr2_div)];
    const uint32_t r = u - e.first * g.lr2;
    const DivU32 nd{e.n, e.m, e.s};
    uint32_t lk, j;
    if (kToPacked && e.pair < 32) {  // the paired walk of copy_units_kernel
      const uint32_t ps = g.parts_shift + 1;
      const uint32_t wi = (r << g.parts_shift) + part, p = divu(wi >> ps, nd);
      const uint32_t r2 = wi - ((p * e.n) << ps), r3 = r2 & ((1u << ps) - 1);
      j = r2 >> ps;
      part = r3 >> 1;
      lk = ((p >> e.pair) << (e.pair + 1)) + (p & ((1u << e.pair) - 1)) + ((r3 & 1) << e.pair);
    } else {
      lk = divu(r, nd);
      j = r - lk * e.n;
    }
    const int32_t id = block_table[e.bt + (int32_t)j];
    char* layer = layers.p[lk];
    __asm__ volatile("" : : "s"(id), "s"(layer));
    if ((uint32_t)id < g.num_blocks) {
      char* pk = packed + e.packed + (uint64_t)(lk * e.n + j) * g.slab;
      move_unit<kToPacked, kLayout, kElem, kOne, T, V>(layer + (uint64_t)(uint32_t)id * g.slab, pk,
                                                       g.n16, g.sg, lk & 1, part);
    } else if (threadIdx.x == 0) {
      atomicOr(err, kErrBadBlock);
    }
    if (!kAgain) return;
    if (kLayout == KVX_LAYOUT_PAGED_ATTN) __syncthreads();  // before the LDS image is reused
    b += stride;
  } while (b < total);
}

// ---- small slabs: several per workgroup ----------------------------------------
//
// A slab of at most kGroupMaxVectors vectors (2 KiB) would leave half of a
// 256-thread workgroup or more idle, and the copy is then bound by the rate at
// which workgroups are dispatched (1.65 per ns measured, so a slab each caps
// 1 KiB slabs at 1.7 TB/s each way). So a workgroup moves `group` = 256 / n16
// consecutive units, one vector per thread; thread t takes vector t % n16 of
// unit t / n16. Where a slab is a whole number of waves (kWave) a wave's unit is
// uniform and its decode stays on the scalar unit; else each lane decodes its
// own. 1 GiB, 32 layers, gather / scatter, a slab per workgroup -> grouped:
// 2 KiB slabs 373 / 378 -> 351 / 372 us, 1 KiB 641 / 588 -> 353 / 372 us,
// 512 bytes 1272 / 1163 -> 366 / 384 us, 256 bytes 2540 / 2320 -> 370 / 384 us.
// (128-thread workgroups holding half as many slabs measured level at 2 KiB
// and 3 to 16 % slower at 1,536 and 1,280 bytes.)

// Where one unit's slab lies, or ok = false: an id outside the pool (reported) or no unit.
struct Place {
  char* paged;
  char* packed;
  char* base;  // at or below this lane's destination, the same or nearby for the wave's lanes
  uint32_t kv;
  bool ok;
};

// Store v at vector w of dst. Lanes of one wave may hold different dst; kWave
// says that they do not. The streaming store takes one base per wave and a
// 32-bit offset per lane, so lanes store relative to the first lane's `base`
// where every lane is less than 4 GiB above it; otherwise (layers far apart in
// one wave) with plain non-temporal stores.
template <bool kWave>
__device__ __forceinline__ void store_grouped(char* base, char* dst, uint32_t n16, uint32_t w,
                                              v4u v) {
  if (kWave) {
    const auto out = stream_dst(reinterpret_cast<v4u*>(dst), n16 * 16u);
    store_stream(out, w, v);
    return;
  }
  const uint64_t b = (uint64_t)base;
  const uint64_t b0 = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(b >> 32)) << 32) |
                      (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
  const uint64_t off = (uint64_t)dst + 16u * w - b0;
  if (__builtin_amdgcn_ballot_w64(off > 0xFFFFFFE0ull) == 0) {
    const auto out = stream_dst(reinterpret_cast<v4u*>(b0), 0xFFFFFFFFu);
    store_stream_at(out, (uint32_t)off, v);
  } else {
    __builtin_nontemporal_store(v, reinterpret_cast<v4u*>(dst) + w);
  }
}

// Unit of this thread in the workgroup, and its vector in the unit's slab.
template <bool kWave>
__device__ __forceinline__ uint32_t grouped_unit(const SlabGeom& g, uint32_t* w) {
  uint32_t i = divmod(threadIdx.x, g.n16, *w);
  return kWave ? (uint32_t)__builtin_amdgcn_readfirstlane((int)i) : i;
}

template <bool kToPacked, int kLayout, bool kWave>
__device__ __forceinline__ void move_grouped(const Place& p, uint32_t w, const SlabGeom& g) {
  const v4u* src = reinterpret_cast<const v4u*>(kToPacked ? p.paged : p.packed);
  char* dst = kToPacked ? p.packed : p.paged;
  const uint32_t from = kLayout == KVX_LAYOUT_HND ? hnd_source(w, g) : w;
  store_grouped<kWave>(p.base, dst, g.n16.d, w, __builtin_nontemporal_load(src + from));
}

// Paged attention: each slab of the group has an LDS image of its own and is one
// tile (gh = heads, dw = v16). Called by every thread of the workgroup. 1 GiB of
// 2 KiB slabs, 8-bit, one head, gather / scatter: 516 / 552 us with a slab per
// workgroup, 404 / 411 grouped with a unit decoded by every lane, 370 / 372 with
// one per wave; 512-byte slabs 1480 / 1526 -> 575 / 513 us (by lane).
template <bool kToPacked, int kElem, bool kWave>
__device__ __forceinline__ void move_grouped_paged(const Place& p, uint32_t i, uint32_t w,
                                                   const SlabGeom& g) {
  typedef typename std::conditional<
      kElem == 1, uint8_t,
      typename std::conditional<kElem == 2, uint16_t,
                                typename std::conditional<kElem == 4, uint32_t,
                                                          uint64_t>::type>::type>::type E;
  unsigned char* image = kvx_lds + 16u * ((p.ok ? i : 0u) * g.image);
  v4u* lds = reinterpret_cast<v4u*>(image);
  if (p.ok)
    lds[lds_slot<kToPacked, kElem>(w, g)] = __builtin_nontemporal_load(
        reinterpret_cast<const v4u*>(kToPacked ? p.paged : p.packed) + w);
  __syncthreads();
  v4u v = {};
  uint32_t to = w;
  const bool turn = p.ok && p.kv != 0;
  if (kElem == 1 && g.v_bytes) {
    // a wave can hold K and V: all of its lanes take part in the transposing reads
    v4u turned = {};
    uint32_t at = 0;
    const bool rows = kToPacked && g.v_bytes == 2;  // as v_bytes_rows_out
    if (__builtin_amdgcn_ballot_w64(turn))
      turned = v_bytes<kToPacked>(w, g, image, rows ? g.row.d : g.prow, &at);
    if (turn) v = turned;
    else if (p.ok) v = lds[lds_slot<kToPacked, kElem>(k_source<kToPacked, false>(w, g), g)];
    if (rows) {
      __syncthreads();
      if (turn) lds[at] = v;
      __syncthreads();
      if (turn) v = lds[w];
    } else if (turn) {
      to = at;
    }
  } else if (turn) {
    v = v_elements<kToPacked, false, E>(w, g, image);
  } else if (p.ok) {
    v = lds[lds_slot<kToPacked, kElem>(k_source<kToPacked, false>(w, g), g)];
  }
  if (p.ok) store_grouped<kWave>(p.base, kToPacked ? p.packed : p.paged, g.n16.d, to, v);
}

// Unit u of a grouped call, in image order (slabs this small take no other:
// small_rows, kvx_walk.cpp).
template <bool kToPacked>
__device__ __forceinline__ Place place_unit(const LayerPtrs& layers, const int32_t* block_table,
                                            const UnitGeom& g, uint32_t u, char* packed, int* err,
                                            bool report) {
  const uint32_t c = divu(u, g.upc_div), first = c * g.bpc;
  const uint32_t r = u - c * g.units_per_chunk, left = g.n_blocks - first;
  const bool full = left >= g.bpc;
  const uint32_t lk = divu(r, full ? g.bpc_div : g.last_div);
  const int32_t id = block_table[first + r - lk * (full ? g.bpc : left)];
  char* layer = layers.p[lk];
  Place p;
  p.ok = (uint32_t)id < g.num_blocks;
  if (!p.ok && report) atomicOr(err, kErrBadBlock);
  p.paged = layer + (uint64_t)(uint32_t)id * g.slab;
  p.packed = packed + (uint64_t)u * g.slab;
  p.base = kToPacked ? p.packed : layer;
  p.kv = lk & 1;
  return p;
}

// kElem: the word size with paged attention, else 0.
template <bool kToPacked, int kLayout, int kElem, bool kWave>
__global__ void __launch_bounds__(kPartThreads)
    copy_unit_groups_kernel(LayerPtrs layers, const int32_t* __restrict__ block_table, UnitGeom g,
                            uint32_t group_base, uint32_t group_count, char* __restrict__ packed,
                            int* __restrict__ err) {
  uint32_t w;
  const uint32_t i = grouped_unit<kWave>(g.sg, &w);
  const uint32_t u = (group_base + (g.linear_walk ? blockIdx.x
                                                  : xcd_contiguous(blockIdx.x, group_count))) *
                         g.group + i;
  Place p = {};
  if (i < g.group && u < g.n_units)
    p = place_unit<kToPacked>(layers, block_table, g, u, packed, err, w == 0);
  if constexpr (kLayout == KVX_LAYOUT_PAGED_ATTN)
    move_grouped_paged<kToPacked, kElem, kWave>(p, i, w, g.sg);
  else if (p.ok)
    move_grouped<kToPacked, kLayout, kWave>(p, w, g.sg);
}

// Unit u of a chunk list's padded unit space (copy_chunks_kernel).
template <bool kToPacked>
__device__ __forceinline__ Place place_chunk_unit(const LayerPtrs& layers,
                                                  const int32_t* block_table,
                                                  const kvx_chunk_ref* refs, const ChunkGeom& g,
                                                  uint32_t u, char* packed, int* err,
                                                  bool report) {
  const uint32_t c = divu(u, g.upc_div), r = u - c * g.upc;
  const uint32_t lk = divu(r, g.bpc_div), j = r - lk * g.bpc;
  const kvx_chunk_ref ref = refs[c];
  Place p = {};
  if (!chunk_ref_ok(ref, g)) {
    if (r == 0 && report) atomicOr(err, kErrBadChunk);
    return p;
  }
  const uint32_t nc = (uint32_t)ref.n_blocks;
  if (j >= nc) return p;
  const int32_t id = block_table[ref.bt_offset + j];
  char* layer = layers.p[lk];
  p.ok = (uint32_t)id < g.num_blocks;
  if (!p.ok && report) atomicOr(err, kErrBadBlock);
  p.paged = layer + (uint64_t)(uint32_t)id * g.slab;
  p.packed = packed + ref.packed_offset + (uint64_t)(lk * nc + j) * g.slab;
  p.base = kToPacked ? packed : layer;
  p.kv = lk & 1;
  return p;
}

template <bool kToPacked, int kLayout, int kElem, bool kWave>
__global__ void __launch_bounds__(kPartThreads)
    copy_chunk_groups_kernel(LayerPtrs layers, const int32_t* __restrict__ block_table,
                             const kvx_chunk_ref* __restrict__ refs, ChunkGeom g,
                             uint32_t group_base, uint32_t group_count, char* __restrict__ packed,
                             int* __restrict__ err) {
  uint32_t w;
  const uint32_t i = grouped_unit<kWave>(g.sg, &w);
  const uint32_t u = (group_base + xcd_contiguous(blockIdx.x, group_count)) * g.group + i;
  Place p = {};
  if (i < g.group && u < g.n_units)
    p = place_chunk_unit<kToPacked>(layers, block_table, refs, g, u, packed, err, w == 0);
  if constexpr (kLayout == KVX_LAYOUT_PAGED_ATTN)
    move_grouped_paged<kToPacked, kElem, kWave>(p, i, w, g.sg);
  else if (p.ok)
    move_grouped<kToPacked, kLayout, kWave>(p, w, g.sg);
}

// The grouped copy over a list without padding.
template <bool kToPacked, bool kLoop, int kLayout, int kElem, bool kWave>
__global__ void __launch_bounds__(kPartThreads)
    copy_list_groups_kernel(LayerPtrs layers, const int32_t* __restrict__ block_table,
                            const ListBlock* __restrict__ blocks,
                            const uint32_t* __restrict__ count, ChunkGeom g, uint32_t first,
                            uint32_t stride, char* __restrict__ packed, int* __restrict__ err) {
  constexpr bool kAgain = kLoop || kLayout != KVX_LAYOUT_PAGED_ATTN;
  const uint32_t units = *count * g.lr2, groups = (units + g.group - 1) / g.group;
  uint32_t w;
  const uint32_t i = grouped_unit<kWave>(g.sg, &w);
  uint32_t b = first + blockIdx.x;
  if (b >= groups) return;
  do {
    const uint32_t u = xcd_contiguous(b, groups) * g.group + i;
    Place p = {};
    if (i < g.group && u < units) {
      const ListBlock e = blocks[divu(u, g.lr2_div)];
      const uint32_t r = u - e.first * g.lr2, lk = divu(r, DivU32{e.n, e.m, e.s});
      const uint32_t j = r - lk * e.n;
      const int32_t id = block_table[e.bt + (int32_t)j];
      char* layer = layers.p[lk];
      p.ok = (uint32_t)id < g.num_blocks;
      if (!p.ok && w == 0) atomicOr(err, kErrBadBlock);
      p.paged = layer + (uint64_t)(uint32_t)id * g.slab;
      p.packed = packed + e.packed + (uint64_t)r * g.slab;
      p.base = kToPacked ? packed : layer;
      p.kv = lk & 1;
    }
    if constexpr (kLayout == KVX_LAYOUT_PAGED_ATTN) {
      move_grouped_paged<kToPacked, kElem, kWave>(p, i, w, g.sg);
      if (!kAgain) return;
      __syncthreads();  // before the LDS images are reused
    } else if (p.ok) {
      move_grouped<kToPacked, kLayout, kWave>(p, w, g.sg);
    }
    b += stride;
  } while (b < groups);
}

// Destination order for a scatter: order[] lists the block-table indexes,
// each with the id it holds, bucketed by destination id, buckets ascending. The id range [0, num_blocks)
// is cut into kBins equal bins (ids outside it go to the last bin; the copy
// kernel skips them). One workgroup counts bin sizes in LDS, scans them into
// bin starts and places each index with an LDS atomic, so order[] is a
// permutation of [0, n) for any table (within a bin the order is
// unspecified, which only matters if destinations repeat, and a scatter's
// destinations must be distinct).
constexpr int kOrderThreads = 1024;
constexpr uint32_t kBins = 4096;  // 4 bins per thread

__device__ __forceinline__ uint32_t bin_of(int32_t id, uint32_t num_blocks, uint32_t bins) {
  const uint32_t u = (uint32_t)id;
  return u >= num_blocks ? bins - 1 : (uint32_t)(((uint64_t)u * bins) / num_blocks);
}

__global__ void __launch_bounds__(kOrderThreads)
    order_kernel(const int32_t* __restrict__ block_table, uint32_t n, uint32_t num_blocks,
                 OrderEntry* __restrict__ order) {
  __shared__ uint32_t cnt[kBins];
  __shared__ uint32_t wave_total[kOrderThreads / 64];
  const uint32_t t = threadIdx.x, lane = t % 64, wave = t / 64;
  const uint32_t bins = num_blocks < kBins ? num_blocks : kBins;
  for (uint32_t b = t; b < kBins; b += kOrderThreads) cnt[b] = 0;
  __syncthreads();
  for (uint32_t i = t; i < n; i += kOrderThreads)
    atomicAdd(&cnt[bin_of(block_table[i], num_blocks, bins)], 1u);
  __syncthreads();
  // exclusive scan of the kBins counts: 4 per thread, then waves, then workgroup
  const uint32_t c0 = cnt[4 * t], c1 = cnt[4 * t + 1], c2 = cnt[4 * t + 2], c3 = cnt[4 * t + 3];
  const uint32_t mine = c0 + c1 + c2 + c3;
  uint32_t incl = mine;
  for (uint32_t off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(incl, off, 64);
    if (lane >= off) incl += y;
  }
  if (lane == 63) wave_total[wave] = incl;
  __syncthreads();
  if (wave == 0) {
    uint32_t w = lane < kOrderThreads / 64 ? wave_total[lane] : 0;
    for (uint32_t off = 1; off < kOrderThreads / 64; off <<= 1) {
      const uint32_t y = __shfl_up(w, off, 64);
      if (lane >= off) w += y;
    }
    if (lane < kOrderThreads / 64) wave_total[lane] = w;  // inclusive over waves
  }
  __syncthreads();
  const uint32_t base = (wave > 0 ? wave_total[wave - 1] : 0u) + incl - mine;
  cnt[4 * t] = base;
  cnt[4 * t + 1] = base + c0;
  cnt[4 * t + 2] = base + c0 + c1;
  cnt[4 * t + 3] = base + c0 + c1 + c2;
  __syncthreads();
  for (uint32_t i = t; i < n; i += kOrderThreads) {
    const int32_t id = block_table[i];
    order[atomicAdd(&cnt[bin_of(id, num_blocks, bins)], 1u)] = OrderEntry{i, id};
  }
}

#define KVX_UNPAREN(...) __VA_ARGS__

constexpr uint64_t kListMinPadding = 1u << 15;
constexpr uint64_t kListMinWork = 1u << 13;
constexpr uint32_t kListTail = 2048;  // eight workgroups a compute unit

// Whether a paged-attention scatter of tiles of at most 256 vectors runs them
// on half as many threads with two vectors each. Twice as many of
// its workgroups then fit a compute unit, which keeps more loads in flight
// across its LDS phases. Measured over 12-18 (cache, packed buffer)
// allocation pairs in one process at the 80k prefix of the 8B shape, against
// one vector on each of 256 threads: 81.2 against 78.9 % of peak with 8
// heads, level with 4 (75.3 / 75.2 %), 69.4 against 69.9 % with 2 and, with
// the linear walk a one-head scatter takes (kvx_walk.cpp), 69.6 against
// 73.2 % with 1. So only slabs of four heads or more take it, and not tiles
// that are pieces of a head (4 heads of 32 tokens x 128 dims: 390 us on half the
// threads, 374 on 256, 1 GiB).
inline bool pa_scatter_on_half_threads(const SlabGeom& sg) {
  return sg.gh * sg.np.d <= (uint32_t)kTransposeThreads && sg.heads >= 4 && sg.dpieces.d == 1;
}

// Dynamic LDS bytes of a workgroup of T threads with V vectors each: the tile's
// image. Tiles that fill two or more vectors a thread reserve enough that six
// workgroups run on a compute unit: eight would keep 64 KiB or more of reads in
// flight there. 1 GiB, 32 layers, gather / scatter, 64-token blocks of 128
// dims: 2 heads bf16 375 / 394 us unheld, 360 / 382 held; 2 heads 8-bit 376 /
// 402 and 365 / 387; 4 heads 8-bit 382 / 389 and 355 / 375 (held to four 373 /
// 384). Tiles with idle lanes lost up to 10 % held (5 x 96 dims 8-bit: 375 / 394
// and 413 / 399).
inline size_t tile_lds(const SlabGeom& sg, uint32_t T, uint32_t V) {
  constexpr size_t kSixPerUnit = 27000;
  const size_t image = 16u * (size_t)sg.image;
  return V > 1 && T == (uint32_t)kTransposeThreads && sg.gh * sg.np.d == T * V
             ? std::max(image, kSixPerUnit)
             : image;
}

// Launch a paged-attention kernel: a tile per workgroup of kTransposeThreads
// with 1, 2, 4 or kVecPerThread vectors a thread, a scatter of four or more
// heads per slab on half the threads (pa_scatter_on_half_threads; the gather
// was no faster that way). PREFIX is the kernel's parenthesized leading
// template arguments; kToPacked is the enclosing launcher's direction.
#define KVX_LAUNCH_TILE(KERNEL, PREFIX, ELEM, ONE, T, V, ...)                               \
  hipLaunchKernelGGL((KERNEL<KVX_UNPAREN PREFIX, KVX_LAYOUT_PAGED_ATTN, ELEM, ONE, T, V>), grid, \
                     dim3(T), tile_lds(sg, T, V), stream, __VA_ARGS__)

#define KVX_LAUNCH_TILES(KERNEL, PREFIX, ELEM, ...)                                         \
  do {                                                                                 \
    const uint32_t tile = sg.gh * sg.np.d;                                             \
    const bool one = sg.gh == 1 && sg.dpieces.d == 1;                                  \
    constexpr int T = kTransposeThreads;                                               \
    if constexpr (!kToPacked) {                                                        \
      if (pa_scatter_on_half_threads(sg)) {                                            \
        if (one)                                                                       \
          KVX_LAUNCH_TILE(KERNEL, PREFIX, ELEM, true, T / 2, 2, __VA_ARGS__);          \
        else                                                                           \
          KVX_LAUNCH_TILE(KERNEL, PREFIX, ELEM, false, T / 2, 2, __VA_ARGS__);         \
        break;                                                                         \
      }                                                                                \
    }                                                                                  \
    if (tile <= (uint32_t)T && one)                                                    \
      KVX_LAUNCH_TILE(KERNEL, PREFIX, ELEM, true, T, 1, __VA_ARGS__);                  \
    else if (tile <= (uint32_t)T)                                                      \
      KVX_LAUNCH_TILE(KERNEL, PREFIX, ELEM, false, T, 1, __VA_ARGS__);                 \
    else if (tile <= 2u * T)                                                           \
      KVX_LAUNCH_TILE(KERNEL, PREFIX, ELEM, false, T, 2, __VA_ARGS__);                 \
    else if (tile <= 4u * T)                                                           \
      KVX_LAUNCH_TILE(KERNEL, PREFIX, ELEM, false, T, 4, __VA_ARGS__);                 \
    else                                                                               \
      KVX_LAUNCH_TILE(KERNEL, PREFIX, ELEM, false, T, kVecPerThread, __VA_ARGS__);     \
  } while (0)

#define KVX_DISPATCH_PAGED(KERNEL, PREFIX, ...)                                             \
  do {                                                                                 \
    if (elem == 1)                                                                     \
      KVX_LAUNCH_TILES(KERNEL, PREFIX, 1, __VA_ARGS__);                                 \
    else if (elem == 2)                                                                \
      KVX_LAUNCH_TILES(KERNEL, PREFIX, 2, __VA_ARGS__);                                 \
    else if (elem == 4)                                                                \
      KVX_LAUNCH_TILES(KERNEL, PREFIX, 4, __VA_ARGS__);                                 \
    else                                                                               \
      KVX_LAUNCH_TILES(KERNEL, PREFIX, 8, __VA_ARGS__);                                 \
  } while (0)

#define KVX_DISPATCH(KERNEL, PREFIX, ...)                                                   \
  do {                                                                                 \
    const uint32_t threads = (sg.piece + 63u) & ~63u;                                  \
    if (layout == KVX_LAYOUT_NHD)                                                      \
      hipLaunchKernelGGL((KERNEL<KVX_UNPAREN PREFIX, KVX_LAYOUT_NHD, 0, false, kPartThreads, 1>), \
                         grid, dim3(threads), 0, stream, __VA_ARGS__);                 \
    else if (layout == KVX_LAYOUT_HND)                                                 \
      hipLaunchKernelGGL((KERNEL<KVX_UNPAREN PREFIX, KVX_LAYOUT_HND, 0, false, kPartThreads, 1>), \
                         grid, dim3(threads), 0, stream, __VA_ARGS__);                 \
    else                                                                               \
      KVX_DISPATCH_PAGED(KERNEL, PREFIX, __VA_ARGS__);                                 \
  } while (0)

// Calls launch(unit_base, part_base, workgroups) for each launch of a copy of
// n_units slabs of `parts` workgroups each: as many whole slabs as fit
// kMaxWorkPerLaunch, or runs of one slab's parts where a slab has more.
template <typename F>
hipError_t each_launch(uint32_t n_units, uint32_t parts, F launch) {
  const uint32_t units = parts < kMaxWorkPerLaunch ? kMaxWorkPerLaunch / parts : 1;
  for (uint64_t u = 0; u < n_units; u += units) {
    const uint32_t nu = n_units - u < units ? (uint32_t)(n_units - u) : units;
    const uint64_t work = (uint64_t)nu * parts;
    for (uint64_t p = 0; p < work; p += kMaxWorkPerLaunch) {
      launch((uint32_t)u, (uint32_t)p,
             (uint32_t)(work - p < kMaxWorkPerLaunch ? work - p : kMaxWorkPerLaunch));
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

// Launch the grouped kernel of a copy of slabs of N16 vectors, GROUP of them per
// workgroup (paged attention: an LDS image each).
#define KVX_LAUNCH_GROUP(KERNEL, PREFIX, LAYOUT, ELEM, LDS, N16, ...)                       \
  do {                                                                                 \
    if ((N16) % 64 == 0)                                                               \
      hipLaunchKernelGGL((KERNEL<KVX_UNPAREN PREFIX, LAYOUT, ELEM, true>), grid,       \
                         dim3(kPartThreads), LDS, stream, __VA_ARGS__);                \
    else                                                                               \
      hipLaunchKernelGGL((KERNEL<KVX_UNPAREN PREFIX, LAYOUT, ELEM, false>), grid,      \
                         dim3(kPartThreads), LDS, stream, __VA_ARGS__);                \
  } while (0)

#define KVX_LAUNCH_GROUPS_PAGED(KERNEL, PREFIX, N16, GROUP, ...)                            \
  do {                                                                                 \
    const size_t lds = 16u * (size_t)sg.image * (GROUP);                               \
    if (elem == 1)                                                                     \
      KVX_LAUNCH_GROUP(KERNEL, PREFIX, KVX_LAYOUT_PAGED_ATTN, 1, lds, N16, __VA_ARGS__); \
    else if (elem == 2)                                                                \
      KVX_LAUNCH_GROUP(KERNEL, PREFIX, KVX_LAYOUT_PAGED_ATTN, 2, lds, N16, __VA_ARGS__); \
    else if (elem == 4)                                                                \
      KVX_LAUNCH_GROUP(KERNEL, PREFIX, KVX_LAYOUT_PAGED_ATTN, 4, lds, N16, __VA_ARGS__); \
    else                                                                               \
      KVX_LAUNCH_GROUP(KERNEL, PREFIX, KVX_LAYOUT_PAGED_ATTN, 8, lds, N16, __VA_ARGS__); \
  } while (0)

#define KVX_LAUNCH_GROUPS(KERNEL, PREFIX, N16, GROUP, ...)                                  \
  do {                                                                                 \
    if (layout == KVX_LAYOUT_NHD)                                                      \
      KVX_LAUNCH_GROUP(KERNEL, PREFIX, KVX_LAYOUT_NHD, 0, 0, N16, __VA_ARGS__);         \
    else if (layout == KVX_LAYOUT_HND)                                                 \
      KVX_LAUNCH_GROUP(KERNEL, PREFIX, KVX_LAYOUT_HND, 0, 0, N16, __VA_ARGS__);         \
    else                                                                               \
      KVX_LAUNCH_GROUPS_PAGED(KERNEL, PREFIX, N16, GROUP, __VA_ARGS__);                \
  } while (0)

template <bool kToPacked, bool kOrdered>
hipError_t launch(const LayerPtrs& lp, const int32_t* bt, const UnitGeom& ug,
                  const OrderEntry* order, char* packed, int* err, int layout, int elem,
                  hipStream_t stream) {
  const SlabGeom& sg = ug.sg;
  if constexpr (!kOrdered) {
    if (ug.group > 1)
      return each_launch((ug.n_units - 1) / ug.group + 1, 1,
                         [&](uint32_t group, uint32_t, uint32_t cnt) {
                           const dim3 grid(cnt);
                           KVX_LAUNCH_GROUPS(copy_unit_groups_kernel, (kToPacked), ug.n16, ug.group,
                                             lp, bt, ug, group, cnt, packed, err);
                         });
  }
  return each_launch(ug.n_units, ug.parts, [&](uint32_t unit, uint32_t part, uint32_t cnt) {
    const dim3 grid(cnt);
    KVX_DISPATCH(copy_units_kernel, (kToPacked, kOrdered), lp, bt, ug, unit, part, cnt,
                 order, packed, err);
  });
}

template <bool kToPacked>
hipError_t launch_chunks(const LayerPtrs& lp, const int32_t* bt, const kvx_chunk_ref* refs,
                         const ChunkGeom& cg, char* packed, int* err, int layout, int elem,
                         hipStream_t stream) {
  const SlabGeom& sg = cg.sg;
  if (cg.group > 1)
    return each_launch((cg.n_units - 1) / cg.group + 1, 1,
                       [&](uint32_t group, uint32_t, uint32_t cnt) {
                         const dim3 grid(cnt);
                         KVX_LAUNCH_GROUPS(copy_chunk_groups_kernel, (kToPacked), cg.n16, cg.group,
                                           lp, bt, refs, cg, group, cnt, packed, err);
                       });
  return each_launch(cg.n_units, cg.parts, [&](uint32_t unit, uint32_t part, uint32_t cnt) {
    const dim3 grid(cnt);
    KVX_DISPATCH(copy_chunks_kernel, (kToPacked), lp, bt, refs, cg, unit, part, cnt, packed, err);
  });
}

// Workgroups `first` and up of a list copy, `n` of them; kLoop: the second launch
// of paged attention.
template <bool kToPacked, bool kLoop>
hipError_t launch_list_copy(const LayerPtrs& lp, const int32_t* bt, const ListBlock* blocks,
                            const uint32_t* count, const ChunkGeom& cg, uint32_t first, uint32_t n,
                            char* packed, int* err, int layout, int elem, hipStream_t stream) {
  const SlabGeom& sg = cg.sg;
  const dim3 grid(n);
  if constexpr (kLoop) {
    if (cg.group > 1)
      KVX_LAUNCH_GROUPS_PAGED(copy_list_groups_kernel, (kToPacked, true), cg.n16, cg.group, lp, bt,
                              blocks, count, cg, first, n, packed, err);
    else
      KVX_DISPATCH_PAGED(copy_list_kernel, (kToPacked, true), lp, bt, blocks, count, cg, first, n,
                         packed, err);
  } else {
    if (cg.group > 1)
      KVX_LAUNCH_GROUPS(copy_list_groups_kernel, (kToPacked, false), cg.n16, cg.group, lp, bt,
                        blocks, count, cg, first, n, packed, err);
    else
      KVX_DISPATCH(copy_list_kernel, (kToPacked, false), lp, bt, blocks, count, cg, first, n,
                   packed, err);
  }
  return hipGetLastError();
}

// The list's blocks counted and listed in `scratch` (a slot's: take_list_slot),
// then one copy over them.
template <bool kToPacked>
hipError_t launch_list(const LayerPtrs& lp, const int32_t* bt, const kvx_chunk_ref* refs,
                       const ChunkGeom& cg, uint32_t* scratch, char* packed, int* err, int layout,
                       int elem, hipStream_t stream) {
  ListBlock* blocks = reinterpret_cast<ListBlock*>(scratch + 64);
  const bool pair = kToPacked && cg.parts_shift < 32 && cg.group == 1;
  hipLaunchKernelGGL(list_kernel, dim3((cg.n_chunks + kListChunks - 1) / kListChunks),
                     dim3(kListThreads), 0, stream, refs, cg, pair ? 1u : 0u, blocks, scratch,
                     err);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = launch_list_copy<kToPacked, false>(lp, bt, blocks, scratch, cg, 0, cg.list_grid, packed, err,
                                         layout, elem, stream);
  if (e == hipSuccess && layout == KVX_LAYOUT_PAGED_ATTN)
    e = launch_list_copy<kToPacked, true>(lp, bt, blocks, scratch, cg, cg.list_grid,
                                          std::min(cg.list_grid, kListTail), packed, err, layout,
                                          elem, stream);
  return e;
}

// Workgroups of a list copy without padding, or 0 where the padded copy is
// taken: few padding workgroups by the table's length (a list's chunks hardly
// ever share table entries); little to move; more blocks than a slot has entries;
// more units than a launch takes; or a capturing stream, whose graph would use a
// slot without waiting for it. The lines at 32,768 padding workgroups and 8,192
// others were drawn when a call's scratch took 12 us of its stream and 24 us of the
// host (65 us padded, 57 listed, with 38,000 padding workgroups). With slots a
// listed call takes 10 us of the host, a padded one 5, and the listed copy is level
// below 16 MiB and ahead from there: chunks of 1 to 16 of 16 blocks, 32 layers of
// 32 KiB slabs, padded / listed, 8 MiB 10.8 / 10.9 us, 24 MiB 17.7 / 17.1, 48 MiB
// 28.7 / 23.9, 128 MiB 57.9 / 54.3, 256 MiB 119.0 / 95.3.
uint32_t list_grid(const ChunkGeom& g, hipStream_t stream) {
  const uint64_t padded = (uint64_t)g.n_chunks * g.bpc, table = (uint64_t)g.table_len;
  if (table >= padded || g.n_chunks > kListMaxChunks || padded > kListMaxBlocks) return 0;
  const auto workgroups = [&](uint64_t blocks) {
    return g.group > 1 ? (blocks * g.lr2 + g.group - 1) / g.group : blocks * g.lr2 * g.parts;
  };
  if (workgroups(padded) - workgroups(table) < kListMinPadding ||
      workgroups(table) < kListMinWork)
    return 0;
  if (workgroups(padded) > 0x7FFFFFFF || workgroups(table) > kMaxWorkPerLaunch) return 0;
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &capture) != hipSuccess ||
      capture != hipStreamCaptureStatusNone) {
    (void)hipGetLastError();
    return 0;
  }
  // a multiple of the XCDs, so that a workgroup that goes round stays on its own
  return (uint32_t)((workgroups(table) + kXcds - 1) / kXcds * kXcds);
}

DivU32 div_u32(uint32_t d) {
  DivU32 f{d, 0u, 0u};
  if (d <= 1) return f;
  uint32_t l = 0;
  while (l < 32 && (1ull << l) < d) ++l;  // ceil(log2 d)
  f.m = (uint32_t)(((1ull << 32) * ((1ull << l) - d)) / d + 1);
  f.s = l - 1;
  return f;
}

FastDiv fast_div(uint32_t d) {
  FastDiv f;
  f.d = d;
  f.m = d <= 1 ? 0u : (uint32_t)(((1ull << 32) + d - 1) / d);
  return f;
}

// Vectors that a workgroup moves of a slab of n16 in the default layout or HND:
// 256, or, where a second piece or a nearly empty third one would follow, the
// slab in equal pieces of whole 128-byte lines, on as many waves as they need.
// 1 GiB, 32 layers, gather: 4,352-byte slabs 459 us in 256s, 390 in halves,
// 5 KiB 409 and 372, 6 KiB 381 and 353, 9 KiB in thirds 365 and 355; a fuller
// third piece is better left short (10 KiB: 358 us in 256s, 366 in thirds), and
// larger slabs measured level either way.
uint32_t piece_vectors(uint32_t n16) {
  const uint32_t parts = (n16 + kPartThreads - 1) / kPartThreads, last = n16 % kPartThreads;
  if (parts == 1 || last == 0 || parts > 3 || (parts == 3 && last >= kPartThreads / 2))
    return kPartThreads;
  return ((n16 + parts - 1) / parts + 7u) & ~7u;
}

// Slab shape and LDS layout, from the stride (in vectors) of a tile's strided
// LDS reads: a gather (cache image in LDS)
// reads paged-attention K vectors and V elements of consecutive dims at
// stride bs, and swizzles with shift log2 of that stride (at least 16)
// rounded up to a power of two; a scatter (packed image in LDS) reads them at
// the stride of a tile's row (K: consecutive tokens; V: the x tokens of one
// output vector) and pads after every row (of at least 8 vectors). HND uses
// no LDS.
SlabGeom slab_geom(const kvx_cache* c, bool to_packed) {
  const uint32_t bs = (uint32_t)c->block_size, h = (uint32_t)c->num_kv_heads,
                 v16 = (uint32_t)((int64_t)c->head_dim * c->elem_bytes / 16),
                 n16 = (uint32_t)((int64_t)bs * h * c->head_dim * c->elem_bytes / 16);
  SlabGeom sg = {};
  sg.bs = fast_div(bs);
  sg.v16 = fast_div(v16 ? v16 : 1);
  sg.nh = bs * v16;
  sg.prow = h * v16;
  sg.heads = h;
  if (c->layout == KVX_LAYOUT_PAGED_ATTN) {
    const TileShape tile = paged_tile(bs, h, v16);
    sg.gh = tile.heads;
    sg.dw = tile.vectors;
    sg.dpieces = fast_div(v16 / tile.vectors);
    sg.row = fast_div(tile.heads * tile.vectors);
    sg.np = fast_div(bs * tile.vectors);
    sg.dwd = fast_div(tile.vectors);
  }
  sg.piece = piece_vectors(n16);
  sg.n16 = fast_div(n16);
  sg.outer = fast_div(to_packed ? sg.prow : sg.nh);
  sg.src_step = to_packed ? sg.nh : sg.prow;
  // V of 2-byte words as row pairs in a gather: token pairs, so an even
  // block size (v_pairs_gather says why not in a scatter)
  sg.v_pairs = c->elem_bytes == 2 && to_packed && bs % 2 == 0 ? 1u : 0u;
  // transpose reads; 2: a gather's rows are not whole 64-byte runs (v_bytes_rows_out)
  sg.v_bytes = c->elem_bytes != 1 || bs % 16 != 0 ? 0u : to_packed && sg.dw % 4 != 0 ? 2u : 1u;
  sg.bs16 = fast_div(bs / 16);
  const uint32_t stride = to_packed ? bs : sg.row.d;
  sg.swz = 4;
  while ((1u << sg.swz) < stride) ++sg.swz;
  sg.pad = fast_div(stride < 8 ? 8 : stride);
  const uint32_t n = sg.gh * sg.np.d;
  sg.image = to_packed ? (n + 15u) & ~15u : n + n / sg.pad.d + 1;
  return sg;
}

}  // namespace

namespace {

// Per device: the table's device address and which stream owns each word.
// Fixed-size (no allocation), open addressing on the stream handle.
constexpr int kMaxDevices = 64;
struct ErrorTable {
  int* base = nullptr;
  hipStream_t owner[kErrorWords] = {};
  bool used[kErrorWords] = {};
};
ErrorTable g_tables[kMaxDevices];
std::mutex g_tables_mu;

// ---- scratch of the list copies without padding --------------------------------
//
// A fixed array, cut into slots (count, then one entry per block): stream-ordered
// allocations made a call wait, on the host, for the list call before it. A stream
// keeps the slot it used last and is in order with itself; a stream without one
// takes the slot that was used longest ago and waits on the device for the copy
// that had it. Calls are so independent on up to kListSlots streams. The event of
// a slot is recorded behind each copy; waiting for it also covers a stream that
// was destroyed and whose handle another one got.
constexpr int kListSlots = 4;
constexpr size_t kListSlotBytes = 256 + kListMaxBlocks * sizeof(ListBlock);
static __device__ __align__(256) unsigned char g_list_scratch[kListSlots * kListSlotBytes];

struct ListSlot {
  hipStream_t stream = nullptr;
  hipEvent_t done = nullptr;
  uint64_t used = 0;  // when, in the device's list copies; 0: never
};

struct ListSlots {
  char* base = nullptr;
  uint64_t copies = 0;
  ListSlot slot[kListSlots];
};

ListSlots g_list_slots[kMaxDevices];
std::mutex g_list_mu;  // held from taking a slot until its event is recorded

// The calling device's slot for a list copy on `stream`, which is made to wait
// for the slot's last copy, and the slot's memory; null if that fails.
ListSlot* take_list_slot(hipStream_t stream, uint32_t** scratch) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  ListSlots& t = g_list_slots[dev];
  if (!t.base) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(g_list_scratch)) != hipSuccess) return nullptr;
    t.base = (char*)p;
  }
  ListSlot* s = t.slot;
  for (ListSlot& c : t.slot) {
    if (c.used && c.stream == stream) {
      s = &c;
      break;
    }
    if (c.used < s->used) s = &c;
  }
  if (!s->done && hipEventCreateWithFlags(&s->done, hipEventDisableTiming) != hipSuccess) {
    s->done = nullptr;
    return nullptr;
  }
  if (s->used && hipStreamWaitEvent(stream, s->done, 0) != hipSuccess) return nullptr;
  s->stream = stream;
  s->used = ++t.copies;
  *scratch = reinterpret_cast<uint32_t*>(t.base + (size_t)(s - t.slot) * kListSlotBytes);
  return s;
}

}  // namespace

int* stream_error_word(hipStream_t stream) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_tables_mu);
  ErrorTable& t = g_tables[dev];
  if (!t.base) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(g_error_words)) != hipSuccess) return nullptr;
    t.base = (int*)p;
  }
  if (!stream) return t.base;
  const uint64_t h = (uint64_t)(uintptr_t)stream * 0x9E3779B97F4A7C15ull;
  uint32_t w = 1 + (uint32_t)(h >> 40) % (kErrorWords - 1);
  for (int probe = 0; probe < kErrorWords - 1; ++probe) {
    if (!t.used[w]) {
      t.used[w] = true;
      t.owner[w] = stream;
      return t.base + w;
    }
    if (t.owner[w] == stream) return t.base + w;
    w = w + 1 == (uint32_t)kErrorWords ? 1u : w + 1;
  }
  return t.base;  // table full: the shared word
}

kvx_status launch_copy(bool to_packed, const kvx_cache* cache, int32_t l0, int32_t l1,
                       const int32_t* block_table, const Geometry& g, void* packed,
                       hipStream_t stream, int* err, void* order_scratch) {
  if (g.n_units == 0) return KVX_OK;
  if (g.n_units > 0x7FFFFFFF || g.slab % 16 != 0) return KVX_EINTERNAL;
  if (!err) return KVX_EHIP;
  LayerPtrs lp = {};
  for (int32_t l = l0; l < l1; ++l) {
    lp.p[2 * (l - l0)] = static_cast<char*>(cache->k[l]);
    lp.p[2 * (l - l0) + 1] = static_cast<char*>(cache->v[l]);
  }
  Walk walk;
  const kvx_status ws = choose_walk(to_packed, cache, g, &walk);
  if (ws != KVX_OK) return ws;
  UnitGeom ug;
  ug.units_per_chunk = (uint32_t)(2 * g.lr * g.bpc);
  ug.bpc = (uint32_t)g.bpc;
  ug.n_blocks = (uint32_t)g.n_blocks;
  ug.num_blocks = (uint32_t)g.num_blocks;
  ug.n_units = (uint32_t)g.n_units;
  ug.n16 = (uint32_t)(g.slab / 16);
  const int layout = copy_layout(cache->layout, cache->num_kv_heads, cache->block_size);
  const int elem = cache->elem_bytes;
  ug.group = copy_group(ug.n16);
  ug.parts = walk.parts;
  ug.parts_shift = walk.parts_shift;
  ug.parts_div = div_u32(ug.parts);
  ug.upc_div = div_u32(ug.units_per_chunk);
  ug.bpc_div = div_u32(ug.bpc);
  ug.last_div = div_u32((uint32_t)(g.n_blocks - (g.n_blocks - 1) / g.bpc * g.bpc));
  ug.nb_div = div_u32(ug.n_blocks);
  ug.slab = (uint64_t)g.slab;
  ug.sg = slab_geom(cache, to_packed);
  const uint32_t n_slices = (uint32_t)(2 * g.lr);
  ug.pair_shift = walk.pair_shift;
  ug.gather_pair_shift = walk.gather_pair_shift;
  ug.half_slices = n_slices / kXcds / 2;
  ug.linear_walk = walk.linear ? 1u : 0u;
  ug.xcd_slices_div = div_u32(n_slices / kXcds ? n_slices / kXcds : 1);
  if (to_packed) {
    hipError_t e = launch<true, false>(lp, block_table, ug, nullptr, (char*)packed, err, layout,
                                       elem, stream);
    return e == hipSuccess ? KVX_OK : KVX_EHIP;
  }
  // Destination-ordered scatter for large calls of multi-block chunks; the
  // order lives in the caller's scratch (order_scratch, n_blocks entries) or
  // else in stream-ordered scratch allocated here. If that allocation fails,
  // fall back to image order (same result, slower).
  OrderEntry* order = nullptr;
  const bool own = order_scratch == nullptr;
  if (walk.ordered) {
    if (!own)
      order = static_cast<OrderEntry*>(order_scratch);
    else if (hipMallocAsync((void**)&order, (size_t)g.n_blocks * sizeof(OrderEntry), stream) !=
             hipSuccess)
      order = nullptr;
  }
  (void)hipGetLastError();
  hipError_t e;
  if (order) {
    hipLaunchKernelGGL(order_kernel, dim3(1), dim3(kOrderThreads), 0, stream, block_table,
                       (uint32_t)g.n_blocks, (uint32_t)g.num_blocks, order);
    e = hipGetLastError();
    if (e == hipSuccess)
      e = launch<false, true>(lp, block_table, ug, order, (char*)packed, err, layout, elem,
                              stream);
    if (own) {
      const hipError_t ef = hipFreeAsync(order, stream);
      if (e == hipSuccess) e = ef;
    }
  } else {
    e = launch<false, false>(lp, block_table, ug, nullptr, (char*)packed, err, layout, elem,
                             stream);
  }
  return e == hipSuccess ? KVX_OK : KVX_EHIP;
}

// Both chunk-list launchers; may_list: the copy may run without padding (list_grid).
static kvx_status copy_chunks(bool may_list, bool to_packed, const kvx_cache* cache, int32_t l0,
                              int32_t l1, const int32_t* block_table, int32_t table_len,
                              const kvx_chunk_ref* refs, int32_t n_chunks, int32_t chunk_tokens,
                              void* packed, int64_t packed_bytes, hipStream_t stream,
                              int* err) {
  if (n_chunks <= 0 || l1 <= l0) return KVX_OK;
  if (!err) return KVX_EHIP;
  const int64_t slab = (int64_t)cache->block_size * cache->num_kv_heads * cache->head_dim *
                       cache->elem_bytes;
  const int64_t bpc = chunk_tokens / cache->block_size;
  const int64_t upc = (int64_t)(l1 - l0) * 2 * bpc;
  const int64_t n_units = upc * n_chunks;
  if (bpc <= 0 || n_units > 0x7FFFFFFF || slab % 16 != 0) return KVX_EINTERNAL;
  LayerPtrs lp = {};
  for (int32_t l = l0; l < l1; ++l) {
    lp.p[2 * (l - l0)] = static_cast<char*>(cache->k[l]);
    lp.p[2 * (l - l0) + 1] = static_cast<char*>(cache->v[l]);
  }
  ChunkGeom cg = {};
  cg.upc = (uint32_t)upc;
  cg.bpc = (uint32_t)bpc;
  cg.lr2 = (uint32_t)(2 * (l1 - l0));
  cg.num_blocks = (uint32_t)cache->num_blocks;
  cg.n_units = (uint32_t)n_units;
  cg.n16 = (uint32_t)(slab / 16);
  const int layout = copy_layout(cache->layout, cache->num_kv_heads, cache->block_size);
  const int elem = cache->elem_bytes;
  copy_parts(cache, cg.n16, &cg.parts, &cg.parts_shift);
  cg.group = copy_group(cg.n16);
  cg.parts_div = div_u32(cg.parts);
  cg.upc_div = div_u32(cg.upc);
  cg.bpc_div = div_u32(cg.bpc);
  cg.table_len = table_len;
  cg.slab = (uint64_t)slab;
  cg.packed_bytes = packed_bytes;
  cg.sg = slab_geom(cache, to_packed);
  cg.n_chunks = (uint32_t)n_chunks;
  cg.lr2_div = div_u32(cg.lr2);
  cg.list_grid = may_list ? list_grid(cg, stream) : 0;
  char* pk = static_cast<char*>(packed);
  hipError_t e;
  if (cg.list_grid) {
    std::lock_guard<std::mutex> lock(g_list_mu);
    uint32_t* scratch = nullptr;
    if (ListSlot* slot = take_list_slot(stream, &scratch)) {
      e = to_packed ? launch_list<true>(lp, block_table, refs, cg, scratch, pk, err, layout, elem,
                                        stream)
                    : launch_list<false>(lp, block_table, refs, cg, scratch, pk, err, layout, elem,
                                         stream);
      hipError_t er = hipEventRecord(slot->done, stream);
      if (er != hipSuccess) (void)hipStreamSynchronize(stream);  // nothing left to wait for
      return e == hipSuccess && er == hipSuccess ? KVX_OK : KVX_EHIP;
    }
    (void)hipGetLastError();  // the padded copy needs no slot
  }
  e = to_packed ? launch_chunks<true>(lp, block_table, refs, cg, pk, err, layout, elem, stream)
                : launch_chunks<false>(lp, block_table, refs, cg, pk, err, layout, elem, stream);
  return e == hipSuccess ? KVX_OK : KVX_EHIP;
}

kvx_status launch_copy_chunks(bool to_packed, const kvx_cache* cache, int32_t l0, int32_t l1,
                              const int32_t* block_table, int32_t table_len,
                              const kvx_chunk_ref* refs, int32_t n_chunks, int32_t chunk_tokens,
                              void* packed, int64_t packed_bytes, hipStream_t stream,
                              int* err) {
  return copy_chunks(false, to_packed, cache, l0, l1, block_table, table_len, refs, n_chunks,
                     chunk_tokens, packed, packed_bytes, stream, err);
}

kvx_status launch_copy_list(bool to_packed, const kvx_cache* cache, int32_t l0, int32_t l1,
                            const int32_t* block_table, int32_t table_len,
                            const kvx_chunk_ref* refs, int32_t n_chunks, int32_t chunk_tokens,
                            void* packed, int64_t packed_bytes, hipStream_t stream, int* err) {
  return copy_chunks(true, to_packed, cache, l0, l1, block_table, table_len, refs, n_chunks,
                     chunk_tokens, packed, packed_bytes, stream, err);
}

}  // namespace kvx

// ---- scatter for callers that cannot allocate --------------------------------
//
// The order entries of a destination-ordered scatter live in this fixed array
// instead of stream-ordered scratch: each GPU the library runs on holds one
// copy (kvx::kNoAllocScratchBytes) until the process ends. Host code reaches a
// device's copy only through the address hipGetSymbolAddress returns for that
// device (resolved once per device, with the device current); the array's
// name on the host is not a device address.
static __device__ __align__(256) unsigned char scratch[kvx::kNoAllocScratchBytes];

namespace {

constexpr int kScratchDevices = 64;
void* g_scratch_ptr[kScratchDevices] = {};
std::mutex g_scratch_mu;

// The calling device's copy of `scratch`, or null.
void* device_scratch() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kScratchDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
    g_scratch_ptr[dev] = p;
  }
  return g_scratch_ptr[dev];
}

}  // namespace

extern "C" kvx_status kvx_scatter_blocks_noalloc(const kvx_cache* cache, int32_t l0, int32_t l1,
                                                 const int32_t* block_table, int32_t n_blocks,
                                                 int32_t chunk_tokens, const void* src,
                                                 hipStream_t stream) {
  try {
    kvx::Geometry g;
    kvx_status st = kvx::validate(cache, l0, l1, n_blocks, chunk_tokens, true, &g);
    if (st != KVX_OK) return st;
    if (n_blocks > KVX_NOALLOC_MAX_BLOCKS) return KVX_EINVAL;
    if (g.n_units == 0) return KVX_OK;
    if (!block_table || !src || ((uintptr_t)src & 15)) return KVX_EINVAL;
    if (kvx::overlaps_cache(cache, l0, l1, src, g.packed)) return KVX_EINVAL;
    void* order = device_scratch();
    int* err = kvx::stream_error_word(stream);
    if (!order || !err) return KVX_EHIP;
    return kvx::launch_copy(false, cache, l0, l1, block_table, g, const_cast<void*>(src), stream,
                            err, order);
  } catch (...) {
    return KVX_EINTERNAL;
  }
}

