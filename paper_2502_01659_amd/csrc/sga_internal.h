// Internal declarations shared by the translation units of libsga.so (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include "sga.h"

namespace sga {

constexpr int kHeadDim = 64;          // head dimension of the tile (MFMA) kernels; the per-row
                                      // kernels also take 32, 128 and 256
constexpr int kWave = 64;             // CDNA wavefront width

// ---- split-row parameters (gather path) -----------------------------------
constexpr int kSplitThreshold = 2048; // rows with more neighbours are split
constexpr int kSplitChunk = 2048;     // target edges per chunk
constexpr int kSplitChunkMin = 256;   // ... of a call with little work in total (split_chunk)
constexpr int kMaxSplit = 64;         // at most this many chunks per row by L2 share, and ranges of an implicit global row
// ... and by edge count: a row of millions of neighbours (one global token of a long sequence
// whose tile does not qualify for the tile path) must spread over the chip, not over 64
// wavefronts (L = 4,194,304, one global token, fp16: 2.65 -> 0.8 ms)
constexpr int kMaxSplitLong = 1024;
// Keys whose K and V rows do not fit one L2 (each of the 8 XCDs has its own 4 MB): rows of at
// least kL2ChunkEdges * n neighbours are then cut into n = l2_chunks() chunks, a multiple of 8, and
// chunk c of every row runs on XCD c % 8.  A chunk of a row's sorted neighbour list covers a
// range of keys, so each L2 then serves about an n-th of K and V instead of all of it (for a
// uniformly random mask exactly that; any other mask is split the same way, only with less to
// gain).  The partial states of this finer split may take up to kL2PartialBudget bytes; a call
// that could need more keeps the coarser split by edge count.
constexpr int64_t kL2FitBytes = int64_t(3) << 20;
constexpr int64_t kL2ShareBytes = int64_t(2) << 20;       // K and V bytes per chunk and XCD aimed at
constexpr int kL2ChunkEdges = 128;
constexpr int64_t kL2PartialBudget = int64_t(64) << 20;
__host__ __device__ inline int l2_chunks(int64_t L, int32_t d, int32_t dtype) {
  const int64_t kv = 2 * L * d * (dtype == SGA_F32 ? 4 : 2);
  if (kv <= kL2FitBytes) return 0;
  int64_t n = 8 * ((kv + 8 * kL2ShareBytes - 1) / (8 * kL2ShareBytes));
  return (int)(n > kMaxSplit ? kMaxSplit : n);
}
constexpr int kMaxImplicitGlobal = 64;  // global rows the implicit non-local kernels can split
// Implicit window masks on few tiles (a short sequence, one head): a tile's key blocks are cut
// into up to kMaxWindowSplit ranges that separate wavefronts reduce to partial states, so that
// the call fills the chip.  The workspace holds the partials of up to kWindowSplitTiles
// (tile, head) pairs; larger calls have tiles enough and are not cut.
constexpr int kMaxWindowSplit = 8;
constexpr int kWindowSplitTiles = 4096;

// ---- tile path parameters -----------------------------------------------------
constexpr int kTile = 32;                 // query rows per tile = keys per block
constexpr int kCutEdges = 16384;          // tiles with fewer edges are never cut into segments
constexpr int kPairEdges = 128;           // a tile qualifies if it averages >= this many edges per block
constexpr int kProbeBlocks = 16;          // ... and a list is given up early if its first kProbeBlocks blocks
constexpr int kProbeEdges = 112;          //     average fewer than kProbeEdges edges (kPairEdges less a margin)
constexpr int kMaxTilePartials = 32768;   // partial states of split tiles per call
constexpr int kTilePartialFloats = kTile * 64 + 2 * kTile;   // o[32][64], m[32], l[32]

// Edges per unit of tile work.  Tile t owns the work items [f(t), f(t+1)) with
// f(t) = t + (edges before tile t)/S, i.e. one item plus one per multiple of S its edge range
// crosses; the first max(1, edges(t)/S) of them are the tile's segments, the rest stay idle.
// The mapping follows from row_ptr alone and needs neither a scan nor atomics.  A dense
// 32x32 block is 1024 edges: S is 32 dense blocks of fp32 MFMA work or 256 of fp16 work.
// S is a power of two (the kernels divide edge counts by it with a shift): 2^15 or 2^18 edges.
// A call with less work in total (nnz * H edges) gets shorter items, down to 2^12 or 2^15
// edges, until it has about 1024 (fp32) or 4096 (fp16) of them: otherwise a call with a few
// dense rows leaves its few long items to a handful of wavefronts while the rest of the chip
// idles.  An item of S edges takes a wavefront S / (nnz * H / 4096) of the time the whole chip
// needs for the call, and the tiles that are cut at all (rows of global tokens) are half empty,
// which doubles that.  (Microbenchmark grid, fp32, one head, a few global tokens at L = 8192:
// 0.76 -> 0.14 ms with 1024 items; the longformer mask with fp16 storage, L = 65,536, H = 8:
// 0.28 -> 0.16 ms with 4096 instead of 1024, L = 262,144, H = 4: 0.65 -> 0.32 ms.  fp32 items
// pay about 5 microseconds between the claim and the first block, as much as 3 blocks of
// matrix work: 4096 items made the global masks of the microbenchmark grid up to 1.5 times
// slower, and 8192 cost workload 2 1.4 %.)
// Edges per chunk of a split row: kSplitChunk, halved down to kSplitChunkMin while the call
// (nnz * H edges) has fewer than about 1024 such chunks, for the same reason as seg_shift.
__host__ __device__ inline int split_chunk(int64_t nnz, int32_t H) {
  int c = kSplitChunk;
  const int64_t e = (nnz < 0 ? 0 : nnz) * (int64_t)H;
  while (c > kSplitChunkMin && e / c < 1024) c >>= 1;
  return c;
}
__host__ __device__ inline int seg_shift_min(int32_t dtype) { return dtype == SGA_F32 ? 12 : 15; }
// fp32 masks that fill a sixteenth of the L x L pairs and more, at d = 64 and 128, whose average tile is
// cut at 2^15 already (kTwiceCutEdges): 2^14 where that makes fewer than 16,384 items, 2^13 where 2^14
// makes fewer than 4096, so that the 512 (d = 64: for four items each) to 1024 resident workgroups
// come out even.  No tile is cut for this: the blocks of a random mask are as thin as its fill, but those
// of a band or of block masks are full, and an item of 2^13 edges is then eight of them and one
// partial state.  16,384 items also bound the partial states, far below kMaxTilePartials (beyond
// which every cut tile would go to the per-row kernels).
// (us, 2^15 / 2^14 / 2^13, prepared, one head where not said.  Inside: random, a quarter, L = 24,576
// 982 / 895 / -, L = 10,972 394 / 330 / 260; half, L = 12,000 356 / 280 / 292; a fifth, L = 14,000
// 522 / 448 / 377; +-4,000, L = 9,000 373 / 383 / 250, d = 128 644 / 708 / 582; +-1,100, L = 14,000
// 186 / 139 / 116; +-2,000, L = 16,000, two heads 289 / 270 / 321; against it +-2,000, L = 9,000
// 175 / 216 / 240.  Outside: +-1,000, L = 20,000, two heads 179 / 241 / 235, eight heads 499 / 827 / 910;
// +-3,000, L = 65,536 720 / 757 / 31,000 (no room for the partial states); 64-token blocks, 5 to 8 per
// row, L = 11,072, eight heads 139 / - / 311; d = 256, +-600, L = 8,192 166 / - / 172.)
// kTwiceCutEdges is 2^16 less a margin for masks of random rows, whose tiles fall on both sides of their
// average (a quarter of the pairs, L = 8,192, four heads, uncut / cut 613 / 468).
constexpr int64_t kTwiceCutEdges = 65024;
__host__ __device__ inline int seg_shift(int32_t dtype, int64_t nnz, int32_t H, int64_t L, int32_t d) {
  int sh = dtype == SGA_F32 ? 15 : 18;
  const int64_t e = (nnz < 0 ? 0 : nnz) * (int64_t)H;
  const int64_t items = dtype == SGA_F32 ? 1024 : 4096;
  if (dtype == SGA_F32 && d <= 2 * kHeadDim && nnz > 0 && nnz / L >= L / 16 && nnz / L * kTile >= kTwiceCutEdges &&
      (e >> 14) < 16384)
    sh = (e >> 14) < 4096 ? 13 : 14;
  while (sh > seg_shift_min(dtype) && (e >> sh) < items) --sh;
  return sh;
}

// ---- workspace layout -------------------------------------------------------
// [0, 256)            counters (uint32): see WsCounter
// long_rows           cap_items x int4 {row, first partial slot, nchunks, chunk_len}   (gather split)
// partials            cap_items x H x kPartialStride floats {acc[d], m, l}
//                     (implicit non-local mask: kMaxImplicitGlobal rows x kMaxSplit chunks)
// items_rec           n_work x TileItem: the work items of the tile path
// tile_bad            n_tiles x int32: != 0 -> tile is left to the gather path
// bad_list            n_tiles x int32: the tiles with tile_bad != 0, in any order (kCtrTilesBad of them)
// tile_pbase          n_tiles x int32: first partial slot of a multi-segment tile
// multi_tiles         cap_tparts x {tile, first partial slot, segments, -}: the multi-segment tiles (merge list, any order)
// pair_blk            cap_pairs x int32: key block id (| full flag); tile t owns slots
//                     [row_ptr[32t]/128, row_ptr[32(t+1)]/128), split evenly among its segments
// pair_mask           cap_pairs x 32 x uint32: bit j of word r = edge (row 32t+r, key 32b+j)
// tpartials           cap_tparts x H x max(1, d / 64) x kTilePartialFloats floats
// work_next           H x uint32: claims of tile work items made so far of each head (dynamic scheduling)
enum WsCounter : int {
  kCtrChunksNeeded = 0,   // sum of chunk counts of all long rows, handing out their partial slots
  kCtrFineNeeded = 1,     // the same for the finer split (see row_split_shape); one 64-bit word with the former
  kCtrTilePartsNeeded = 3,  // sum of segment counts of all multi-segment tiles
  kCtrTilePartsAlloc = 4,   // bump allocator over tile partial slots
  kCtrTilesBad = 5,         // tiles whose block lists overflowed (left to the gather path)
  kCtrMultiTiles = 6,       // multi-segment tiles recorded in the merge list
  kCtrMultiItems = 11,      // groups of up to four segment items (see TileItem::group)
  kCtrLongestRow = 12,      // neighbours of the longest row (written when a graph is prepared)
  kCtrLengthSquares = 14,   // sum of the squares of the rows' lengths, 64 bits (likewise)
  // (the second cache line: atomics on one line wait for each other)
  kCtrLongRows = 32,        // number of long rows recorded
  kCtrMaxChunks = 34,       // most chunks any split row has (bounds the chunk kernel's unit loop), ...
  kCtrMaxChunksFine = 35,   // ... in the finer split; one 64-bit word with the former
  kNumCounters = 64
};

// One work item of the tile path, written by the CSR -> tile graph pass and read (one record,
// one load) by the attention kernel.
struct alignas(32) TileItem {
  int32_t tile;     // tile index, or -1 for an idle item
  int32_t nblk;     // key blocks in the item's list, or -1 if the list overflowed its slots
  int32_t seg;      // segment of the tile's key-block span ...
  int32_t nseg;     // ... out of this many
  int64_t slot0;    // first (tile, key block) pair slot of the list
  int64_t group;    // (no part of this item: entry of the list of groups, see tile_attend_f32_kernel)
};

struct WorkspacePlan {
  // gather split
  int64_t cap_items;
  size_t off_long, off_partials;
  // tile path
  int64_t n_tiles;        // ceil(L / 32)
  int64_t n_work;         // tile work items (segments)
  int64_t cap_pairs;      // capacity of the (tile, key block) pair arrays
  int64_t cap_tparts;     // capacity of tile partial states
  int seg_shift;          // log2 of S, the edges per work item of the tile path
  int split_chunk;        // target edges per chunk of a split row
  int l2_chunks;          // != 0: rows of >= kL2ChunkEdges * l2_chunks neighbours are cut into this many chunks
  size_t off_items_rec, off_tile_bad, off_bad_list, off_tile_pbase, off_multi_tiles, off_pair_blk, off_pair_mask,
      off_tpartials, off_work_next, off_wparts;
  int64_t cap_wparts;     // (tile, head) pairs whose window partials fit (implicit masks)
  size_t total_bytes;
};

// A row partial of the split-row path is d + 4 floats: acc[d], m, l, 2 pad.

// Sizes every region for (L, H, nnz, dtype); nnz < 0 means implicit mask (no tile lists).
// Evaluated identically on the host (sga_workspace_bytes) and inside the kernels
// (with nnz = row_ptr[L]), so no layout has to be passed around.  (force_shift: the size of a
// layout with that log2 S and the shortest row chunks instead of those the arguments select.)
__host__ __device__ inline WorkspacePlan plan_workspace(int64_t L, int32_t H, int64_t nnz,
                                                        int32_t dtype, int32_t d = kHeadDim,
                                                        int force_shift = -1) {
  WorkspacePlan p{};
  p.seg_shift = force_shift >= 0 ? force_shift : seg_shift(dtype, nnz, H, L, d);
  p.split_chunk = force_shift >= 0 ? kSplitChunkMin : split_chunk(nnz, H);
  size_t off = 256;   // counters
  const int64_t e = nnz < 0 ? 0 : nnz;
  int64_t n_long = e / (kSplitThreshold + 1);
  if (n_long > L) n_long = L;
  int64_t cap = e / p.split_chunk + n_long;
  if (cap > (int64_t)kMaxSplitLong * n_long) cap = (int64_t)kMaxSplitLong * n_long;
  p.l2_chunks = nnz < 0 ? 0 : l2_chunks(L, d, dtype);
  if (p.l2_chunks) {
    int64_t rows = e / ((int64_t)kL2ChunkEdges * p.l2_chunks);      // rows that can qualify
    if (rows > L) rows = L;
    const int64_t cap_l2 = rows * p.l2_chunks;
    if (cap_l2 * H * (d + 4) * (int64_t)sizeof(float) > kL2PartialBudget) p.l2_chunks = 0;
    else if (cap_l2 > cap) cap = cap_l2;
  }
  // implicit masks: only the dense rows of the global (non-local) mask are split
  if (nnz < 0) cap = (int64_t)kMaxImplicitGlobal * kMaxSplit;
  p.cap_items = cap;
  p.off_long = off;
  off = (off + (size_t)cap * 32 + 255) & ~size_t(255);      // (the records of the finer split follow the cap records)
  p.off_partials = off;
  off = (off + (size_t)cap * H * (d + 4) * sizeof(float) + 255) & ~size_t(255);
  // tile path
  const bool tiles = nnz >= 0;
  p.n_tiles = tiles ? (L + kTile - 1) / kTile : 0;
  p.n_work = tiles ? p.n_tiles + (e >> p.seg_shift) : 0;
  p.cap_pairs = tiles ? e / kPairEdges + 1 : 0;
  p.cap_tparts = tiles ? (e >> p.seg_shift) + 1 : 0;
  if (p.cap_tparts > kMaxTilePartials) p.cap_tparts = kMaxTilePartials;
  p.off_items_rec = off;
  off = (off + (size_t)p.n_work * sizeof(TileItem) + 255) & ~size_t(255);
  p.off_tile_bad = off;
  off = (off + (size_t)p.n_tiles * 4 + 255) & ~size_t(255);
  p.off_bad_list = off;
  off = (off + (size_t)p.n_tiles * 4 + 255) & ~size_t(255);
  p.off_tile_pbase = off;
  off = (off + (size_t)p.n_tiles * 4 + 255) & ~size_t(255);
  p.off_multi_tiles = off;
  off = (off + (size_t)p.cap_tparts * 16 + 255) & ~size_t(255);     // {tile, first partial slot, segments, -}
  p.off_pair_blk = off;
  off = (off + (size_t)p.cap_pairs * sizeof(int32_t) + 255) & ~size_t(255);
  p.off_pair_mask = off;
  off = (off + (size_t)p.cap_pairs * kTile * sizeof(uint32_t) + 255) & ~size_t(255);
  p.off_tpartials = off;
  const int64_t slices = d > kHeadDim ? d / kHeadDim : 1;   // a wide tile leaves one record per 64 channels
  off = (off + (size_t)p.cap_tparts * H * slices * kTilePartialFloats * sizeof(float) + 255) & ~size_t(255);
  p.off_work_next = off;
  off = (off + (tiles ? (size_t)H * 4 : 0) + 255) & ~size_t(255);
  // implicit window masks: partial states of cut tiles (short sequences only)
  p.cap_wparts = 0;
  if (nnz < 0 && d >= kHeadDim) {
    const int64_t pairs = ((L + kTile - 1) / kTile + 256) * H;     // (tiles of every class: + a margin) x heads
    if (pairs <= kWindowSplitTiles) p.cap_wparts = pairs;
  }
  p.off_wparts = off;
  off = (off + (size_t)p.cap_wparts * kMaxWindowSplit * slices * kTilePartialFloats * sizeof(float) + 255) &
        ~size_t(255);
  p.total_bytes = off;
  return p;
}

// Rows the per-row kernels split into chunks (partial states + ordered merge): more than
// kSplitThreshold neighbours, or enough of them for the split by L2 share (see l2_chunks).
__host__ __device__ inline bool row_is_split(int64_t deg, const WorkspacePlan& p) {
  return deg > kSplitThreshold || (p.l2_chunks && deg >= (int64_t)kL2ChunkEdges * p.l2_chunks);
}
// ... into nchunks chunks of len edges (the last one shorter), len a multiple of 32 where they are cut by edge count.
// The slots are sized for chunks of split_chunk edges with every row of the mask split; where
// the split rows hold a small part of the edges (a few dense rows beside a window), the same
// slots take chunks of kSplitChunkMin edges: the call uses this finer split (fine = true)
// if the chunks of all its rows then still fit, else the coarser one for every row.  (One
// global token at L = 65,536, 8 heads, fp32: 32 chunks of 2,048 edges per head kept 256
// wavefronts busy for 0.29 ms, each waiting for its own gathers.)
__host__ __device__ inline void row_split_shape(int64_t deg, const WorkspacePlan& p, bool fine, int32_t& nchunks,
                                                int32_t& len) {
  const int chunk = fine ? kSplitChunkMin : p.split_chunk;
  int64_t n = (deg + chunk - 1) / chunk;
  if (n > kMaxSplitLong) n = kMaxSplitLong;
  // (a row of more than kMaxSplit chunks by edge count keeps them: there are few such rows in a
  // call, and each has to spread over the chip before it can share an L2 with its neighbours)
  // By share every row has n chunks: in multiples of 32, 1,106 neighbours would be 7 chunks of 160, which leave
  // an XCD idle and shift the chunks of one row against the key ranges of the next (random 4.5 %, L = 24,576, fp32,
  // us: 648 with chunk 7 missing, 1,191 with the rows' seven in turn on all XCDs, 620 so).
  const bool by_share = n <= kMaxSplit && p.l2_chunks && deg >= (int64_t)kL2ChunkEdges * p.l2_chunks;
  if (by_share) n = p.l2_chunks;
  int64_t l = (deg + n - 1) / n;
  if (!by_share) l = (l + 31) / 32 * 32;
  len = (int32_t)l;
  nchunks = (int32_t)((deg + l - 1) / l);
}

// The XCD of chunk 0 of split row s, which has z chunks (chunk c follows c XCDs further on).  Up to four chunks would
// leave half the XCDs or more without work, so such rows take them in turn; rows of more chunks all
// start at XCD 0, where the same part of the keys stays in an L2 for every row.  (us, all rows from XCD 0 / in
// turn, 3,200 rows of L = 51,200 split, fp32, d = 64, four heads: 2 chunks 6,021 / 2,777, 3 5,428 / 4,705,
// 4 5,995 / 4,468, 5 5,173 / 7,664, 1,600 rows: 6 2,354 / 3,994, 7 2,217 / 4,983, 9 4,124 / 6,607, 12 4,151 / 5,376,
// 15 4,128 / 9,669; L = 20,000, fp16, eight heads: 2 2,180 / 1,066, 4 2,162 / 1,241, 5 2,051 / 2,796.)
constexpr int kXcdTurnChunks = 4;
__host__ __device__ inline uint32_t first_xcd(uint32_t s, int32_t z) {
  return z <= kXcdTurnChunks ? s * (uint32_t)z & 7u : 0u;
}

// fp16 windows staged in LDS: key blocks that a workgroup of 128 consecutive queries of a class of Lc tokens copies, and
// blocks that one of its 32-query sub-tiles meets
// (blocks start at the first key of the workgroup's window, or at key 0 where that cuts it).  A class holds
// ceil(Lc / 32): in 2-D dilated masks W = Lc - 1, and LDS and registers for 2W keys halved the
// workgroups per CU (L = 262,144, 4 heads, us, band kernel / sized by W / so: Lc = 130 175 / 153 / 136, 160 133 / 167 / 121,
// 192 133 / 161 / 120, 257 221 / 219 / 176).  sets: LDS blocks per key block (2: K beside V; 1: K and V in turn).  The four
// output tiles leave through the same space, 4.5 blocks.
constexpr int kStagedBlockBytes = kTile * kHeadDim * 2;
constexpr int kOutTileBytes = kTile * (kHeadDim * 2 + 16);
__host__ __device__ inline int64_t staged_blocks(int64_t W, int64_t Lc, int sets) {
  const int64_t window = (4 * kTile - 1 + 2 * W) / kTile + 1, held = (Lc + kTile - 1) / kTile;
  const int64_t out = (4 * kOutTileBytes + sets * kStagedBlockBytes - 1) / (sets * kStagedBlockBytes);
  const int64_t keys = window < held ? window : held;
  return keys < out ? out : keys;
}
__host__ __device__ inline int64_t subtile_blocks(int64_t W, int64_t Lc) {
  const int64_t window = 2 * ((W + kTile - 1) / kTile) + 1, held = (Lc + kTile - 1) / kTile;
  return window < held ? window : held;
}

// Workgroups (of four wavefronts) of a head that stride over what the tile path leaves over: about one chip-full over
// the heads, a multiple of 8 so that workgroup i runs on XCD i % 8 behind any other such number; fewer where a prepared
// graph knows that there are not so many rows (one global token, L = 1,000, fp32, d = 256, 32 heads, us: 243 -> 210).
__host__ __device__ inline int64_t leftover_workgroups(int64_t rows_left, int32_t H) {
  const int64_t rows = (rows_left + 3) / 4, full = 2048 / H > 256 ? 2048 / H : 256;
  return ((rows < full ? rows : full) + 7) & ~int64_t(7);
}

// Calls on a prepared graph of even rows (no tile, none split, none longer than twice the average and 64 neighbours, at most
// 256 on average) that gather_even_rows_kernel takes: K and V of a head beyond one L2 and rows for four wavefronts per SIMD
// (fp32, d = 64).  Longer rows gain nothing (3 %, L = 16,000: fp32, d = 64 183 / 182, fp16, d = 128 194.6 / 198.4).
// The lengths vary no more than evenly spread ones do (a variance of a third of the squared average; random neighbours add
// the average), since a wavefront stays until the longest of its rows ends and a small call until its longest row does:
// rows of 0.05 and of 1.95 times the average, 64 of each in turn, average 128, L = 16,500, fp32, d = 64 68 / 87,
// d = 128 139 / 200, average 245 208 / 353.
// (us, a wavefront per row / that.  Equal lengths, average 35, fp32, d = 64, L = 8,192, two heads 25.8 / 19.5, L = 24,576
// 48.7 / 43.7, L = 100,000 236 / 234; random neighbours, average 70, L = 24,576, fp32, d = 64 88 / 77, d = 128 206 / 195, fp16,
// d = 128 88 / 77, d = 256 206 / 195; L = 100,000, in that order 462 / 456, 974 / 943, 462 / 458, 963 / 946.  Lengths between 0.4 and
// 1.6 times the average, fp32, d = 64: average 70, L = 35,000 143 / 136; average 245, L = 8,192, two heads, where the longest
// rows decide 98 / 110.)
inline bool rows_of_one_length(int64_t nnz, int64_t L, int64_t longest, uint64_t squares) {
  const double mean = (double)nnz / (double)L;
  return nnz / L <= 256 && longest <= 2 * (nnz / L) + 64 && (double)squares / (double)L <= mean * mean * 4.0 / 3.0 + mean;
}
inline bool even_rows(int64_t L, int32_t H, int32_t d, int32_t dtype) {
  const int64_t bytes = L * d * (dtype == SGA_F32 ? 4 : 2);
  return L * H >= 16384 && 2 * bytes > kL2FitBytes && bytes < int64_t(1) << 32;      // (32-bit offsets)
}

// The finer split is taken if all its chunks fit (ctr: the counters of the workspace).
__host__ __device__ inline bool split_is_fine(const WorkspacePlan& p, const uint32_t* ctr) {
  return (int64_t)ctr[kCtrFineNeeded] <= p.cap_items;
}

// Which calls run shared_chunk_kernel: those of dense enough random rows.  The host asks whether the mask may be one
// (shared_chunks_possible), the chunk kernels of such a call then look at the mask itself (shared_chunks); a plan knows.
// Where rows are cut by L2 share the other kernel reads K and V from its XCD's L2, and the line lies at an 18th of
// the pairs for fp32 (us, that / this kernel, L = 24,576, d = 64: 4.5 % 620 / 651, 5 % 627 / 625, 5.5 % 675 / 655,
// 10 % 1,287 / 880; L = 12,001, 10 % 317 / 259; d = 128, L = 13,001, 10 % 668 / 603); fp16 stays there (L = 24,576,
// d = 64, 10 % 765 / 880; d = 128, L = 13,001, 8 % 393 / 480).  Where the partial states of that split have no room,
// this kernel is the faster one down to a 25th for fp16 and below a 30th for fp32 (fp32 / fp16, d = 64, two heads,
// L = 24,576, 10 % 4,700 -> 1,535 / 1,909 -> 1,611; one head, L = 44,001, 5 % 3,975 -> 1,949 / 2,560 -> 1,999; L = 65,001,
// 3.4 % 6,947 -> 3,313 / 3,825 -> 3,900; d = 128, L = 24,576, 10 % 4,971 -> 1,627 / 2,844 -> 1,360); with fewer edges
// to a step the sums lose accuracy (L = 90,001, 2.5 %, fp32: 3.7e-7 against 3.4e-7).
// A unit of it (a chunk of 64 rows and a head) is a workgroup's work of 100 to 250 us, and few of them leave the chip idle
// where the other kernel has a wavefront per chunk.  Rows of 10 % below window rows, prepared, us, that / this kernel by the
// share of its places that the units fill.  Chunks of 2,048 edges (two a row): fp32, d = 64, a quarter 642 / 599, 3/8
// 476 / 476, a half 588 / 483 and 1,125 / 615; d = 128, all 4,095 / 1,445; fp16, d = 64, a quarter 409 / 544, a half
// 387 / 442 and 716 / 570, all 678 / 659; d = 128, all 686 / 590.  The finer split of a few rows, ten chunks and more, each on
// its XCD: fp32, d = 64, 0.8 328 / 341, 1.25 457 / 390; d = 128, 5 1,724 / 1,265; fp16 0.8 199 / 289, 1.25 272 / 325, d = 128,
// 2.5 450 / 483.
constexpr int64_t kSharedMaxKeys = int64_t(1) << 16;
constexpr uint32_t kSharedMinRows = 2048;
constexpr int64_t kSharedFillByShare = 18;
constexpr int kSharedRows = 64;          // rows of a workgroup
__host__ __device__ constexpr int64_t shared_fill(int32_t dtype) { return dtype == SGA_F32 ? 30 : 25; }
__host__ __device__ constexpr unsigned shared_places(int32_t d) { return d == 64 ? 512 : 256; }   // workgroups that the chip holds
__host__ __device__ inline bool shared_chunks(const WorkspacePlan& pl, int64_t nnz, int64_t L, int32_t H, int32_t d,
                                              int32_t dtype, const uint32_t* ctr) {
  const bool fine = split_is_fine(pl, ctr), finer = fine && !pl.l2_chunks;      // (by L2 share both splits are one)
  if ((pl.l2_chunks || finer) && dtype == SGA_F16) return false;
  const int64_t chunks = (int64_t)ctr[fine ? kCtrFineNeeded : kCtrChunksNeeded] * H;
  return ctr[fine ? kCtrMaxChunksFine : kCtrMaxChunks] <= (uint32_t)kMaxSplit && ctr[kCtrLongRows] >= kSharedMinRows &&
         chunks * (dtype == SGA_F32 && !finer ? 4 : 1) >= (int64_t)kSharedRows * shared_places(d) &&
         nnz / L >= L / (pl.l2_chunks ? kSharedFillByShare : shared_fill(dtype));
}
// False where no mask that this workspace was sized for can take shared_chunks: an empty launch costs a
// small call 2 us.  The fewest edges that can are, with the split by L2 share, those of its line (fp32 only), and
// without it those of the other line or the first for which that split has no room; every workspace of
// sga_workspace_bytes for such a mask, or larger, answers true.
inline bool shared_chunks_possible(int64_t L, int32_t H, int32_t d, int32_t dtype, size_t ws_bytes) {
  const int n = l2_chunks(L, d, dtype);
  if (!(d == 64 || d == 128) || L > kSharedMaxKeys || n == 0) return false;
  auto room = [&](int64_t nnz, bool by_share) {
    const WorkspacePlan p = plan_workspace(L, H, nnz, dtype, d, seg_shift_min(dtype));
    return (p.l2_chunks != 0) == by_share && p.total_bytes <= ws_bytes;
  };
  if (dtype == SGA_F32 && room(L * (L / kSharedFillByShare), true)) return true;
  const int64_t rows = kL2PartialBudget / ((int64_t)n * H * (d + 4) * (int64_t)sizeof(float)) + 1;
  const int64_t without = rows * kL2ChunkEdges * n, least = L * (L / shared_fill(dtype));
  return rows <= L && room(without > least ? without : least, false);
}

// ... and over the chunks of its split rows: two rounds of the 1,024 that the chip holds of leftovers_kernel
__host__ __device__ inline int64_t leftover_chunk_workgroups(int32_t H) {
  const int64_t full = 2048 / H > 128 ? 2048 / H : 128;
  return (full + 7) & ~int64_t(7);
}

// First work item of tile t: f(t) = t + row_ptr[min(32t, L)] / S.
__device__ __forceinline__ int64_t work_first(const int64_t* __restrict__ row_ptr, int64_t L,
                                              int sh, int64_t t) {
  const int64_t r = t * kTile;
  return t + (row_ptr[r < L ? r : L] >> sh);
}

// Segments tile t is cut into: max(1, edges(t) / S); a tile below kCutEdges edges (every tile of
// a window mask up to +-255) stays whole also where a small call has S below that.
//
// Four neighbouring tiles 4g .. 4g+3 of similar size (the largest at most twice the smallest) are
// cut into the same number of segments, so that segment s of the four covers the same range of keys:
// four consecutive work items, starting at a multiple of four, hold the same segment of the four
// tiles, and a workgroup streams or shares the key blocks of one range.  Of the items the four
// own, [f(4g), f(4g+4)), item first + 4 s + i then is segment s of tile 4g + i and the others are idle.
struct TileCut {
  int32_t nseg;
  bool together;       // the four tiles are cut alike
  int64_t first;       // ... and this is their first item (nseg > 1 only)
};
__device__ __forceinline__ TileCut tile_cut(const int64_t* __restrict__ row_ptr, int64_t L, int sh, int64_t t) {
  const int64_t g = t & ~int64_t(3);
  int64_t r[5];
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    const int64_t row = (g + i) * kTile;
    r[i] = row_ptr[row < L ? row : L];
  }
  int64_t least = r[1] - r[0], most = least, own = least;
#pragma unroll
  for (int i = 1; i < 4; ++i) {
    const int64_t e = r[i + 1] - r[i];
    least = e < least ? e : least;
    most = e > most ? e : most;
    if (t - g == i) own = e;
  }
  TileCut cut{1, false, 0};
  if ((g + 3) * kTile < L && 2 * least >= most) {
    cut.together = true;
    cut.first = (g + (r[0] >> sh) + 3) & ~int64_t(3);
    const int64_t room = (((g + 4 + (r[4] >> sh)) & ~int64_t(3)) - cut.first) / 4;
    int64_t n = ((r[4] - r[0]) >> 2) >> sh;
    n = n < room ? n : room;
    if (n > 1 && most >= kCutEdges) cut.nseg = (int32_t)n;
  } else {
    const int64_t n = own >> sh;
    if (n > 1 && own >= kCutEdges) cut.nseg = (int32_t)n;
  }
  return cut;
}
__device__ __forceinline__ int32_t tile_segments(const int64_t* __restrict__ row_ptr, int64_t L, int sh, int64_t t) {
  return tile_cut(row_ptr, L, sh, t).nseg;
}

// True when the tile path of this call produces the rows of tile t: its block lists fitted
// their slots and, if it is a multi-segment tile, the call's partial states fitted theirs.
__device__ __forceinline__ bool tile_handled(const WorkspacePlan& pl, const void* ws,
                                             const int64_t* __restrict__ row_ptr, int64_t L, int64_t t) {
  const char* base = static_cast<const char*>(ws);
  if (reinterpret_cast<const int32_t*>(base + pl.off_tile_bad)[t] != 0) return false;
  if (tile_segments(row_ptr, L, pl.seg_shift, t) == 1) return true;
  return (int64_t) reinterpret_cast<const uint32_t*>(ws)[kCtrTilePartsNeeded] <= pl.cap_tparts;
}

// True when the tile path of this call left no row to the gather path.
__device__ __forceinline__ bool tiles_cover_everything(const WorkspacePlan& pl, const void* ws) {
  const uint32_t* ctr = reinterpret_cast<const uint32_t*>(ws);
  return ctr[kCtrTilesBad] == 0 && (int64_t)ctr[kCtrTilePartsNeeded] <= pl.cap_tparts;
}

// The per-row path's preparation of a wavefront's rows (lane: row i, if mine): those that are split reserve their
// partial slots and enter the list of long rows.  All lanes call it.  Atomics on one counter follow each other
// 12 ns apart whatever they come from, so a wavefront issues two, and two more where it raises a maximum (24,576
// split rows, the CSR -> tile pass, us: none recorded 28, seven atomics per wavefront 89, so 60).
__device__ __forceinline__ void record_split_rows(const int64_t* __restrict__ row_ptr, int64_t i, bool mine,
                                                  const WorkspacePlan& pl, void* ws) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t deg = mine ? row_ptr[i + 1] - row_ptr[i] : 0;
  int32_t n = 0, len = 0, nf = 0, lenf = 0;
  if (row_is_split(deg, pl)) {
    row_split_shape(deg, pl, false, n, len);
    row_split_shape(deg, pl, true, nf, lenf);
    if (nf <= n) {
      nf = n;
      lenf = len;
    }
  }
  if (!__any(n > 0)) return;
  int32_t sum = n, sumf = nf, most = n, mostf = nf;      // up to this lane
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int32_t t = __shfl_up(sum, off, kWave), tf = __shfl_up(sumf, off, kWave);
    const int32_t u = __shfl_up(most, off, kWave), uf = __shfl_up(mostf, off, kWave);
    if (lane >= off) {
      sum += t;
      sumf += tf;
      most = max(most, u);
      mostf = max(mostf, uf);
    }
  }
  uint32_t* ctr = reinterpret_cast<uint32_t*>(ws);
  uint32_t base = 0, basef = 0, slot = 0;
  if (lane == kWave - 1) {
    const unsigned long long both = atomicAdd(reinterpret_cast<unsigned long long*>(&ctr[kCtrChunksNeeded]),
                                              (unsigned long long)(uint32_t)sumf << 32 | (uint32_t)sum);
    base = (uint32_t)both;
    basef = (uint32_t)(both >> 32);
    const unsigned long long seen = __hip_atomic_load(reinterpret_cast<unsigned long long*>(&ctr[kCtrMaxChunks]),
                                                      __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((uint32_t)seen < (uint32_t)most) atomicMax(&ctr[kCtrMaxChunks], (uint32_t)most);
    if ((uint32_t)(seen >> 32) < (uint32_t)mostf) atomicMax(&ctr[kCtrMaxChunksFine], (uint32_t)mostf);
  }
  base = __shfl(base, kWave - 1, kWave) + (uint32_t)(sum - n);
  basef = __shfl(basef, kWave - 1, kWave) + (uint32_t)(sumf - nf);
  const bool fits = n > 0 && (int64_t)base + n <= pl.cap_items;
  const uint64_t all = __ballot(fits);
  if (lane == 0) slot = atomicAdd(&ctr[kCtrLongRows], (uint32_t)__popcll(all));
  slot = __shfl(slot, 0, kWave) + (uint32_t)__popcll(all & ((uint64_t(1) << lane) - 1));
  if (!fits) return;
  int4* lr = reinterpret_cast<int4*>(static_cast<char*>(ws) + pl.off_long);
  lr[slot] = make_int4((int)i, (int)base, n, len);
  // (read only if the finer chunks of every row fit, and then basef + nf <= cap_items)
  lr[pl.cap_items + slot] = make_int4((int)i, (int)basef, nf, lenf);
}

// The split rows that the tile path leaves over are recorded by the CSR -> tile pass where it gives a tile
// up.  Whether the partial states of the multi-segment tiles fit is known only after it: they do
// unless the call has more edges than kMaxTilePartials items hold, and such a call records its rows in a
// launch of its own behind that pass (split_prepass_kernel).
__host__ __device__ inline bool tile_parts_in_doubt(const WorkspacePlan& p) { return p.cap_tparts >= kMaxTilePartials; }
// What the host can tell of a call whose edge count it does not know: that many edges make items of the
// longest kind, whatever L, H and d, and a workspace that holds their pair lists.
inline bool tile_parts_may_be_in_doubt(int32_t dtype, size_t ws_bytes) {
  const size_t least = size_t(kMaxTilePartials - 1) << (dtype == SGA_F32 ? 15 : 18);
  return ws_bytes >= least / kPairEdges * (sizeof(int32_t) + kTile * sizeof(uint32_t));
}

template <typename T> struct DtypeOf;
template <> struct DtypeOf<float> { static constexpr int32_t code = SGA_F32; };
template <> struct DtypeOf<__half> { static constexpr int32_t code = SGA_F16; };

struct AttnArgs {
  const void* Q;
  const void* K;
  const void* V;
  void* O;
  float* lse;
  int64_t L;
  int32_t H;
  float scale;
  int32_t dtype;
  int32_t d;           // head dimension
  hipStream_t stream;
  // explicit
  const int64_t* row_ptr;
  const int32_t* col_idx;
  // implicit (window family): neighbours j = i + stride*k, |k| <= window
  int32_t window;
  int32_t stride;
  int32_t mask_kind;   // implicit: sga_mask_kind
  int32_t n_global;    // implicit non-local mask
  int32_t block;       // implicit 2-D dilated mask
  // continue from the (O, lse) state already in the output buffers instead of overwriting it
  bool accumulate;
  // fp32 storage: products as three fp16 matrix-core terms instead of fp32 MFMA (tile path)
  bool split;
  // implicit non-local mask: the tile kernels may be used (the caller did not ask for the
  // per-row kernels)
  bool tiles_allowed;
  // workspace
  void* ws;
  size_t ws_bytes;
  // prepared graph (sga_graph_prepare): the workspace already holds the tile graph and the
  // chunk items of the split rows, and the host knows what they contain
  bool prepared;
  uint32_t plan_multi_tiles;   // multi-segment tiles whose partial states fit (0: no merge launch)
  bool plan_tiles_cover_all;   // no row is left to the per-row kernels
  int64_t plan_rows_left;      // at most so many rows are left to the per-row kernels
  bool plan_no_tiles;          // no tile qualified: the tile kernels have nothing to do
  uint32_t plan_long_rows;     // split rows among the leftover rows whose chunk items fit
  bool plan_rows_even;         // every row is left to them, none is split and all are of about one length
  bool plan_rows_share;        // ... and shared_chunk_kernel computes them
};

// Global -> LDS copy of 16 bytes per lane without passing through registers: lane l's 16 bytes
// land at dst + 16*l (dst is wave-uniform).  Completion is tracked by vmcnt.
__device__ __forceinline__ void copy16_to_lds(const void* src, char* dst) {
  __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)src,
                                   (void __attribute__((address_space(3)))*)dst, 16, 0, 0);
}
// copy16_to_lds issued behind the compiler's back.  While it knows of copies in flight, the
// compiler waits for all of them before any LDS read it cannot prove to be elsewhere; the
// caller of this one orders the reads itself, by counted waits.
__device__ __forceinline__ void copy16_to_lds_untracked(const void* src, char* dst) {
  const uint32_t at = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(char __attribute__((address_space(3)))*)dst);
  uint32_t m0_kept;    // (M0 holds the LDS address of the copy; the compiler's own value is put back)
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, off\n\t"
               "s_mov_b32 m0, %0"
               : "=&s"(m0_kept) : "s"(at), "v"(src) : "memory");
}

// gather path (attention_gather.hip)
// Zeroes the counters (and, when row_ptr is given, the per-tile flags of the tile path).
void clear_workspace(const AttnArgs& a, bool tile_flags);
// skip_tiled: rows whose 32-row tile was produced by the tile path (tile_bad == 0 in the
// workspace) are skipped, and a small grid strides over the rows; without a prepared graph the same
// launch merges the tiles' segments.
void launch_row_lengths(const AttnArgs& a);
sga_status launch_gather_explicit(const AttnArgs& a, bool allow_split, bool skip_tiled);
sga_status launch_gather_implicit(const AttnArgs& a);

// tile path (attention_tile.hip)
sga_status launch_tile_explicit(const AttnArgs& a);
// CSR -> tile graph pass alone (sga_graph_prepare); a.ws holds a full workspace
void launch_tile_analyze(const AttnArgs& a);
// records the split rows that this pass has not (after_tiles), or all of a call without tiles
void launch_split_prepass(const AttnArgs& a, bool after_tiles);
sga_status launch_tile_implicit(const AttnArgs& a);
// Implicit non-local mask on the tile kernels (d = 64, 128, 256): the rows >= g against the global keys,
// and the partial states of the g global rows over *n_chunks ranges of the key blocks, in the
// layout nonlocal_merge_kernel reads (the caller launches that merge).
void launch_tile_nonlocal(const AttnArgs& a, int64_t g, float* partials, int32_t* n_chunks);

// mask builder (mask_builder.hip)
sga_status mask_validate(const sga_mask_desc* d);
int64_t mask_total_edges(const sga_mask_desc& d);
sga_status launch_build_mask(const sga_mask_desc& d, int64_t* row_ptr, int32_t* col_idx,
                             hipStream_t stream);
// Enqueues the checks of sga_validate_csr; verdict[0] and verdict[1] (uint64) end as the smallest bad row
// found in the row offsets and in the columns, or ~0.
sga_status launch_validate_csr(const int64_t* row_ptr, const int32_t* col_idx, int64_t L, int64_t col_capacity,
                               unsigned long long* verdict, hipStream_t stream);

// Benchmark hook (api.hip): when enabled, brackets the dominant attention kernel of a forward
// call with a pair of events on the call's stream.
void profile_mark_begin(hipStream_t stream, const char* kernel);
void profile_mark_end(hipStream_t stream);

// Sequential composition on one shared state (Section V-F runs a local, a global and a CSR
// kernel one after another on the same O, l, m of Algorithm 1).  The state handed from call to
// call is the normalised O_i and lse_i = m_i + ln l_i of the edges visited so far (the two
// statistics only ever enter the recurrence through this sum).  Given the earlier state and the
// (O, lse) of the edges this call visited, the continued state is
//   lse' = ln(e^lse_prev + e^lse_now),  O' = w_prev O_prev + w_now O_now,  w_x = e^(lse_x - lse').
struct CarryWeights {
  float w_prev, w_now, lse;
};
__device__ __forceinline__ CarryWeights carry_weights(float lse_prev, float lse_now) {
  const float M = fmaxf(lse_prev, lse_now);
  if (!(M > -INFINITY)) return {0.f, 0.f, -INFINITY};     // no edge visited so far
  constexpr float kLog2eC = 1.4426950408889634f, kLn2C = 0.6931471805599453f;
  const float a = __builtin_amdgcn_exp2f((lse_prev - M) * kLog2eC);
  const float b = __builtin_amdgcn_exp2f((lse_now - M) * kLog2eC);
  const float inv = 1.0f / (a + b);
  return {a * inv, b * inv, M + __builtin_amdgcn_logf(a + b) * kLn2C};
}

inline sga_status hip_status(hipError_t e) { return e == hipSuccess ? SGA_OK : SGA_ERR_HIP; }

}  // namespace sga
