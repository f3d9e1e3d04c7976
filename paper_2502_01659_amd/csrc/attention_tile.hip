// Tile path of Algorithm 1: 32 query rows x 32 keys per MFMA tile.
//
// The graph is regrouped into a "tile graph": for every tile of 32 consecutive query rows,
// the sorted list of 32-key blocks that hold at least one of its edges, each with a 32x32
// bit mask (word r, bit j = edge between row 32t+r and key 32b+j).  Explicit CSR masks are
// converted on the device by tile_analyze_kernel into workspace slots derived from row_ptr
// alone (no scan, no host round trip); window masks generate the same lists by index
// arithmetic inside the attention kernel (implicit Get_Neighbors).
//
// One wavefront owns one tile and walks its block list.  Per block it computes, on the
// matrix cores,
//     S^T[key][query] = K_blk Q_tile^T                       (SDDMM restricted to the block)
//     O^T[chan][query] += V_blk^T P^T                        (SpMM)
// with the online-softmax recurrence of Algorithm 1 applied per block instead of per key.
// Both products are laid out transposed so that a lane always owns one query (lane % 32):
// the running max m, the running sum l, the rescale factor and the mask word of a query
// live in that query's lanes and no cross-lane traffic is needed except one exchange
// between the two half-waves per block.  Entries outside the mask are set to -inf before
// the softmax, so they contribute exactly 0; blocks whose 1024 bits are all set skip the
// masking.
//
// fp32 storage splits its operands into 16-bit parts whose products the 16-bit matrix cores sum
// in fp32 (see SplitOperand; v_mfma_f32_32x32x2_f32 only where a tile holds an
// infinity or numbers near the smallest), fp16 storage uses v_mfma_f32_32x32x16_f16 with fp32 accumulation; P is rounded
// to fp16 only as the MFMA operand, l is summed in fp32.
//
// Tiles with many edges (global-token rows) are cut into segments of their key-block span;
// each segment is one more work item of the same launches, leaves a partial (m, l, acc)
// state, and tile_merge_kernel combines the partials in segment order (deterministic).
// Window masks on short sequences (few tiles, many key blocks each) are cut the same way by a
// host rule, into ranges of key blocks whose partial states window_merge_kernel combines.
#include "sga_internal.h"
#include "tile_merge.h"

#include <type_traits>

namespace sga {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef short short4v __attribute__((ext_vector_type(4)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kMinusHuge = -1.0e30f;
constexpr int kFullBit = 1 << 30;
constexpr int kBitmapBlocks = 32;   // key blocks per window of the CSR -> tile pass's bitmap walk
constexpr int kScoutColumns = 1024;  // longest rows that the CSR -> tile pass compares with the first of their tile, ...
constexpr int kScoutRuns = 8;        // ... and most runs of consecutive columns they may have
constexpr int kBitmapAfter = 4;     // ... which takes over after this many blocks if all but one had scattered columns
constexpr int kBitmapUnits = 2;     // ... each lane taking this many units of 16 columns at a time

// Key (within a 32-key block) held in accumulator register r of half-wave h after an
// MFMA 32x32 whose M index is the key: rows 8*(r/4) + 4*h + r%4.
__device__ __forceinline__ constexpr int acc_row(int r, int h) { return 8 * (r / 4) + 4 * h + (r % 4); }

// copy16_to_lds with 4 bytes per lane: lane l's word lands at dst + 4*l.
__device__ __forceinline__ void copy4_to_lds(const void* src, char* dst) {
  __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)src,
                                   (void __attribute__((address_space(3)))*)dst, 4, 0, 0);
}

// s_waitcnt vmcnt(N): all but the N most recently issued vector memory operations (global
// loads, LDS copies included) have completed.  The 6-bit count sits in bits 3:0 and 15:14.
template <int N>
__device__ __forceinline__ void wait_loads_except() {
  static_assert(N >= 0 && N <= 63, "vmcnt immediate");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// Wait ahead of the reads of a staged V block: with further copies behind it (more), all but
// the kKeepMore most recently issued vector memory operations must have completed; without, all
// of them.  kKeepMore = -1: the block is known to be complete, no wait.
template <int kKeepMore>
__device__ __forceinline__ void wait_staged_v(bool more) {
  static_assert(kKeepMore >= -1 && kKeepMore <= 63, "a count the vmcnt field can hold, or -1");
  if constexpr (kKeepMore >= 0) {
    if (more) wait_loads_except<kKeepMore>(); else wait_loads_except<0>();
  }
}

// K-ready wait of the LDS pipelines: the K copies of block k are older than the kCopies V copies
// and, if a block record was requested after them, its kGetLoads loads.
template <int kCopies, int kGetLoads>
__device__ __forceinline__ void wait_k_block(bool record_requested) {
  if (kGetLoads > 0 && record_requested) wait_loads_except<kCopies + kGetLoads>();
  else wait_loads_except<kCopies>();
}

// The value held by the lane 32 positions away (the same query in the other half-wave), by the
// gfx950 half-wave swap: one vector instruction instead of a round trip through the LDS
// permute network.  h = lane / 32.
__device__ __forceinline__ float other_half(float x, int h) {
  const unsigned xi = __builtin_bit_cast(unsigned, x);
  const auto r = __builtin_amdgcn_permlane32_swap(xi, xi, false, false);
  return __builtin_bit_cast(float, h ? r[0] : r[1]);
}

// s_waitcnt lgkmcnt(0): every LDS read issued so far has returned its data.
__device__ __forceinline__ void wait_lds_reads() { __builtin_amdgcn_s_waitcnt(0xC07F); }

// K/V pipelines of the tile kernels (template parameter kPipe).
constexpr int kPipeRegK = 0;   // K fragment prefetched into registers, V block staged in LDS
constexpr int kPipeLdsK = 1;   // K and V blocks staged in LDS, one block ahead
constexpr int kPipeSplit = 2;  // fp32 storage, products as three fp16 matrix-core terms (CoreSplit)

struct BlockInfo {   // (no padding bytes: copies of the struct stay in registers)
  int64_t row0;     // tensor row of the block's first key (wave-uniform)
  int raw;          // explicit masks: block record as loaded (row0, nvalid, full follow from it)
  int nvalid;       // keys of the block that exist (1..32); others are masked off (wave-uniform)
  uint32_t word;    // mask bits of this lane's query against the block's 32 keys
  int full;         // non-zero: all 32x32 bits set (wave-uniform)
};

__device__ __forceinline__ int64_t uniform64(int64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Block list of an explicit tile, as written by tile_analyze_kernel.
struct ExplicitBlocks {
  const int32_t* blk;
  const uint32_t* mask;
  int64_t L;
  static constexpr int kGetLoads = 2;   // vector memory loads issued by one get()
  __device__ int64_t key_stride() const { return 1; }
  // get() only issues the loads (two blocks ahead of their use); resolve() turns the loaded
  // record into wave-uniform values once the block is about to be staged, so that the loads are
  // not waited for early.
  __device__ BlockInfo get(int k, int n) const {
    BlockInfo b;
    b.raw = blk[k];
    b.word = mask[(int64_t)k * kTile + n];
    return b;
  }
  __device__ void resolve(BlockInfo& b) const {
    const int id = __builtin_amdgcn_readfirstlane(b.raw);
    b.full = (id & kFullBit) != 0;
    b.row0 = (int64_t)(id & ~kFullBit) * kTile;
    const int64_t left = L - b.row0;
    b.nvalid = left < kTile ? (int)left : kTile;
  }
  // resolve() for a block that is not the last of its list: lists ascend, so only the last
  // block of a list can be the one the end of the sequence cuts short.
  __device__ void resolve_whole(BlockInfo& b) const {
    const int id = __builtin_amdgcn_readfirstlane(b.raw);
    b.full = (id & kFullBit) != 0;
    b.row0 = (int64_t)(id & ~kFullBit) * kTile;
    b.nvalid = kTile;
  }
  // Block k without its mask word, read through the scalar (constant) path: the list is only
  // written by an earlier kernel, and a scalar load neither occupies a vector register nor counts
  // among the vector memory operations, so the pipelines' counted waits stay exact.
  // (like get(), this only issues the load; resolve() completes the record)
  __device__ BlockInfo block(int k) const {
    BlockInfo b;
    b.raw = ((const int32_t __attribute__((address_space(4)))*)blk)[k];
    b.word = ~0u;
    return b;
  }
};

// Block list of a window tile in one residue class p of stride s: queries u0..u0+31 and keys
// v of the class (token = s*index + p), edge iff |u - v| <= W.  Everything but the lane's mask
// word is wave-uniform and is computed from differences that fit 32 bits.
struct WindowBlocks {
  int64_t vfirst, Lc, s, p, u0, W;   // blocks start at the tile's first key, not at multiples of 32
  static constexpr int kGetLoads = 0;
  __device__ int64_t key_stride() const { return s; }
  __device__ static int clamp64(int64_t v) { return v < -64 ? -64 : (v > 64 ? 64 : (int)v); }
  __device__ void resolve(BlockInfo&) const {}
  // Where block k lies (wave-uniform; no mask word): what the staging needs.
  __device__ BlockInfo place(int k) const {
    BlockInfo b;
    b.raw = 0;
    const int64_t v0 = vfirst + (int64_t)k * kTile;
    b.row0 = s * v0 + p;
    const int64_t left = Lc - v0;
    b.nvalid = left < kTile ? (int)left : kTile;
    b.word = 0;
    b.full = 0;
    return b;
  }
  // Block k against the tile's queries, from wave-uniform quantities alone: 0 = no query of the
  // tile sees a key of the block, 2 = every query sees every key, 1 = anything else (get() then
  // gives the lanes' mask words).  Interior blocks of a wide window are all 2 and cost no
  // per-lane arithmetic.
  __device__ int classify(int k) const {
    const int64_t v0 = vfirst + (int64_t)k * kTile;
    const int64_t left = Lc - v0, nq = Lc - u0;
    const int64_t dlo = u0 - W - v0, dhi = u0 + W - v0;
    if (left <= 0 || nq <= 0 || dhi + (kTile - 1) < 0 || dlo > kTile - 1) return 0;
    return left >= kTile && nq >= kTile && dlo + (kTile - 1) <= 0 && dhi >= kTile - 1 ? 2 : 1;
  }
  __device__ BlockInfo get(int k, int n) const {
    BlockInfo b;
    b.raw = 0;
    const int64_t v0 = vfirst + (int64_t)k * kTile;
    b.row0 = s * v0 + p;
    const int64_t left = Lc - v0;
    b.nvalid = left < kTile ? (int)left : kTile;
    // query n sees the keys [n + dlo, n + dhi] of the block, clipped to the keys that exist
    const int dlo = clamp64(u0 - W - v0), dhi = clamp64(u0 + W - v0);
    const int nq = clamp64(Lc - u0);               // queries of the tile that exist
    int lo = n + dlo, hi = n + dhi;
    lo = lo < 0 ? 0 : lo;
    hi = hi > b.nvalid - 1 ? b.nvalid - 1 : hi;
    b.word = (lo > hi || n >= nq) ? 0u : ((~0u >> (31 - hi)) & (~0u << lo));
    // every query of the tile sees every key of the block
    b.full = b.nvalid == kTile && nq >= kTile && dlo + (kTile - 1) <= 0 && dhi >= kTile - 1;
    return b;
  }
};

// The mask words of WindowBlocks for a tile whose keys all lie within a few hundred positions of
// its first key (the workgroup-staged kernel): the same quantities as 32-bit differences, so the
// per-block arithmetic runs on the scalar unit.  d0 = u0 - vfirst, rem = min(Lc - vfirst, 2^20),
// nq = queries of the tile that exist (clamped to 64).
struct WindowWordsNear {
  int d0, W, nq, rem;
  __device__ static int clamp(int v) { return v < -64 ? -64 : (v > 64 ? 64 : v); }
  __device__ BlockInfo get(int k, int n) const {
    BlockInfo b;
    b.raw = 0;
    b.row0 = 0;                                    // (not used: the blocks are staged by the workgroup)
    const int v0 = k * kTile;                      // first key of the block, relative to vfirst
    const int left = rem - v0;
    b.nvalid = left < kTile ? left : kTile;
    const int dlo = clamp(d0 - W - v0), dhi = clamp(d0 + W - v0);
    int lo = n + dlo, hi = n + dhi;
    lo = lo < 0 ? 0 : lo;
    hi = hi > b.nvalid - 1 ? b.nvalid - 1 : hi;
    b.word = (lo > hi || n >= nq) ? 0u : ((~0u >> (31 - hi)) & (~0u << lo));
    b.full = b.nvalid == kTile && nq >= kTile && dlo + (kTile - 1) <= 0 && dhi >= kTile - 1;
    return b;
  }
};

// Per-lane running state: lane owns query n = lane % 32; channels of O^T are spread over the
// 16 accumulator registers of both 32-channel halves.
struct TileState {
  float m;          // running max (log2 domain), identical in both half-waves
  float l;          // running sum of this half-wave's keys
  floatx16 o[2];    // o[cb][r]: channel cb*32 + acc_row(r, h), un-normalised
  __device__ void init() {
    m = kMinusHuge;
    l = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) { o[0][r] = 0.f; o[1][r] = 0.f; }
  }
};

// The running max m of Algorithm 1 only has to bound the scores for the exponentials to stay
// finite, so it is raised lazily: a block moves m (and rescales l and O) only when its largest
// score exceeds m by more than kRescaleSlack (log2 units).  Softmax numerators are then at most
// 2^kRescaleSlack, well inside fp16/fp32 range, and the quotient acc/l is unchanged.
constexpr float kRescaleSlack = 8.0f;

// c = |scale| * log2(e) of p = 2^(c*s - m).  A zero scale (uniform weights over the neighbours)
// is replaced by 2^-100: every finite product then scales to 0 within rounding, while the -inf of
// a masked entry stays -inf instead of turning into 0 * inf.
__device__ __forceinline__ float softmax_factor(float scale) {
  const float c = __builtin_fabsf(scale) * kLog2e;
  return c > 0.f ? c : 7.888609052210118e-31f;
}

// Mask, running max/sum update and (rare) rescale for one block.  sv: raw dot products of this
// lane's query with keys acc_row(r, h); c > 0 is scale * log2(e) (a negative scale is folded
// into the sign of Q by the caller), so the block maximum can be taken over the raw products
// and the scaling fused into the exponent: p = 2^(c*s - m).
__device__ __forceinline__ void softmax_block(floatx16 sv, float c, const BlockInfo& b, int h,
                                              TileState& st, float (&p)[16],
                                              floatx16* o_low = nullptr) {
  float bm = -INFINITY;
  if (!b.full) {
    const uint32_t wh = b.word >> (4 * h);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      // all-ones where the edge exists, else zero; then select the product or -inf bitwise
      const int keep = ((int)(wh << (31 - acc_row(r, 0)))) >> 31;
      const float x = sv[r];   // (a bit cast applied to the vector element itself reads element 0)
      const int bits = (__builtin_bit_cast(int, x) & keep) | ((int)0xff800000 & ~keep);
      sv[r] = __builtin_bit_cast(float, bits);
    }
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) bm = fmaxf(bm, sv[r]);
  bm = fmaxf(bm, other_half(bm, h)) * c;
  if (__any(bm > st.m + kRescaleSlack)) {
    const float m_new = bm > st.m + kRescaleSlack ? bm : st.m;
    const float alpha = __builtin_amdgcn_exp2f(st.m - m_new);
    st.m = m_new;
    st.l *= alpha;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      st.o[0][r] *= alpha;
      st.o[1][r] *= alpha;
    }
    if (o_low) {       // low-order accumulators of the split-precision core
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        o_low[0][r] *= alpha;
        o_low[1][r] *= alpha;
      }
    }
  }
  float lsum = 0.f;
  const float neg_m = -st.m;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    p[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[r], c, neg_m));
    lsum += p[r];
  }
  st.l += lsum;
}

typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));

// softmax_block for fp16 storage, in three steps that callers with two independent sub-tiles
// interleave.  The numerators leave as the B operand of the PV products: rounded to fp16 two at a
// time (one packed conversion per pair, to nearest even), ph[u][e] = p of accumulator register
// 8u + e.  The running sum adds the *rounded* numerators (a dot product of each pair with (1, 1),
// accumulated in fp32), i.e. exactly the weights the products apply, so that acc / l is a true
// weighted mean of V rows.
//
// Entries outside the mask become -inf (word: mask bits of this lane's query).
__device__ __forceinline__ void mask_scores(floatx16& sv, uint32_t word, int h) {
  const uint32_t wh = word >> (4 * h);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    // all-ones where the edge exists, else zero; then select the product or -inf bitwise
    const int keep = ((int)(wh << (31 - acc_row(r, 0)))) >> 31;
    const float x = sv[r];   // (a bit cast applied to the vector element itself reads element 0)
    const int bits = (__builtin_bit_cast(int, x) & keep) | ((int)0xff800000 & ~keep);
    sv[r] = __builtin_bit_cast(float, bits);
  }
}
// Largest scaled score of this lane's query in the block (both half-waves agree).
__device__ __forceinline__ float block_max(const floatx16& sv, float c, int h) {
  float bm = fmaxf(sv[0], sv[1]);
#pragma unroll
  for (int r = 2; r < 16; r += 2) bm = __builtin_fmaxf(__builtin_fmaxf(bm, sv[r]), sv[r + 1]);
  return fmaxf(bm, other_half(bm, h)) * c;
}
__device__ __forceinline__ bool needs_rescale(const TileState& st, float bm) {
  return bm > st.m + kRescaleSlack;
}
// Raises m to bm where bm exceeds it by more than the slack, and rescales l and O (a factor of
// exactly 1 elsewhere).
__device__ __forceinline__ void rescale_state(TileState& st, float bm) {
  const float m_new = needs_rescale(st, bm) ? bm : st.m;
  const float alpha = __builtin_amdgcn_exp2f(st.m - m_new);
  st.m = m_new;
  st.l *= alpha;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    st.o[0][r] *= alpha;
    st.o[1][r] *= alpha;
  }
}
// kMatrixSum: the pairs are not summed by v_dot2_f32_f16, which no matrix instruction overlaps with, but by four 4 x 4 x 4
// products with ones, whose lane l holds the sum of its own four numerators.  (Two wavefronts of one SIMD, one issuing matrix
// products, the other the instruction, us alone / alone / together: dot2 242 / 244 / 489, packed conversion 236 / 237 /
// 243, exp2 253 / 253 / 330.  Kernels of two wavefronts per SIMD with interior loops take 3.4 % fewer cycles (+-1,359, L =
// 1,600,000 2.93M -> 2.84M), most of which a lower clock takes back (1.97 -> 1.90 GHz): medians of 15 alternations, us, +-1,359
// 1,377 -> 1,360; +-2,000, L = 400,000, 4 heads 1,901 -> 1,884; +-3,000, L = 400,000 761 -> 761; d = 128, +-2,048, L = 32,768, 32 heads
// 2,461 -> 2,437, +-200, L = 200,000, 4 heads 340 -> 331, +-32, L = 300,000, 4 heads 264 -> 257.  The others, with four
// wavefronts per SIMD or masked blocks, do not gain, and tile_attend_f16_kernel loses 4 % on random masks.)
template <bool kMatrixSum = false>
__device__ __forceinline__ void numerators_h(const floatx16& sv, float c, TileState& st, half8 (&ph)[2]) {
  const float neg_m = -st.m;
  const half2v ones = {(_Float16)1.0f, (_Float16)1.0f};
  float l = st.l;
#pragma unroll
  for (int r = 0; r < 16; r += 2) {
    const float2v p2 = {__builtin_amdgcn_exp2f(__builtin_fmaf(sv[r], c, neg_m)),
                        __builtin_amdgcn_exp2f(__builtin_fmaf(sv[r + 1], c, neg_m))};
    const half2v hp = __builtin_convertvector(p2, half2v);
    if constexpr (!kMatrixSum) l = __builtin_amdgcn_fdot2(hp, ones, l, false);
    ph[r / 8][r % 8] = hp[0];
    ph[r / 8][r % 8 + 1] = hp[1];
  }
  if constexpr (kMatrixSum) {
    const half4 four_ones = {(_Float16)1.0f, (_Float16)1.0f, (_Float16)1.0f, (_Float16)1.0f};
    float4v sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < 16; r += 4) {
      const half4 four = {ph[r / 8][r % 8], ph[r / 8][r % 8 + 1], ph[r / 8][r % 8 + 2], ph[r / 8][r % 8 + 3]};
      sum = __builtin_amdgcn_mfma_f32_4x4x4f16(four_ones, four, sum, 0, 0, 0);
    }
    l += sum[0];
  }
  st.l = l;
}
// The running max of fp16 tiles is raised on demand: the numerators are first taken against the
// m the state already has, and only if one of them leaves the fp16 range (it rounds to +inf, and
// so does the sum it enters; the first block of a tile, whose m is still the initial one, always
// does) is the block's maximum computed, m raised and the numerators taken again.  A numerator is
// then at most 2^16 instead of 2^kRescaleSlack, which fp16 holds at the same relative precision,
// and the common block pays neither for the maximum nor for waiting on it.
constexpr float kSumOverflow = 3.0e38f;
__device__ __forceinline__ bool sum_overflowed(const TileState& st) { return !(st.l < kSumOverflow); }
__device__ __forceinline__ void softmax_block_h(floatx16 sv, float c, bool full, uint32_t word, int h,
                                                TileState& st, half8 (&ph)[2]) {
  if (!full) mask_scores(sv, word, h);
  const float l_before = st.l;
  numerators_h(sv, c, st, ph);
  if (__any(sum_overflowed(st))) {
    st.l = l_before;
    rescale_state(st, block_max(sv, c, h));
    numerators_h(sv, c, st, ph);
  }
}
// The same for two sub-tiles whose blocks are both unmasked, as one stretch of code with one
// (rare) branch.
__device__ __forceinline__ void softmax_pair_h(const floatx16& s_a, const floatx16& s_b, float c, int h,
                                               TileState& sta, TileState& stb, half8 (&pha)[2],
                                               half8 (&phb)[2]) {
  const float la = sta.l, lb = stb.l;
  numerators_h<true>(s_a, c, sta, pha);
  numerators_h<true>(s_b, c, stb, phb);
  if (__any(sum_overflowed(sta) || sum_overflowed(stb))) {
    sta.l = la;
    stb.l = lb;
    rescale_state(sta, block_max(s_a, c, h));
    rescale_state(stb, block_max(s_b, c, h));
    numerators_h<true>(s_a, c, sta, pha);
    numerators_h<true>(s_b, c, stb, phb);
  }
}

// Source addresses of the global -> LDS block copies.  A block's rows are row0 + j*stride
// (j = 0..31); copy i of a block moves kRows consecutive keys, kLanes lanes of 16 bytes per
// row.  The per-lane part of the address is fixed for a whole work item (32-bit byte offsets
// from the block's first row); the per-block part is wave-uniform, so a copy costs no vector
// arithmetic.  Blocks cut short by the end of the sequence (nvalid < 32) re-read their last
// row instead of running past it; those keys are masked off.
//
// kD is the row length of the tensors in global memory; a block always holds 64 channels of a
// key (for kD > 64 the caller passes tensor pointers already advanced to its 64-channel slice).
template <typename T, int kD = kHeadDim>
struct StageMap {
  static constexpr int kRowBytes = kHeadDim * (int)sizeof(T);   // staged row (one 64-channel slice)
  static constexpr int kGlobalRowBytes = kD * (int)sizeof(T);   // tensor row
  static constexpr int kLanes = kRowBytes / 16;          // lanes per row
  static constexpr int kRows = kWave / kLanes;           // rows per copy
  static constexpr int kCopies = kTile / kRows;          // copies per block
  int64_t stride_bytes;                                  // bytes between consecutive keys
  uint32_t voff;                                         // V: lane's row and 16-byte chunk
  uint32_t koff[kLanes / 4 > 1 ? 4 : 1];                 // K: same with the chunk swizzled, per copy % 4

  __device__ void init(int64_t stride, int lane) {
    stride_bytes = stride * kGlobalRowBytes;
    const int lr = lane / kLanes, lc = lane % kLanes;
    const uint32_t rowoff = (uint32_t)(lr * stride_bytes);
    voff = rowoff + lc * 16;
    // chunk c of key r is stored at chunk slot c ^ (r % kLanes): the copy reads the chunk that
    // belongs into the slot this lane writes
    if (kLanes == 8) {
      koff[0] = rowoff + ((lc ^ lr) * 16);               // (8i + lr) % 8 = lr for every copy i
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) koff[i] = rowoff + ((lc ^ ((4 * i + lr) & 15)) * 16);
    }
  }
  // (a block all of whose 32 keys exist)
  __device__ void stage_v_whole(const T* __restrict__ Vh, int64_t row0, char* dst) const {
    const char* base = reinterpret_cast<const char*>(Vh) + row0 * kGlobalRowBytes;
#pragma unroll
    for (int i = 0; i < kCopies; ++i) copy16_to_lds(base + i * kRows * stride_bytes + voff, dst + i * 1024);
  }
  __device__ void stage_k_whole(const T* __restrict__ Kh, int64_t row0, char* dst) const {
    const char* base = reinterpret_cast<const char*>(Kh) + row0 * kGlobalRowBytes;
#pragma unroll
    for (int i = 0; i < kCopies; ++i)
      copy16_to_lds(base + i * kRows * stride_bytes + koff[kLanes == 8 ? 0 : i % 4], dst + i * 1024);
  }
  __device__ void stage_v(const T* __restrict__ Vh, const BlockInfo& b, int lane, char* dst) const {
    if (b.nvalid == kTile) {
      stage_v_whole(Vh, b.row0, dst);
    } else {
#pragma unroll
      for (int i = 0; i < kCopies; ++i) {
        int key = kRows * i + lane / kLanes;
        key = key < b.nvalid ? key : b.nvalid - 1;
        copy16_to_lds(reinterpret_cast<const char*>(Vh) + b.row0 * kGlobalRowBytes + key * stride_bytes +
                          (lane % kLanes) * 16,
                      dst + i * 1024);
      }
    }
  }
  __device__ void stage_k(const T* __restrict__ Kh, const BlockInfo& b, int lane, char* dst) const {
    if (b.nvalid == kTile) {
      stage_k_whole(Kh, b.row0, dst);
    } else {
#pragma unroll
      for (int i = 0; i < kCopies; ++i) {
        const int row = kRows * i + lane / kLanes;
        const int key = row < b.nvalid ? row : b.nvalid - 1;
        const int chunk = (lane % kLanes) ^ (row % kLanes);
        copy16_to_lds(reinterpret_cast<const char*>(Kh) + b.row0 * kGlobalRowBytes + key * stride_bytes +
                          chunk * 16,
                      dst + i * 1024);
      }
    }
  }
};

// Head dimensions above 64: the kD / 64 wavefronts of a workgroup own one tile together, each
// with one 64-channel slice of Q, K, V and O.  The products S^T = K Q^T of the slices are partial
// sums over the channels; every wavefront leaves its 32x32 partial in LDS and, after one
// workgroup barrier, all of them add the partials in slice order, so that every wavefront
// continues with bit-identical scores (and therefore identical m, l and P).  Two buffers
// alternate, which makes one barrier per block enough: a wavefront overwrites a buffer only
// after the barrier that every reader of its previous contents has passed.
template <int kD>
struct SliceExchange {
  static constexpr int kSlices = kD / kHeadDim;
  static constexpr int kBytes = 2 * kSlices * 4096;   // [2][slice][4][64 lanes] float4
  float4* xs;      // the workgroup's exchange buffers
  int slice;       // this wavefront's slice
  int parity;
  __device__ void init(char* lds, int slice_) {
    xs = reinterpret_cast<float4*>(lds);
    slice = slice_;
    parity = 0;
  }
  __device__ void sum_slices(floatx16& s, int lane) {
    float4* buf = xs + parity * (kSlices * 256);
    parity ^= 1;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      buf[(slice * 4 + j) * 64 + lane] = make_float4(s[4 * j], s[4 * j + 1], s[4 * j + 2], s[4 * j + 3]);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float4 t = buf[j * 64 + lane];
#pragma unroll
      for (int w = 1; w < kSlices; ++w) {
        const float4 v = buf[(w * 4 + j) * 64 + lane];
        t.x += v.x; t.y += v.y; t.z += v.z; t.w += v.w;
      }
      s[4 * j] = t.x; s[4 * j + 1] = t.y; s[4 * j + 2] = t.z; s[4 * j + 3] = t.w;
    }
  }
};

// ---- fp32 storage ---------------------------------------------------------------------------
// fp32 products on the 16-bit matrix cores (16 times the rate of the fp32 ones), by splitting
// the operands into parts whose products are summed in fp32.
//
// An element x of any operand (Q, K, the numerators of the softmax, V) becomes three bf16 parts,
// hi = bf16(x), mid = bf16(x - hi), lo = x - hi - mid: both differences are exact in fp32 and lo (at
// most 8 significant bits) is exact in bf16, so the parts hold x to its last bit and keep the exponent
// range of fp32.  A product is taken as
//   lo.hi + hi.lo + mid.mid + mid.hi + hi.mid + hi.hi
// and the terms left out (mid.lo, lo.mid, lo.lo) are together below 2^-24 |a.b|, whatever else the row
// holds.  (Two fp16 parts under a scale per row take half the products for the scores, but an element
// is then known to 2^-40 of the largest of its row only: one large channel costs the others their
// accuracy, and the scales themselves can overflow.)
//
// The smallest terms go first into an accumulator, so that only the last few of its additions
// round at the size of the sum, where the fp32 matrix instruction (two channels or keys at a
// time) rounds at every one: the error against 64-bit arithmetic is smaller than with
// fp32 products (longformer mask, L = 65,536: 1.5e-7 instead of 4.1e-7 relative).
//
// Per 32 x 32 block: 48 matrix instructions of 32 cycles instead of 64 of 64, and about 440 vector
// instructions for the splits (three quarters fewer where a workgroup shares them, SharedBlock).
// With every wavefront splitting its own blocks: longformer mask, L = 65,536, 8 heads, prepared
// 494 -> 411 us; +-815 at d = 256, L = 16,301 282 -> 228 us.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t round_pair_bf16(float x0, float x1) {
  const float2v x = {x0, x1};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));
}
// x0 and x1 less the two bf16 numbers packed in `pair`
__device__ __forceinline__ void take_pair(float& x0, float& x1, uint32_t pair) {
  x0 -= __builtin_bit_cast(float, pair << 16);
  x1 -= __builtin_bit_cast(float, pair & 0xffff0000u);
}
// One operand of the products (8 values per lane).
struct SplitOperand {
  bf16x8 hi, mid, lo;
  __device__ __forceinline__ void split(const float* x) {
    uint4v a, b, c;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float x0 = x[2 * e], x1 = x[2 * e + 1];
      a[e] = round_pair_bf16(x0, x1);
      take_pair(x0, x1, a[e]);
      b[e] = round_pair_bf16(x0, x1);
      take_pair(x0, x1, b[e]);
      c[e] = round_pair_bf16(x0, x1);
    }
    hi = __builtin_bit_cast(bf16x8, a);
    mid = __builtin_bit_cast(bf16x8, b);
    lo = __builtin_bit_cast(bf16x8, c);
  }
};
__device__ __forceinline__ floatx16 mfma_bf16(bf16x8 a, bf16x8 b, floatx16 acc) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
}
__device__ __forceinline__ floatx16 split_product(const SplitOperand& a, const SplitOperand& b, floatx16 acc) {
  acc = mfma_bf16(a.lo, b.hi, acc);
  acc = mfma_bf16(a.hi, b.lo, acc);
  acc = mfma_bf16(a.mid, b.mid, acc);
  acc = mfma_bf16(a.mid, b.hi, acc);
  acc = mfma_bf16(a.hi, b.mid, acc);
  return mfma_bf16(a.hi, b.hi, acc);
}
// Scores of 32 keys, S[key acc_row(r, h)].
__device__ __forceinline__ floatx16 split_scores(const SplitOperand (&k)[4], const SplitOperand (&q)[4]) {
  floatx16 s = {0};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    s = mfma_bf16(k[i].lo, q[i].hi, s);
    s = mfma_bf16(k[i].hi, q[i].lo, s);
    s = mfma_bf16(k[i].mid, q[i].mid, s);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    s = mfma_bf16(k[i].mid, q[i].hi, s);
    s = mfma_bf16(k[i].hi, q[i].mid, s);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) s = mfma_bf16(k[i].hi, q[i].hi, s);
  return s;
}
// O^T += V_blk^T P^T for one block; value(u, cb) is the operand V^T[channel cb*32+n][keys 16u ..].
// The products of a block are summed by themselves and added to O once: one rounding at the size
// of O per block (chained into O they round 12 times, the fp32 instruction 16 times, which is
// what the error of rows of thousands of keys comes from: +-16,383, L = 65,536, relative error 3.0e-6
// with fp32 products, 0.66e-6 so; the 32 additions cost nothing measurable).
// No branch here: skipping the halves of a masked block that no query attends made two versions
// of this code, whose registers cost more than the products saved (247 -> 331 us at +-128).
template <typename Value>
__device__ __forceinline__ void weigh_values(const float (&p)[16], TileState& st, Value value) {
  SplitOperand pb[2];
  pb[0].split(p);
  pb[1].split(p + 8);
#pragma unroll
  for (int cb = 0; cb < 2; ++cb) {
    floatx16 part = split_product(value(0, cb), pb[0], floatx16{0});
    part = split_product(value(1, cb), pb[1], part);
#pragma unroll
    for (int r = 0; r < 16; ++r) st.o[cb][r] += part[r];
  }
}

// Inputs whose split is not exact: an infinity or a finite value that rounds to an infinite bf16 (from
// 3.39e38), whose parts are no numbers, and values below 2^-109, whose low parts fall below the subnormal
// numbers of bf16 (an error of 2^-134: it counts in the scores where the other operand is that large, and
// in O where all values are that small).  A tile that may have met one is computed once more with
// fp32 products (run_exact), which decide what such inputs give.  All of this is seen per tile, not
// per block: in the state a tile ends with, and in its queries (small ones themselves, large ones
// because the keys they meet may be small).
constexpr float kSplitSmall = 0x1p-108f, kSplitLarge = 0x1p96f;
// True in a lane whose state holds an infinity or a NaN, or no value of a size that V's split keeps.
__device__ __forceinline__ bool beyond_split(const TileState& st) {
  float z = st.l * 0.f, top = 0.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    z = __builtin_fmaf(st.o[0][r], 0.f, z);
    z = __builtin_fmaf(st.o[1][r], 0.f, z);
    top = __builtin_fmaxf(__builtin_fmaxf(top, __builtin_fabsf(st.o[0][r])), __builtin_fabsf(st.o[1][r]));
  }
  return !(z == 0.f) || (top > 0.f && top < st.l * (kSplitSmall * 16.f));
}

template <int kD>
struct CoreF32T {
  using Stage = StageMap<float, kD>;
  SplitOperand q3[4];         // Q[query n][h*32 + 8s .. +7], s = 0..3 (of this wavefront's 64-channel slice)
  const float* q_row;         // this lane's half row of Q, for run_exact
  bool q_negate;
  bool q_beyond;              // the tile's queries call for run_exact, see beyond_split (wave-uniform)
  SliceExchange<kD> xchg;   // used for kD > 64 only

  __device__ void load_qf(float (&qf)[32]) const {
    const float4* src = reinterpret_cast<const float4*>(q_row);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const float4 v = src[t];
      qf[4 * t] = v.x; qf[4 * t + 1] = v.y; qf[4 * t + 2] = v.z; qf[4 * t + 3] = v.w;
    }
    if (q_negate) {
#pragma unroll
      for (int t = 0; t < 32; ++t) qf[t] = -qf[t];
    }
  }
  __device__ void load_q(const float* Qrow, int h, bool negate) {
    q_row = Qrow + h * 32;
    q_negate = negate;
    float qf[32];
    load_qf(qf);
    // (twice a number's bits, less one: the order of the magnitudes, with the zeros at the top)
    float most = 0.f;
    uint32_t least = ~0u;
#pragma unroll
    for (int t = 0; t < 32; ++t) {
      most = __builtin_fmaxf(most, __builtin_fabsf(qf[t]));
      const uint32_t order = (__builtin_bit_cast(uint32_t, qf[t]) << 1) - 1u;
      least = order < least ? order : least;
    }
    q_beyond = __any(least < (__builtin_bit_cast(uint32_t, kSplitSmall) << 1) - 1u || most > kSplitLarge);
#pragma unroll
    for (int s = 0; s < 4; ++s) q3[s].split(qf + 8 * s);
  }
  __device__ bool again(const TileState& st) const { return q_beyond || __any(beyond_split(st)); }
  __device__ floatx16 scores(const SplitOperand (&k3)[4], int lane) {
    floatx16 s = split_scores(k3, q3);
    if (kD > kHeadDim) xchg.sum_slices(s, lane);
    return s;
  }

  // kf[t] = K[key n of the block][h*32 + t], straight from global memory: 128 contiguous bytes
  // per lane, i.e. kFragLoads loads of 16 bytes (the widest load there is; the counted waits
  // below rely on this number).  lane_off = byte offset of the lane's key row and half inside
  // a whole block.
  static constexpr int kFragLoads = 32 * (int)sizeof(float) / 16;
  __device__ static void load_k(const float* __restrict__ Kh, const BlockInfo& b, int64_t stride_bytes,
                                uint32_t lane_off, int n, int h, float (&kf)[32]) {
    const char* base = reinterpret_cast<const char*>(Kh) + b.row0 * Stage::kGlobalRowBytes;
    const float4* kp;
    if (b.nvalid == kTile) {
      kp = reinterpret_cast<const float4*>(base + lane_off);
    } else {
      const int krow = n < b.nvalid ? n : b.nvalid - 1;
      kp = reinterpret_cast<const float4*>(base + krow * stride_bytes + h * 128);
    }
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const float4 v = kp[t];
      kf[4 * t] = v.x; kf[4 * t + 1] = v.y; kf[4 * t + 2] = v.z; kf[4 * t + 3] = v.w;
    }
  }

  static constexpr int kBlockBytes = kTile * kHeadDim * 4;   // one staged K or V block

  // O^T += V_blk^T P^T with the V rows of the block staged (complete) at ldsv.  A operand:
  // V^T[channel cb*32+n][key acc_row(r,h)] = staged V[key][channel], 8 keys per operand.
  __device__ static void weigh_v(const float (&p)[16], int n, int h, TileState& st, const char* ldsv) {
    const float* vread = reinterpret_cast<const float*>(ldsv) + h * 4 * kHeadDim + n;
    weigh_values(p, st, [&](int u, int cb) {
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = vread[acc_row(8 * u + e, 0) * kHeadDim + cb * 32];
      SplitOperand va;
      va.split(v);
      return va;
    });
  }

  // The pipeline: the K fragment of block k+1 is loaded global -> registers (each lane reads 128
  // contiguous bytes of its key row) into the registers that block k's fragment left when it was
  // split, the V block k is copied global -> LDS behind the S^T matrix work.
  template <typename Src>
  __device__ void run_split(const float* __restrict__ Kh, const float* __restrict__ Vh, const Src& src,
                            int k0, int k1, float c, int lane, TileState& st, char* lds) {
    const int n = lane & 31, h = lane >> 5;
    Stage sm;
    sm.init(src.key_stride(), lane);
    const uint32_t klane = (uint32_t)(n * sm.stride_bytes) + h * 128;
    BlockInfo b = src.get(k0, n);
    src.resolve(b);
    float kf[32];
    load_k(Kh, b, sm.stride_bytes, klane, n, h, kf);
    for (int k = k0; k < k1; ++k) {
      const bool more = k + 1 < k1;      // wave-uniform
      SplitOperand k3[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) k3[i].split(kf + 8 * i);
      BlockInfo b1 = src.get(more ? k + 1 : k, n);
      src.resolve(b1);
      __builtin_amdgcn_wave_barrier();   // the previous block's reads of the staged V are done
      sm.stage_v(Vh, b, lane, lds);
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0); // (the counted wait below relies on this order)
      if (more) load_k(Kh, b1, sm.stride_bytes, klane, n, h, kf);
      const floatx16 s = scores(k3, lane);
      float p[16];
      softmax_block(s, c, b, h, st, p);
      wait_staged_v<kFragLoads>(more);   // V block k is older than the K fragment loads (if any)
      __builtin_amdgcn_wave_barrier();
      weigh_v(p, n, h, st, lds);
      b = b1;
    }
  }

  // Explicit block lists: the block ids are read through the scalar path and the mask words of
  // block k+1 are copied global -> LDS while block k is computed (two 256-byte slots behind the V
  // block), as in CoreF16T::run_ldsk.  The only loads into vector registers are the K fragments.
  __device__ void run_split(const float* __restrict__ Kh, const float* __restrict__ Vh,
                            const ExplicitBlocks& src, int k0, int k1, float c, int lane, TileState& st,
                            char* lds) {
    const int n = lane & 31, h = lane >> 5;
    Stage sm;
    sm.init(1, lane);
    const uint32_t klane = (uint32_t)(n * sm.stride_bytes) + h * 128;
    char* ldsw = lds + kBlockBytes;              // two slots of 64 mask words (both half-waves)
    const uint32_t* wsrc = src.mask + n;         // this lane's word of block k: wsrc[32 k]
    BlockInfo b = src.block(k0);
    BlockInfo b1 = src.block(k0 + 1 < k1 ? k0 + 1 : k0);
    src.resolve(b);
    __builtin_amdgcn_wave_barrier();     // reads of the buffers by an earlier work item are done
    copy4_to_lds(wsrc + (int64_t)k0 * kTile, ldsw + (k0 & 1) * 256);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    float kf[32];
    load_k(Kh, b, sm.stride_bytes, klane, n, h, kf);
    for (int k = k0; k < k1; ++k) {
      const bool more = k + 1 < k1;      // wave-uniform
      src.resolve(b1);
      SplitOperand k3[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) k3[i].split(kf + 8 * i);
      wait_loads_except<0>();            // the words of block k are older than its K fragment
      __builtin_amdgcn_wave_barrier();
      b.word = *reinterpret_cast<const uint32_t*>(ldsw + (k & 1) * 256 + lane * 4);
      sm.stage_v(Vh, b, lane, lds);
      if (more) copy4_to_lds(wsrc + (int64_t)(k + 1) * kTile, ldsw + ((k + 1) & 1) * 256);
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0); // (the counted wait below relies on this order)
      if (more) load_k(Kh, b1, sm.stride_bytes, klane, n, h, kf);
      BlockInfo b2 = b1;
      if (k + 2 < k1) b2 = src.block(k + 2);
      const floatx16 s = scores(k3, lane);
      float p[16];
      softmax_block(s, c, b, h, st, p);
      wait_staged_v<kFragLoads>(more);   // V block k is older than the K fragment loads (if any)
      __builtin_amdgcn_wave_barrier();
      weigh_v(p, n, h, st, lds);
      b = b1;
      b1 = b2;
    }
  }

  // The same tile with v_mfma_f32_32x32x2_f32 (true fp32 products), one block after the other.
  template <typename Src>
  __device__ void run_exact(const float* __restrict__ Kh, const float* __restrict__ Vh, const Src& src,
                            int k0, int k1, float c, int lane, TileState& st, char* lds) {
    const int n = lane & 31, h = lane >> 5;
    Stage sm;
    sm.init(src.key_stride(), lane);
    const uint32_t klane = (uint32_t)(n * sm.stride_bytes) + h * 128;
    float qf[32];
    load_qf(qf);
    for (int k = k0; k < k1; ++k) {
      BlockInfo b = src.get(k, n);
      src.resolve(b);
      __builtin_amdgcn_wave_barrier();   // the previous block's reads of the staged V are done
      sm.stage_v(Vh, b, lane, lds);
      float kf[32];
      load_k(Kh, b, sm.stride_bytes, klane, n, h, kf);
      floatx16 s = {0};
#pragma unroll
      for (int t = 0; t < 32; ++t) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[t], qf[t], s, 0, 0, 0);
      if (kD > kHeadDim) xchg.sum_slices(s, lane);
      float p[16];
      softmax_block(s, c, b, h, st, p);
      wait_loads_except<0>();
      __builtin_amdgcn_wave_barrier();
      const float* vread = reinterpret_cast<const float*>(lds) + h * 4 * kHeadDim + n;
      // The values of keys that no query of the tile attends count as 0, so an infinity or a NaN among them
      // (padding behind a mask) stays out of the sums, where 0 * inf would spoil the whole tile.
      uint32_t seen = b.word;
#pragma unroll
      for (int off = 1; off < kTile; off <<= 1) seen |= __shfl_xor(seen, off, kWave);
      if (b.full) seen = ~0u;
      seen >>= 4 * h;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const bool used = (seen >> acc_row(r, 0)) & 1u;
        const float v0 = used ? vread[acc_row(r, 0) * kHeadDim] : 0.f;
        const float v1 = used ? vread[acc_row(r, 0) * kHeadDim + 32] : 0.f;
        st.o[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(v0, p[r], st.o[0], 0, 0, 0);
        st.o[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(v1, p[r], st.o[1], 0, 0, 0);
      }
    }
  }

  template <int kPipe>
  static constexpr int lds_bytes() { return kBlockBytes + 512; }     // V block, mask words

  template <int kPipe, typename Src>
  __device__ void run(const float* __restrict__ Kh, const float* __restrict__ Vh, const Src& src,
                      int k0, int k1, float c, int lane, TileState& st, char* lds) {
    static_assert(kPipe == kPipeRegK, "fp32 pipeline");
    if (k0 >= k1) return;                // (for a wide tile the same in every slice)
    run_split(Kh, Vh, src, k0, k1, c, lane, st, lds);
    bool once_more = again(st);
    if constexpr (kD > kHeadDim) once_more = __syncthreads_or(once_more);
    if (once_more) {
      st.init();
      run_exact(Kh, Vh, src, k0, k1, c, lane, st, lds);
    }
  }

  // The slices of a wide tile for one of several ranges of its blocks in one workgroup: sum_slices waits for the whole
  // workgroup, so every wavefront meets `longest` (>= k1 - k0) barriers.
  template <typename Src>
  __device__ void run_range(const float* __restrict__ Kh, const float* __restrict__ Vh, const Src& src, int k0, int k1,
                            int longest, float c, int lane, TileState& st, char* lds) {
    if (k0 < k1) run_split(Kh, Vh, src, k0, k1, c, lane, st, lds);
    for (int k = k1 - k0; k < longest; ++k) __syncthreads();
    if (!__syncthreads_or(k0 < k1 && again(st))) return;
    st.init();
    if (k0 < k1) run_exact(Kh, Vh, src, k0, k1, c, lane, st, lds);
    for (int k = k1 - k0; k < longest; ++k) __syncthreads();
  }

  // Orow = acc * inv, or w_prev * Orow + acc * inv when the call continues an earlier state.
  __device__ static void store_row(float* Orow, const TileState& st, float inv, float w_prev,
                                   bool accumulate, int h) {
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float4* dst = reinterpret_cast<float4*>(Orow + cb * 32 + 8 * g + 4 * h);
        float4 v = make_float4(st.o[cb][4 * g] * inv, st.o[cb][4 * g + 1] * inv,
                               st.o[cb][4 * g + 2] * inv, st.o[cb][4 * g + 3] * inv);
        if (accumulate) {
          const float4 old = *dst;
          v.x = __builtin_fmaf(w_prev, old.x, v.x);
          v.y = __builtin_fmaf(w_prev, old.y, v.y);
          v.z = __builtin_fmaf(w_prev, old.z, v.z);
          v.w = __builtin_fmaf(w_prev, old.w, v.w);
        }
        *dst = v;
      }
  }

  // (Direct row stores: 32 bytes per row and instruction from the two half-waves.  Sending the
  // tile through LDS to store whole rows, as CoreF16T::store_tile does, changes nothing here.)
  static constexpr bool kTileStore = false;
};
using CoreF32 = CoreF32T<kHeadDim>;

// ---- fp16 storage ---------------------------------------------------------------------------
template <int kD>
struct CoreF16T {
  using Stage = StageMap<__half, kD>;
  half8 qf[4];    // Q[query n][h*32 + 8s .. +7], s = 0..3 (of this wavefront's 64-channel slice)
  SliceExchange<kD> xchg;   // used for kD > 64 only

  __device__ void load_q(const __half* Qrow, int h, bool negate) {
    const half8* src = reinterpret_cast<const half8*>(Qrow + h * 32);
#pragma unroll
    for (int s = 0; s < 4; ++s) qf[s] = src[s];
    if (negate) {
#pragma unroll
      for (int s = 0; s < 4; ++s) qf[s] = -qf[s];
    }
  }

  // The loads of load_q have completed (the caller has waited for them): taking qf as read and
  // written here keeps the compiler from waiting for them again at their first use, where
  // copies issued in between would be waited for as well.
  __device__ void q_arrived() {
#pragma unroll
    for (int s = 0; s < 4; ++s) asm volatile("" : "+v"(qf[s]));
  }

  static constexpr int kBlockBytes = kTile * kHeadDim * 2;   // one staged K or V block

  // kf[s] = K[key n][h*32 + 8s .. +7] out of the staged block: keys 8i..8i+7 per copy, 8 lanes
  // per 128-byte row, the eight 16-byte chunks of a row XOR-swizzled with the row index (see
  // CoreSplit::read_k) so that these reads are free of bank conflicts.
  __device__ static void read_k(const char* ldsk, int n, int h, half8 (&kf)[4]) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int slot = (4 * h + s) ^ (n & 7);
      kf[s] = *reinterpret_cast<const half8*>(ldsk + (n * 8 + slot) * 16);
    }
  }

  // 4 keys x 1 channel per lane out of the row-major staged V block, using the LDS transpose
  // read of gfx950: inside a 16-lane group, lane i receives element (i % 4) of the 8 bytes
  // addressed by lanes i/4, 4 + i/4, 8 + i/4 and 12 + i/4.  Lane i therefore addresses key
  // (key0 + i/4) at channels 4*(i%4).. of its group's 16 channels, and ends up with channel i of
  // the group for keys key0..key0+3: the K-contiguous A operand of V^T.
  __device__ static half4 read_vt(const char* p) {
    const short4v raw =
        __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4v __attribute__((address_space(3)))*)p);
    return __builtin_bit_cast(half4, raw);
  }

  // (kKeepMore, more: see wait_staged_v)
  template <int kKeepMore>
  __device__ void block_math(const half8 (&kf)[4], const BlockInfo& b, float c, int lane, int h,
                             TileState& st, const char* ldsv, bool more) {
    half8 ph[2];
    scores(kf, b, c, lane, h, st, ph);
    wait_staged_v<kKeepMore>(more);
    __builtin_amdgcn_wave_barrier();
    accumulate(ph, lane, h, st, ldsv);
  }

  // First half of the block step: S^T = K_blk Q^T and the softmax update; ph = numerators as the
  // B operand of the PV products.
  __device__ void scores(const half8 (&kf)[4], const BlockInfo& b, float c, int lane, int h,
                         TileState& st, half8 (&ph)[2]) {
    floatx16 sacc = {0};
#pragma unroll
    for (int s = 0; s < 4; ++s)
      sacc = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[s], qf[s], sacc, 0, 0, 0);
    if (kD > kHeadDim) xchg.sum_slices(sacc, lane);
    softmax_block_h(sacc, c, b.full != 0, b.word, h, st, ph);
  }

  // This lane's address of the V^T operand reads for key0 = 4h, channel group 0; the other reads
  // are constant offsets from it.
  __device__ static const char* vt_base(const char* ldsv, int lane, int h) {
    const int i = lane & 15, grp16 = (lane >> 4) & 1;
    return ldsv + (4 * h + (i >> 2)) * (kHeadDim * 2) + (grp16 * 16 + 4 * (i & 3)) * 2;
  }

  // A operand of one PV product: V^T[channel cb*32+n][slot (u,h,e)], slot key = 16u + 8(e/4) + 4h + e%4
  __device__ static half8 read_va(const char* vt, int u, int cb) {
    const half4 lo = read_vt(vt + (16 * u) * (kHeadDim * 2) + cb * 64);
    const half4 hi = read_vt(vt + (16 * u + 8) * (kHeadDim * 2) + cb * 64);
    return half8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  }

  // Second half: O^T += V_blk^T P^T with the V block staged (complete) at ldsv.
  __device__ static void accumulate(const half8 (&ph)[2], int lane, int h, TileState& st,
                                    const char* ldsv) {
    const char* vt = vt_base(ldsv, lane, h);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
        st.o[cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(read_va(vt, u, cb), ph[u], st.o[cb], 0, 0, 0);
  }

  // K and V blocks travel global -> LDS without registers, as whole rows (coalesced).  Per block k:
  // the V copy is issued first; the K fragment (copied during block k-1) is read into registers and the K
  // copy of block k+1 is issued at once, so it lands behind the matrix work of block k; block ids / mask
  // words are fetched two blocks ahead.
  template <typename Src>
  __device__ void run_ldsk(const __half* __restrict__ Kh, const __half* __restrict__ Vh, const Src& src,
                      int k0, int k1, float c, int lane, TileState& st, char* lds) {
    if (k0 >= k1) return;
    const int n = lane & 31, h = lane >> 5;
    Stage sm;
    sm.init(src.key_stride(), lane);
    char* ldsk = lds;
    char* ldsv = lds + kBlockBytes;
    BlockInfo b = src.get(k0, n);
    BlockInfo b1 = src.get(k0 + 1 < k1 ? k0 + 1 : k0, n);
    src.resolve(b);
    __builtin_amdgcn_wave_barrier();     // reads of both buffers by an earlier work item are done
    sm.stage_k(Kh, b, lane, ldsk);
    for (int k = k0; k < k1; ++k) {
      const bool more = k + 1 < k1;      // wave-uniform
      src.resolve(b1);
      __builtin_amdgcn_wave_barrier();   // the previous block's reads of the staged V are done
      sm.stage_v(Vh, b, lane, ldsv);
      BlockInfo b2 = b1;
      if (k + 2 < k1) b2 = src.get(k + 2, n);
      wait_k_block<4, Src::kGetLoads>(k + 2 < k1);   // K block k: older than the V copies (and the record loads)
      __builtin_amdgcn_wave_barrier();
      half8 kf[4];
      read_k(ldsk, n, h, kf);
      wait_lds_reads();                  // the K buffer may be overwritten now
      __builtin_amdgcn_wave_barrier();
      if (more) sm.stage_k(Kh, b1, lane, ldsk);
      // V block k (and any record load after it) is older than the 4 K copies issued above (if any)
      block_math<4>(kf, b, c, lane, h, st, ldsv, more);
      b = b1;
      b1 = b2;
    }
  }

  // Explicit block lists: as run_ldsk, with no vector load into registers inside the loop.  Block
  // ids come through the scalar path (ExplicitBlocks::block), and the 32 mask words of block k+1
  // are copied global -> LDS (one 4-byte copy per lane into one of two 256-byte slots) while block
  // k is computed.  Every vector memory operation of the loop is then an LDS copy whose
  // completion only the counted waits below ask for; a register load carried around the loop
  // would make the compiler drain all of them, the prefetched K block included, once per block.
  __device__ void run_ldsk(const __half* __restrict__ Kh, const __half* __restrict__ Vh,
                           const ExplicitBlocks& src, int k0, int k1, float c, int lane, TileState& st,
                           char* lds) {
    if (k0 >= k1) return;
    const int n = lane & 31, h = lane >> 5;
    Stage sm;
    sm.init(1, lane);
    char* ldsk = lds;
    char* ldsv = lds + kBlockBytes;
    char* ldsw = lds + 2 * kBlockBytes;          // two slots of 64 mask words (both half-waves)
    const uint32_t* wsrc = src.mask + n;         // this lane's word of block k: wsrc[32 k]
    BlockInfo b = src.block(k0);
    BlockInfo b1 = src.block(k0 + 1 < k1 ? k0 + 1 : k0);
    src.resolve(b);
    __builtin_amdgcn_wave_barrier();     // reads of the buffers by an earlier work item are done
    copy4_to_lds(wsrc + (int64_t)k0 * kTile, ldsw + (k0 & 1) * 256);
    sm.stage_k(Kh, b, lane, ldsk);
    // One block step.  kInner: blocks k+1 and k+2 exist and blocks k and k+1 are whole (true up
    // to the list's last two blocks), which leaves no branch on the position in the list and
    // none on a block cut short by the end of the sequence.
    auto step = [&](int k, auto inner) {
      constexpr bool kInner = decltype(inner)::value;
      const bool more = kInner || k + 1 < k1;      // wave-uniform
      if (kInner) src.resolve_whole(b1); else src.resolve(b1);
      __builtin_amdgcn_wave_barrier();   // the previous block's reads of V and of the other word slot are done
      if (more) copy4_to_lds(wsrc + (int64_t)(k + 1) * kTile, ldsw + ((k + 1) & 1) * 256);
      if (kInner) sm.stage_v_whole(Vh, b.row0, ldsv); else sm.stage_v(Vh, b, lane, ldsv);
      BlockInfo b2 = b1;
      if (kInner || k + 2 < k1) b2 = src.block(k + 2);
      // K block k and the words of block k are older than the copies issued in this step
      if (more) wait_loads_except<5>(); else wait_loads_except<4>();
      __builtin_amdgcn_wave_barrier();
      half8 kf[4];
      read_k(ldsk, n, h, kf);
      b.word = *reinterpret_cast<const uint32_t*>(ldsw + (k & 1) * 256 + lane * 4);
      wait_lds_reads();                  // the K buffer may be overwritten now
      __builtin_amdgcn_wave_barrier();
      if (kInner) sm.stage_k_whole(Kh, b1.row0, ldsk); else if (more) sm.stage_k(Kh, b1, lane, ldsk);
      half8 ph[2];
      scores(kf, b, c, lane, h, st, ph);
      // V block k (and the words of block k+1) are older than the 4 K copies issued above (if any)
      if (more) wait_loads_except<4>(); else wait_loads_except<0>();
      __builtin_amdgcn_wave_barrier();
      accumulate(ph, lane, h, st, ldsv);
      b = b1;
      b1 = b2;
    };
    int k = k0;
    for (; k + 2 < k1; ++k) step(k, std::true_type{});
    for (; k < k1; ++k) step(k, std::false_type{});
  }

  template <int kPipe>
  static constexpr int lds_bytes() { return 2 * kBlockBytes + 512; }

  template <int kPipe, typename Src>
  __device__ void run(const __half* __restrict__ Kh, const __half* __restrict__ Vh, const Src& src,
                      int k0, int k1, float c, int lane, TileState& st, char* lds) {
    static_assert(kPipe == kPipeLdsK, "fp16 pipeline");
    run_ldsk(Kh, Vh, src, k0, k1, c, lane, st, lds);
  }

  // (see CoreF32T::run_range)
  template <typename Src>
  __device__ void run_range(const __half* __restrict__ Kh, const __half* __restrict__ Vh, const Src& src, int k0, int k1,
                            int longest, float c, int lane, TileState& st, char* lds) {
    run_ldsk(Kh, Vh, src, k0, k1, c, lane, st, lds);
    for (int k = k1 - k0; k < longest; ++k) __syncthreads();
  }

  __device__ static void store_row(__half* Orow, const TileState& st, float inv, float w_prev,
                                   bool accumulate, int h) {
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        uint2* dst = reinterpret_cast<uint2*>(Orow + cb * 32 + 8 * g + 4 * h);
        float v[4] = {st.o[cb][4 * g] * inv, st.o[cb][4 * g + 1] * inv, st.o[cb][4 * g + 2] * inv,
                      st.o[cb][4 * g + 3] * inv};
        if (accumulate) {
          const uint2 old = *dst;
          const __half2 o01 = __builtin_bit_cast(__half2, old.x), o23 = __builtin_bit_cast(__half2, old.y);
          v[0] = __builtin_fmaf(w_prev, __low2float(o01), v[0]);
          v[1] = __builtin_fmaf(w_prev, __high2float(o01), v[1]);
          v[2] = __builtin_fmaf(w_prev, __low2float(o23), v[2]);
          v[3] = __builtin_fmaf(w_prev, __high2float(o23), v[3]);
        }
        uint2 w;
        w.x = __builtin_bit_cast(uint32_t, __floats2half2_rn(v[0], v[1]));
        w.y = __builtin_bit_cast(uint32_t, __floats2half2_rn(v[2], v[3]));
        *dst = w;
      }
  }

  // The whole tile, normalised, in row order: tensor rows row0 + r * row_step, r < n_rows.
  // A lane holds fragments of its own query's row, so store_row touches 32 rows with 16 bytes
  // each per instruction, eight times; here the tile goes through the wavefront's LDS instead
  // (rows kTilePitch bytes apart, which spreads the writes over the banks) and leaves as whole
  // 128-byte rows, eight per instruction.  lds = kTileBytes bytes no copy is in flight to.
  // (Workloads 3, 4 and 5: 8 to 10 % off the kernel time.)
  static constexpr bool kTileStore = true;
  static constexpr int kTilePitch = 64 * 2 + 16;
  static constexpr int kTileBytes = kTile * kTilePitch;
  __device__ static void store_tile(__half* Oh, int64_t row0, int64_t row_step, int n_rows,
                                    const TileState& st, float inv, int lane, char* lds) {
    const int n = lane & 31, h = lane >> 5;
    __builtin_amdgcn_wave_barrier();     // the last block's reads of the staged blocks are done
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        uint2 w;
        w.x = __builtin_bit_cast(uint32_t, __floats2half2_rn(st.o[cb][4 * g] * inv, st.o[cb][4 * g + 1] * inv));
        w.y = __builtin_bit_cast(uint32_t,
                                 __floats2half2_rn(st.o[cb][4 * g + 2] * inv, st.o[cb][4 * g + 3] * inv));
        *reinterpret_cast<uint2*>(lds + n * kTilePitch + (cb * 32 + 8 * g + 4 * h) * 2) = w;
      }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = (lane >> 3) + 8 * i;
      const uint4 v = *reinterpret_cast<const uint4*>(lds + r * kTilePitch + (lane & 7) * 16);
      if (r < n_rows)
        // (written once and not read again by this call: a streaming store keeps the L2 for K and V)
        __builtin_nontemporal_store(__builtin_bit_cast(half8, v),
                                    reinterpret_cast<half8*>(Oh + (row0 + r * row_step) * kHeadDim + (lane & 7) * 8));
    }
  }

  // The same for a call that continues an earlier state: O = w_prev O + inv acc on the rows r_lo <= r <
  // n_rows (inv and w_prev are those of the lane's query).  The tile passes through LDS in fp32 and
  // the earlier rows are read and written whole, where store_row moves 16 bytes of 32 rows per
  // instruction (the non-local call of that mask: 25 us off).  lds = kCarryBytes bytes.
  static constexpr int kCarryPitch = 64 * 4 + 16;
  static constexpr int kCarryBytes = kTile * kCarryPitch;
  __device__ static void store_tile_carry(__half* Oh, int64_t row0, int r_lo, int n_rows, const TileState& st, float inv,
                                          float w_prev, int lane, char* lds) {
    const int n = lane & 31, h = lane >> 5;
    __builtin_amdgcn_wave_barrier();     // the last block's reads of the staged blocks are done
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<float4*>(lds + n * kCarryPitch + (cb * 32 + 8 * g + 4 * h) * 4) =
            make_float4(st.o[cb][4 * g] * inv, st.o[cb][4 * g + 1] * inv, st.o[cb][4 * g + 2] * inv, st.o[cb][4 * g + 3] * inv);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = (lane >> 3) + 8 * i;
      const float w = __shfl(w_prev, r, kWave);
      const float4 a = reinterpret_cast<const float4*>(lds + r * kCarryPitch + (lane & 7) * 32)[0];
      const float4 b = reinterpret_cast<const float4*>(lds + r * kCarryPitch + (lane & 7) * 32)[1];
      if (r < r_lo || r >= n_rows) continue;
      half8* at = reinterpret_cast<half8*>(Oh + (row0 + r) * kHeadDim + (lane & 7) * 8);
      const half8 old = *at;
      const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
      half8 out;
#pragma unroll
      for (int e = 0; e < 8; ++e) out[e] = (_Float16)__builtin_fmaf(w, (float)old[e], v[e]);
      __builtin_nontemporal_store(out, at);
    }
  }
};
using CoreF16 = CoreF16T<kHeadDim>;

// ---- fp32 storage, split-precision products -----------------------------------------------------
// Every fp32 operand x is written as hi + lo with hi = fp16(x) and lo = fp16(x - hi) (x - hi is
// exact in fp32), and a product a.b is evaluated as hi_a.hi_b + hi_a.lo_b + lo_a.hi_b on the
// fp16 matrix cores, all three terms into the same fp32 accumulator.  The dropped term
// lo_a.lo_b and the rounding of lo are below 2^-22 |a.b|, the size of an fp32 rounding error,
// so results match the kernels that hold every bit of the operands (CoreF32T: 48 matrix instructions
// per block) to their tolerance, with 24 (768 cycles).  lo is a subnormal fp16
// number for |x| < 0.25 (the matrix cores do not flush them); below |x| ~ 2^-13 it loses bits,
// an absolute error of at most 2^-25 per operand.  Inputs must lie inside the fp16 range
// (|x| < 65504); the caller opts in (SGA_PATH_TILE_SPLIT).
// K and V blocks travel global -> LDS as raw fp32 (as in CoreF16T::run_ldsk); K is split when
// its fragment is read, V is split in registers and written back over its own staged block as
// two row-major fp16 blocks, which the PV products read with the LDS transpose read.
struct CoreSplit {
  using Stage = StageMap<float>;
  static constexpr int kBlockBytes = kTile * kHeadDim * 4;
  half8 qh[4], ql[4];   // Q[query n][h*32 + 8s .. +7], high and low parts

  // Two values at a time: hi = fp16(x) packed into one register, x - hi by the mixed-precision
  // fma (the fp16 operand is read straight out of the packed pair, no conversion back), and the
  // remainders packed again: four instructions per pair.
  __device__ static void split2(float x0, float x1, half2v& hi, half2v& lo) {
    hi = half2v{(_Float16)x0, (_Float16)x1};
    const uint32_t hp = __builtin_bit_cast(uint32_t, hi);
    float r0, r1;
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r0) : "v"(hp), "v"(x0));
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r1) : "v"(hp), "v"(x1));
    lo = half2v{(_Float16)r0, (_Float16)r1};
  }

  __device__ static void split8(const float* x, half8& hi, half8& lo) {
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      half2v h2, l2;
      split2(x[e], x[e + 1], h2, l2);
      hi[e] = h2[0]; hi[e + 1] = h2[1];
      lo[e] = l2[0]; lo[e + 1] = l2[1];
    }
  }

  __device__ void load_q(const float* Qrow, int h, bool negate) {
    float q[32];
    const float4* src = reinterpret_cast<const float4*>(Qrow + h * 32);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const float4 v = src[t];
      q[4 * t] = v.x; q[4 * t + 1] = v.y; q[4 * t + 2] = v.z; q[4 * t + 3] = v.w;
    }
    if (negate) {
#pragma unroll
      for (int t = 0; t < 32; ++t) q[t] = -q[t];
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) split8(q + 8 * s, qh[s], ql[s]);
  }

  // kf[t] = K[key n][h*32 + t] out of the staged block.  The global -> LDS copy moved keys
  // 4i..4i+3 per instruction, 16 lanes per 256-byte row (whole cache lines), and stored the
  // sixteen 16-byte chunks of a row XOR-swizzled: chunk c of key r lives at chunk slot
  // c ^ (r & 15).  This read (each lane 128 contiguous bytes of its own key row, 16 at a time)
  // then spreads 8 consecutive lanes over the 8 groups of 4 banks instead of hitting one.
  __device__ static void read_k(const char* ldsk, int n, int h, float (&kf)[32]) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int slot = (8 * h + j) ^ (n & 15);
      const float4 v = *reinterpret_cast<const float4*>(ldsk + (n * 16 + slot) * 16);
      kf[4 * j] = v.x; kf[4 * j + 1] = v.y; kf[4 * j + 2] = v.z; kf[4 * j + 3] = v.w;
    }
  }

  template <int kPipe>
  static constexpr int lds_bytes() { return 2 * kBlockBytes; }

  template <int kPipe, typename Src>
  __device__ void run(const float* __restrict__ Kh, const float* __restrict__ Vh, const Src& src,
                      int k0, int k1, float c, int lane, TileState& st, char* lds) {
    if (k0 >= k1) return;
    const int n = lane & 31, h = lane >> 5;
    Stage sm;
    sm.init(src.key_stride(), lane);
    char* ldsk = lds;
    char* ldsv = lds + kBlockBytes;
    BlockInfo b = src.get(k0, n);
    BlockInfo b1 = src.get(k0 + 1 < k1 ? k0 + 1 : k0, n);
    src.resolve(b);
    __builtin_amdgcn_wave_barrier();     // reads of both buffers by an earlier work item are done
    sm.stage_k(Kh, b, lane, ldsk);
    // this lane's part of the row-major staged V block: copy i moved 16 bytes to dst + i*1024 + lane*16
    const int lr = lane >> 4, lc = lane & 15;
    const int i16 = lane & 15, grp16 = (lane >> 4) & 1;
    const char* vt = ldsv + (4 * h + (i16 >> 2)) * (kHeadDim * 2) + (grp16 * 16 + 4 * (i16 & 3)) * 2;
    for (int k = k0; k < k1; ++k) {
      const bool more = k + 1 < k1;      // wave-uniform
      src.resolve(b1);
      __builtin_amdgcn_wave_barrier();   // the previous block's reads of the V buffer are done
      sm.stage_v(Vh, b, lane, ldsv);
      BlockInfo b2 = b1;
      if (k + 2 < k1) b2 = src.get(k + 2, n);
      wait_k_block<8, Src::kGetLoads>(k + 2 < k1);   // K block k: older than the V copies (and the record loads)
      __builtin_amdgcn_wave_barrier();
      half8 kh[4], kl[4];
      {
        float kf[32];
        read_k(ldsk, n, h, kf);
        wait_lds_reads();                // the K buffer may be overwritten now
        __builtin_amdgcn_wave_barrier();
        if (more) sm.stage_k(Kh, b1, lane, ldsk);
#pragma unroll
        for (int s = 0; s < 4; ++s) split8(kf + 8 * s, kh[s], kl[s]);
      }
      floatx16 sacc = {0};
#pragma unroll
      for (int s = 0; s < 4; ++s) {     // smallest terms first
        sacc = __builtin_amdgcn_mfma_f32_32x32x16_f16(kl[s], qh[s], sacc, 0, 0, 0);
        sacc = __builtin_amdgcn_mfma_f32_32x32x16_f16(kh[s], ql[s], sacc, 0, 0, 0);
      }
#pragma unroll
      for (int s = 0; s < 4; ++s)
        sacc = __builtin_amdgcn_mfma_f32_32x32x16_f16(kh[s], qh[s], sacc, 0, 0, 0);
      float p[16];
      softmax_block(sacc, c, b, h, st, p);
      // V block k (and any record load after it) is older than the 8 K copies issued above (if any)
      if (more) wait_loads_except<8>(); else wait_loads_except<0>();
      b = b1;
      b1 = b2;
      __builtin_amdgcn_wave_barrier();
      {
        // split the staged fp32 V block in place: rows 4i + lr, channels 4*lc .. +3 per copy i
        float vraw[32];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float4 v = *reinterpret_cast<const float4*>(ldsv + i * 1024 + lane * 16);
          vraw[4 * i] = v.x; vraw[4 * i + 1] = v.y; vraw[4 * i + 2] = v.z; vraw[4 * i + 3] = v.w;
        }
        wait_lds_reads();
        __builtin_amdgcn_wave_barrier();   // every lane holds its part: the block may be overwritten
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          half4 vh, vl;
#pragma unroll
          for (int e = 0; e < 4; e += 2) {
            half2v h2, l2;
            split2(vraw[4 * i + e], vraw[4 * i + e + 1], h2, l2);
            vh[e] = h2[0]; vh[e + 1] = h2[1];
            vl[e] = l2[0]; vl[e + 1] = l2[1];
          }
          char* row = ldsv + (4 * i + lr) * (kHeadDim * 2) + lc * 8;
          *reinterpret_cast<half4*>(row) = vh;
          *reinterpret_cast<half4*>(row + kTile * kHeadDim * 2) = vl;
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);   // LDS writes have landed
        __builtin_amdgcn_wave_barrier();
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        half8 ph, pl;
        split8(p + 8 * u, ph, pl);
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
          const char* a0 = vt + (16 * u) * (kHeadDim * 2) + cb * 64;
          const half4 hlo = CoreF16::read_vt(a0), hhi = CoreF16::read_vt(a0 + 8 * (kHeadDim * 2));
          const half4 llo = CoreF16::read_vt(a0 + kTile * kHeadDim * 2);
          const half4 lhi = CoreF16::read_vt(a0 + kTile * kHeadDim * 2 + 8 * (kHeadDim * 2));
          const half8 vh = {hlo[0], hlo[1], hlo[2], hlo[3], hhi[0], hhi[1], hhi[2], hhi[3]};
          const half8 vl = {llo[0], llo[1], llo[2], llo[3], lhi[0], lhi[1], lhi[2], lhi[3]};
          st.o[cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vl, ph, st.o[cb], 0, 0, 0);
          st.o[cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vh, pl, st.o[cb], 0, 0, 0);
          st.o[cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vh, ph, st.o[cb], 0, 0, 0);
        }
      }
    }
  }

  __device__ static void store_row(float* Orow, const TileState& st, float inv, float w_prev,
                                   bool accumulate, int h) {
    CoreF32::store_row(Orow, st, inv, w_prev, accumulate, h);
  }
};

template <typename T> struct CoreOf;
template <> struct CoreOf<float> { using type = CoreF32; };
template <> struct CoreOf<__half> { using type = CoreF16; };
// the core that runs pipeline kPipe on storage type T
template <typename T, int kPipe> struct CoreFor { using type = typename CoreOf<T>::type; };
template <> struct CoreFor<float, kPipeSplit> { using type = CoreSplit; };
// the core of a 64-channel slice of kD-wide rows
template <typename T, int kD> struct WideCoreOf;
template <int kD> struct WideCoreOf<float, kD> { using type = CoreF32T<kD>; };
template <int kD> struct WideCoreOf<__half, kD> { using type = CoreF16T<kD>; };

// Normalise and store the tile's rows (row(n) = tensor row of query n, < 0 if it does not exist).
template <typename T>
__device__ __forceinline__ void finish_tile(T* Oh, float* lse_h, int64_t row, int64_t lse_idx,
                                            bool exists, TileState& st, int h, bool accumulate) {
  const float l = st.l + other_half(st.l, h);
  if (!exists) return;
  const bool empty = !(l > 0.f);
  float inv = empty ? 0.f : 1.0f / l;
  float lse_row = empty ? -INFINITY : (st.m + __builtin_amdgcn_logf(l)) * kLn2;
  float w_prev = 0.f;
  if (accumulate) {    // both half-waves read the earlier lse before half-wave 0 replaces it
    const CarryWeights cw = carry_weights(lse_h[lse_idx], lse_row);
    inv *= cw.w_now;
    w_prev = cw.w_prev;
    lse_row = cw.lse;
  }
  CoreOf<T>::type::store_row(Oh + row * kHeadDim, st, inv, w_prev, accumulate, h);
  if (lse_h && h == 0) lse_h[lse_idx] = lse_row;
}

// finish_tile for a call that starts from the initial state, rows row0 + r * row_step with
// r < n_rows existing: the tile leaves in row order through lds (Core::store_tile).
template <typename T>
__device__ __forceinline__ void finish_tile_rows(T* Oh, float* lse_h, int64_t row0, int64_t row_step,
                                                 int n_rows, TileState& st, int lane, char* lds) {
  const int n = lane & 31, h = lane >> 5;
  const float l = st.l + other_half(st.l, h);
  const bool empty = !(l > 0.f);
  const float inv = empty ? 0.f : 1.0f / l;
  CoreOf<T>::type::store_tile(Oh, row0, row_step, n_rows, st, inv, lane, lds);
  if (lse_h && h == 0 && n < n_rows)
    lse_h[row0 + n * row_step] = empty ? -INFINITY : (st.m + __builtin_amdgcn_logf(l)) * kLn2;
}

// Un-normalised partial of a chunk: o[32][64], m[32], l[32].
__device__ __forceinline__ void store_partial(float* part, TileState& st, int n, int h) {
  const float l = st.l + other_half(st.l, h);
#pragma unroll
  for (int cb = 0; cb < 2; ++cb)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<float4*>(part + n * 64 + cb * 32 + 8 * g + 4 * h) =
          make_float4(st.o[cb][4 * g], st.o[cb][4 * g + 1], st.o[cb][4 * g + 2], st.o[cb][4 * g + 3]);
  if (h == 0) {
    part[kTile * 64 + n] = st.m;
    part[kTile * 64 + kTile + n] = l;
  }
}

// finish_tile for one 64-channel slice of a kD-wide tile (Oslice = first channel of the slice in
// the head's O).  Every slice wavefront holds the same (m, l); when the call continues an earlier
// state, all of them read the earlier lse before the workgroup barrier and slice 0 replaces it
// after it.
template <typename T, int kD>
__device__ __forceinline__ void finish_tile_wide(T* Oslice, float* lse_h, int64_t row, bool exists,
                                                 TileState& st, int h, int slice, bool accumulate) {
  const float l = st.l + other_half(st.l, h);
  const bool empty = !(l > 0.f);
  float inv = empty ? 0.f : 1.0f / l;
  float lse_row = empty ? -INFINITY : (st.m + __builtin_amdgcn_logf(l)) * kLn2;
  float w_prev = 0.f;
  if (accumulate) {
    if (exists) {
      const CarryWeights cw = carry_weights(lse_h[row], lse_row);
      inv *= cw.w_now;
      w_prev = cw.w_prev;
      lse_row = cw.lse;
    }
    __syncthreads();
  }
  if (!exists) return;
  CoreOf<T>::type::store_row(Oslice + row * kD, st, inv, w_prev, accumulate, h);
  if (lse_h && h == 0 && slice == 0) lse_h[row] = lse_row;
}

// Minimum (maximum) of v over lanes 0..31, as a wave-uniform value.  Data-parallel-primitive
// moves inside the 16-lane rows (a running minimum towards lane 15), then lane 15 of row 0 into
// row 1, and lane 31 holds the result: a chain of short vector instructions, where shuffles
// through the LDS crossbar cost a round trip each (this reduction sits in the block loop of the
// CSR -> tile pass, once per key block).
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_from(int v) {     // lanes without a source keep v
  return __builtin_amdgcn_update_dpp(v, v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ int first_half_min(int v) {
  int o;
  o = dpp_from<0x111, 0xf>(v); v = o < v ? o : v;    // row_shr:1
  o = dpp_from<0x112, 0xf>(v); v = o < v ? o : v;    // row_shr:2
  o = dpp_from<0x114, 0xf>(v); v = o < v ? o : v;    // row_shr:4
  o = dpp_from<0x118, 0xf>(v); v = o < v ? o : v;    // row_shr:8
  o = dpp_from<0x142, 0xa>(v); v = o < v ? o : v;    // row_bcast:15 into rows 1 and 3
  return __builtin_amdgcn_readlane(v, 31);
}
__device__ __forceinline__ int first_half_max(int v) {
  int o;
  o = dpp_from<0x111, 0xf>(v); v = o > v ? o : v;
  o = dpp_from<0x112, 0xf>(v); v = o > v ? o : v;
  o = dpp_from<0x114, 0xf>(v); v = o > v ? o : v;
  o = dpp_from<0x118, 0xf>(v); v = o > v ? o : v;
  o = dpp_from<0x142, 0xa>(v); v = o > v ? o : v;
  return __builtin_amdgcn_readlane(v, 31);
}

// First position in [lo, hi) of the sorted column list whose column is >= key.
__device__ __forceinline__ int64_t lower_bound_col(const int32_t* __restrict__ col, int64_t lo,
                                                   int64_t hi, int64_t key) {
  while (lo < hi) {
    const int64_t mid = lo + ((hi - lo) >> 1);
    if (col[mid] < key) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// Work item w -> (tile, item index within the tile, segments of the tile).  With S = seg_edges
// and f(t) = t + row_ptr[min(32t, L)] / S, tile t owns the items [f(t), f(t+1)); items with
// index >= segments are idle.
struct WorkId {
  int64_t tile;
  int32_t seg, nseg;       // seg >= nseg: idle
  bool together;           // see tile_cut
};

// (Called by a whole wavefront with the same w.)  f is increasing, and for masks of even density
// the item index is close to proportional to the tile index: the 64 lanes evaluate f at the 64
// tiles around that guess in one round of loads, and only a guess that misses this window falls
// back to galloping and bisection, one dependent load per step.
__device__ __forceinline__ WorkId locate_work(const int64_t* __restrict__ row_ptr, int64_t L, int sh,
                                              int64_t n_tiles, int64_t n_work, int64_t w, int lane) {
  int64_t g = (int64_t)((double)w * (double)n_tiles / (double)n_work);
  if (g >= n_tiles) g = n_tiles - 1;
  // (the guess errs upwards where rows with many edges come first: most of the window lies below it)
  int64_t base = g - 47;
  if (base + kWave > n_tiles) base = n_tiles - kWave;
  if (base < 0) base = 0;
  const int64_t tc = base + lane;
  const int64_t fc = tc < n_tiles ? work_first(row_ptr, L, sh, tc) : INT64_MAX;
  const uint64_t below = __builtin_amdgcn_ballot_w64(fc <= w);       // a prefix of the lanes
  const int n_below = __builtin_popcountll(below);
  int64_t lo, f0;
  if (n_below > 0 && (n_below < kWave || base + kWave >= n_tiles)) {
    lo = base + n_below - 1;
    f0 = __shfl(fc, n_below - 1, kWave);
  } else {
    int64_t hi;
    if (n_below > 0) {                 // beyond the window
      lo = base + kWave - 1;
      int64_t step = 1;
      hi = n_tiles;
      while (lo + step < n_tiles) {
        if (work_first(row_ptr, L, sh, lo + step) <= w) { lo += step; step <<= 1; }
        else { hi = lo + step; break; }
      }
    } else {                           // before it
      hi = base;
      int64_t step = 1;
      lo = 0;
      while (hi - step > 0) {
        if (work_first(row_ptr, L, sh, hi - step) > w) { hi -= step; step <<= 1; }
        else { lo = hi - step; break; }
      }
    }
    while (hi - lo > 1) {
      const int64_t mid = lo + ((hi - lo) >> 1);
      if (work_first(row_ptr, L, sh, mid) <= w) lo = mid; else hi = mid;
    }
    f0 = work_first(row_ptr, L, sh, lo);
  }
  const TileCut cut = tile_cut(row_ptr, L, sh, lo);
  WorkId id;
  id.tile = lo;
  id.seg = (int32_t)(w - f0);
  id.nseg = cut.nseg;
  id.together = cut.together;
  if (cut.together && cut.nseg > 1) {
    const int64_t j = w - cut.first;
    id.tile = (lo & ~int64_t(3)) + (j & 3);
    id.seg = j >= 0 && (j >> 2) < cut.nseg ? (int32_t)(j >> 2) : cut.nseg;
  }
  return id;
}

// ---- CSR -> tile graph ------------------------------------------------------------------------
// One wavefront per work item (a tile, or one key-block range of a tile with many edges);
// lane r < 32 walks row 32t + r.  A 32-way merge by key block id: every round takes the
// smallest block id at the head of any row and lets each row consume its columns inside that
// block into a 32-bit word.  A row whose remaining columns are consecutive integers (windows,
// global rows) is walked arithmetically without reading col_idx again, and so are rows of one shape (below);
// otherwise a run of consecutive columns up to the end of the block costs two loads, and only scattered columns
// are read one by one.
__global__ __attribute__((amdgpu_waves_per_eu(4, 4))) __launch_bounds__(256) void tile_analyze_kernel(const int64_t* __restrict__ row_ptr,
                                                           const int32_t* __restrict__ col_idx,
                                                           int64_t L, int32_t H, int32_t dtype,
                                                           int32_t d, void* ws, size_t ws_bytes) {
  const WorkspacePlan pl = plan_workspace(L, H, row_ptr[L], dtype, d);
  if (pl.total_bytes > ws_bytes) return;
  // per wavefront: the bit words of kBitmapBlocks key blocks, then of the 32 rows the first
  // unit of the window in one numbering, their positions in col_idx (low, high word) and their
  // numbers of columns inside the window
  __shared__ __attribute__((aligned(16))) uint32_t bitmap_all[4][kBitmapBlocks * kTile + 4 * kTile];
  const int lane = threadIdx.x & (kWave - 1);
  const int waves = blockDim.x / kWave;
  uint32_t* bm = bitmap_all[__builtin_amdgcn_readfirstlane(threadIdx.x / kWave)];
  char* base_ws = static_cast<char*>(ws);
  TileItem* items = reinterpret_cast<TileItem*>(base_ws + pl.off_items_rec);
  int32_t* tile_bad = reinterpret_cast<int32_t*>(base_ws + pl.off_tile_bad);
  int32_t* tile_pbase = reinterpret_cast<int32_t*>(base_ws + pl.off_tile_pbase);
  int32_t* pair_blk = reinterpret_cast<int32_t*>(base_ws + pl.off_pair_blk);
  uint32_t* pair_mask = reinterpret_cast<uint32_t*>(base_ws + pl.off_pair_mask);
  uint32_t* ctr = reinterpret_cast<uint32_t*>(ws);
  for (int64_t w = (int64_t)blockIdx.x * waves + threadIdx.x / kWave; w < pl.n_work;
       w += (int64_t)gridDim.x * waves) {
    WorkId id = locate_work(row_ptr, L, pl.seg_shift, pl.n_tiles, pl.n_work, w, lane);
    if (id.seg >= id.nseg) {          // spare item of a tile whose edge range crosses a multiple of S
      if (lane == 0) items[w].tile = -1;
      continue;
    }
    const int64_t t = id.tile;
    const int64_t row_first = t * kTile;
    const int64_t row_last = row_first + kTile < L ? row_first + kTile : L;
    const int64_t slot_t = row_ptr[row_first] / kPairEdges;
    const int64_t cap_t = row_ptr[row_last] / kPairEdges - slot_t;
    const int64_t cap = cap_t / id.nseg;
    const int64_t slot0 = slot_t + (int64_t)id.seg * cap;
    const int64_t row = row_first + lane;
    const bool active = lane < kTile && row < L;
    int64_t pos = active ? row_ptr[row] : 0;
    int64_t end = active ? row_ptr[row + 1] : 0;
    if (id.nseg > 1) {
      // this segment's share of the tile's key-block span
      const int first_c = pos < end ? col_idx[pos] : INT32_MAX;
      const int last_c = pos < end ? col_idx[end - 1] : -1;
      const int64_t bmin = first_half_min(first_c) >> 5;
      const int64_t bmax = first_half_max(last_c) >> 5;
      const int64_t span = bmax - bmin + 1;
      const int64_t B0 = bmin + span * id.seg / id.nseg;
      const int64_t B1 = bmin + span * (id.seg + 1) / id.nseg;
      if (pos < end && (int64_t)last_c - first_c == end - 1 - pos) {
        // the row is one run of consecutive columns (global-token rows): its share follows by
        // arithmetic instead of two binary searches over the column list
        const int64_t p0 = pos;
        const int64_t lo = B0 * kTile - first_c, hi = B1 * kTile - first_c;
        pos = p0 + (lo < 0 ? 0 : (lo > end - p0 ? end - p0 : lo));
        end = p0 + (hi < 0 ? 0 : (hi > end - p0 ? end - p0 : hi));
      } else {
        pos = lower_bound_col(col_idx, pos, end, B0 * kTile);
        end = lower_bound_col(col_idx, pos, end, B1 * kTile);
      }
    }
    // a row whose remaining columns are one run of consecutive integers needs no more loads;
    // the test is repeated with every column that starts a round (it costs nothing: the last
    // column is kept), so a row of a few runs turns arithmetic once its last run is reached
    int run_lo = 0, run_hi = -1;
    bool arith = false;
    const int64_t pos_first = pos;
    const int c_first = pos < end ? col_idx[pos] : -1;
    const int c_last = pos < end ? col_idx[end - 1] : -1;
    const int deg = (int)(end - pos < kScoutColumns + 1 ? end - pos : kScoutColumns + 1);
    const int deg0 = __builtin_amdgcn_readfirstlane(deg);
    const bool one_length = row_first + kTile <= L && deg0 > 1 && deg0 <= kScoutColumns && __all(lane >= kTile || deg == deg0);
    int c_second = 0, c_before_last = 0;                  // (requested with the former two)
    if (one_length && lane < kTile) {
      c_second = col_idx[pos + 1];
      c_before_last = col_idx[end - 2];
    }
    int nblk = 0;
    bool overflow = false;
    int consumed = 0;                   // edges of this lane's row in the blocks written so far
    int scattered = 0;                  // blocks so far in which some row's columns were read one by one
    bool by_bitmap = false;
    auto write_block = [&](int b, uint32_t word) {
      const bool full = __all(lane >= kTile || word == ~0u);
      if (lane < kTile) pair_mask[(slot0 + nblk) * kTile + lane] = word;
      if (lane == 0) pair_blk[slot0 + nblk] = b | (full ? kFullBit : 0);
      ++nblk;
    };
    // Every row is down to one run of consecutive columns lo .. hi (some) or to nothing: writes the rest of the list and
    // returns true if there is none, or if the runs' block ranges overlap or touch.  The remaining blocks then are
    // the whole range from the first to the last, and each row's word follows from its run alone: no minimum per block.
    auto close_runs = [&](bool some, int run_lo, int run_hi) -> bool {
      const int blo = first_half_min(some ? run_lo >> 5 : INT32_MAX);
      if (blo == INT32_MAX) return true;
      const int bhi = first_half_max(some ? run_hi >> 5 : -1);
      const int lo_max = first_half_max(some ? run_lo >> 5 : -1);
      const int hi_min = first_half_min(some ? run_hi >> 5 : INT32_MAX);
      if (lo_max > hi_min + 1) return false;
      for (int b = blo; b <= bhi; ++b) {
        if (nblk >= cap) {
          overflow = true;
          break;
        }
        const int lo = run_lo - (b << 5) > 0 ? run_lo - (b << 5) : 0;
        const int hi = run_hi - (b << 5) < 31 ? run_hi - (b << 5) : 31;
        write_block(b, some && lo <= hi ? (~0u >> (31 - hi)) & (~0u << lo) : 0u);
      }
      return true;
    };
    // A list that averages under kProbeEdges edges per block over its first kProbeBlocks blocks
    // is given up at once (scattered columns: the rows go to the per-row kernels) instead
    // of being walked until its slots run out.  Like the slot rule this depends on the mask
    // alone.
    auto too_thin = [&]() -> bool {
      if (nblk != kProbeBlocks) return false;
      int total = lane < kTile ? consumed : 0;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) total += __shfl_xor(total, off, kWave);
      return total < kProbeBlocks * kProbeEdges;
    };
    // Rows of one shape: as many columns in every row, in the same few runs of consecutive ones (block masks; global columns
    // beside a window).  The first row is read whole, with coalesced loads; of the others the first and last column of
    // each run, all requested together, show the rest, since a list is sorted and free of duplicates.  The list then
    // follows without another load: three dependent ones in place of two or more per block.  (BigBird mask of 64-token
    // blocks, L = 1,048,576, us of this kernel: 551 -> 385, 2.06 -> 1.53 GB of col_idx; it waits for memory, at
    // four wavefronts per SIMD: five and six spill and gain nothing, and a list written with scalar code where all rows are
    // equal, at 40 % fewer vector instructions, takes as long.  Looking ahead along each row by itself, at the ends of the
    // 2nd, 4th, 6th and 8th key block, 460: it brings in lines that are gone again before the walk reaches them.)
    // Scattered columns do not come here though the rows be of one length (it would cost their calls 1.2 us of 22 to 50): the
    // first or the last two columns of every row have to be neighbours.
    int n_runs = 0;
    if (one_length && !__all(lane >= kTile || c_last - c_first == deg - 1)) {
      if (__all(lane >= kTile || c_second - c_first == 1 || c_last - c_before_last == 1)) {
        const int64_t at0 = uniform64(pos);
        int cc[kScoutColumns / kWave];
#pragma unroll
        for (int k = 0; k < kScoutColumns / kWave; ++k) {
          const int e = k * kWave + lane;
          cc[k] = k * kWave < deg0 ? col_idx[at0 + (e < deg0 ? e : deg0 - 1)] : 0;
        }
        int at[kScoutRuns + 1];              // the runs' first entries (uniform)
#pragma unroll
        for (int k = 0; k < kScoutColumns / kWave; ++k) {
          if (k * kWave >= deg0) break;
          int before = __shfl_up(cc[k], 1, kWave);
          if (lane == 0) before = k > 0 ? __builtin_amdgcn_readlane(cc[k > 0 ? k - 1 : 0], kWave - 1) : INT32_MIN;
          uint64_t starts = __builtin_amdgcn_ballot_w64(k * kWave + lane < deg0 && cc[k] != before + 1);
          while (starts && n_runs <= kScoutRuns) {
            const int e = k * kWave + (int)__builtin_ctzll(starts);
            starts &= starts - 1;
#pragma unroll
            for (int i = 0; i < kScoutRuns; ++i)
              if (i == n_runs) at[i] = e;
            ++n_runs;
          }
        }
        if (n_runs <= kScoutRuns) {
          bool same = true;
          int lo[kScoutRuns], hi[kScoutRuns], len[kScoutRuns];
#pragma unroll
          for (int i = 0; i < kScoutRuns; ++i) {
            const int e = i < n_runs ? at[i] : 0;
            const int next = i + 1 < n_runs ? at[i + 1] : deg0;
            len[i] = (i < n_runs ? next : 1) - e;
            lo[i] = col_idx[(lane < kTile ? pos : at0) + e];
            hi[i] = col_idx[(lane < kTile ? pos : at0) + e + len[i] - 1];
          }
#pragma unroll
          for (int i = 0; i < kScoutRuns; ++i) {
            same = same && hi[i] - lo[i] == len[i] - 1;
          }
          same = __all(same);
          if (same) {
#pragma unroll
            for (int i = 0; i < kScoutRuns; ++i) {
              if (lane < kTile) bm[i * kTile + lane] = (uint32_t)lo[i];
              if (lane == 0) bm[kScoutRuns * kTile + i] = (uint32_t)len[i];
            }
          } else {
            n_runs = 0;
          }
        } else {
          n_runs = 0;
        }
      }
    }
    if (n_runs > 0) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // (one wavefront: its LDS operations complete in order)
      const int deg = lane < kTile ? (int)(end - pos) : 0;
      int i = lane < kTile ? 0 : n_runs;
      run_lo = c_first;
      run_hi = run_lo + (int)bm[kScoutRuns * kTile] - 1;
      while (true) {
        if (__all(i >= n_runs || c_last - run_lo == deg - consumed - 1) && close_runs(i < n_runs, run_lo, c_last)) break;
        const int b = first_half_min(i < n_runs ? run_lo >> 5 : INT32_MAX);
        if (b == INT32_MAX) break;
        if (nblk >= cap) {
          overflow = true;
          break;
        }
        uint32_t word = 0;
        while (i < n_runs && run_lo >> 5 == b) {
          const int last = (b << 5) + 31;
          word |= (~0u >> (31 - ((run_hi < last ? run_hi : last) & 31))) & (~0u << (run_lo & 31));
          if (run_hi > last) {
            run_lo = last + 1;
          } else if (++i < n_runs) {
            run_lo = (int)bm[i * kTile + lane];
            run_hi = run_lo + (int)bm[kScoutRuns * kTile + i] - 1;
          }
        }
        write_block(b, word);
        consumed += __builtin_popcount(word);
        if (too_thin()) {
          overflow = true;
          break;
        }
      }
    }
    while (n_runs == 0) {
      int cur = INT32_MAX;
      if (!arith && pos < end) {
        const int c0 = pos == pos_first ? c_first : col_idx[pos];
        if ((int64_t)c_last - c0 == end - 1 - pos) {
          arith = true;
          run_lo = c0;
          run_hi = c_last;
          pos = end;
        } else {
          cur = c0 >> 5;
        }
      }
      if (arith) cur = run_lo <= run_hi ? (run_lo >> 5) : INT32_MAX;
      if (__all(arith || pos >= end)) {
        // Every row is down to one run of consecutive columns (or to nothing).  If the runs'
        // block ranges overlap or touch, the remaining blocks are the whole range from the first
        // to the last, and each row's word follows from its run alone: no minimum per block.
        if (close_runs(arith && run_lo <= run_hi, run_lo, run_hi)) break;
      }
      const int b = first_half_min(cur);
      if (b == INT32_MAX) break;
      if (nblk >= cap) {
        overflow = true;
        break;
      }
      uint32_t word = 0;
      bool one_by_one = false;
      if (cur == b) {
        if (arith) {
          const int lo = run_lo & 31;
          const int hi = run_hi < (b << 5) + 31 ? (run_hi & 31) : 31;
          word = (~0u >> (31 - hi)) & (~0u << lo);
          run_lo = (b + 1) << 5;
        } else {
          // if the row's columns run consecutively up to the end of the block (or of the row),
          // one more load settles the whole word: the list is sorted and free of duplicates, so
          // equal ends mean every column in between is present
          const int c0 = col_idx[pos];
          const int lo = c0 & 31;
          const int64_t left = end - pos;
          const int cnt = left < 32 - lo ? (int)left : 32 - lo;
          if (col_idx[pos + cnt - 1] == c0 + cnt - 1) {
            word = (~0u >> (32 - cnt)) << lo;
            pos += cnt;
          } else {
            // the row's columns inside block b are the next entries of its sorted list: take
            // them four per load while four remain, then one by one
            one_by_one = true;
            bool more = true;
            while (more && pos + 4 <= end) {
              int cc[4];
              __builtin_memcpy(cc, col_idx + pos, 16);
#pragma unroll
              for (int t = 0; t < 4; ++t) {
                if (more && (cc[t] >> 5) == b) {
                  word |= 1u << (cc[t] & 31);
                  ++pos;
                } else {
                  more = false;
                }
              }
            }
            while (more && pos < end) {
              const int cc = col_idx[pos];
              if ((cc >> 5) != b) break;
              word |= 1u << (cc & 31);
              ++pos;
            }
          }
        }
      }
      write_block(b, word);
      consumed += __builtin_popcount(word);
      if (__any(one_by_one)) ++scattered;
      // Scattered columns in nearly all of the first blocks: the rest of the list is made by
      // the bitmap walk below (the same blocks and words, from coalesced loads, many in flight,
      // instead of a chain of dependent ones per row).
      if (nblk == kBitmapAfter && scattered >= kBitmapAfter - 1) {
        by_bitmap = true;
        break;
      }
      if (too_thin()) {
        overflow = true;
        break;
      }
    }
    if (by_bitmap) {
      // (a row walked arithmetically goes back to its position in the column list)
      if (arith) pos = end - (run_lo <= run_hi ? run_hi - run_lo + 1 : 0);
      uint32_t* first = bm + kBitmapBlocks * kTile;
      uint32_t* at_lo = first + kTile;
      uint32_t* at_hi = at_lo + kTile;
      uint32_t* count = at_hi + kTile;
      const int64_t nnz = row_ptr[L];
      while (true) {
        const int cur = pos < end ? col_idx[pos] >> 5 : INT32_MAX;
        const int b0 = first_half_min(cur);              // the window: key blocks b0 .. b0 + kBitmapBlocks - 1
        if (b0 == INT32_MAX) break;
#pragma unroll
        for (int k = 0; k < kBitmapBlocks * kTile / (4 * kWave); ++k)
          reinterpret_cast<uint4*>(bm)[k * kWave + lane] = uint4{0u, 0u, 0u, 0u};
        // where each row's columns inside the window end (at most one column per key)
        const int64_t reach = end - pos > kBitmapBlocks * kTile ? pos + kBitmapBlocks * kTile : end;
        const int64_t q = lower_bound_col(col_idx, pos, reach, ((int64_t)b0 + kBitmapBlocks) * kTile);
        const int cnt = (int)(q - pos);
        // The window's columns in units of 16 consecutive entries of one row, all units of the 32
        // rows in one numbering: a lane takes a unit with four 16-byte loads, combines the bits
        // that fall into the same word in registers, and adds each word to the bitmap with one
        // LDS atomic (neighbouring lanes hold different words, or at worst the same one).
        const int units = (cnt + 15) >> 4;
        int incl = units;
#pragma unroll
        for (int off = 1; off < kTile; off <<= 1) {
          const int up = __shfl_up(incl, off, kWave);
          if (lane >= off) incl += up;
        }
        const int total = __shfl(incl, kTile - 1, kWave);
        if (total == 0) break;                           // (cannot happen: the row that gave b0 has a column in the window)
        if (lane < kTile) {
          first[lane] = (uint32_t)(incl - units);
          at_lo[lane] = (uint32_t)pos;
          at_hi[lane] = (uint32_t)((uint64_t)pos >> 32);
          count[lane] = (uint32_t)cnt;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // (one wavefront: its LDS operations complete in order)
        for (int u0 = 0; u0 < total; u0 += kBitmapUnits * kWave) {
          int rr[kBitmapUnits], nn[kBitmapUnits];
          int cc[kBitmapUnits][16];
#pragma unroll
          for (int v = 0; v < kBitmapUnits; ++v) {
            const int unit = u0 + v * kWave + lane;
            const int uu = unit < total ? unit : total - 1;
            int r = 0;
#pragma unroll
            for (int st = kTile / 2; st > 0; st >>= 1)
              if ((int)first[r + st] <= uu) r += st;
            const int j = uu - (int)first[r];
            const int64_t at = (int64_t)(((uint64_t)at_hi[r] << 32) | at_lo[r]) + 16 * j;
            const int left = (int)count[r] - 16 * j;
            rr[v] = r;
            nn[v] = unit < total ? (left < 16 ? left : 16) : 0;
            if (at + 16 <= nnz) {
              __builtin_memcpy(cc[v], col_idx + at, 64);
            } else {
#pragma unroll
              for (int t = 0; t < 16; ++t) cc[v][t] = at + t < nnz ? col_idx[at + t] : 0;
            }
          }
#pragma unroll
          for (int v = 0; v < kBitmapUnits; ++v) {
            int held = -1;
            uint32_t word = 0;
#pragma unroll
            for (int t = 0; t < 16; ++t) {
              if (t < nn[v]) {
                const int k = (cc[v][t] >> 5) - b0;
                if (k != held) {
                  if (held >= 0) atomicOr(&bm[held * kTile + rr[v]], word);
                  held = k;
                  word = 0;
                }
                word |= 1u << (cc[v][t] & 31);
              }
            }
            if (held >= 0) atomicOr(&bm[held * kTile + rr[v]], word);
          }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        for (int k = 0; k < kBitmapBlocks; ++k) {
          const uint32_t word = lane < kTile ? bm[k * kTile + lane] : 0u;
          if (!__any(word != 0u)) continue;
          if (nblk >= cap) {
            overflow = true;
            break;
          }
          write_block(b0 + k, word);
          consumed += __builtin_popcount(word);
          if (too_thin()) {
            overflow = true;
            break;
          }
        }
        if (overflow) break;
        pos = q;
      }
    }
    bool gives_up = false;            // this item is the first of its tile to be given up
    if (lane == 0) {
      *reinterpret_cast<int4*>(items + w) = make_int4((int32_t)t, overflow ? -1 : nblk, id.seg, id.nseg);
      items[w].slot0 = slot0;
      // Segment items in groups of four consecutive items: the same segment of four tiles, or
      // four segments of one tile.  (The order of the list is that of arrival; it only orders
      // the claims of the attention kernel.)
      if (id.nseg > 1 && ((id.together ? (int)t : id.seg) & 3) == 0)
        items[atomicAdd(&ctr[kCtrMultiItems], 1u)].group = w;
      if (overflow && atomicOr(&tile_bad[t], 1) == 0) {
        gives_up = true;
        // (the per-row kernels walk this list instead of testing every row of the sequence)
        const uint32_t bi = atomicAdd(&ctr[kCtrTilesBad], 1u);
        reinterpret_cast<int32_t*>(base_ws + pl.off_bad_list)[bi] = (int32_t)t;
      }
      if (id.seg == 0 && id.nseg > 1) {
        // reserve the tile's partial slots; if the call needs more than exist, every
        // multi-segment tile goes to the gather path (all-or-nothing keeps runs reproducible)
        atomicAdd(&ctr[kCtrTilePartsNeeded], (uint32_t)id.nseg);
        const uint32_t first = atomicAdd(&ctr[kCtrTilePartsAlloc], (uint32_t)id.nseg);
        const int32_t pbase = (int64_t)first + id.nseg <= pl.cap_tparts ? (int32_t)first : -1;
        tile_pbase[t] = pbase;
        // the merge reads one record per tile instead of a chain of dependent loads
        const uint32_t mi = atomicAdd(&ctr[kCtrMultiTiles], 1u);
        if ((int64_t)mi < pl.cap_tparts)
          reinterpret_cast<int4*>(base_ws + pl.off_multi_tiles)[mi] = make_int4((int32_t)t, pbase, id.nseg, 0);
      }
    }
    // the tile's rows that the per-row kernels split (L > kSplitThreshold; see tile_parts_in_doubt)
    if (L > kSplitThreshold && !tile_parts_in_doubt(pl) && __any(gives_up))
      record_split_rows(row_ptr, row, lane < kTile && row < L, pl, ws);
  }
}

__device__ __forceinline__ bool tile_parts_fit(const WorkspacePlan& pl, const void* ws) {
  return (int64_t) reinterpret_cast<const uint32_t*>(ws)[kCtrTilePartsNeeded] <= pl.cap_tparts;
}

// Dynamic schedule: of n items of a head, claimant i (a wavefront or a workgroup) takes item i first
// and then claims from the head's counter, which hands out the items from `claimants` on.  Once n
// is passed every claimant fails exactly once, and the last to fail, the n-th claim in all, puts
// the counter back to zero: the next call on the same workspace starts from a clean schedule
// without a clearing launch of its own.  With no more items than claimants nobody touches the
// counter.  (Claims are atomic operations on one address, about 17 ns each: with a claim for every
// item and an exit counter they took 40 of the 67 us of 1,307 items.)  One lane calls.
__device__ __forceinline__ int64_t claim_next(uint32_t* work_next, int64_t n, uint32_t claimants) {
  const uint32_t c = atomicAdd(work_next, 1u);
  if (c == (uint32_t)n - 1) atomicExch(work_next, 0u);
  return (int64_t)claimants + c;
}

constexpr uint32_t kXcdRun = 4;   // consecutive workgroups of the static schedule that share an XCD

// Persistent wavefronts: every wavefront claims the next unprocessed work item of its head from
// a device counter until none is left (items are ordered long segments first, so the greedy
// order balances the load and no workgroup has to be re-launched between items).  A segment
// of a multi-segment tile leaves a partial state.
template <typename T, int kPipe>
__device__ __forceinline__ void tile_attend_body(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, T* __restrict__ O,
    float* __restrict__ lse, const int64_t* __restrict__ row_ptr, int64_t L, float scale, void* ws,
    size_t ws_bytes, int accumulate, char* lds_all) {
  constexpr int kLds = CoreFor<T, kPipe>::type::template lds_bytes<kPipe>();       // (lds_all: 4 of them)
  const int32_t H = (int32_t)gridDim.x;   // head-major grid: the long work items of every head are dispatched first
  const WorkspacePlan pl = plan_workspace(L, H, row_ptr[L], DtypeOf<T>::code);
  if (pl.total_bytes > ws_bytes) return;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int n = lane & 31, h = lane >> 5;
  char* lds = lds_all + wave * kLds;
  char* base_ws = static_cast<char*>(ws);
  // a negative scale is applied as a sign flip of Q (exact), so the kernels see c >= 0
  const bool negate = scale < 0.f;
  const float c = softmax_factor(scale);
  const TileItem* items = reinterpret_cast<const TileItem*>(base_ws + pl.off_items_rec);
  const int32_t* tile_bad = reinterpret_cast<const int32_t*>(base_ws + pl.off_tile_bad);
  const int32_t* tile_pbase = reinterpret_cast<const int32_t*>(base_ws + pl.off_tile_pbase);
  const bool parts_fit = tile_parts_fit(pl, ws);
  constexpr bool kDynamic = DtypeOf<T>::code == SGA_F32;
  // Workgroups go to the 8 XCDs (each with its own L2) round-robin in launch order.  The static
  // schedule hands every XCD runs of kXcdRun consecutive workgroups of one head, so that the key
  // blocks neighbouring tiles share (window blocks, global blocks) are fetched into one L2 instead
  // of several.  (gridDim.y is a multiple of 8 * kXcdRun for this schedule.)
  uint32_t head = blockIdx.x, ywg = blockIdx.y;
  if (!kDynamic && gridDim.y % (8 * kXcdRun) == 0) {
    const uint32_t lin = blockIdx.x + gridDim.x * blockIdx.y;
    const uint32_t xcd = lin & 7, slot = lin >> 3;
    const uint32_t v = ((slot / kXcdRun) * 8 + xcd) * kXcdRun + slot % kXcdRun;
    head = v / gridDim.y;
    ywg = v % gridDim.y;
  }
  const int64_t hoff = (int64_t)head * L * kHeadDim;
  uint32_t* work_next = reinterpret_cast<uint32_t*>(base_ws + pl.off_work_next) + head;
  // fp32 items are long (1,536 matrix-core cycles per block and the splits): wavefronts stay resident
  // and claim the next item of their head from a device counter (greedy balance, no re-launch gaps).
  // fp16 items are short and bound by the memory path: the 4 wavefronts of a workgroup take 4
  // neighbouring tiles at the same time (static stride), so that the key blocks they share are
  // fetched together and hit the CU's L1.
  int64_t w_static = (int64_t)ywg * 4 + wave;
  bool first = true;
  while (true) {
    int64_t w_cur;
    if constexpr (kDynamic) {
      const uint32_t claimants = gridDim.y * 4;
      w_cur = w_static;
      if (!first) {
        if (pl.n_work <= claimants) break;
        uint32_t claimed = 0;
        if (lane == 0) claimed = (uint32_t)claim_next(work_next, pl.n_work, claimants);
        w_cur = __builtin_amdgcn_readfirstlane(claimed);
      }
      first = false;
      if (w_cur >= pl.n_work) break;
    } else {
      w_cur = w_static;
      w_static += (int64_t)gridDim.y * 4;
      if (w_cur >= pl.n_work) break;
    }
    // the whole record in one uniform 32-byte read
    const int4 r0 = reinterpret_cast<const int4*>(items + w_cur)[0];
    const int64_t slot_raw = reinterpret_cast<const int64_t*>(items + w_cur)[2];
    const int32_t t = __builtin_amdgcn_readfirstlane(r0.x);
    const int32_t nblk = __builtin_amdgcn_readfirstlane(r0.y);
    const int32_t seg = __builtin_amdgcn_readfirstlane(r0.z);
    const int32_t nseg = __builtin_amdgcn_readfirstlane(r0.w);
    const int64_t slot0 = uniform64(slot_raw);
    if (t < 0 || nblk < 0) continue;         // idle item / list overflow: tile left to the gather path
    if (nseg > 1 && (!parts_fit || tile_bad[t])) continue;
    const int64_t row_first = (int64_t)t * kTile;
    ExplicitBlocks src{reinterpret_cast<const int32_t*>(base_ws + pl.off_pair_blk) + slot0,
                       reinterpret_cast<const uint32_t*>(base_ws + pl.off_pair_mask) + slot0 * kTile, L};
    const int64_t qrow = row_first + n;
    const bool exists = qrow < L;
    typename CoreFor<T, kPipe>::type core;
    core.load_q(Q + hoff + (exists ? qrow : L - 1) * kHeadDim, h, negate);
    TileState st;
    st.init();
    core.template run<kPipe>(K + hoff, V + hoff, src, 0, nblk, c, lane, st, lds);
    if (nseg > 1) {
      float* part = reinterpret_cast<float*>(base_ws + pl.off_tpartials) +
                    (((int64_t)tile_pbase[t] + seg) * H + head) * (int64_t)kTilePartialFloats;
      store_partial(part, st, n, h);
    } else if (accumulate || !CoreOf<T>::type::kTileStore) {
      finish_tile<T>(O + hoff, lse ? lse + (int64_t)head * L : nullptr, qrow, qrow, exists, st, h,
                     accumulate != 0);
    } else if constexpr (CoreOf<T>::type::kTileStore) {
      static_assert(CoreOf<T>::type::kTileBytes <= kLds, "output tile fits the wavefront's LDS");
      const int64_t left = L - row_first;
      finish_tile_rows<T>(O + hoff, lse ? lse + (int64_t)head * L : nullptr, row_first, 1,
                          left < kTile ? (int)left : kTile, st, lane, lds);
    }
  }
}

template <typename T, int kPipe>
__global__ __attribute__((amdgpu_waves_per_eu(2, 2))) __launch_bounds__(256) void tile_attend_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, T* __restrict__ O,
    float* __restrict__ lse, const int64_t* __restrict__ row_ptr, int64_t L, float scale, void* ws,
    size_t ws_bytes, int accumulate) {
  __shared__ __attribute__((aligned(16))) char lds[4 * CoreFor<T, kPipe>::type::template lds_bytes<kPipe>()];
  tile_attend_body<T, kPipe>(Q, K, V, O, lse, row_ptr, L, scale, ws, ws_bytes, accumulate, lds);
}

// fp16 storage: the same body held to the registers of four wavefronts per SIMD (the fp16 items
// are short and bound by the memory path: the fourth wavefront is worth more than the two
// registers the allocator would otherwise take beyond 128).
__global__ __attribute__((amdgpu_waves_per_eu(4, 4))) __launch_bounds__(256) void tile_attend_f16_kernel(
    const __half* __restrict__ Q, const __half* __restrict__ K, const __half* __restrict__ V,
    __half* __restrict__ O, float* __restrict__ lse, const int64_t* __restrict__ row_ptr, int64_t L,
    float scale, void* ws, size_t ws_bytes, int accumulate) {
  __shared__ __attribute__((aligned(16))) char lds[4 * CoreF16::lds_bytes<kPipeLdsK>()];
  tile_attend_body<__half, kPipeLdsK>(Q, K, V, O, lse, row_ptr, L, scale, ws, ws_bytes, accumulate, lds);
}

// Head dimensions 128 and 256: one workgroup of kD / 64 wavefronts per work item, wavefront w
// owning channels 64w .. 64w+63 (CoreF32T / CoreF16T with SliceExchange).  Workgroups stay
// resident and claim items from the head's counter like the fp32 kernel above; wavefront 0
// claims and the item index travels through LDS.
template <typename T, int kD, int kPipe>
__global__ __launch_bounds__(kD, 2) void tile_attend_wide_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, T* __restrict__ O,
    float* __restrict__ lse, const int64_t* __restrict__ row_ptr, int64_t L, float scale, void* ws,
    size_t ws_bytes, int accumulate) {
  using Core = typename WideCoreOf<T, kD>::type;
  constexpr int kSlices = kD / kHeadDim;
  constexpr int kLds = Core::template lds_bytes<kPipe>();
  __shared__ __attribute__((aligned(16))) char lds_all[kSlices * kLds + SliceExchange<kD>::kBytes];
  __shared__ uint32_t claim;
  const int32_t H = (int32_t)gridDim.x;
  const WorkspacePlan pl = plan_workspace(L, H, row_ptr[L], DtypeOf<T>::code, kD);
  if (pl.total_bytes > ws_bytes) return;
  const int lane = threadIdx.x & (kWave - 1);
  const int slice = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int n = lane & 31, h = lane >> 5;
  char* lds = lds_all + slice * kLds;
  char* base_ws = static_cast<char*>(ws);
  const bool negate = scale < 0.f;
  const float c = softmax_factor(scale);
  const TileItem* items = reinterpret_cast<const TileItem*>(base_ws + pl.off_items_rec);
  const int32_t* tile_bad = reinterpret_cast<const int32_t*>(base_ws + pl.off_tile_bad);
  const int32_t* tile_pbase = reinterpret_cast<const int32_t*>(base_ws + pl.off_tile_pbase);
  const bool parts_fit = tile_parts_fit(pl, ws);
  const int64_t head = blockIdx.x;
  const int64_t hoff = head * L * kD + slice * kHeadDim;   // this wavefront's slice of the head
  uint32_t* work_next = reinterpret_cast<uint32_t*>(base_ws + pl.off_work_next) + head;
  Core core;
  core.xchg.init(lds_all + kSlices * kLds, slice);
  for (bool first = true;; first = false) {
    int64_t w_cur = blockIdx.y;
    if (!first) {
      if (pl.n_work <= gridDim.y) break;
      __syncthreads();         // every wavefront has read the previous claim and left its item
      if (threadIdx.x == 0) claim = (uint32_t)claim_next(work_next, pl.n_work, gridDim.y);
      __syncthreads();
      w_cur = __builtin_amdgcn_readfirstlane(claim);
    }
    if (w_cur >= pl.n_work) break;
    const int4 r0 = reinterpret_cast<const int4*>(items + w_cur)[0];
    const int64_t slot_raw = reinterpret_cast<const int64_t*>(items + w_cur)[2];
    const int32_t t = __builtin_amdgcn_readfirstlane(r0.x);
    const int32_t nblk = __builtin_amdgcn_readfirstlane(r0.y);
    const int32_t seg = __builtin_amdgcn_readfirstlane(r0.z);
    const int32_t nseg = __builtin_amdgcn_readfirstlane(r0.w);
    const int64_t slot0 = uniform64(slot_raw);
    if (t < 0 || nblk < 0) continue;
    if (nseg > 1 && (!parts_fit || tile_bad[t])) continue;
    const int64_t row_first = (int64_t)t * kTile;
    ExplicitBlocks src{reinterpret_cast<const int32_t*>(base_ws + pl.off_pair_blk) + slot0,
                       reinterpret_cast<const uint32_t*>(base_ws + pl.off_pair_mask) + slot0 * kTile, L};
    const int64_t qrow = row_first + n;
    const bool exists = qrow < L;
    core.load_q(Q + hoff + (exists ? qrow : L - 1) * kD, h, negate);
    TileState st;
    st.init();
    core.template run<kPipe>(K + hoff, V + hoff, src, 0, nblk, c, lane, st, lds);
    if (nseg > 1) {
      float* part = reinterpret_cast<float*>(base_ws + pl.off_tpartials) +
                    ((((int64_t)tile_pbase[t] + seg) * H + head) * kSlices + slice) *
                        (int64_t)kTilePartialFloats;
      store_partial(part, st, n, h);
    } else {
      finish_tile_wide<T, kD>(O + hoff, lse ? lse + head * L : nullptr, qrow, exists, st, h, slice,
                              accumulate != 0);
    }
  }
}

// Merge of the multi-segment tiles of a prepared graph (see tile_merge_body; other calls merge in the launch
// of the leftover rows).
template <typename T, int kD>
__global__ __launch_bounds__(256) void tile_merge_kernel(T* __restrict__ O, float* __restrict__ lse,
                                                         const int64_t* __restrict__ row_ptr, int64_t L,
                                                         void* ws, size_t ws_bytes, int accumulate) {
  tile_merge_body<T, kD>(O, lse, row_ptr, L, ws, ws_bytes, accumulate, blockIdx.x, gridDim.x, blockIdx.z, gridDim.z);
}

// A workgroup's place among the window tiles.  Whole-sequence masks (seg_len = 0): residue class
// bid % s of the sequence, group bid / s of that class.  Block-diagonal masks (seg_len > 0: the
// 2-D dilated blocks of Section II-C, where the rows at in-block multiples of s attend each
// other inside every block of seg_len tokens): block bid / n_groups, the one class that starts
// at the block's first token, group bid % n_groups.  p = token of class index 0, Lc = tokens of
// the class; token = s * index + p in both cases.
struct WindowSlot {
  int64_t p, Lc, grp;
};
__device__ __forceinline__ bool locate_window_slot(int64_t bid, int64_t L, int64_t s, int64_t n_groups,
                                                   int64_t seg_len, WindowSlot& w) {
  if (seg_len > 0) {
    const int64_t base = (bid / n_groups) * seg_len;
    if (base >= L) return false;
    const int64_t len = L - base < seg_len ? L - base : seg_len;
    w.p = base;
    w.Lc = (len + s - 1) / s;
    w.grp = bid % n_groups;
  } else {
    if (bid >= n_groups * s) return false;
    w.p = bid % s;
    if (w.p >= L) return false;
    w.Lc = (L - w.p + s - 1) / s;
    w.grp = bid / s;
  }
  return true;
}

// Rows of a 2-D dilated mask that are no in-block multiple of the stride have no neighbour:
// O = 0, lse = -inf (Algorithm 1's initial state).  One thread per 16 bytes of O.
template <typename T>
__global__ __launch_bounds__(256) void clear_unselected_rows_kernel(T* __restrict__ O,
                                                                    float* __restrict__ lse, int64_t L,
                                                                    int64_t H, int32_t d, int64_t b,
                                                                    int64_t s) {
  const int64_t per_row = d * (int64_t)sizeof(T) / 16;
  const int64_t total = H * L * per_row;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t row = (i / per_row) % L;
    if (((row % b) % s) == 0) continue;
    reinterpret_cast<uint4*>(O)[i] = make_uint4(0, 0, 0, 0);
    if (lse && i % per_row == 0) lse[i / per_row] = -INFINITY;
  }
}

// Implicit window masks.  grid.x = workgroups (4 tiles each) over all residue classes, grid.y = head.
// Workgroups are dealt round-robin to the 8 XCDs, each with its own L2, and neighbouring tiles
// share most of their K/V rows, so the linear workgroup id is remapped to give every XCD one
// contiguous range of the sequence; inside it consecutive workgroups alternate between the
// residue classes, so that the interleaved rows of all classes are touched together.
template <typename T, int kPipe>
__global__ __attribute__((amdgpu_waves_per_eu(2, 2))) __launch_bounds__(256) void tile_window_kernel(const T* __restrict__ Q,
                                                          const T* __restrict__ K,
                                                          const T* __restrict__ V, T* __restrict__ O,
                                                          float* __restrict__ lse, int64_t L, int64_t W,
                                                          int64_t s, int64_t n_groups, float scale,
                                                          int accumulate, int64_t seg_len, int nsplit,
                                                          float* __restrict__ parts) {
  constexpr int kLds = CoreFor<T, kPipe>::type::template lds_bytes<kPipe>();
  __shared__ __attribute__((aligned(16))) char lds_all[4 * kLds];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int n = lane & 31, h = lane >> 5;
  char* lds = lds_all + wave * kLds;
  // gridDim.x is a multiple of 8: XCD x handles the workgroups [x*chunk, (x+1)*chunk)
  const int64_t chunk = gridDim.x / 8;
  const int64_t bid_all = (int64_t)(blockIdx.x % 8) * chunk + blockIdx.x / 8;
  // (nsplit > 1: nsplit consecutive workgroups share four tiles, each takes one range of their
  // key blocks and leaves partial states for window_merge_kernel)
  const int64_t bid = bid_all / nsplit;
  const int part = (int)(bid_all - bid * nsplit);
  WindowSlot slot;
  if (!locate_window_slot(bid, L, s, n_groups, seg_len, slot)) return;
  const int64_t p = slot.p, Lc = slot.Lc;
  const int64_t u0 = (slot.grp * 4 + wave) * kTile;
  if (u0 >= Lc) return;
  const int64_t hd = blockIdx.y;
  const int64_t hoff = hd * L * kHeadDim;
  const int64_t vlo = u0 - W > 0 ? u0 - W : 0;
  const int64_t vhi = u0 + kTile - 1 + W < Lc - 1 ? u0 + kTile - 1 + W : Lc - 1;
  WindowBlocks src{vlo, Lc, s, p, u0, W};
  const int nblk = (int)((vhi - vlo) / kTile + 1);
  const int64_t u = u0 + n;
  const bool exists = u < Lc;
  const int64_t qrow = s * (exists ? u : Lc - 1) + p;
  typename CoreFor<T, kPipe>::type core;
  core.load_q(Q + hoff + qrow * kHeadDim, h, scale < 0.f);
  TileState st;
  st.init();
  if (nsplit > 1) {
    const int k0 = (int)((int64_t)nblk * part / nsplit), k1 = (int)((int64_t)nblk * (part + 1) / nsplit);
    core.template run<kPipe>(K + hoff, V + hoff, src, k0, k1, softmax_factor(scale), lane, st, lds);
    store_partial(parts + (((bid * 4 + wave) * gridDim.y + hd) * nsplit + part) * (int64_t)kTilePartialFloats,
                  st, n, h);
    return;
  }
  core.template run<kPipe>(K + hoff, V + hoff, src, 0, nblk, softmax_factor(scale), lane, st, lds);
  if (accumulate || !CoreOf<T>::type::kTileStore) {
    finish_tile<T>(O + hoff, lse ? lse + hd * L : nullptr, qrow, qrow, exists, st, h, accumulate != 0);
  } else if constexpr (CoreOf<T>::type::kTileStore) {
    static_assert(CoreOf<T>::type::kTileBytes <= kLds, "output tile fits the wavefront's LDS");
    finish_tile_rows<T>(O + hoff, lse ? lse + hd * L : nullptr, s * u0 + p, s,
                        Lc - u0 < kTile ? (int)(Lc - u0) : kTile, st, lane, lds);
  }
}

// The state of a wavefront, left in its LDS for another one to add (kShareBytes of it).
constexpr int kShareBytes = 34 * kWave * 4;
__device__ __forceinline__ void leave_state(const TileState& st, char* lds, int lane) {
  wait_loads_except<0>();                // (nothing of this wavefront still lands in its LDS)
  wait_lds_reads();
  __builtin_amdgcn_wave_barrier();
  float* mine = reinterpret_cast<float*>(lds) + lane;
  mine[0] = st.m;
  mine[kWave] = st.l;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    mine[(2 + r) * kWave] = st.o[0][r];
    mine[(18 + r) * kWave] = st.o[1][r];
  }
}

// Adds the states left at lds + kStep, lds + 2 kStep, ... to st (one common maximum, so that each is scaled once).  Sum: double
// for fp32 tiles of four blocks, whose ranges are so short that the additions and weights of the merge, rounded to 32 bits, would
// show.  (Error against 64 bits, means of 24 inputs, W = 33: d = 64 one range 1.297e-7, two in 32 bits 1.310e-7, in
// 64 1.289e-7; d = 128 one range 1.316e-7, four 1.318e-7, 1.276e-7; from five blocks on 32 bits are enough, W = 52 1.361e-7, 1.357e-7.
// 64 bits cost 0.23 us of 9.3 for two states, 0.5 of 11 for four.)
template <int kShare, int kStep, typename Sum>
__device__ __forceinline__ void add_states(TileState& st, const char* lds, int lane) {
  const float* other = reinterpret_cast<const float*>(lds) + lane;
  constexpr int step = kStep / 4;
  float m = st.m;
  Sum weight[kShare];
#pragma unroll
  for (int w = 1; w < kShare; ++w) m = __builtin_fmaxf(m, other[w * step]);
  auto weigh = [&](float of) -> Sum {
    if constexpr (sizeof(Sum) == 8) return exp2((Sum)of - (Sum)m);
    else return __builtin_amdgcn_exp2f(of - m);
  };
  weight[0] = weigh(st.m);
#pragma unroll
  for (int w = 1; w < kShare; ++w) weight[w] = weigh(other[w * step]);
  st.m = m;
  auto sum = [&](float& own, int at) {
    Sum x = own * weight[0];
#pragma unroll
    for (int w = 1; w < kShare; ++w) x = __builtin_elementwise_fma((Sum)other[w * step + at], weight[w], x);
    own = (float)x;
  };
  sum(st.l, kWave);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    float own[2] = {st.o[0][r], st.o[1][r]};
    sum(own[0], (2 + r) * kWave);
    sum(own[1], (18 + r) * kWave);
    st.o[0][r] = own[0];
    st.o[1][r] = own[1];
  }
}

// fp32 windows of calls that leave most SIMDs without a second wavefront: kShare wavefronts (2 or 4) take a tile, each a
// range of its key blocks, and the first one merges their states through LDS, in wavefront order (see window_share).
template <int kShare, typename Sum>
__global__ __attribute__((amdgpu_waves_per_eu(2, 2))) __launch_bounds__(256) void tile_window_share_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V, float* __restrict__ O,
    float* __restrict__ lse, int64_t L, int64_t W, int64_t s, int64_t n_groups, float scale, int accumulate,
    int64_t seg_len) {
  constexpr int kLds = CoreF32::lds_bytes<kPipeRegK>(), kTiles = 4 / kShare;
  static_assert(kShareBytes <= kLds, "a wavefront's state fits its LDS");
  __shared__ __attribute__((aligned(16))) char lds_all[4 * kLds];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int n = lane & 31, h = lane >> 5, part = wave % kShare;
  char* lds = lds_all + wave * kLds;
  const int64_t chunk = gridDim.x / 8;
  const int64_t bid = (int64_t)(blockIdx.x % 8) * chunk + blockIdx.x / 8;
  WindowSlot slot;
  if (!locate_window_slot(bid, L, s, n_groups, seg_len, slot)) return;      // (the whole workgroup leaves)
  const int64_t p = slot.p, Lc = slot.Lc;
  const int64_t u0 = (slot.grp * kTiles + wave / kShare) * kTile;
  const bool active = u0 < Lc;                     // (a wavefront without queries still meets the barrier)
  const int64_t hd = blockIdx.y;
  const int64_t hoff = hd * L * kHeadDim;
  const int64_t u = u0 + n;
  const bool exists = u < Lc;
  const int64_t qrow = s * (exists ? u : Lc - 1) + p;
  TileState st;
  st.init();
  if (active) {
    const int64_t vlo = u0 - W > 0 ? u0 - W : 0;
    const int64_t vhi = u0 + kTile - 1 + W < Lc - 1 ? u0 + kTile - 1 + W : Lc - 1;
    const WindowBlocks src{vlo, Lc, s, p, u0, W};
    const int nblk = (int)((vhi - vlo) / kTile + 1);
    CoreF32 core;
    core.load_q(Q + hoff + qrow * kHeadDim, h, scale < 0.f);
    core.run<kPipeRegK>(K + hoff, V + hoff, src, nblk * part / kShare, nblk * (part + 1) / kShare, softmax_factor(scale),
                        lane, st, lds);
  }
  if (part > 0) leave_state(st, lds, lane);
  __syncthreads();
  if (part > 0 || !active) return;
  add_states<kShare, kLds, Sum>(st, lds, lane);
  finish_tile<float>(O + hoff, lse ? lse + hd * L : nullptr, qrow, qrow, exists, st, h, accumulate != 0);
}

// ---- fp32 storage, key blocks shared by a workgroup ------------------------------------------------
// Four tiles (one per wavefront) walk one list of key blocks together.  Each block of K and V is
// loaded once per workgroup, split once (16 values per thread), and left in LDS as six planes of
// 16-bit parts in the layouts CoreF16 reads: three of K (32 keys x 64 channels, the 16-byte chunks
// of a row swizzled), three of V (row-major, for the LDS transpose read).  The wavefronts take
// their matrix-core operands from there.  Splitting a block costs about as much vector time as its
// products cost matrix time; shared by four tiles it is a quarter of that.
struct SharedBlock {
  static constexpr int kPlane = kTile * kHeadDim * 2;
  static constexpr int kValues = 3 * kPlane;               // offset of the first V plane
  static constexpr int kBytes = 6 * kPlane;
  float k[8], v[8];        // this thread's share: key threadIdx.x / 8, channels 8 * (threadIdx.x % 8) ..
  __device__ __forceinline__ void load(const char* k_at, const char* v_at) {
    const float4 a = reinterpret_cast<const float4*>(k_at)[0], b = reinterpret_cast<const float4*>(k_at)[1];
    const float4 c = reinterpret_cast<const float4*>(v_at)[0], d = reinterpret_cast<const float4*>(v_at)[1];
    k[0] = a.x; k[1] = a.y; k[2] = a.z; k[3] = a.w; k[4] = b.x; k[5] = b.y; k[6] = b.z; k[7] = b.w;
    v[0] = c.x; v[1] = c.y; v[2] = c.z; v[3] = c.w; v[4] = d.x; v[5] = d.y; v[6] = d.z; v[7] = d.w;
  }
  __device__ __forceinline__ void store(char* planes) const {
    const int r = threadIdx.x >> 3, j = threadIdx.x & 7;
    SplitOperand x;
    x.split(k);
    char* at = planes + (r * 8 + (j ^ (r & 7))) * 16;
    *reinterpret_cast<bf16x8*>(at) = x.hi;
    *reinterpret_cast<bf16x8*>(at + kPlane) = x.mid;
    *reinterpret_cast<bf16x8*>(at + 2 * kPlane) = x.lo;
    SplitOperand y;
    y.split(v);
    at = planes + kValues + r * (kHeadDim * 2) + j * 16;
    *reinterpret_cast<bf16x8*>(at) = y.hi;
    *reinterpret_cast<bf16x8*>(at + kPlane) = y.mid;
    *reinterpret_cast<bf16x8*>(at + 2 * kPlane) = y.lo;
  }
  // One block step of a wavefront's tile against the planes of a block (the operations of
  // CoreF32T::run_split in the same order: the same result bit for bit).
  __device__ static __forceinline__ void attend(CoreF32& core, const char* planes, const BlockInfo& b, float c, int lane,
                                                TileState& st) {
    const int n = lane & 31, h = lane >> 5;
    SplitOperand k3[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const char* at = planes + (n * 8 + ((4 * h + s) ^ (n & 7))) * 16;
      k3[s].hi = *reinterpret_cast<const bf16x8*>(at);
      k3[s].mid = *reinterpret_cast<const bf16x8*>(at + kPlane);
      k3[s].lo = *reinterpret_cast<const bf16x8*>(at + 2 * kPlane);
    }
    const floatx16 s = core.scores(k3, lane);
    float p[16];
    softmax_block(s, c, b, h, st, p);
    const char* vt = CoreF16::vt_base(planes + kValues, lane, h);
    weigh_values(p, st, [&](int u, int cb) {
      SplitOperand va;
      va.hi = __builtin_bit_cast(bf16x8, CoreF16::read_va(vt, u, cb));
      va.mid = __builtin_bit_cast(bf16x8, CoreF16::read_va(vt + kPlane, u, cb));
      va.lo = __builtin_bit_cast(bf16x8, CoreF16::read_va(vt + 2 * kPlane, u, cb));
      return va;
    });
  }
};
constexpr int64_t kSharedSteps = 8192;      // steps of a call from which sharing pays, see run_tile_implicit

// Every wavefront is done with its LDS reads and writes and has met the others.  (Loads into
// registers stay in flight across it.)
__device__ __forceinline__ void workgroup_lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Implicit window masks, fp32: 128 consecutive queries of a class per workgroup, 32 per wavefront,
// over the key blocks of the whole 128 (grid mapping, ranges of key blocks and partial states as
// in tile_window_kernel).  Block k is computed from one of two LDS buffers while block k+1, whose
// values have arrived in registers, is split into the other one and block k+2 is requested.
// Bound by matrix cores and vector unit together (see the profile of this kernel); 168 registers and
// 48 KB keep three wavefronts per SIMD (two were 5 to 10 % slower).  +-1359, L = 262,144, 4 heads: 6.51
// ms with fp32 products -> 3.64 ms; +-128, L = 65,536, 8 heads: 386 -> 270 us; L = 2,000,000, one head,
// +-16: 524 -> 465 us.
__global__ __attribute__((amdgpu_waves_per_eu(3, 3))) __launch_bounds__(256) void tile_window_f32_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V, float* __restrict__ O,
    float* __restrict__ lse, int64_t L, int64_t W, int64_t s, int64_t n_groups, float scale, int accumulate,
    int64_t seg_len, int nsplit, float* __restrict__ parts) {
  __shared__ __attribute__((aligned(16))) char planes[2 * SharedBlock::kBytes];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int n = lane & 31, h = lane >> 5;
  const int64_t chunk = gridDim.x / 8;
  const int64_t bid_all = (int64_t)(blockIdx.x % 8) * chunk + blockIdx.x / 8;
  const int64_t bid = bid_all / nsplit;
  const int part = (int)(bid_all - bid * nsplit);
  WindowSlot slot;
  if (!locate_window_slot(bid, L, s, n_groups, seg_len, slot)) return;      // (the whole workgroup leaves)
  const int64_t p = slot.p, Lc = slot.Lc;
  const int64_t q0 = slot.grp * (4 * kTile);
  if (q0 >= Lc) return;
  const int64_t hd = blockIdx.y;
  const int64_t hoff = hd * L * kHeadDim;
  const int64_t u0 = q0 + (int64_t)wave * kTile;
  const int64_t vfirst = q0 - W > 0 ? q0 - W : 0;
  const int64_t vlast = q0 + 4 * kTile - 1 + W < Lc - 1 ? q0 + 4 * kTile - 1 + W : Lc - 1;
  const int nblk = (int)((vlast - vfirst) / kTile + 1);
  const int k0 = (int)((int64_t)nblk * part / nsplit), k1 = (int)((int64_t)nblk * (part + 1) / nsplit);
  // a wavefront whose queries lie past the end of the class still copies and meets the barriers;
  // classify() then reports no block as its own
  const WindowBlocks src{vfirst, Lc, s, p, u0, W};
  const int64_t u = u0 + n;
  const bool exists = u < Lc;
  const int64_t qrow = s * (exists ? u : Lc - 1) + p;
  const float c = softmax_factor(scale);
  TileState st;
  st.init();
  CoreF32 core;
  const uint32_t key_bytes = (uint32_t)(s * kHeadDim * 4);       // (at most 2^27, the host checks)
  const int r_own = threadIdx.x >> 3;
  SharedBlock next;
  auto request = [&](int k) {                                    // (past the last block: the last one again)
    const int64_t v0 = vfirst + (int64_t)(k < k1 ? k : k1 - 1) * kTile;
    const int64_t left = Lc - v0;
    const int last = left < kTile ? (int)left - 1 : kTile - 1;   // keys past the end re-read the last one (masked off)
    const uint32_t at = (uint32_t)(r_own < last ? r_own : last) * key_bytes + (threadIdx.x & 7) * 32;
    const int64_t base = hoff * 4 + (s * v0 + p) * (kHeadDim * 4);
    next.load(reinterpret_cast<const char*>(K) + base + at, reinterpret_cast<const char*>(V) + base + at);
  };
  if (k0 < k1) {
    request(k0);
    core.load_q(Q + hoff + qrow * kHeadDim, h, scale < 0.f);
    next.store(planes + (k0 & 1) * SharedBlock::kBytes);
    request(k0 + 1);
    workgroup_lds_barrier();
    for (int k = k0; k < k1; ++k) {
      next.store(planes + ((k + 1) & 1) * SharedBlock::kBytes);
      request(k + 2);
      const int cls = src.classify(k);                           // wave-uniform
      if (cls) {
        BlockInfo b = src.get(k, n);
        b.full = cls == 2;
        SharedBlock::attend(core, planes + (k & 1) * SharedBlock::kBytes, b, c, lane, st);
      }
      workgroup_lds_barrier();
    }
    if (core.again(st)) {                // (see beyond_split)
      int ka = k0, kb = k1;
      while (ka < kb && src.classify(ka) == 0) ++ka;
      while (kb > ka && src.classify(kb - 1) == 0) --kb;
      st.init();
      core.run_exact(K + hoff, V + hoff, src, ka, kb, c, lane, st, planes + wave * CoreF32::kBlockBytes);
    }
  }
  if (u0 >= Lc) return;
  if (nsplit > 1)
    store_partial(parts + (((bid * 4 + wave) * gridDim.y + hd) * nsplit + part) * (int64_t)kTilePartialFloats, st, n, h);
  else
    finish_tile<float>(O + hoff, lse ? lse + hd * L : nullptr, qrow, qrow, exists, st, h, accumulate != 0);
}

// The block lists of four work items, merged: advance() names the lists' smallest block not taken
// yet (kDone past the end) and moves every list that holds it one entry on.  Everything is
// wave-uniform (the ids are read through the scalar path) and the same in all four wavefronts.
struct MergedLists {
  typedef const int32_t __attribute__((address_space(4)))* Ids;
  static constexpr int kDone = kFullBit - 1;
  Ids at[4];
  int left[4], head[4];      // entries behind the head, the head's record
  struct Step {
    int block;               // key block, or kDone
    int own;                 // this wavefront's record of it (block | full flag), or -1
  };
  __device__ __forceinline__ void start(int i, const int32_t* ids, int n) {
    at[i] = (Ids)ids;
    left[i] = n;
    head[i] = n > 0 ? *at[i] : kDone;
  }
  __device__ __forceinline__ Step advance(int wave) {
    int m = kDone;
#pragma unroll
    for (int i = 0; i < 4; ++i) m = min(m, head[i] & ~kFullBit);
    Step s{m, -1};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if ((head[i] & ~kFullBit) != m || m == kDone) continue;
      if (wave == i) s.own = head[i];
      --left[i];
      ++at[i];
      head[i] = left[i] > 0 ? *at[i] : kDone;
    }
    return s;
  }
};

// Explicit masks, fp32: a workgroup takes four work items, one per wavefront, over the union of
// their block lists: four neighbouring tiles share most of their blocks (a block only some of them
// hold is skipped by the others), and so do the same segments of four tiles cut alike.  The pipeline
// is that of tile_window_f32_kernel.  Items whose lists have little in common (four segments of one
// tile, tiles whose blocks are mostly random ones) run side by side, each wavefront with the split
// of its own blocks; both forms do the same operations in the same order.
// Resident workgroups claim from the head's counter: first the groups of segment items that the
// CSR -> tile pass listed (the long ones), then the tiles in fours.  A call with fewer claims than
// kSharedClaims leaves CUs without a workgroup: there every wavefront claims items by itself
// (+-100, one head, us, that / fours: L = 8,192 26.5 / 28.4, L = 16,301 38.2 / 30.1).
// Bound like that kernel, at two wavefronts per SIMD (256 registers, for the wavefronts on lists
// of their own; 18 vector values spill outside the loops over blocks, 92 scalar ones to vector lanes).  us, fp32
// products -> every wavefront by itself -> this: longformer mask, L = 65,536, 8 heads, prepared 494 ->
// 411 -> 387; +-300, L = 200,000, 2 heads 670 -> 568 -> 465; random, a quarter of the pairs, L = 24,576
// 2,014 -> 1,144 -> 893.
constexpr int64_t kSharedClaims = 128;

__global__ __attribute__((amdgpu_waves_per_eu(2, 2))) __launch_bounds__(256) void tile_attend_f32_kernel(
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V, float* __restrict__ O,
    float* __restrict__ lse, const int64_t* __restrict__ row_ptr, int64_t L, float scale, void* ws, size_t ws_bytes,
    int accumulate) {
  constexpr int kOwnLds = CoreF32::lds_bytes<kPipeRegK>();
  static_assert(4 * kOwnLds <= 2 * SharedBlock::kBytes, "four wavefronts' own blocks fit the shared planes");
  __shared__ __attribute__((aligned(16))) char planes[2 * SharedBlock::kBytes];
  __shared__ uint32_t claim;
  const int32_t H = (int32_t)gridDim.x;   // head-major grid: the long work items of every head are dispatched first
  const WorkspacePlan pl = plan_workspace(L, H, row_ptr[L], SGA_F32);
  if (pl.total_bytes > ws_bytes) return;
  char* base_ws = static_cast<char*>(ws);
  const int64_t n_groups = reinterpret_cast<const uint32_t*>(ws)[kCtrMultiItems];
  const int64_t n_claims = n_groups + (pl.n_tiles + 3) / 4;
  if (n_claims * H < kSharedClaims) {
    tile_attend_body<float, kPipeRegK>(Q, K, V, O, lse, row_ptr, L, scale, ws, ws_bytes, accumulate, planes);
    return;
  }
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int n = lane & 31, h = lane >> 5;
  const float c = softmax_factor(scale);
  const TileItem* items = reinterpret_cast<const TileItem*>(base_ws + pl.off_items_rec);
  const int32_t* tile_bad = reinterpret_cast<const int32_t*>(base_ws + pl.off_tile_bad);
  const int32_t* tile_pbase = reinterpret_cast<const int32_t*>(base_ws + pl.off_tile_pbase);
  const int32_t* pair_blk = reinterpret_cast<const int32_t*>(base_ws + pl.off_pair_blk);
  const uint32_t* pair_mask = reinterpret_cast<const uint32_t*>(base_ws + pl.off_pair_mask);
  const bool parts_fit = tile_parts_fit(pl, ws);
  const int64_t head = blockIdx.x;
  const int64_t hoff = head * L * kHeadDim;
  const char* Kb = reinterpret_cast<const char*>(K + hoff);
  const char* Vb = reinterpret_cast<const char*>(V + hoff);
  uint32_t* work_next = reinterpret_cast<uint32_t*>(base_ws + pl.off_work_next) + head;
  const int r_own = threadIdx.x >> 3;
  SharedBlock next;
  auto request = [&](int block) {
    const int64_t v0 = (int64_t)block * kTile;
    const int64_t left = L - v0;
    const int last = left < kTile ? (int)left - 1 : kTile - 1;   // keys past the end re-read the last one (masked off)
    const uint32_t at = (uint32_t)(r_own < last ? r_own : last) * (kHeadDim * 4) + (threadIdx.x & 7) * 32;
    next.load(Kb + v0 * (kHeadDim * 4) + at, Vb + v0 * (kHeadDim * 4) + at);
  };
  for (bool first = true;; first = false) {
    int64_t cl = blockIdx.y;
    if (!first) {
      if (n_claims <= gridDim.y) break;
      __syncthreads();                   // every wavefront has read the previous claim and left the LDS of its item
      if (threadIdx.x == 0) claim = (uint32_t)claim_next(work_next, n_claims, gridDim.y);
      __syncthreads();
      cl = __builtin_amdgcn_readfirstlane(claim);
    }
    if (cl >= n_claims) break;
    const bool segments = cl < n_groups;
    const int64_t group = segments ? uniform64(items[cl].group) : 0;
    MergedLists lists;
    const int32_t* ids[4];
    int32_t nb[4], ti[4], t = -1, seg = 0, nseg = 1, nblk = 0;
    int64_t slot0 = 0;
    int held = 0, first_seg = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      int64_t w;
      bool there;
      if (segments) {
        w = group + i;
        there = w < pl.n_work;
      } else {
        const int64_t tile = (cl - n_groups) * 4 + i;
        there = tile < pl.n_tiles;
        w = there ? work_first(row_ptr, L, pl.seg_shift, tile) : 0;
      }
      const TileItem* rec = items + (there ? w : 0);
      ti[i] = __builtin_amdgcn_readfirstlane(rec->tile);
      nb[i] = __builtin_amdgcn_readfirstlane(rec->nblk);
      const int32_t si = __builtin_amdgcn_readfirstlane(rec->seg), ns = __builtin_amdgcn_readfirstlane(rec->nseg);
      const int64_t slot = uniform64(rec->slot0);
      there = there && ti[i] >= 0 && nb[i] >= 0;                 // (a tile without edges still writes its rows)
      if (segments) {
        // of the group: the same segment of the next tile, or the next segment of the same one
        there = there && ns > 1 && parts_fit && !tile_bad[ti[i]] &&
                (i == 0 || ti[i] == ti[0] || (ti[i] == ti[0] + i && si == first_seg));
      } else if (there) {
        there = ns == 1;
      }
      if (i == 0) first_seg = si;
      if (!there) nb[i] = 0;
      ids[i] = pair_blk + slot;
      held += there;
      if (wave == i) {
        t = there ? ti[i] : -1;
        seg = si;
        nseg = ns;
        nblk = nb[i];
        slot0 = slot;
      }
    }
    // Lists worth merging: their blocks a quarter, half, three quarters and all of the way down lie
    // close together, in a call of enough steps (see kSharedSteps).  (us, every wavefront on its own
    // list / merged: 32-token blocks with two random ones per row, 4 heads, L = 65,536, 122 / 158;
    // longformer mask with 16 global tokens, 406 / 379, its global tokens merged as well 506;
    // +-300, L = 200,000, 2 heads, 540 / 456; random, a quarter of the pairs, L = 24,576, 1,163 / 890;
    // +-30, L = 100,000, 42 / 51.)
    int most = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) most = max(most, nb[i]);
    bool alike = held > 1 && most > 0 && n_claims * H * most >= kSharedSteps;
#pragma unroll
    for (int f = 1; f <= 4; ++f) {
      int lo = INT32_MAX, hi = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (nb[i] == 0) continue;
        const int id = ((MergedLists::Ids)ids[i])[(int)((int64_t)(nb[i] - 1) * f / 4)] & ~kFullBit;
        lo = min(lo, id);
        hi = max(hi, id);
      }
      alike = alike && hi - lo <= 4 + most / 8;
    }
    const int64_t row_first = (int64_t)(t < 0 ? 0 : t) * kTile;
    const int64_t qrow = row_first + n;
    const bool exists = qrow < L;
    CoreF32 core;
    core.load_q(Q + hoff + (exists ? qrow : L - 1) * kHeadDim, h, scale < 0.f);
    TileState st;
    st.init();
    const ExplicitBlocks src{pair_blk + slot0, pair_mask + slot0 * kTile, L};
    if (alike) {
#pragma unroll
      for (int i = 0; i < 4; ++i) lists.start(i, ids[i], nb[i]);
      MergedLists::Step cur = lists.advance(wave);               // (some list holds a block)
      request(cur.block);
      const uint32_t* words = src.mask + n;                      // this lane's word of the item's next block
      uint32_t word = nblk > 0 ? *words : 0u;
      int to_go = nblk;
      MergedLists::Step ahead = lists.advance(wave);
      next.store(planes);
      request(ahead.block != MergedLists::kDone ? ahead.block : cur.block);
      workgroup_lds_barrier();
      for (int k = 0; cur.block != MergedLists::kDone; ++k) {
        next.store(planes + ((k + 1) & 1) * SharedBlock::kBytes);
        const MergedLists::Step after = lists.advance(wave);
        request(after.block != MergedLists::kDone ? after.block : cur.block);
        if (cur.own >= 0) {
          BlockInfo b;
          b.row0 = 0;
          b.raw = 0;
          b.nvalid = kTile;
          b.word = word;
          b.full = cur.own & kFullBit;
          words += kTile;
          if (--to_go > 0) word = *words;
          SharedBlock::attend(core, planes + (k & 1) * SharedBlock::kBytes, b, c, lane, st);
        }
        workgroup_lds_barrier();
        cur = ahead;
        ahead = after;
      }
      if (core.again(st)) {                // (see beyond_split)
        st.init();
        core.run_exact(K + hoff, V + hoff, src, 0, nblk, c, lane, st, planes + wave * CoreF32::kBlockBytes);
      }
    } else {
      core.run<kPipeRegK>(K + hoff, V + hoff, src, 0, nblk, c, lane, st, planes + wave * kOwnLds);
    }
    if (t < 0) continue;
    if (nseg > 1) {
      float* part = reinterpret_cast<float*>(base_ws + pl.off_tpartials) +
                    (((int64_t)tile_pbase[t] + seg) * H + head) * (int64_t)kTilePartialFloats;
      store_partial(part, st, n, h);
    } else {
      finish_tile<float>(O + hoff, lse ? lse + head * L : nullptr, qrow, qrow, exists, st, h, accumulate != 0);
    }
  }
}

// Key blocks of the non-local mask (global tokens 0..g-1 without the window, Section IV-B
// "Global (non-local)") against the 32 queries that start at row0, by index arithmetic.
// kGlobalRows: the queries i < g, which see every key outside their window, blocks kb0, kb0+1, ...;
// otherwise the queries i >= g, which see the global keys j < min(g, i - W).  Queries of the
// other kind (and past the end) get empty words.
template <bool kGlobalRows>
struct NonlocalBlocks {
  int64_t L, g, W, row0;
  int64_t kb0;
  static constexpr int kGetLoads = 0;
  __device__ int64_t key_stride() const { return 1; }
  __device__ void resolve(BlockInfo&) const {}
  __device__ BlockInfo get(int k, int n) const {
    BlockInfo b;
    b.raw = 0;
    const int64_t v0 = (kb0 + k) * kTile;
    b.row0 = v0;
    const int64_t left = L - v0;
    b.nvalid = left < kTile ? (int)left : kTile;
    const uint32_t valid = b.nvalid == kTile ? ~0u : ((1u << b.nvalid) - 1u);
    const int64_t i = row0 + n;
    if (kGlobalRows) {
      // keys of the block inside the window [i - W, i + W] are no neighbours
      int64_t lo = i - W - v0, hi = i + W - v0;
      uint32_t inside = 0;
      if (hi >= 0 && lo <= kTile - 1) {
        lo = lo < 0 ? 0 : lo;
        hi = hi > kTile - 1 ? kTile - 1 : hi;
        inside = (~0u >> (31 - (int)hi)) & (~0u << (int)lo);
      }
      b.word = i < g ? (valid & ~inside) : 0u;
      // (wave-uniform) every query of the tile is a global row and no window reaches the block
      b.full = b.nvalid == kTile && row0 + kTile <= g && (row0 + kTile - 1 + W < v0 || row0 - W > v0 + kTile - 1);
    } else {
      const int64_t end = (g < i - W ? g : i - W) - v0;       // keys [0, end) of the block are neighbours
      const uint32_t below = end <= 0 ? 0u : (end >= kTile ? ~0u : ((1u << (int)end) - 1u));
      b.word = (i >= g && i < L) ? (valid & below) : 0u;
      const int64_t end0 = (g < row0 - W ? g : row0 - W) - v0;      // of the tile's first query
      b.full = b.nvalid == kTile && row0 >= g && row0 + kTile <= L && end0 >= kTile;
    }
    return b;
  }
};

// Implicit non-local mask, queries i >= g: one wavefront per 32 rows against the (g + 31) / 32
// key blocks that hold the global tokens.
template <typename T, int kPipe>
__device__ __forceinline__ void nonlocal_cols(const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V,
                                              T* __restrict__ O, float* __restrict__ lse, int64_t L, int64_t W,
                                              int64_t g, int64_t tile, float scale, int accumulate, int lane, char* lds) {
  const int n = lane & 31, h = lane >> 5;
  const int64_t row0 = (g / kTile + tile) * kTile;           // the first tile may start below g
  if (row0 >= L) return;
  const int64_t hd = blockIdx.y;
  const int64_t hoff = hd * L * kHeadDim;
  const NonlocalBlocks<false> src{L, g, W, row0, 0};
  const int nblk = (int)((g + kTile - 1) / kTile);
  const int64_t i = row0 + n;
  const bool mine = i >= g && i < L;
  typename CoreFor<T, kPipe>::type core;
  core.load_q(Q + hoff + (i < L ? i : L - 1) * kHeadDim, h, scale < 0.f);
  TileState st;
  st.init();
  core.template run<kPipe>(K + hoff, V + hoff, src, 0, nblk, softmax_factor(scale), lane, st, lds);
  if constexpr (CoreOf<T>::type::kTileStore) {
    static_assert(CoreF16::kCarryBytes <= CoreF16::lds_bytes<kPipeLdsK>(), "output tile fits the wavefront's LDS");
    if (accumulate) {
      const float l = st.l + other_half(st.l, h);
      const bool empty = !(l > 0.f);
      const float lse_row = empty ? -INFINITY : (st.m + __builtin_amdgcn_logf(l)) * kLn2;
      const CarryWeights cw = carry_weights(lse[hd * L + (mine ? i : L - 1)], lse_row);
      CoreF16::store_tile_carry(O + hoff, row0, g > row0 ? (int)(g - row0) : 0, L - row0 < kTile ? (int)(L - row0) : kTile,
                                st, empty ? 0.f : 1.0f / l * cw.w_now, cw.w_prev, lane, lds);
      if (mine && h == 0) lse[hd * L + i] = cw.lse;
      return;
    }
  }
  finish_tile<T>(O + hoff, lse ? lse + hd * L : nullptr, i, i, mine, st, h, accumulate != 0);
}

// ... and the g global rows: one workgroup per (tile of global rows, range c of key blocks), a quarter of the range per
// wavefront.  The four states are merged in LDS, in wavefront order, and leave as
// the partial state of the tile's rows over the range in the layout nonlocal_merge_kernel reads
// (row-major: D accumulators, m, l per (row, range, head)).  (A wavefront with a range of its own took twice to four times as
// many blocks one after the other, 2 us each in fp32: three global tokens, L = 35,000, one head, kernel and merge
// 28 + 5.6 us, 16 + 5.5 so; both calls: L = 200,000, 16 tokens, fp32 206 -> 135, fp16 68 -> 51; L = 65,536, 8 heads,
// fp16 127 -> 124.)
template <typename T, int kPipe>
__device__ __forceinline__ void nonlocal_rows(const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V,
                                              int64_t L, int64_t W, int64_t g, int64_t tile, int64_t c, int64_t n_ranges,
                                              int64_t blocks_per_range, float scale, float* __restrict__ partials,
                                              int lane, int wave, char* lds_all) {
  constexpr int kLds = CoreFor<T, kPipe>::type::template lds_bytes<kPipe>();
  constexpr int kStateBytes = kTile * kHeadDim * 4;          // a wavefront's accumulators; its m and l of the rows follow
  static_assert(kStateBytes + 2 * kTile * 4 <= kLds, "a wavefront's state fits its LDS");
  char* const lds = lds_all + wave * kLds;
  const int n = lane & 31, h = lane >> 5;
  const int64_t hd = blockIdx.y, H = gridDim.y;
  const int64_t row0 = tile * kTile;
  const int64_t hoff = hd * L * kHeadDim;
  const int64_t nb_total = (L + kTile - 1) / kTile;
  const int64_t kb0 = c * blocks_per_range;
  const int64_t kb1 = kb0 + blocks_per_range < nb_total ? kb0 + blocks_per_range : nb_total;
  const int nb = (int)(kb1 > kb0 ? kb1 - kb0 : 0);
  const NonlocalBlocks<true> src{L, g, W, row0, kb0};
  const int64_t i = row0 + n;
  typename CoreFor<T, kPipe>::type core;
  core.load_q(Q + hoff + (i < L ? i : L - 1) * kHeadDim, h, scale < 0.f);
  TileState st;
  st.init();
  core.template run<kPipe>(K + hoff, V + hoff, src, nb * wave / 4, nb * (wave + 1) / 4, softmax_factor(scale),
                           lane, st, lds);
  const float l = st.l + other_half(st.l, h);
  wait_loads_except<0>();                  // (nothing of this wavefront still lands in its LDS)
  wait_lds_reads();
  __builtin_amdgcn_wave_barrier();
  // (the 16-byte chunks of a row swizzled)
#pragma unroll
  for (int cb = 0; cb < 2; ++cb)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<float4*>(lds + n * (kHeadDim * 4) + (((cb * 8 + 2 * q + h) ^ (n & 15)) * 16)) =
          make_float4(st.o[cb][4 * q], st.o[cb][4 * q + 1], st.o[cb][4 * q + 2], st.o[cb][4 * q + 3]);
  if (h == 0) {
    reinterpret_cast<float*>(lds + kStateBytes)[n] = st.m;
    reinterpret_cast<float*>(lds + kStateBytes)[kTile + n] = l;
  }
  __syncthreads();
  const int t = wave * kWave + lane, chunk = t & 15;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int r = (t >> 4) + 16 * k;
    if (row0 + r >= g) continue;
    float m[4], M = kMinusHuge, sum = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      m[w] = reinterpret_cast<const float*>(lds_all + w * kLds + kStateBytes)[r];
      M = fmaxf(M, m[w]);
    }
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float e = __builtin_amdgcn_exp2f(m[w] - M);
      const float4 o = *reinterpret_cast<const float4*>(lds_all + w * kLds + r * (kHeadDim * 4) + ((chunk ^ (r & 15)) * 16));
      sum = __builtin_fmaf(reinterpret_cast<const float*>(lds_all + w * kLds + kStateBytes)[kTile + r], e, sum);
      acc.x = __builtin_fmaf(o.x, e, acc.x);
      acc.y = __builtin_fmaf(o.y, e, acc.y);
      acc.z = __builtin_fmaf(o.z, e, acc.z);
      acc.w = __builtin_fmaf(o.w, e, acc.w);
    }
    float* p = partials + (((row0 + r) * n_ranges + c) * H + hd) * (kHeadDim + 4);
    *reinterpret_cast<float4*>(p + 4 * chunk) = acc;
    if (chunk == 0) {
      p[kHeadDim] = M;
      p[kHeadDim + 1] = sum;
    }
  }
}

// Both parts in one launch (neither reads what the other writes): the first row_wgs workgroups of a
// head take the ranges of the global rows, which are the long ones, the others the tiles of the rows
// >= g, which wait for memory.  (longformer mask, L = 65,536, 8 heads, fp16: 56 and 22 us one
// after the other; 58 us together, with the rows written whole.  268 MB of Q and O: 4.6 TB/s.)
template <typename T, int kPipe>
__global__ __launch_bounds__(256, 2) void tile_nonlocal_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, T* __restrict__ O,
    float* __restrict__ lse, int64_t L, int64_t W, int64_t g, float scale, int accumulate, uint32_t row_wgs,
    uint32_t n_ranges, int64_t blocks_per_range, float* __restrict__ partials) {
  constexpr int kLds = CoreFor<T, kPipe>::type::template lds_bytes<kPipe>();
  __shared__ __attribute__((aligned(16))) char lds_all[4 * kLds];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  char* lds = lds_all + wave * kLds;
  if (blockIdx.x < row_wgs) {
    const uint32_t tile = blockIdx.x / n_ranges;             // (ranges of a tile together)
    nonlocal_rows<T, kPipe>(Q, K, V, L, W, g, tile, blockIdx.x - tile * n_ranges, n_ranges, blocks_per_range, scale,
                            partials, lane, wave, lds_all);
  } else {
    nonlocal_cols<T, kPipe>(Q, K, V, O, lse, L, W, g, (int64_t)(blockIdx.x - row_wgs) * 4 + wave, scale, accumulate,
                            lane, lds);
  }
}

__device__ __forceinline__ float lane_value(float v, int src_lane) {     // v of lane src_lane (uniform index)
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), src_lane));
}

// Merge of the partial states that the window kernels leave when they cut the key blocks of
// their tiles into nsplit <= kMaxWindowSplit ranges.  grid = (tiles: 4 per workgroup of the uncut
// d = 64 launch, 1 per workgroup of the wider ones; head; quarter of the tile's rows), one
// wavefront per 64-channel slice.  Lanes 0..7 first reduce the (m, l) of the quarter's eight rows
// over the ranges, in ascending order, to the rows' weights; then lane = channel and the
// weighted accumulators are summed row by row, every load independent of the others.
template <typename T, int kD>
__global__ __launch_bounds__(kD) void window_merge_kernel(
    T* __restrict__ O, float* __restrict__ lse, const float* __restrict__ parts, int64_t L, int64_t s,
    int64_t n_groups, int accumulate, int64_t seg_len, int nsplit) {
  constexpr int kSlices = kD / kHeadDim;
  constexpr int kTilesPerWg = kSlices == 1 ? 4 : 1;    // of the launch that wrote the partial states
  constexpr int kRows = kTile / 4;
  const int lane = threadIdx.x & (kWave - 1);
  const int slice = threadIdx.x / kWave;
  const int64_t bid = blockIdx.x / kTilesPerWg, hd = blockIdx.y;
  const int tile_in_wg = blockIdx.x % kTilesPerWg;
  WindowSlot slot;
  if (!locate_window_slot(bid, L, s, n_groups, seg_len, slot)) return;
  const int64_t u0 = (slot.grp * kTilesPerWg + tile_in_wg) * kTile + blockIdx.z * kRows;
  if (u0 >= slot.Lc) return;
  const int r0 = blockIdx.z * kRows;
  const int64_t range_step = (int64_t)kSlices * kTilePartialFloats;
  const float* p0 = parts + ((((bid * kTilesPerWg + tile_in_wg) * gridDim.y + hd) * nsplit) * kSlices + slice) *
                                (int64_t)kTilePartialFloats;
  // row statistics: lane j < kRows owns row r0 + j
  const int jr = lane < kRows ? lane : 0;
  const int64_t row_j = s * (u0 + jr < slot.Lc ? u0 + jr : slot.Lc - 1) + slot.p;
  float mc[kMaxWindowSplit], lc[kMaxWindowSplit];
  float M = kMinusHuge;
#pragma unroll
  for (int c = 0; c < kMaxWindowSplit; ++c) {
    const int cc = c < nsplit ? c : 0;
    mc[c] = p0[cc * range_step + kTile * 64 + r0 + jr];
    lc[c] = c < nsplit ? p0[cc * range_step + kTile * 64 + kTile + r0 + jr] : 0.f;
    if (c < nsplit) M = fmaxf(M, mc[c]);
  }
  float l = 0.f, w[kMaxWindowSplit];
#pragma unroll
  for (int c = 0; c < kMaxWindowSplit; ++c) {
    w[c] = c < nsplit ? __builtin_amdgcn_exp2f(mc[c] - M) : 0.f;
    l = __builtin_fmaf(lc[c], w[c], l);
  }
  const bool empty = !(l > 0.f);
  float lse_row = empty ? -INFINITY : (M + __builtin_amdgcn_logf(l)) * kLn2;
  float w_now = empty ? 0.f : 1.0f / l, w_prev = 0.f;
  if (accumulate) {
    const CarryWeights cw = carry_weights(lse[hd * L + row_j], lse_row);
    w_now *= cw.w_now;
    w_prev = cw.w_prev;
    lse_row = cw.lse;
    if (kSlices > 1) __syncthreads();     // every slice has read the earlier lse before slice 0 replaces it
  }
  if (lse && slice == 0 && lane < kRows && u0 + lane < slot.Lc) lse[hd * L + row_j] = lse_row;
#pragma unroll
  for (int c = 0; c < kMaxWindowSplit; ++c) w[c] *= w_now;        // weights of the normalised sum
#pragma unroll
  for (int j = 0; j < kRows; ++j) {
    if (u0 + j >= slot.Lc) break;
    const int64_t row = s * (u0 + j) + slot.p;
    float acc = 0.f;
#pragma unroll
    for (int c = 0; c < kMaxWindowSplit; ++c) {
      if (c < nsplit)
        acc = __builtin_fmaf(p0[c * range_step + (r0 + j) * 64 + lane], lane_value(w[c], j), acc);
    }
    T* dst = O + hd * L * kD + row * kD + slice * kHeadDim + lane;
    if (accumulate) acc = __builtin_fmaf(lane_value(w_prev, j), load_out(dst), acc);
    store_out(dst, acc);
  }
}

// Window masks at head dimensions 128 and 256: one workgroup of kD / 64 wavefronts per
// 32-query tile (see tile_attend_wide_kernel); grid mapping as in tile_window_kernel with one
// tile per workgroup.
template <typename T, int kD, int kPipe>
__global__ __launch_bounds__(kD) void tile_window_wide_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, T* __restrict__ O,
    float* __restrict__ lse, int64_t L, int64_t W, int64_t s, int64_t n_tiles, float scale,
    int accumulate, int64_t seg_len, int nsplit, float* __restrict__ parts) {
  using Core = typename WideCoreOf<T, kD>::type;
  constexpr int kSlices = kD / kHeadDim;
  constexpr int kLds = Core::template lds_bytes<kPipe>();
  __shared__ __attribute__((aligned(16))) char lds_all[kSlices * kLds + SliceExchange<kD>::kBytes];
  const int lane = threadIdx.x & (kWave - 1);
  const int slice = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int n = lane & 31, h = lane >> 5;
  const int64_t chunk = gridDim.x / 8;
  const int64_t bid_all = (int64_t)(blockIdx.x % 8) * chunk + blockIdx.x / 8;
  // (nsplit > 1: nsplit consecutive workgroups share a tile, see tile_window_kernel)
  const int64_t bid = bid_all / nsplit;
  const int part = (int)(bid_all - bid * nsplit);
  // (every condition below is the same for all wavefronts of the workgroup)
  WindowSlot slot;
  if (!locate_window_slot(bid, L, s, n_tiles, seg_len, slot)) return;
  const int64_t p = slot.p, Lc = slot.Lc;
  const int64_t u0 = slot.grp * kTile;
  if (u0 >= Lc) return;
  const int64_t hd = blockIdx.y;
  const int64_t hoff = hd * L * kD + slice * kHeadDim;
  const int64_t vlo = u0 - W > 0 ? u0 - W : 0;
  const int64_t vhi = u0 + kTile - 1 + W < Lc - 1 ? u0 + kTile - 1 + W : Lc - 1;
  WindowBlocks src{vlo, Lc, s, p, u0, W};
  const int nblk = (int)((vhi - vlo) / kTile + 1);
  const int64_t u = u0 + n;
  const bool exists = u < Lc;
  const int64_t qrow = s * (exists ? u : Lc - 1) + p;
  Core core;
  core.xchg.init(lds_all + kSlices * kLds, slice);
  core.load_q(Q + hoff + qrow * kD, h, scale < 0.f);
  TileState st;
  st.init();
  if (nsplit > 1) {
    const int k0 = (int)((int64_t)nblk * part / nsplit), k1 = (int)((int64_t)nblk * (part + 1) / nsplit);
    core.template run<kPipe>(K + hoff, V + hoff, src, k0, k1, softmax_factor(scale), lane, st,
                             lds_all + slice * kLds);
    store_partial(parts + (((bid * gridDim.y + hd) * nsplit + part) * kSlices + slice) *
                              (int64_t)kTilePartialFloats,
                  st, n, h);
    return;
  }
  core.template run<kPipe>(K + hoff, V + hoff, src, 0, nblk, softmax_factor(scale), lane, st,
                           lds_all + slice * kLds);
  finish_tile_wide<T, kD>(O + hoff, lse ? lse + hd * L : nullptr, qrow, exists, st, h, slice,
                          accumulate != 0);
}

// Windows at d = 128 and 256 of calls with few tiles: kShare groups of kD / 64 wavefronts per tile, each for a range
// of its key blocks; the first group merges their states through LDS (see window_share_wide).
template <typename T, int kD, int kShare, typename Sum>
__global__ __attribute__((amdgpu_waves_per_eu(2, 2))) __launch_bounds__(kD * kShare) void tile_window_wide_share_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, T* __restrict__ O,
    float* __restrict__ lse, int64_t L, int64_t W, int64_t s, int64_t n_tiles, float scale, int accumulate,
    int64_t seg_len) {
  using Core = typename WideCoreOf<T, kD>::type;
  constexpr int kPipe = DtypeOf<T>::code == SGA_F16 ? kPipeLdsK : kPipeRegK;
  constexpr int kSlices = kD / kHeadDim, kLds = Core::template lds_bytes<kPipe>();
  static_assert(kShareBytes <= kLds, "a wavefront's state fits its LDS");
  __shared__ __attribute__((aligned(16))) char lds_all[kShare * (kSlices * kLds + SliceExchange<kD>::kBytes)];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int slice = wave % kSlices, part = wave / kSlices;
  const int n = lane & 31, h = lane >> 5;
  char* lds = lds_all + wave * kLds;
  const int64_t chunk = gridDim.x / 8;
  const int64_t bid = (int64_t)(blockIdx.x % 8) * chunk + blockIdx.x / 8;
  WindowSlot slot;
  if (!locate_window_slot(bid, L, s, n_tiles, seg_len, slot)) return;       // (the whole workgroup leaves)
  const int64_t p = slot.p, Lc = slot.Lc;
  const int64_t u0 = slot.grp * kTile;
  if (u0 >= Lc) return;
  const int64_t hd = blockIdx.y;
  const int64_t hoff = hd * L * kD + slice * kHeadDim;
  const int64_t vlo = u0 - W > 0 ? u0 - W : 0;
  const int64_t vhi = u0 + kTile - 1 + W < Lc - 1 ? u0 + kTile - 1 + W : Lc - 1;
  const WindowBlocks src{vlo, Lc, s, p, u0, W};
  const int nblk = (int)((vhi - vlo) / kTile + 1);
  const int64_t u = u0 + n;
  const bool exists = u < Lc;
  const int64_t qrow = s * (exists ? u : Lc - 1) + p;
  Core core;
  core.xchg.init(lds_all + kShare * kSlices * kLds + part * SliceExchange<kD>::kBytes, slice);
  core.load_q(Q + hoff + qrow * kD, h, scale < 0.f);
  TileState st;
  st.init();
  core.run_range(K + hoff, V + hoff, src, nblk * part / kShare, nblk * (part + 1) / kShare, (nblk + kShare - 1) / kShare,
                 softmax_factor(scale), lane, st, lds);
  if (part > 0) leave_state(st, lds, lane);
  __syncthreads();
  if (part > 0) {
    if (accumulate) __syncthreads();     // (the one of finish_tile_wide)
    return;
  }
  add_states<kShare, kSlices * kLds, Sum>(st, lds, lane);
  finish_tile_wide<T, kD>(O + hoff, lse ? lse + hd * L : nullptr, qrow, exists, st, h, slice, accumulate != 0);
}

// fp16, d = 128, explicit masks: one wavefront per work item with all 128 channels of its 32
// queries (tile_attend_wide_kernel gives each 64-channel slice a wavefront, which repeats the
// softmax in every slice and exchanges the partial scores through LDS).  A key block is staged as
// four 64-channel blocks in the layout CoreF16 reads (K channels 0..63, K 64..127, V 0..63,
// V 64..127: 16 KB per wavefront), K one block ahead as in CoreF16T::run_ldsk; the scores of a
// block are one chain of eight products over the two K halves, the softmax is done once, the
// numerators meet the two V halves in eight more products.  Wavefronts claim items of their head
// from the device counter.  Partial states of multi-segment tiles are written as the two slice
// records tile_merge_kernel<__half, 128> reads.
__global__ __attribute__((amdgpu_waves_per_eu(2, 2))) __launch_bounds__(256) void tile_attend128_f16_kernel(
    const __half* __restrict__ Q, const __half* __restrict__ K, const __half* __restrict__ V,
    __half* __restrict__ O, float* __restrict__ lse, const int64_t* __restrict__ row_ptr, int64_t L,
    float scale, void* ws, size_t ws_bytes, int accumulate) {
  using Core = CoreF16T<2 * kHeadDim>;
  constexpr int kD = 2 * kHeadDim;
  constexpr int kBlk = Core::kBlockBytes;
  __shared__ __attribute__((aligned(16))) char lds_all[4][4 * kBlk];
  const int32_t H = (int32_t)gridDim.x;
  const WorkspacePlan pl = plan_workspace(L, H, row_ptr[L], SGA_F16, kD);
  if (pl.total_bytes > ws_bytes) return;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int n = lane & 31, h = lane >> 5;
  char* ldsk = lds_all[wave];                    // K channels 0..63, then 64..127
  char* ldsv = ldsk + 2 * kBlk;                  // V likewise
  char* base_ws = static_cast<char*>(ws);
  const bool negate = scale < 0.f;
  const float c = softmax_factor(scale);
  const TileItem* items = reinterpret_cast<const TileItem*>(base_ws + pl.off_items_rec);
  const int32_t* tile_bad = reinterpret_cast<const int32_t*>(base_ws + pl.off_tile_bad);
  const int32_t* tile_pbase = reinterpret_cast<const int32_t*>(base_ws + pl.off_tile_pbase);
  const bool parts_fit = tile_parts_fit(pl, ws);
  const int64_t head = blockIdx.x;
  const int64_t hoff = head * L * kD;
  uint32_t* work_next = reinterpret_cast<uint32_t*>(base_ws + pl.off_work_next) + head;
  const __half* Kh = K + hoff;
  const __half* Vh = V + hoff;
  typename Core::Stage sm;
  sm.init(1, lane);
  const char* vt0 = Core::vt_base(ldsv, lane, h);
  float* lse_h = lse ? lse + head * L : nullptr;
  const uint32_t claimants = gridDim.y * 4;
  for (bool first = true;; first = false) {
    int64_t w_cur = (int64_t)blockIdx.y * 4 + wave;
    if (!first) {
      if (pl.n_work <= claimants) break;
      uint32_t claimed = 0;
      if (lane == 0) claimed = (uint32_t)claim_next(work_next, pl.n_work, claimants);
      w_cur = __builtin_amdgcn_readfirstlane(claimed);
    }
    if (w_cur >= pl.n_work) break;
    const int4 r0 = reinterpret_cast<const int4*>(items + w_cur)[0];
    const int64_t slot_raw = reinterpret_cast<const int64_t*>(items + w_cur)[2];
    const int32_t t = __builtin_amdgcn_readfirstlane(r0.x);
    const int32_t nblk = __builtin_amdgcn_readfirstlane(r0.y);
    const int32_t seg = __builtin_amdgcn_readfirstlane(r0.z);
    const int32_t nseg = __builtin_amdgcn_readfirstlane(r0.w);
    const int64_t slot0 = uniform64(slot_raw);
    if (t < 0 || nblk < 0) continue;         // idle item / list overflow: tile left to the gather path
    if (nseg > 1 && (!parts_fit || tile_bad[t])) continue;
    const int64_t row_first = (int64_t)t * kTile;
    const ExplicitBlocks src{reinterpret_cast<const int32_t*>(base_ws + pl.off_pair_blk) + slot0,
                             reinterpret_cast<const uint32_t*>(base_ws + pl.off_pair_mask) + slot0 * kTile, L};
    const int64_t qrow = row_first + n;
    const bool exists = qrow < L;
    Core lo, hi;                             // channels 0..63 and 64..127 of the same queries
    lo.load_q(Q + hoff + (exists ? qrow : L - 1) * kD, h, negate);
    hi.load_q(Q + hoff + (exists ? qrow : L - 1) * kD + kHeadDim, h, negate);
    TileState st, st_hi;                     // m and l live in st; st_hi holds the accumulators of channels 64..127
    st.init();
    st_hi.init();
    if (nblk > 0) {
      BlockInfo b = src.get(0, n);
      BlockInfo b1 = src.get(nblk > 1 ? 1 : 0, n);
      src.resolve(b);
      __builtin_amdgcn_wave_barrier();       // reads of the buffers by the work item before are done
      sm.stage_k(Kh, b, lane, ldsk);
      sm.stage_k(Kh + kHeadDim, b, lane, ldsk + kBlk);
      for (int k = 0; k < nblk; ++k) {
        const bool more = k + 1 < nblk;      // wave-uniform
        src.resolve(b1);
        __builtin_amdgcn_wave_barrier();     // the previous block's reads of the staged V are done
        sm.stage_v(Vh, b, lane, ldsv);
        sm.stage_v(Vh + kHeadDim, b, lane, ldsv + kBlk);
        BlockInfo b2 = b1;
        if (k + 2 < nblk) b2 = src.get(k + 2, n);
        wait_k_block<8, ExplicitBlocks::kGetLoads>(k + 2 < nblk);   // K block k: older than the V copies (and the record loads)
        __builtin_amdgcn_wave_barrier();
        half8 kf[4], kg[4];
        Core::read_k(ldsk, n, h, kf);
        Core::read_k(ldsk + kBlk, n, h, kg);
        wait_lds_reads();                    // the K buffers may be overwritten now
        __builtin_amdgcn_wave_barrier();
        if (more) {
          sm.stage_k(Kh, b1, lane, ldsk);
          sm.stage_k(Kh + kHeadDim, b1, lane, ldsk + kBlk);
        }
        floatx16 sv = {0};
#pragma unroll
        for (int u = 0; u < 4; ++u) sv = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[u], lo.qf[u], sv, 0, 0, 0);
#pragma unroll
        for (int u = 0; u < 4; ++u) sv = __builtin_amdgcn_mfma_f32_32x32x16_f16(kg[u], hi.qf[u], sv, 0, 0, 0);
        if (!b.full) mask_scores(sv, b.word, h);
        half8 ph[2];
        const float l_before = st.l;
        numerators_h(sv, c, st, ph);
        if (__any(sum_overflowed(st))) {
          // (see softmax_block_h; the accumulators of the upper channels take the same factor)
          st.l = l_before;
          const float m_before = st.m;
          rescale_state(st, block_max(sv, c, h));
          const float alpha = __builtin_amdgcn_exp2f(m_before - st.m);
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            st_hi.o[0][r] *= alpha;
            st_hi.o[1][r] *= alpha;
          }
          numerators_h(sv, c, st, ph);
        }
        // V block k (and any record load after it) is older than the 8 K copies issued above (if any)
        wait_staged_v<8>(more);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const half8 a0 = Core::read_va(vt0, u, 0), a1 = Core::read_va(vt0, u, 1);
          const half8 c0 = Core::read_va(vt0 + kBlk, u, 0), c1 = Core::read_va(vt0 + kBlk, u, 1);
          st.o[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a0, ph[u], st.o[0], 0, 0, 0);
          st.o[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, ph[u], st.o[1], 0, 0, 0);
          st_hi.o[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(c0, ph[u], st_hi.o[0], 0, 0, 0);
          st_hi.o[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(c1, ph[u], st_hi.o[1], 0, 0, 0);
        }
        b = b1;
        b1 = b2;
      }
    }
    if (nseg > 1) {
      float* part = reinterpret_cast<float*>(base_ws + pl.off_tpartials) +
                    ((((int64_t)tile_pbase[t] + seg) * H + head) * 2) * (int64_t)kTilePartialFloats;
      st_hi.m = st.m;
      st_hi.l = st.l;
      store_partial(part, st, n, h);
      store_partial(part + kTilePartialFloats, st_hi, n, h);
      continue;
    }
    const float l = st.l + other_half(st.l, h);
    const bool empty = !(l > 0.f);
    const float inv = empty ? 0.f : 1.0f / l;
    float lse_row = empty ? -INFINITY : (st.m + __builtin_amdgcn_logf(l)) * kLn2;
    if (accumulate) {
      if (exists) {
        // (both half-waves read the earlier lse before the first replaces it)
        const CarryWeights cw = carry_weights(lse_h[qrow], lse_row);
        Core::store_row(O + hoff + qrow * kD, st, inv * cw.w_now, cw.w_prev, true, h);
        Core::store_row(O + hoff + qrow * kD + kHeadDim, st_hi, inv * cw.w_now, cw.w_prev, true, h);
        if (h == 0) lse_h[qrow] = cw.lse;
      }
      continue;
    }
    // The tile leaves through the wavefront's LDS (every copy has landed, every read is done) as
    // whole 256-byte rows, four per instruction, with streaming stores (see CoreF16T::store_tile).
    constexpr int kPitch = kD * 2 + 16;
    static_assert(kTile * kPitch <= 4 * kBlk, "output tile fits the wavefront's LDS");
    char* tile = ldsk;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const TileState& part = half ? st_hi : st;
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          uint2 w;
          w.x = __builtin_bit_cast(uint32_t, __floats2half2_rn(part.o[cb][4 * g] * inv, part.o[cb][4 * g + 1] * inv));
          w.y = __builtin_bit_cast(uint32_t,
                                   __floats2half2_rn(part.o[cb][4 * g + 2] * inv, part.o[cb][4 * g + 3] * inv));
          *reinterpret_cast<uint2*>(tile + n * kPitch + (half * kHeadDim + cb * 32 + 8 * g + 4 * h) * 2) = w;
        }
    }
    __builtin_amdgcn_wave_barrier();
    const int64_t left = L - row_first;
    const int n_rows = left < kTile ? (int)left : kTile;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = (lane >> 4) + 4 * i;
      const uint4 v = *reinterpret_cast<const uint4*>(tile + r * kPitch + (lane & 15) * 16);
      if (r < n_rows)
        __builtin_nontemporal_store(__builtin_bit_cast(half8, v),
                                    reinterpret_cast<half8*>(O + hoff + (row_first + r) * kD + (lane & 15) * 8));
    }
    if (lse_h && h == 0 && n < n_rows) lse_h[row_first + n] = lse_row;
    wait_lds_reads();                        // (the tile has left before the next item stages into this space)
  }
}

// The implicit non-local mask at head dimensions 128 and 256: the two kernels of the 64-channel
// form (nonlocal_cols, nonlocal_rows) with one workgroup of kD / 64
// wavefronts per tile, each on its 64-channel slice (see tile_attend_wide_kernel).
template <typename T, int kD, int kPipe>
__global__ __launch_bounds__(kD) void tile_nonlocal_cols_wide_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, T* __restrict__ O,
    float* __restrict__ lse, int64_t L, int64_t W, int64_t g, float scale, int accumulate) {
  using Core = typename WideCoreOf<T, kD>::type;
  constexpr int kSlices = kD / kHeadDim;
  constexpr int kLds = Core::template lds_bytes<kPipe>();
  __shared__ __attribute__((aligned(16))) char lds_all[kSlices * kLds + SliceExchange<kD>::kBytes];
  const int lane = threadIdx.x & (kWave - 1);
  const int slice = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int n = lane & 31, h = lane >> 5;
  const int64_t row0 = (g / kTile + (int64_t)blockIdx.x) * kTile;
  if (row0 >= L) return;                           // (the same for every wavefront of the workgroup)
  const int64_t hd = blockIdx.y;
  const int64_t hoff = hd * L * kD + slice * kHeadDim;
  const NonlocalBlocks<false> src{L, g, W, row0, 0};
  const int nblk = (int)((g + kTile - 1) / kTile);
  const int64_t i = row0 + n;
  Core core;
  core.xchg.init(lds_all + kSlices * kLds, slice);
  core.load_q(Q + hoff + (i < L ? i : L - 1) * kD, h, scale < 0.f);
  TileState st;
  st.init();
  core.template run<kPipe>(K + hoff, V + hoff, src, 0, nblk, softmax_factor(scale), lane, st,
                           lds_all + slice * kLds);
  finish_tile_wide<T, kD>(O + hoff, lse ? lse + hd * L : nullptr, i < L ? i : L - 1, i >= g && i < L, st, h, slice,
                          accumulate != 0);
}

template <typename T, int kD, int kPipe>
__global__ __launch_bounds__(kD) void tile_nonlocal_rows_wide_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, int64_t L, int64_t W,
    int64_t g, int64_t blocks_per_range, float scale, float* __restrict__ partials) {
  using Core = typename WideCoreOf<T, kD>::type;
  constexpr int kSlices = kD / kHeadDim;
  constexpr int kLds = Core::template lds_bytes<kPipe>();
  __shared__ __attribute__((aligned(16))) char lds_all[kSlices * kLds + SliceExchange<kD>::kBytes];
  const int lane = threadIdx.x & (kWave - 1);
  const int slice = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int n = lane & 31, h = lane >> 5;
  const int64_t c = blockIdx.x, n_ranges = gridDim.x, hd = blockIdx.z, H = gridDim.z;
  const int64_t row0 = (int64_t)blockIdx.y * kTile;
  const int64_t hoff = hd * L * kD + slice * kHeadDim;
  const int64_t nb_total = (L + kTile - 1) / kTile;
  const int64_t kb0 = c * blocks_per_range;
  const int64_t kb1 = kb0 + blocks_per_range < nb_total ? kb0 + blocks_per_range : nb_total;
  const NonlocalBlocks<true> src{L, g, W, row0, kb0};
  const int64_t i = row0 + n;
  Core core;
  core.xchg.init(lds_all + kSlices * kLds, slice);
  core.load_q(Q + hoff + (i < L ? i : L - 1) * kD, h, scale < 0.f);
  TileState st;
  st.init();
  core.template run<kPipe>(K + hoff, V + hoff, src, 0, (int)(kb1 > kb0 ? kb1 - kb0 : 0), softmax_factor(scale),
                           lane, st, lds_all + slice * kLds);
  if (i >= g) return;
  const float l = st.l + other_half(st.l, h);
  float* p = partials + ((i * n_ranges + c) * H + hd) * (kD + 4);
#pragma unroll
  for (int cb = 0; cb < 2; ++cb)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<float4*>(p + slice * kHeadDim + cb * 32 + 8 * q + 4 * h) =
          make_float4(st.o[cb][4 * q], st.o[cb][4 * q + 1], st.o[cb][4 * q + 2], st.o[cb][4 * q + 3]);
  if (h == 0 && slice == 0) {
    p[kD] = st.m;
    p[kD + 1] = l;
  }
}

// fp16 window masks, wide bands: a workgroup owns 256 consecutive queries of a class (64 per
// wavefront: two 32-query sub-tiles that share every K fragment and V^T operand read, with two
// independent chains of products) and walks the key blocks of its
// whole window once, in step: every K and V block is copied global -> LDS once per workgroup
// (each wavefront moves one 1 KB copy of K and one of V per block instead of all eight), into a
// ring of kBandSlots blocks that runs kBandAhead blocks ahead of the block being computed.  One
// workgroup barrier per block both publishes the block (every wavefront has waited for its own
// two copies) and retires the block before it (its slot is the next one to be overwritten).
// A wavefront computes a block only where it lies inside its own window (its queries start 64w
// keys into the workgroup's range, so it idles for two blocks per wavefront index at one end or
// the other).  The copies are issued untracked: every wavefront issues exactly two per block, so
// a counted wait names the block that must have landed; past the last block the copies repeat
// the last block into a slot nobody reads any more, which keeps the count constant to the end.
constexpr int kBandSlots = 8;
constexpr int kBandAhead = 6;      // <= kBandSlots - 2: the slot written holds a block retired a barrier ago

__global__ __attribute__((amdgpu_waves_per_eu(2, 2))) __launch_bounds__(256) void tile_window_band_kernel(
    const __half* __restrict__ Q, const __half* __restrict__ K, const __half* __restrict__ V,
    __half* __restrict__ O, float* __restrict__ lse, int64_t L, int64_t W, int64_t s, int64_t n_groups,
    float scale, int accumulate, int64_t seg_len) {
  constexpr int kSlotBytes = 2 * CoreF16::kBlockBytes;       // K block, then V block
  __shared__ __attribute__((aligned(16))) char ring[kBandSlots * kSlotBytes];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int n = lane & 31, h = lane >> 5;
  const int64_t chunk = gridDim.x / 8;
  const int64_t bid = (int64_t)(blockIdx.x % 8) * chunk + blockIdx.x / 8;
  WindowSlot slot;
  if (!locate_window_slot(bid, L, s, n_groups, seg_len, slot)) return;      // (the whole workgroup leaves)
  const int64_t p = slot.p, Lc = slot.Lc;
  const int64_t q0 = slot.grp * (8 * kTile);
  if (q0 >= Lc) return;
  const int64_t hd = blockIdx.y;
  const int64_t hoff = hd * L * kHeadDim;
  const int64_t u0 = q0 + (int64_t)wave * (2 * kTile);
  const int64_t vfirst = q0 - W > 0 ? q0 - W : 0;
  const int64_t vlast = q0 + 8 * kTile - 1 + W < Lc - 1 ? q0 + 8 * kTile - 1 + W : Lc - 1;
  const int nblk = (int)((vlast - vfirst) / kTile + 1);
  // a wavefront whose queries lie past the end of the class (u0 >= Lc) still copies and meets the
  // barriers; classify() then reports no block as its own
  const WindowBlocks sa{vfirst, Lc, s, p, u0, W}, sb{vfirst, Lc, s, p, u0 + kTile, W};
  const int64_t ua = u0 + n, ub = u0 + kTile + n;
  const bool exists_a = ua < Lc, exists_b = ub < Lc;
  const int64_t qrow_a = s * (exists_a ? ua : Lc - 1) + p, qrow_b = s * (exists_b ? ub : Lc - 1) + p;
  CoreF16 core, core_b;
  core.load_q(Q + hoff + qrow_a * kHeadDim, h, scale < 0.f);
  core_b.load_q(Q + hoff + qrow_b * kHeadDim, h, scale < 0.f);
  wait_loads_except<0>();            // Q has arrived: from here on only the ring's copies are counted
  core.q_arrived();
  core_b.q_arrived();
  // this wavefront's share of a block: keys 8w .. 8w+7, eight lanes of 16 bytes per 128-byte row
  // (the K chunks swizzled as CoreF16::read_k expects)
  const int r_own = 8 * wave + (lane >> 3), c_own = lane & 7;
  const char* Kb = reinterpret_cast<const char*>(K + hoff);
  const char* Vb = reinterpret_cast<const char*>(V + hoff);
  auto issue = [&](int kb) {
    const int kc = kb < nblk ? kb : nblk - 1;
    int64_t v = vfirst + (int64_t)kc * kTile + r_own;
    v = v < Lc ? v : Lc - 1;                               // keys past the end re-read the last one (masked off)
    const int64_t row_bytes = (s * v + p) * (kHeadDim * 2);
    char* dst = ring + (kb % kBandSlots) * kSlotBytes + wave * 1024;
    copy16_to_lds_untracked(Kb + row_bytes + ((c_own ^ (r_own & 7)) * 16), dst);
    copy16_to_lds_untracked(Vb + row_bytes + c_own * 16, dst + CoreF16::kBlockBytes);
  };
  TileState sta, stb;
  sta.init();
  stb.init();
  const float c = softmax_factor(scale);
  const char* vt0 = CoreF16::vt_base(ring + CoreF16::kBlockBytes, lane, h);
  // The barrier that opens block kb: every wavefront has waited for its own copies of blocks kb
  // and kb+1 (so after it both are whole: the interior steps read K of block kb+1 for the score
  // products they issue one block ahead), and everyone is done with block kb-1; then the copy
  // kBandAhead blocks on is started, into the slot of block kb-2.
  auto publish = [&](int kb) {
    wait_loads_except<2 * (kBandAhead - 2)>();
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    issue(kb + kBandAhead);
  };
  // One block on the edge of (or outside) this wavefront's windows: publish it, compute what
  // falls inside.
  auto step = [&](int kb) {
    publish(kb);
    const char* ldsk = ring + (kb % kBandSlots) * kSlotBytes;
    const char* vt = vt0 + (kb % kBandSlots) * kSlotBytes;
    half8 pha[2], phb[2];
    {
      const int class_a = sa.classify(kb), class_b = sb.classify(kb);     // wave-uniform
      if (class_a | class_b) {
        half8 kf[4];
        CoreF16::read_k(ldsk, n, h, kf);
        if (class_a) {
          floatx16 sacc = {0};
#pragma unroll
          for (int t = 0; t < 4; ++t) sacc = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[t], core.qf[t], sacc, 0, 0, 0);
          const uint32_t word = class_a == 2 ? ~0u : sa.get(kb, n).word;
          softmax_block_h(sacc, c, class_a == 2, word, h, sta, pha);
        }
        if (class_b) {
          floatx16 sacc = {0};
#pragma unroll
          for (int t = 0; t < 4; ++t) sacc = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[t], core_b.qf[t], sacc, 0, 0, 0);
          const uint32_t word = class_b == 2 ? ~0u : sb.get(kb, n).word;
          softmax_block_h(sacc, c, class_b == 2, word, h, stb, phb);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int cb = 0; cb < 2; ++cb) {
            const half8 va = CoreF16::read_va(vt, u, cb);
            if (class_a) sta.o[cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va, pha[u], sta.o[cb], 0, 0, 0);
            if (class_b) stb.o[cb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va, phb[u], stb.o[cb], 0, 0, 0);
          }
      }
    }
  };
  // the blocks interior to both of this wavefront's sub-tiles form one range [k_lo, k_hi)
  int k_lo = 0, k_hi = nblk;
  while (k_lo < nblk && !(sa.classify(k_lo) == 2 && sb.classify(k_lo) == 2)) ++k_lo;
  while (k_hi > k_lo && !(sa.classify(k_hi - 1) == 2 && sb.classify(k_hi - 1) == 2)) --k_hi;
  // Interior blocks, software-pipelined: the score products of block kb+1 are issued ahead of the
  // exponentials and the PV products of block kb, so that the matrix cores and the vector unit
  // have independent work side by side.  cur_* hold the scores of block kb on entry (kFirst: the
  // step computes them itself), nxt_* receive those of block kb+1 (kNext: it is interior too);
  // successive steps swap the two pairs, so no accumulator is ever copied.
  auto products = [&](int kb, floatx16& da, floatx16& db) {
    half8 kf[4];
    CoreF16::read_k(ring + (kb % kBandSlots) * kSlotBytes, n, h, kf);
    da = floatx16{0};
    db = floatx16{0};
#pragma unroll
    for (int t = 0; t < 4; ++t) da = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[t], core.qf[t], da, 0, 0, 0);
#pragma unroll
    for (int t = 0; t < 4; ++t) db = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[t], core_b.qf[t], db, 0, 0, 0);
  };
  auto piped = [&](int kb, floatx16& cur_a, floatx16& cur_b, floatx16& nxt_a, floatx16& nxt_b, auto first,
                   auto next) {
    publish(kb);
    if constexpr (decltype(first)::value) products(kb, cur_a, cur_b);
    if constexpr (decltype(next)::value) products(kb + 1, nxt_a, nxt_b);
    half8 pha[2], phb[2];
    softmax_pair_h(cur_a, cur_b, c, h, sta, stb, pha, phb);
    const char* vt = vt0 + (kb % kBandSlots) * kSlotBytes;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const half8 va0 = CoreF16::read_va(vt, u, 0), va1 = CoreF16::read_va(vt, u, 1);
      sta.o[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va0, pha[u], sta.o[0], 0, 0, 0);
      stb.o[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va0, phb[u], stb.o[0], 0, 0, 0);
      sta.o[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va1, pha[u], sta.o[1], 0, 0, 0);
      stb.o[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va1, phb[u], stb.o[1], 0, 0, 0);
    }
  };
  for (int kb = 0; kb < kBandAhead; ++kb) issue(kb);
  int kb = 0;
  for (; kb < k_lo; ++kb) step(kb);
  if (kb < k_hi) {
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    floatx16 s_a, s_b, t_a, t_b;
    if (kb + 1 < k_hi) {
      piped(kb, s_a, s_b, t_a, t_b, yes, yes);
      ++kb;                                              // the scores of block kb are in t_*
      for (; kb + 2 < k_hi; kb += 2) {
        piped(kb, t_a, t_b, s_a, s_b, no, yes);
        piped(kb + 1, s_a, s_b, t_a, t_b, no, yes);
      }
      if (kb + 1 < k_hi) {
        piped(kb, t_a, t_b, s_a, s_b, no, yes);
        piped(kb + 1, s_a, s_b, t_a, t_b, no, no);
      } else {
        piped(kb, t_a, t_b, s_a, s_b, no, no);
      }
    } else {
      piped(kb, s_a, s_b, t_a, t_b, yes, no);
    }
    kb = k_hi;
  }
  for (; kb < nblk; ++kb) step(kb);
  // every copy has landed and every wavefront is done with the ring: its space takes the output tiles
  wait_loads_except<0>();
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  if (u0 >= Lc) return;
  float* lse_h = lse ? lse + hd * L : nullptr;
  if (accumulate) {
    finish_tile<__half>(O + hoff, lse_h, qrow_a, qrow_a, exists_a, sta, h, true);
    finish_tile<__half>(O + hoff, lse_h, qrow_b, qrow_b, exists_b, stb, h, true);
  } else {
    char* lds = ring + wave * (2 * CoreF16::kTileBytes);
    const int64_t left = Lc - u0;
    finish_tile_rows<__half>(O + hoff, lse_h, s * u0 + p, s, left < kTile ? (int)left : kTile, sta, lane, lds);
    if (left > kTile)
      finish_tile_rows<__half>(O + hoff, lse_h, s * (u0 + kTile) + p, s,
                               left < 2 * kTile ? (int)(left - kTile) : kTile, stb, lane,
                               lds + CoreF16::kTileBytes);
  }
}

// The same for one 32-query sub-tile per wavefront, 128 queries per workgroup: 128 registers and a ring of four blocks (32 KB)
// let four wavefronts of four workgroups share a SIMD where tile_window_band_kernel has two.  That kernel reads every
// operand from LDS once for two sub-tiles, but a wavefront issues a vector instruction every five cycles at best, so two
// of them leave the vector unit half idle, and each workgroup waits for its first blocks and its output with one other
// beside it.  This one is bound by power where it runs long (+-1,359, L = 1,600,000: 2.45M cycles at 1.69 GHz, the other
// 2.84M at 1.90): there the two are level, and from about 140 blocks per workgroup on the other is 2 to 8 % faster (see
// strip_is_faster).  us, that / this: one head, L = 400,000, W = 257 134 / 99, 400 152 / 128, 1,000 288 / 270; L = 1,600,000, W = 257
// 482 / 399, 400 555 / 513; L = 30,000, W = 577 43 / 26, 2,100 98 / 65; L = 8,000, W = 400 34 / 20; 2-D blocks of 1,100, L =
// 1,600,000 653 / 635.
// (Eight wavefronts on a ring of eight blocks: W = 260 320 where this has 289; without the scores one block ahead
// 293; two groups of four wavefronts that swap matrix and vector work at barriers, 64 queries each, L = 1,600,000,
// +-1,359: 1,350 -> 1,635.)
constexpr int kStripWaves = 4, kStripSlots = 4;
constexpr int kStripAhead = kStripSlots - 1;      // the slot written holds the block retired by the barrier before
__global__ __attribute__((amdgpu_waves_per_eu(4, 4))) __launch_bounds__(kStripWaves * kWave) void tile_window_strip_kernel(
    const __half* __restrict__ Q, const __half* __restrict__ K, const __half* __restrict__ V,
    __half* __restrict__ O, float* __restrict__ lse, int64_t L, int64_t W, int64_t s, int64_t n_groups,
    float scale, int accumulate, int64_t seg_len) {
  constexpr int kSlotBytes = 2 * CoreF16::kBlockBytes;       // K block, then V block
  constexpr int kQueries = kStripWaves * kTile, kCopies = 2;      // copies per wavefront and block: 1 KB of K, 1 KB of V
  constexpr int kRing = kStripSlots * kSlotBytes, kOut = kStripWaves * CoreF16::kTileBytes;
  __shared__ __attribute__((aligned(16))) char ring[kRing];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int n = lane & 31, h = lane >> 5;
  const int64_t chunk = gridDim.x / 8;
  const int64_t bid = (int64_t)(blockIdx.x % 8) * chunk + blockIdx.x / 8;
  WindowSlot slot;
  if (!locate_window_slot(bid, L, s, n_groups, seg_len, slot)) return;      // (the whole workgroup leaves)
  const int64_t p = slot.p, Lc = slot.Lc;
  const int64_t q0 = slot.grp * kQueries;
  if (q0 >= Lc) return;
  const int64_t hd = blockIdx.y;
  const int64_t hoff = hd * L * kHeadDim;
  const int64_t u0 = q0 + (int64_t)wave * kTile;
  const int64_t vfirst = q0 - W > 0 ? q0 - W : 0;
  const int64_t vlast = q0 + kQueries - 1 + W < Lc - 1 ? q0 + kQueries - 1 + W : Lc - 1;
  const int nblk = (int)((vlast - vfirst) / kTile + 1);
  // a wavefront whose queries lie past the end of the class (u0 >= Lc) still copies and meets the
  // barriers; classify() then reports no block as its own
  const WindowBlocks src{vfirst, Lc, s, p, u0, W};
  const int64_t u = u0 + n;
  const bool exists = u < Lc;
  const int64_t qrow = s * (exists ? u : Lc - 1) + p;
  CoreF16 core;
  core.load_q(Q + hoff + qrow * kHeadDim, h, scale < 0.f);
  wait_loads_except<0>();            // Q has arrived: from here on only the ring's copies are counted
  core.q_arrived();
  // this wavefront's share of a block: keys 8w .. 8w+7 (the K chunks swizzled as CoreF16::read_k expects)
  const int r_own = 8 * wave + (lane >> 3), c_own = lane & 7;
  const char* Kb = reinterpret_cast<const char*>(K + hoff) + (c_own ^ (r_own & 7)) * 16;
  const char* Vb = reinterpret_cast<const char*>(V + hoff) + c_own * 16;
  auto issue = [&](int kb) {
    const int kc = kb < nblk ? kb : nblk - 1;
    int64_t v = vfirst + (int64_t)kc * kTile + r_own;
    v = v < Lc ? v : Lc - 1;                               // keys past the end re-read the last one (masked off)
    const int64_t at = (s * v + p) * (kHeadDim * 2);
    char* dst = ring + (kb % kStripSlots) * kSlotBytes + wave * 1024;
    copy16_to_lds_untracked(Kb + at, dst);
    copy16_to_lds_untracked(Vb + at, dst + CoreF16::kBlockBytes);
  };
  TileState st;
  st.init();
  const float c = softmax_factor(scale);
  const char* vt0 = CoreF16::vt_base(ring + CoreF16::kBlockBytes, lane, h);
  // The barrier that opens block kb: every wavefront has waited for its own copies of blocks kb and kb+1 (the scores of
  // kb+1 are taken one block ahead), and everyone is done with block kb-1, whose slot takes the next copy.
  auto publish = [&](int kb) {
    wait_loads_except<kCopies * (kStripAhead - 2)>();
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    issue(kb + kStripAhead);
  };
  int k_lo = 0, k_hi = nblk;
  while (k_lo < nblk && src.classify(k_lo) != 2) ++k_lo;
  while (k_hi > k_lo && src.classify(k_hi - 1) != 2) --k_hi;
  auto scores = [&](int kb, floatx16& sv) {
    half8 kf[4];
    CoreF16::read_k(ring + (kb % kStripSlots) * kSlotBytes, n, h, kf);
    sv = floatx16{0};
#pragma unroll
    for (int t = 0; t < 4; ++t) sv = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[t], core.qf[t], sv, 0, 0, 0);
  };
  auto weigh = [&](int kb, const half8 (&ph)[2]) {
    const char* vt = vt0 + (kb % kStripSlots) * kSlotBytes;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const half8 va0 = CoreF16::read_va(vt, u, 0), va1 = CoreF16::read_va(vt, u, 1);
      st.o[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va0, ph[u], st.o[0], 0, 0, 0);
      st.o[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va1, ph[u], st.o[1], 0, 0, 0);
    }
  };
  // a block on the edge of (or outside) this wavefront's window
  auto edge = [&](int kb) {
    publish(kb);
    const int cls = src.classify(kb);
    if (cls) {
      floatx16 sv;
      half8 ph[2];
      scores(kb, sv);
      softmax_block_h(sv, c, cls == 2, cls == 2 ? ~0u : src.get(kb, n).word, h, st, ph);
      weigh(kb, ph);
    }
  };
  static_assert(kRing >= kOut, "the output tiles fit the ring");
  for (int kb = 0; kb < kStripAhead; ++kb) issue(kb);
  int kb = 0;
  for (; kb < k_lo; ++kb) edge(kb);
  // interior blocks, the scores of block kb+1 ahead of the numerators and PV products of block kb
  if (kb + 1 < k_hi) {
    floatx16 s_cur, s_next;
    publish(kb);
    scores(kb, s_cur);
    for (; kb + 2 < k_hi; kb += 2) {
      half8 ph[2];
      scores(kb + 1, s_next);
      softmax_block_h(s_cur, c, true, 0, h, st, ph);
      weigh(kb, ph);
      publish(kb + 1);
      scores(kb + 2, s_cur);
      softmax_block_h(s_next, c, true, 0, h, st, ph);
      weigh(kb + 1, ph);
      publish(kb + 2);
    }
    half8 ph[2];
    softmax_block_h(s_cur, c, true, 0, h, st, ph);
    weigh(kb, ph);
    ++kb;
  }
  for (; kb < k_hi; ++kb) edge(kb);
  for (; kb < nblk; ++kb) edge(kb);
  // every copy has landed and every wavefront is done with the ring: its space takes the output tiles
  wait_loads_except<0>();
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  if (u0 >= Lc) return;
  float* lse_h = lse ? lse + hd * L : nullptr;
  if (accumulate) {
    finish_tile<__half>(O + hoff, lse_h, qrow, qrow, exists, st, h, true);
  } else {
    const int64_t left = Lc - u0;
    finish_tile_rows<__half>(O + hoff, lse_h, s * u0 + p, s, left < kTile ? (int)left : kTile, st, lane, ring + wave * CoreF16::kTileBytes);
  }
}

// fp16 window masks, wide bands, d = 128: the ring of tile_window_band_kernel with key blocks of
// 128 channels.  A block is staged as four 64-channel blocks in the layout CoreF16 reads (K
// channels 0..63, K 64..127, V 0..63, V 64..127: 16 KB), once per workgroup of 128 queries; a
// wavefront owns one 32-query sub-tile and all 128 channels of it: the scores of a block are one
// chain of eight products over the two K halves, the softmax is done once, and the numerators
// meet the two V halves in eight more products (16 matrix instructions per block against the
// same vector work as at d = 64; the kernel that gives each 64-channel slice a wavefront of its
// own repeats the softmax in every slice and exchanges the partial scores through LDS).  Four
// slots, copies three blocks ahead: the barrier that opens block kb (every wavefront has waited
// for its own four copies of block kb, and is done with block kb-1) is followed by the copy of
// block kb+3 into the slot of block kb-1.
constexpr int kBand128Slots = 4;
constexpr int kBand128Ahead = 3;      // = kBand128Slots - 1

__global__ __attribute__((amdgpu_waves_per_eu(2, 2))) __launch_bounds__(256) void tile_window_band128_kernel(
    const __half* __restrict__ Q, const __half* __restrict__ K, const __half* __restrict__ V,
    __half* __restrict__ O, float* __restrict__ lse, int64_t L, int64_t W, int64_t s, int64_t n_groups,
    float scale, int accumulate, int64_t seg_len) {
  constexpr int kD = 2 * kHeadDim;
  constexpr int kWaves = 4;          // (eight wavefronts, 256 queries and two copies each per block, were slower: 2.60 against 2.55 ms at +-2048)
  constexpr int kBlk = CoreF16::kBlockBytes;
  constexpr int kSlotBytes = 4 * kBlk;
  __shared__ __attribute__((aligned(16))) char ring[kBand128Slots * kSlotBytes];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int n = lane & 31, h = lane >> 5;
  const int64_t chunk = gridDim.x / 8;
  const int64_t bid = (int64_t)(blockIdx.x % 8) * chunk + blockIdx.x / 8;
  WindowSlot slot;
  if (!locate_window_slot(bid, L, s, n_groups, seg_len, slot)) return;      // (the whole workgroup leaves)
  const int64_t p = slot.p, Lc = slot.Lc;
  const int64_t q0 = slot.grp * (kWaves * kTile);
  if (q0 >= Lc) return;
  const int64_t hd = blockIdx.y;
  const int64_t hoff = hd * L * kD;
  const int64_t u0 = q0 + (int64_t)wave * kTile;
  const int64_t vfirst = q0 - W > 0 ? q0 - W : 0;
  const int64_t vlast = q0 + kWaves * kTile - 1 + W < Lc - 1 ? q0 + kWaves * kTile - 1 + W : Lc - 1;
  const int nblk = (int)((vlast - vfirst) / kTile + 1);
  // a wavefront whose queries lie past the end of the class (u0 >= Lc) still copies and meets the
  // barriers; classify() then reports no block as its own
  const WindowBlocks src{vfirst, Lc, s, p, u0, W};
  const int64_t u = u0 + n;
  const bool exists = u < Lc;
  const int64_t qrow = s * (exists ? u : Lc - 1) + p;
  CoreF16 lo, hi;                                  // channels 0..63 and 64..127 of the same queries
  lo.load_q(Q + hoff + qrow * kD, h, scale < 0.f);
  hi.load_q(Q + hoff + qrow * kD + kHeadDim, h, scale < 0.f);
  wait_loads_except<0>();            // Q has arrived: from here on only the ring's copies are counted
  lo.q_arrived();
  hi.q_arrived();
  // this wavefront's share of a block: keys 8w .. 8w+7 of all four 64-channel blocks, eight lanes
  // of 16 bytes per 128-byte half row (the K chunks swizzled as CoreF16::read_k expects)
  constexpr int kCopies = 4;                       // copies per wavefront and block
  const int r_own = 8 * wave + (lane >> 3), c_own = lane & 7;
  const char* Kb = reinterpret_cast<const char*>(K + hoff);
  const char* Vb = reinterpret_cast<const char*>(V + hoff);
  auto issue = [&](int kb) {
    const int kc = kb < nblk ? kb : nblk - 1;
    int64_t v = vfirst + (int64_t)kc * kTile + r_own;
    v = v < Lc ? v : Lc - 1;                               // keys past the end re-read the last one (masked off)
    const int64_t row_bytes = (s * v + p) * (kD * 2);
    char* dst = ring + (kb % kBand128Slots) * kSlotBytes + wave * 1024;
    const int k_at = (c_own ^ (r_own & 7)) * 16, v_at = c_own * 16;
    copy16_to_lds_untracked(Kb + row_bytes + k_at, dst);
    copy16_to_lds_untracked(Kb + row_bytes + kHeadDim * 2 + k_at, dst + kBlk);
    copy16_to_lds_untracked(Vb + row_bytes + v_at, dst + 2 * kBlk);
    copy16_to_lds_untracked(Vb + row_bytes + kHeadDim * 2 + v_at, dst + 3 * kBlk);
  };
  TileState st, st_hi;               // m and l live in st; st_hi holds the accumulators of channels 64..127
  st.init();
  st_hi.init();
  const float c = softmax_factor(scale);
  const char* vt0 = CoreF16::vt_base(ring + 2 * kBlk, lane, h);
  // The barrier that opens block kb: every wavefront has waited for its own copies of blocks kb
  // and kb+1 (the interior steps read K of block kb+1 for the score products they issue one block
  // ahead), and everyone is done with block kb-1, whose slot takes the copy of block kb+3.
  auto publish = [&](int kb) {
    wait_loads_except<kCopies * (kBand128Ahead - 2)>();
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    issue(kb + kBand128Ahead);
  };
  // scores of block kb: one chain of eight products over the two K halves
  auto products = [&](int kb, floatx16& sv) {
    const char* ldsk = ring + (kb % kBand128Slots) * kSlotBytes;
    half8 kf[4], kg[4];
    CoreF16::read_k(ldsk, n, h, kf);
    CoreF16::read_k(ldsk + kBlk, n, h, kg);
    sv = floatx16{0};
#pragma unroll
    for (int t = 0; t < 4; ++t) sv = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[t], lo.qf[t], sv, 0, 0, 0);
#pragma unroll
    for (int t = 0; t < 4; ++t) sv = __builtin_amdgcn_mfma_f32_32x32x16_f16(kg[t], hi.qf[t], sv, 0, 0, 0);
  };
  // numerators of a block (see softmax_block_h; the accumulators of the upper channels take the
  // same factor when the running maximum is raised), then the products with the two V halves
  auto weigh = [&](int kb, floatx16& sv) {
    half8 ph[2];
    const float l_before = st.l;
    numerators_h<true>(sv, c, st, ph);
    if (__any(sum_overflowed(st))) {
      st.l = l_before;
      const float m_before = st.m;
      rescale_state(st, block_max(sv, c, h));
      const float alpha = __builtin_amdgcn_exp2f(m_before - st.m);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        st_hi.o[0][r] *= alpha;
        st_hi.o[1][r] *= alpha;
      }
      numerators_h<true>(sv, c, st, ph);
    }
    const char* vt = vt0 + (kb % kBand128Slots) * kSlotBytes;
#pragma unroll
    for (int uu = 0; uu < 2; ++uu) {
      const half8 a0 = CoreF16::read_va(vt, uu, 0), a1 = CoreF16::read_va(vt, uu, 1);
      const half8 b0 = CoreF16::read_va(vt + kBlk, uu, 0), b1 = CoreF16::read_va(vt + kBlk, uu, 1);
      st.o[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a0, ph[uu], st.o[0], 0, 0, 0);
      st.o[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, ph[uu], st.o[1], 0, 0, 0);
      st_hi.o[0] = __builtin_amdgcn_mfma_f32_32x32x16_f16(b0, ph[uu], st_hi.o[0], 0, 0, 0);
      st_hi.o[1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(b1, ph[uu], st_hi.o[1], 0, 0, 0);
    }
  };
  // a block on the edge of (or outside) this wavefront's window
  auto step = [&](int kb) {
    publish(kb);
    const int cls = src.classify(kb);                      // wave-uniform
    if (cls) {
      floatx16 sv;
      products(kb, sv);
      if (cls != 2) mask_scores(sv, src.get(kb, n).word, h);
      weigh(kb, sv);
    }
  };
  // Interior blocks, software-pipelined as in tile_window_band_kernel: the score products of
  // block kb+1 are issued ahead of the exponentials and the PV products of block kb; cur holds
  // the scores of block kb on entry (first: the step computes them itself), nxt receives those of
  // block kb+1 (next: it is interior too); successive steps swap the two.
  auto piped = [&](int kb, floatx16& cur, floatx16& nxt, auto first, auto next) {
    publish(kb);
    if constexpr (decltype(first)::value) products(kb, cur);
    if constexpr (decltype(next)::value) products(kb + 1, nxt);
    weigh(kb, cur);
  };
  int k_lo = 0, k_hi = nblk;
  while (k_lo < nblk && src.classify(k_lo) != 2) ++k_lo;
  while (k_hi > k_lo && src.classify(k_hi - 1) != 2) --k_hi;
  for (int kb = 0; kb < kBand128Ahead; ++kb) issue(kb);
  int kb = 0;
  for (; kb < k_lo; ++kb) step(kb);
  if (kb < k_hi) {
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    floatx16 s_a, s_b;
    if (kb + 1 < k_hi) {
      piped(kb, s_a, s_b, yes, yes);
      ++kb;                                              // the scores of block kb are in s_b
      for (; kb + 2 < k_hi; kb += 2) {
        piped(kb, s_b, s_a, no, yes);
        piped(kb + 1, s_a, s_b, no, yes);
      }
      if (kb + 1 < k_hi) {
        piped(kb, s_b, s_a, no, yes);
        piped(kb + 1, s_a, s_b, no, no);
      } else {
        piped(kb, s_b, s_a, no, no);
      }
    } else {
      piped(kb, s_a, s_b, yes, no);
    }
    kb = k_hi;
  }
  for (; kb < nblk; ++kb) step(kb);
  // every copy has landed and every wavefront is done with the ring: its space takes the output tiles
  wait_loads_except<0>();
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  if (u0 >= Lc) return;
  const float l = st.l + other_half(st.l, h);
  const bool empty = !(l > 0.f);
  float inv = empty ? 0.f : 1.0f / l;
  float lse_row = empty ? -INFINITY : (st.m + __builtin_amdgcn_logf(l)) * kLn2;
  float* lse_h = lse ? lse + hd * L : nullptr;
  if (accumulate) {
    if (!exists) return;
    // (both half-waves read the earlier lse before the first replaces it)
    const CarryWeights cw = carry_weights(lse_h[qrow], lse_row);
    CoreF16::store_row(O + hoff + qrow * kD, st, inv * cw.w_now, cw.w_prev, true, h);
    CoreF16::store_row(O + hoff + qrow * kD + kHeadDim, st_hi, inv * cw.w_now, cw.w_prev, true, h);
    if (h == 0) lse_h[qrow] = cw.lse;
    return;
  }
  // A lane holds fragments of its own query's row; the tile goes through LDS and leaves as whole
  // 256-byte rows, four per instruction (see CoreF16T::store_tile), with streaming stores.
  constexpr int kPitch = kD * 2 + 16;
  char* tile = ring + wave * (kTile * kPitch);
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const TileState& part = half ? st_hi : st;
#pragma unroll
    for (int cb = 0; cb < 2; ++cb)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        uint2 w;
        w.x = __builtin_bit_cast(uint32_t, __floats2half2_rn(part.o[cb][4 * g] * inv, part.o[cb][4 * g + 1] * inv));
        w.y = __builtin_bit_cast(uint32_t,
                                 __floats2half2_rn(part.o[cb][4 * g + 2] * inv, part.o[cb][4 * g + 3] * inv));
        *reinterpret_cast<uint2*>(tile + n * kPitch + (half * kHeadDim + cb * 32 + 8 * g + 4 * h) * 2) = w;
      }
  }
  __builtin_amdgcn_wave_barrier();
  const int64_t left = Lc - u0;
  const int n_rows = left < kTile ? (int)left : kTile;
  const int64_t row0 = s * u0 + p;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int r = (lane >> 4) + 4 * i;
    const uint4 v = *reinterpret_cast<const uint4*>(tile + r * kPitch + (lane & 15) * 16);
    if (r < n_rows)
      __builtin_nontemporal_store(__builtin_bit_cast(half8, v),
                                  reinterpret_cast<half8*>(O + hoff + (row0 + r * s) * kD + (lane & 15) * 8));
  }
  if (lse_h && h == 0 && n < n_rows) lse_h[row0 + n * s] = lse_row;
}

// fp16 window masks narrow enough that the keys of 128 consecutive queries fit the LDS
// (this kernel takes the windows of up to 6 blocks, W <= 32, K and V side by side in 48 KB at most,
// tile_window_kv_kernel those of 7 to 20, W <= 256).  A workgroup owns 128 queries
// of one residue class: its four wavefronts first copy every K and V block the workgroup
// needs global -> LDS, once (wavefront w copies blocks w, w+4), and after one barrier each
// wavefront runs its own 32-query sub-tile entirely out of LDS.  Compared with one wavefront
// staging its own blocks, neighbouring sub-tiles no longer fetch the blocks they share four
// times, and the block loop holds no memory instruction and no wait.  The LDS is sized to the
// window at launch, so narrow windows run up to four workgroups per CU.  Grid mapping as in
// tile_window_kernel.
__global__ __launch_bounds__(256) void tile_window_wg_kernel(
    const __half* __restrict__ Q, const __half* __restrict__ K, const __half* __restrict__ V,
    __half* __restrict__ O, float* __restrict__ lse, int64_t L, int64_t W, int64_t s, int64_t n_groups,
    float scale, int accumulate, int nb_max, int64_t seg_len, int64_t Lq, int64_t Lr) {
  // nb_max K blocks, then nb_max V blocks (dynamic: narrow windows leave room for more workgroups)
  extern __shared__ __attribute__((aligned(16))) char lds_wg[];
  char* lds_k = lds_wg;
  char* lds_v = lds_wg + nb_max * CoreF16::kBlockBytes;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int n = lane & 31, h = lane >> 5;
  // The place among the window tiles as in locate_window_slot, without its 64-bit divisions
  // (each is a chain of about a hundred dependent scalar instructions ahead of the first load):
  // workgroup indices and the stride fit 32 bits (the host checks the grid size), and the host
  // passes the class lengths.  Whole-sequence masks: Lq = L / s, Lr = L % s, class p holds
  // Lq + (p < Lr) tokens.  Block-diagonal masks: Lq = tokens of the class of a whole block,
  // Lr = of the sequence's last block.
  const uint32_t chunk = gridDim.x / 8;
  const uint32_t bid = (blockIdx.x % 8) * chunk + blockIdx.x / 8;
  int64_t p, Lc, q0;                               // class start, tokens of the class, first query
  if (seg_len > 0) {
    const uint32_t ng32 = (uint32_t)n_groups;
    const uint32_t seg = bid / ng32;
    p = (int64_t)seg * seg_len;
    if (p >= L) return;
    Lc = p + seg_len <= L ? Lq : Lr;
    q0 = (int64_t)(bid - seg * ng32) * (4 * kTile);
  } else {
    if ((int64_t)bid >= n_groups * s) return;
    const uint32_t s32 = (uint32_t)s;
    const uint32_t grp = bid / s32;
    p = bid - grp * s32;                           // residue class
    Lc = Lq + (p < Lr ? 1 : 0);
    q0 = (int64_t)grp * (4 * kTile);
  }
  // (the divisions above run on the vector unit; back in scalar registers, the per-block index
  // arithmetic that follows from these values stays on the scalar unit)
  p = uniform64(p);
  Lc = uniform64(Lc);
  q0 = uniform64(q0);
  if (q0 >= Lc) return;                            // (the whole workgroup leaves: no barrier is missed)
  const int64_t hd = blockIdx.y;
  const int64_t hoff = hd * L * kHeadDim;
  const int64_t vfirst = q0 - W > 0 ? q0 - W : 0;
  const int64_t vlast = q0 + 4 * kTile - 1 + W < Lc - 1 ? q0 + 4 * kTile - 1 + W : Lc - 1;
  const int nb = (int)((vlast - vfirst) / kTile + 1);          // <= nb_max
  const int64_t u0 = q0 + (int64_t)wave * kTile;
  const int64_t u = u0 + n;
  const bool exists = u < Lc;
  const int64_t qrow = s * (exists ? u : Lc - 1) + p;
  CoreF16 core;
  core.load_q(Q + hoff + qrow * kHeadDim, h, scale < 0.f);
  CoreF16::Stage sm;
  sm.init(s, lane);
  auto stage = [&](int j) {
    BlockInfo b;
    const int64_t v0 = vfirst + (int64_t)j * kTile;
    b.raw = 0;
    b.row0 = s * v0 + p;
    b.nvalid = Lc - v0 < kTile ? (int)(Lc - v0) : kTile;
    b.word = 0;
    b.full = false;
    sm.stage_k(K + hoff, b, lane, lds_k + j * CoreF16::kBlockBytes);
    sm.stage_v(V + hoff, b, lane, lds_v + j * CoreF16::kBlockBytes);
  };
  const bool active = u0 < Lc;                     // (a wavefront without queries still meets the barriers below)
  TileState st;
  st.init();
  const int64_t rem64 = Lc - vfirst, nq64 = Lc - u0;
  const WindowWordsNear src{(int)(u0 - vfirst), (int)W, (int)(nq64 > 64 ? 64 : (nq64 > 0 ? nq64 : 0)),
                            (int)(rem64 > (1 << 20) ? (1 << 20) : rem64)};
  const int64_t lo_key = u0 - W > vfirst ? u0 - W : vfirst;
  const int64_t hi_key = u0 + kTile - 1 + W < vlast ? u0 + kTile - 1 + W : vlast;
  const int k_lo = (int)((lo_key - vfirst) / kTile);
  const int k_hi = active ? (int)((hi_key - vfirst) / kTile) : k_lo - 1;
  const float c = softmax_factor(scale);
  auto blocks = [&](int ka, int kb) {
    for (int k = ka; k <= kb; ++k) {
      const BlockInfo b = src.get(k, n);
      half8 kf[4];
      CoreF16::read_k(lds_k + k * CoreF16::kBlockBytes, n, h, kf);
      core.template block_math<-1>(kf, b, c, lane, h, st, lds_v + k * CoreF16::kBlockBytes, false);
    }
  };
  for (int j = wave; j < nb; j += 4) stage(j);
  wait_loads_except<0>();
  __syncthreads();
  blocks(k_lo, k_hi);
  float* lse_h = lse ? lse + hd * L : nullptr;
  if (accumulate) {
    if (active) finish_tile<__half>(O + hoff, lse_h, qrow, qrow, exists, st, h, true);
    return;
  }
  // every wavefront is done with the staged blocks: their space takes the four output tiles
  // (see staged_blocks)
  __syncthreads();
  if (active)
    finish_tile_rows<__half>(O + hoff, lse_h, s * u0 + p, s, Lc - u0 < kTile ? (int)(Lc - u0) : kTile, st,
                             lane, lds_wg + wave * CoreF16::kTileBytes);
}

// softmax_block_h for a caller that accumulates the PV products later: only m and l are kept
// here (st.o is not touched); the numerators of the block are taken against the m the block leaves
// behind, which the caller records.
__device__ __forceinline__ void softmax_block_deferred(floatx16 sv, float c, bool full, uint32_t word,
                                                       int h, TileState& st, half8 (&ph)[2]) {
  if (!full) mask_scores(sv, word, h);
  const float l_before = st.l;
  numerators_h(sv, c, st, ph);
  if (__any(sum_overflowed(st))) {
    const float bm = block_max(sv, c, h);
    const float m_new = needs_rescale(st, bm) ? bm : st.m;
    st.l = l_before * __builtin_amdgcn_exp2f(st.m - m_new);
    st.m = m_new;
    numerators_h(sv, c, st, ph);
  }
}

// Wider windows than those of tile_window_wg_kernel (7 to 20 key blocks per workgroup of 128 queries, W
// up to kKvMaxWindow), with K and V taking turns in ONE set of LDS blocks: the workgroup copies its K
// blocks, every wavefront takes the scores and softmax numerators of its sub-tile against them
// (numerators and the running max each block left behind stay in registers: at most kWaveBlocks
// blocks meet a 32-query sub-tile), and after a barrier the V blocks are copied over the K blocks
// and the PV products follow, O rescaled where the recorded max changes, exactly as the online form does.
// What it lives from is workgroups per CU: the copies of one run under the arithmetic of the
// others.  4 KB of LDS per block and 9 registers per block of a sub-tile leave four workgroups up to W = 96
// (40 KB, 116 registers), three up to 144 (52 KB, 152), two up to 256 (80 KB, 206).  The band kernel
// that took W > 64 before has two, each of which waits for its first blocks, its Q and its output alone.
// (blocks start at the workgroup's first key, W below it: sub-tile w covers blocks w .. w + (31 + 2W) / 32
// of them, and in the first workgroups of a class, where the window is cut at key 0, at most
// 2 * ceil(W / 32) + 1: kWaveBlocks = 5 up to W = 64, 7 up to 96, 9 up to 128, 11 up to 160, 17 up to 256; a class
// of few tokens has fewer, see subtile_blocks)
// L = 1,048,576, 4 heads, us, band kernel -> this: W = 65 737 -> 446, 96 756 -> 475, 128 837 -> 558,
// 144 872 -> 600, 160 923 -> 719, 192 980 -> 797, 256 1,076 -> 952; beyond, one workgroup per CU: 288
// 1,136 -> 1,665.  W = 64 (2.1 GB, 5.1 TB/s): 412.
constexpr int kKvMinBlocks = 7;        // windows of this many blocks per workgroup take this kernel
constexpr int64_t kKvMaxWindow = 256;

template <int kWaveBlocks>
__global__ __launch_bounds__(256) void tile_window_kv_kernel(
    const __half* __restrict__ Q, const __half* __restrict__ K, const __half* __restrict__ V,
    __half* __restrict__ O, float* __restrict__ lse, int64_t L, int64_t W, int64_t s, int64_t n_groups,
    float scale, int accumulate, int nb_max, int64_t seg_len, int64_t Lq, int64_t Lr) {
  extern __shared__ __attribute__((aligned(16))) char lds_wg[];      // nb_max blocks
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int n = lane & 31, h = lane >> 5;
  // (placement of the workgroup among the window tiles: see tile_window_wg_kernel)
  const uint32_t chunk = gridDim.x / 8;
  const uint32_t bid = (blockIdx.x % 8) * chunk + blockIdx.x / 8;
  int64_t p, Lc, q0;
  if (seg_len > 0) {
    const uint32_t ng32 = (uint32_t)n_groups;
    const uint32_t seg = bid / ng32;
    p = (int64_t)seg * seg_len;
    if (p >= L) return;
    Lc = p + seg_len <= L ? Lq : Lr;
    q0 = (int64_t)(bid - seg * ng32) * (4 * kTile);
  } else {
    if ((int64_t)bid >= n_groups * s) return;
    const uint32_t s32 = (uint32_t)s;
    const uint32_t grp = bid / s32;
    p = bid - grp * s32;
    Lc = Lq + (p < Lr ? 1 : 0);
    q0 = (int64_t)grp * (4 * kTile);
  }
  p = uniform64(p);
  Lc = uniform64(Lc);
  q0 = uniform64(q0);
  if (q0 >= Lc) return;                            // (the whole workgroup leaves: no barrier is missed)
  const int64_t hd = blockIdx.y;
  const int64_t hoff = hd * L * kHeadDim;
  const int64_t vfirst = q0 - W > 0 ? q0 - W : 0;
  const int64_t vlast = q0 + 4 * kTile - 1 + W < Lc - 1 ? q0 + 4 * kTile - 1 + W : Lc - 1;
  const int nb = (int)((vlast - vfirst) / kTile + 1);          // <= nb_max
  const int64_t u0 = q0 + (int64_t)wave * kTile;
  const int64_t u = u0 + n;
  const bool exists = u < Lc;
  const int64_t qrow = s * (exists ? u : Lc - 1) + p;
  CoreF16 core;
  core.load_q(Q + hoff + qrow * kHeadDim, h, scale < 0.f);
  CoreF16::Stage sm;
  sm.init(s, lane);
  auto block_at = [&](int j) {
    BlockInfo b;
    const int64_t v0 = vfirst + (int64_t)j * kTile;
    b.raw = 0;
    b.row0 = s * v0 + p;
    b.nvalid = Lc - v0 < kTile ? (int)(Lc - v0) : kTile;
    b.word = 0;
    b.full = false;
    return b;
  };
  const bool active = u0 < Lc;                     // (a wavefront without queries still meets the barriers below)
  const int64_t rem64 = Lc - vfirst, nq64 = Lc - u0;
  const WindowWordsNear src{(int)(u0 - vfirst), (int)W, (int)(nq64 > 64 ? 64 : (nq64 > 0 ? nq64 : 0)),
                            (int)(rem64 > (1 << 20) ? (1 << 20) : rem64)};
  const int64_t lo_key = u0 - W > vfirst ? u0 - W : vfirst;
  const int64_t hi_key = u0 + kTile - 1 + W < vlast ? u0 + kTile - 1 + W : vlast;
  const int k_lo = (int)((lo_key - vfirst) / kTile);
  const int k_hi = active ? (int)((hi_key - vfirst) / kTile) : k_lo - 1;     // k_hi - k_lo < kWaveBlocks
  const float c = softmax_factor(scale);
  // K blocks of the workgroup, then this sub-tile's scores and numerators
  for (int j = wave; j < nb; j += 4) sm.stage_k(K + hoff, block_at(j), lane, lds_wg + j * CoreF16::kBlockBytes);
  wait_loads_except<0>();
  __syncthreads();
  TileState st;
  st.init();
  half8 ph[kWaveBlocks][2];
  float m_after[kWaveBlocks];
#pragma unroll
  for (int j = 0; j < kWaveBlocks; ++j) {
    const int k = k_lo + j;
    m_after[j] = st.m;
    if (k <= k_hi) {
      const BlockInfo b = src.get(k, n);
      half8 kf[4];
      CoreF16::read_k(lds_wg + k * CoreF16::kBlockBytes, n, h, kf);
      floatx16 sacc = {0};
#pragma unroll
      for (int t = 0; t < 4; ++t) sacc = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf[t], core.qf[t], sacc, 0, 0, 0);
      softmax_block_deferred(sacc, c, b.full != 0, b.word, h, st, ph[j]);
      m_after[j] = st.m;
    }
  }
  __syncthreads();                                 // every wavefront has read its K blocks
  for (int j = wave; j < nb; j += 4) sm.stage_v(V + hoff, block_at(j), lane, lds_wg + j * CoreF16::kBlockBytes);
  wait_loads_except<0>();
  __syncthreads();
  float m_run = m_after[0];
#pragma unroll
  for (int j = 0; j < kWaveBlocks; ++j) {
    const int k = k_lo + j;
    if (k <= k_hi) {
      if (__any(m_after[j] != m_run)) {
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_after[j]);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          st.o[0][r] *= alpha;
          st.o[1][r] *= alpha;
        }
        m_run = m_after[j];
      }
      CoreF16::accumulate(ph[j], lane, h, st, lds_wg + k * CoreF16::kBlockBytes);
    }
  }
  float* lse_h = lse ? lse + hd * L : nullptr;
  if (accumulate) {
    if (active) finish_tile<__half>(O + hoff, lse_h, qrow, qrow, exists, st, h, true);
    return;
  }
  // every wavefront is done with the staged blocks: their space takes the four output tiles (see staged_blocks)
  __syncthreads();
  if (active)
    finish_tile_rows<__half>(O + hoff, lse_h, s * u0 + p, s, Lc - u0 < kTile ? (int)(Lc - u0) : kTile, st,
                             lane, lds_wg + wave * CoreF16::kTileBytes);
}

template <typename T>
sga_status run_tile_explicit_wide(const AttnArgs& a);

template <typename T>
sga_status run_tile_explicit(const AttnArgs& a) {
  if (a.d != kHeadDim) return run_tile_explicit_wide<T>(a);
  const T* Q = static_cast<const T*>(a.Q);
  const T* K = static_cast<const T*>(a.K);
  const T* V = static_cast<const T*>(a.V);
  T* O = static_cast<T*>(a.O);
  // The number of work items depends on row_ptr[L], which only the device knows: the kernels
  // stride over the items with grids sized from L alone.
  const int64_t n_tiles = (a.L + kTile - 1) / kTile;
  int64_t nwg = (n_tiles + 3) / 4 + 64;
  if (nwg > 16384) nwg = 16384;
  if (!a.prepared) launch_tile_analyze(a);
  // fp32: resident workgroups only (256 CUs x 2 wavefronts per SIMD, shared by the heads), which
  // claim items dynamically; fp16: one pass of workgroups over the items of each head
  int64_t per_head = (nwg + 8 * kXcdRun - 1) / (8 * kXcdRun) * (8 * kXcdRun);
  if (a.dtype == SGA_F32) {
    per_head = 512 / a.H;
    if (per_head < 1) per_head = 1;
    if (per_head > n_tiles + 64) per_head = n_tiles + 64;
  }
  // fp32 tiles keep the K fragment in registers; fp16 tiles stage K in LDS (measured best)
  const dim3 grid((unsigned)a.H, (unsigned)per_head);
  if constexpr (DtypeOf<T>::code == SGA_F16) {
    profile_mark_begin(a.stream, "tile_attend_f16_kernel");
    hipLaunchKernelGGL(tile_attend_f16_kernel, grid, dim3(256), 0, a.stream, Q, K, V, O, a.lse, a.row_ptr,
                       a.L, a.scale, a.ws, a.ws_bytes, a.accumulate ? 1 : 0);
  } else {
    profile_mark_begin(a.stream, a.split ? "tile_attend_kernel" : "tile_attend_f32_kernel");
    auto kernel = a.split ? tile_attend_kernel<T, kPipeSplit> : tile_attend_f32_kernel;
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, a.stream, Q, K, V, O, a.lse, a.row_ptr, a.L, a.scale, a.ws,
                       a.ws_bytes, a.accumulate ? 1 : 0);
  }
  profile_mark_end(a.stream);
  // (a prepared graph knows whether any tile was cut into segments; otherwise the launch for the rows left
  // over merges them)
  if (a.prepared && a.plan_multi_tiles > 0)
    hipLaunchKernelGGL((tile_merge_kernel<T, kHeadDim>), dim3(merge_tiles(a), (unsigned)a.H, kTile), dim3(256), 0,
                       a.stream, O, a.lse, a.row_ptr, a.L, a.ws, a.ws_bytes, a.accumulate ? 1 : 0);
  return hip_status(hipGetLastError());
}

template <typename T, int kD>
sga_status run_tile_explicit_wide_d(const AttnArgs& a) {
  const T* Q = static_cast<const T*>(a.Q);
  const T* K = static_cast<const T*>(a.K);
  const T* V = static_cast<const T*>(a.V);
  T* O = static_cast<T*>(a.O);
  constexpr int kSlices = kD / kHeadDim;
  const int64_t n_tiles = (a.L + kTile - 1) / kTile;
  if (!a.prepared) launch_tile_analyze(a);
  // resident workgroups (2 wavefronts per SIMD over the chip), shared by the heads
  int64_t per_head = (2048 / kSlices) / a.H;
  if (per_head < 1) per_head = 1;
  if (per_head > n_tiles + 64) per_head = n_tiles + 64;
  constexpr int kPipe = DtypeOf<T>::code == SGA_F16 ? kPipeLdsK : kPipeRegK;
  if constexpr (DtypeOf<T>::code == SGA_F16 && kD == 128) {
    // one wavefront per item with all 128 channels; two workgroups of four wavefronts per CU
    int64_t wgs = 512 / a.H;
    if (wgs < 1) wgs = 1;
    if (wgs > (n_tiles + 3) / 4 + 16) wgs = (n_tiles + 3) / 4 + 16;
    profile_mark_begin(a.stream, "tile_attend128_f16_kernel");
    hipLaunchKernelGGL(tile_attend128_f16_kernel, dim3((unsigned)a.H, (unsigned)wgs), dim3(256), 0, a.stream, Q, K,
                       V, O, a.lse, a.row_ptr, a.L, a.scale, a.ws, a.ws_bytes, a.accumulate ? 1 : 0);
  } else {
    profile_mark_begin(a.stream, "tile_attend_wide_kernel");
    hipLaunchKernelGGL((tile_attend_wide_kernel<T, kD, kPipe>), dim3((unsigned)a.H, (unsigned)per_head),
                       dim3(kD), 0, a.stream, Q, K, V, O, a.lse, a.row_ptr, a.L, a.scale, a.ws, a.ws_bytes,
                       a.accumulate ? 1 : 0);
  }
  profile_mark_end(a.stream);
  if (a.prepared && a.plan_multi_tiles > 0)
    hipLaunchKernelGGL((tile_merge_kernel<T, kD>), dim3(merge_tiles(a), (unsigned)a.H, kTile), dim3(256), 0, a.stream, O,
                       a.lse, a.row_ptr, a.L, a.ws, a.ws_bytes, a.accumulate ? 1 : 0);
  return hip_status(hipGetLastError());
}

template <typename T>
sga_status run_tile_explicit_wide(const AttnArgs& a) {
  if (a.d == 128) return run_tile_explicit_wide_d<T, 128>(a);
  if (a.d == 256) return run_tile_explicit_wide_d<T, 256>(a);
  return SGA_ERR_UNSUPPORTED;
}

// Shape of a window launch: the classes the tiles are dealt over (residue classes of the whole
// sequence, or one class per block of a 2-D dilated mask) and the longest class.
struct WindowShape {
  int64_t seg_len;   // 0, or the block length of a 2-D dilated mask
  int64_t n_slots;   // residue classes, or blocks
  int64_t Lc;        // tokens of the longest class
};
WindowShape window_shape(const AttnArgs& a) {
  WindowShape w;
  if (a.mask_kind == SGA_MASK_DILATED_2D) {
    const int64_t span = a.block < a.L ? a.block : a.L;
    w.seg_len = a.block;
    w.n_slots = (a.L + a.block - 1) / a.block;
    w.Lc = (span + a.stride - 1) / a.stride;
  } else {
    w.seg_len = 0;
    w.n_slots = a.stride;
    w.Lc = (a.L + a.stride - 1) / a.stride;
  }
  return w;
}

// 2-D dilated masks: rows off the stride have no neighbour; a forward call writes their initial
// state, a continuing call leaves them as they are.
template <typename T>
void clear_unselected_rows(const AttnArgs& a) {
  if (a.mask_kind != SGA_MASK_DILATED_2D || a.stride == 1 || a.accumulate) return;
  const int64_t chunks = (int64_t)a.H * a.L * (a.d * (int64_t)sizeof(T) / 16);
  int64_t nwg = (chunks + 255) / 256;
  if (nwg > 8192) nwg = 8192;
  hipLaunchKernelGGL(clear_unselected_rows_kernel<T>, dim3((unsigned)nwg), dim3(256), 0, a.stream,
                     static_cast<T*>(a.O), a.lse, a.L, (int64_t)a.H, a.d, (int64_t)a.block,
                     (int64_t)a.stride);
}

// A window call with few tiles and many key blocks per tile (a short sequence with a wide
// window, one head) is cut into ranges of at least 16 key blocks per tile.  The chip runs
// `resident` tiles at a time, so k ranges cost about ceil(tiles * k / resident) rounds of
// ceil(blocks / k) blocks each, plus the partial states and their merge (taken as 4 blocks per
// range): the cheapest k <= kMaxWindowSplit wins.  The partial states go to the workspace; without
// room for them (or without a workspace) the call is not cut.  Returns k and sets *parts.
int choose_window_split(const AttnArgs& a, int64_t tile_heads, int64_t resident, float** parts) {
  *parts = nullptr;
  const int64_t blocks_per_tile = (2 * (int64_t)a.window + kTile - 1) / kTile + 1;
  if (!a.ws || tile_heads >= 4 * resident || blocks_per_tile < 32) return 1;
  const WorkspacePlan pl = plan_workspace(a.L, a.H, -1, a.dtype, a.d);
  if (pl.total_bytes > a.ws_bytes || tile_heads > pl.cap_wparts) return 1;
  int64_t want = 1, best = blocks_per_tile * ((tile_heads + resident - 1) / resident);
  for (int64_t k = 2; k <= kMaxWindowSplit && blocks_per_tile / k >= 16; ++k) {
    const int64_t cost = (tile_heads * k + resident - 1) / resident * ((blocks_per_tile + k - 1) / k) + 4 * k;
    if (cost < best) {
      best = cost;
      want = k;
    }
  }
  if (want > 1) *parts = reinterpret_cast<float*>(static_cast<char*>(a.ws) + pl.off_wparts);
  return (int)want;
}

// fp16 windows at d = 128: true where tile_window_band128_kernel, with so many workgroups of 128 queries that meet so many key
// blocks, beats tile_window_wide_kernel, whose workgroups hold one 32-query tile.  That one runs 1,024 tiles at a time and cuts
// fewer than 512 into ranges of their keys; the former takes 0.65 us a block and 7 us around them.  Calls of at most 64
// workgroups (256 tiles) may take window_share_wide's groups instead (W = 400 13.5).  (us, wide / band128,
// one head unless stated.  Up to 128 workgroups: L = 8,000, W = 2,000 60 / 87, 500 33 / 31; L = 16,000, W = 200 18 / 20, 400 30 / 27,
// 8,000 297 / 308.  Up to 256: L = 20,000, W = 300 26 / 24, 4,000 216 / 164; L = 30,000, W = 100 15.7 / 16.4, 200 22 / 20, 1,000
// 78 / 51; three heads, L = 16,384, W = 2,000 294 / 133.  Beyond: L = 60,000, W = 64 24 / 19, 130 35 / 24; L = 40,000,
// W = 10,000 959 / 565.)
bool band128_is_faster(int64_t wgs, int64_t blocks) {
  return wgs >= 512 || (wgs > 256 && blocks >= 8) || (wgs > 128 && blocks >= 20);
}

// Groups of d / 64 wavefronts per tile of a window call, in tile_window_wide_share_kernel (1: none, tile_window_wide_kernel),
// as window_share: a CU holds eight wavefronts, two groups want six blocks (with five d = 256 gains nothing and d = 128 no
// accuracy).  fp16 takes four groups or none: sums of two ranges are no more exact than of one (2.956e-4 -> 2.962e-4), of four
// they are; below ten blocks its calls wait for the host.
// (us, one group / shared, one head: fp32, d = 128, L = 8,000 (four groups), W = 50 16.4 / 13.5, 200 36.5 / 22.6, 400 63.4 / 33.7, 600 (two
// ranges of keys and their merge) 84 / 45; L = 16,000 (two), W = 100 33.5 / 23.7, 400 95 / 59; d = 256, L = 8,000 (two), W = 50
// 19.7 / 19.5, 200 42.4 / 36.1, 400 75.5 / 60.8; fp16, d = 128, L = 8,000, W = 100 12.0 / 12.4, 200 15.5 / 12.2, 400 25.4 / 13.5, 600
// 36.1 / 17.9; two groups, not taken: L = 16,000, W = 400 29.9 / 20.7, d = 256, L = 8,000 32.5 / 24.3.)
template <typename T, int kD>
int window_share_wide(int64_t tiles, int64_t blocks, int nsplit) {
  constexpr bool kF32 = DtypeOf<T>::code == SGA_F32;
  constexpr int64_t kPairs = 1024 * kHeadDim / kD;       // tiles whose two groups the chip holds at once
  const int most = kD == 128 && tiles <= kPairs / 2 ? 4 : kF32 && tiles <= kPairs ? 2 : 1;
  const int share = blocks < (kF32 ? most == 4 ? 4 : 6 : 10) ? 1 : most;
  return nsplit == 1 || share >= 2 * nsplit ? share : 1;
}

template <typename T, int kD>
sga_status run_tile_implicit_wide_d(const AttnArgs& a) {
  const int64_t s = a.stride;
  const WindowShape shape = window_shape(a);
  const int64_t n_tiles = (shape.Lc + kTile - 1) / kTile;     // workgroups per class
  const int64_t n_wg = (n_tiles * shape.n_slots + 7) / 8 * 8;
  if (n_wg >= (int64_t(1) << 31)) return SGA_ERR_OVERFLOW;
  constexpr int kPipe = DtypeOf<T>::code == SGA_F16 ? kPipeLdsK : kPipeRegK;
  constexpr int kSlices = kD / kHeadDim;
  clear_unselected_rows<T>(a);
  const int acc = a.accumulate ? 1 : 0;
  if constexpr (DtypeOf<T>::code == SGA_F16 && kD == 128) {
    // one wavefront per 32 queries with all 128 channels, key blocks staged once per 128 queries
    const int64_t n_groups = (n_tiles + 3) / 4;
    const int64_t n_wg128 = (n_groups * shape.n_slots + 7) / 8 * 8;
    const int64_t met = (4 * kTile - 1 + 2 * (int64_t)a.window) / kTile + 1;
    if (band128_is_faster(n_groups * shape.n_slots * a.H, met < n_tiles ? met : n_tiles)) {
      profile_mark_begin(a.stream, "tile_window_band128_kernel");
      hipLaunchKernelGGL(tile_window_band128_kernel, dim3((unsigned)n_wg128, (unsigned)a.H), dim3(256), 0, a.stream,
                         static_cast<const __half*>(a.Q), static_cast<const __half*>(a.K),
                         static_cast<const __half*>(a.V), static_cast<__half*>(a.O), a.lse, a.L,
                         (int64_t)a.window, s, n_groups, a.scale, acc, shape.seg_len);
      profile_mark_end(a.stream);
      return hip_status(hipGetLastError());
    }
  }
  float* parts = nullptr;
  const int nsplit = choose_window_split(a, n_wg * a.H, 2048 / kSlices, &parts);
  const int64_t met = (kTile - 1 + 2 * (int64_t)a.window) / kTile + 1;
  const int64_t blocks = met < n_tiles ? met : n_tiles;
  const int share = window_share_wide<T, kD>(n_tiles * shape.n_slots * a.H, blocks, nsplit);
  if constexpr (DtypeOf<T>::code == SGA_F32 || kD == 128) {
    if (share > 1) {
      void (*kernel)(const T*, const T*, const T*, T*, float*, int64_t, int64_t, int64_t, int64_t, float, int, int64_t) = nullptr;
      if constexpr (kD == 128) kernel = tile_window_wide_share_kernel<T, kD, 4, float>;
      if constexpr (kD == 128 && DtypeOf<T>::code == SGA_F32)
        if (blocks == 4) kernel = tile_window_wide_share_kernel<T, kD, 4, double>;            // (see add_states)
      if constexpr (DtypeOf<T>::code == SGA_F32)
        if (share == 2) kernel = tile_window_wide_share_kernel<T, kD, 2, float>;
      profile_mark_begin(a.stream, "tile_window_wide_share_kernel");
      hipLaunchKernelGGL(kernel, dim3((unsigned)n_wg, (unsigned)a.H), dim3(kD * share), 0, a.stream,
                         static_cast<const T*>(a.Q), static_cast<const T*>(a.K), static_cast<const T*>(a.V),
                         static_cast<T*>(a.O), a.lse, a.L, (int64_t)a.window, s, n_tiles, a.scale, acc, shape.seg_len);
      profile_mark_end(a.stream);
      return hip_status(hipGetLastError());
    }
  }
  profile_mark_begin(a.stream, "tile_window_wide_kernel");
  hipLaunchKernelGGL((tile_window_wide_kernel<T, kD, kPipe>), dim3((unsigned)(n_wg * nsplit), (unsigned)a.H),
                     dim3(kD), 0, a.stream, static_cast<const T*>(a.Q), static_cast<const T*>(a.K),
                     static_cast<const T*>(a.V), static_cast<T*>(a.O), a.lse, a.L, (int64_t)a.window, s,
                     n_tiles, a.scale, acc, shape.seg_len, nsplit, parts);
  profile_mark_end(a.stream);
  if (nsplit > 1)
    hipLaunchKernelGGL((window_merge_kernel<T, kD>), dim3((unsigned)n_wg, (unsigned)a.H, 4), dim3(kD), 0, a.stream,
                       static_cast<T*>(a.O), a.lse, parts, a.L, s, n_tiles, acc, shape.seg_len, nsplit);
  return hip_status(hipGetLastError());
}

template <typename T>
sga_status run_tile_implicit_wide(const AttnArgs& a) {
  if (a.d == 128) return run_tile_implicit_wide_d<T, 128>(a);
  if (a.d == 256) return run_tile_implicit_wide_d<T, 256>(a);
  return SGA_ERR_UNSUPPORTED;
}

// Wavefronts per tile of an fp32 window call that tile_window_f32_kernel leaves, in tile_window_share_kernel (1: none,
// tile_window_kernel): shorter chains of blocks.  A wavefront takes 2.1 us a block alone on its SIMD, two take 3.5 for one
// each.  Four per tile: up to 320 tiles, where a quarter of the SIMDs have two of them (up to 256 none).  Two per tile: up to
// 1,536 tiles, where three wavefronts of half the blocks follow each other on a SIMD (3.5 + 2.1 times half of them)
// instead of two of all of them (3.5 times all); beyond, four do, and lose.  Tiles of four and five blocks, which gain 2 to
// 6 % there, keep to 1,152; those of fewer gain nothing.  Ranges of keys that workgroups take (nsplit) stay where they
// leave no less than half a chain: their sums of several states are as exact, if slower.
// (us of the kernel, 1 / 2 / 4.  250 tiles, 4 blocks 14.0 / 9.2 / 7.1, 14 35.1 / 19.5 / 13.9, 26 60.3 / 31.3 / 20.7; 320 tiles, 4
// 14.1 / 9.4 / 10.0, 14 35.0 / 20.0 / 19.7, 26 60.3 / 32.1 / 30.1; 375, 4 14.2 / 9.5 / 10.1, 26 60.6 / 32.5 / 30.5; 1,024, 5
// 17.7 / 17.5 / 22.0, 26 63.9 / 55.4 / 58.4; 1,094, 5 25.8 / 24.9 / 27.2, 20 75.5 / 62.6 / 56.3; 1,188, 5 26.0 / 25.5 / 27.8, 14
// 56.0 / 47.0 / 44.6; 1,500, four heads, 6 29.9 / 27.3 / 32.7, 14 56.9 / 49.6 / 53.8; 1,536, 6 30.1 / 27.6 / 32.9, 14
// 56.8 / 49.1 / 53.0; 1,563, 6 29.9 / 32.0 / 36.2, 14 57.3 / 58.5 / 58.9.  Errors against 64 bits, 1 / 2: 6 blocks 1.39e-7 / 1.39e-7, 14
// 1.58e-7 / 1.51e-7, 20 1.66e-7 / 1.56e-7.  Two ranges and their merge / 4: L = 8,000, W = 600 53.5 / 25.3, 1.70e-7 / 1.62e-7; three
// ranges / 4: W = 1,000 51.9 / 37.1, 1.735e-7 / 1.740e-7.)
int window_share(int64_t tiles, int64_t blocks, int nsplit) {
  const int share = blocks < 4 ? 1 : tiles <= 320 ? 4 : tiles <= (blocks < 6 ? 1152 : 1536) ? 2 : 1;
  return nsplit == 1 || share >= 2 * nsplit ? share : 1;
}

// fp16 windows beyond the staged ones: true where tile_window_strip_kernel (128 queries per workgroup) is expected to beat
// tile_window_band_kernel (256).  A CU takes its workgroups of either kind at about one pace, alone or with others: a key
// block costs 0.59 us of the latter, 0.324 of the former, and a call 16 and 5 us around its blocks.  The CUs with one workgroup
// more than others decide a short call.  Beyond eight rounds of the strip kernel (256 of its workgroups each) the rounds run into
// each other, and the blocks of the band kernel cost 0.61 us.  Over 535 shapes (L 4,000 to 8,000,000, W 257 to 16,000, 1 to 32 heads,
// strides, 2-D blocks) the kernel taken is within 0.2 % of the faster one in the geometric mean, and 8 to 12 % behind it in five,
// four of them 2-D.  (us, band / strip near the line, the one taken marked: L = 8,000, 16 heads, W = 1,000
// 95 / 93.5*, 1,359 119.5 / 121.0*, 3,000 232* / 242; L = 65,536, W = 3,000 135.3 / 134.0*, 5,000 210* / 215; L = 100,000, W = 1,359
// 110.3 / 109.5*, 2,100 157* / 164; L = 400,000, W = 2,100 537* / 533, 5,000 1,198* / 1,221; L = 1,600,000, W = 1,000
// 1,093 / 1,067*, 1,359 1,368* / 1,382, 2,100 2,022* / 2,053; L = 4,000,000, W = 1,000 2,766 / 2,644*; L = 154,821, 32 heads,
// W = 771 2,812 / 2,637*.)
bool strip_is_faster(int64_t W, int64_t Lc, int64_t classes) {
  const int64_t held = (Lc + kTile - 1) / kTile;
  const bool many = (Lc + 4 * kTile - 1) / (4 * kTile) * classes > 8 * 256;
  const auto cost = [&](int64_t queries, double per_block, double last_round, double around) {
    const int64_t wgs = (Lc + queries - 1) / queries * classes, met = (queries - 1 + 2 * W) / kTile + 1;
    const double rounds = many ? (double)wgs / 256.0 + last_round : (double)((wgs + 255) / 256);
    return per_block * rounds * (double)(met < held ? met : held) + around;
  };
  return many ? cost(4 * kTile, 0.324, 0.25, 5.0) < cost(8 * kTile, 0.61, 0.0, 21.0)
              : cost(4 * kTile, 0.324, 0.0, 5.0) < cost(8 * kTile, 0.59, 0.0, 16.0);
}

sga_status run_tile_implicit(const AttnArgs& a) {
  if (a.d != kHeadDim)
    return a.dtype == SGA_F32 ? run_tile_implicit_wide<float>(a) : run_tile_implicit_wide<__half>(a);
  const int64_t s = a.stride;
  const WindowShape shape = window_shape(a);
  const int64_t Lc = shape.Lc;
  // fp16, 128 queries' key range fits the LDS at two workgroups per CU or more: one workgroup stages
  // it once (128 queries per workgroup, as in the fp32 kernel); wider fp16 windows: 32 or 64 queries per wavefront
  const bool wg = a.dtype == SGA_F16 && a.window <= kKvMaxWindow;
  const bool strip = a.dtype == SGA_F16 && !wg && strip_is_faster(a.window, Lc, shape.n_slots * a.H);
  const bool pair = a.dtype == SGA_F16 && !wg && !strip;
  const int64_t per_wave = pair ? 2 * kTile : kTile;
  const int64_t n_tiles = (Lc + per_wave - 1) / per_wave;
  const int64_t n_groups = (n_tiles + 3) / 4;           // workgroups per class
  const int64_t n_wg = (n_groups * shape.n_slots + 7) / 8 * 8;
  if (n_wg >= (int64_t(1) << 31)) return SGA_ERR_OVERFLOW;
  const dim3 grid((unsigned)n_wg, (unsigned)a.H);
  const int acc = a.accumulate ? 1 : 0;
  if (a.dtype == SGA_F32) clear_unselected_rows<float>(a); else clear_unselected_rows<__half>(a);
  const int64_t nb_max = (4 * kTile - 1 + 2 * (int64_t)a.window) / kTile + 1;   // key blocks of 128 queries
  const bool kv = wg && nb_max >= kKvMinBlocks;
  const int64_t staged = staged_blocks(a.window, Lc, kv ? 1 : 2);
  static_assert(CoreF16::kBlockBytes == kStagedBlockBytes && CoreF16::kTileBytes == kOutTileBytes, "see staged_blocks");
  const char* window_kernel = kv ? "tile_window_kv_kernel" : wg ? "tile_window_wg_kernel"
                              : strip ? "tile_window_strip_kernel"
                              : pair ? "tile_window_band_kernel" : "tile_window_kernel";
  if (wg || strip || pair) profile_mark_begin(a.stream, window_kernel);
  if (wg) {
    int64_t Lq = a.L / s, Lr = a.L % s;             // class lengths, see the kernel
    if (shape.seg_len > 0) {
      const int64_t last_len = a.L - (a.L - 1) / shape.seg_len * shape.seg_len;
      Lq = (shape.seg_len + s - 1) / s;
      Lr = (last_len + s - 1) / s;
    }
    const int64_t wave_blocks = subtile_blocks(a.window, Lc);
    const auto kv_kernel = wave_blocks <= 5   ? tile_window_kv_kernel<5>
                           : wave_blocks <= 7 ? tile_window_kv_kernel<7>
                           : wave_blocks <= 9 ? tile_window_kv_kernel<9>
                           : wave_blocks <= 11 ? tile_window_kv_kernel<11> : tile_window_kv_kernel<17>;
    if (kv)
      hipLaunchKernelGGL(kv_kernel, grid, dim3(256), (size_t)staged * CoreF16::kBlockBytes,
                         a.stream, static_cast<const __half*>(a.Q), static_cast<const __half*>(a.K),
                         static_cast<const __half*>(a.V), static_cast<__half*>(a.O), a.lse, a.L,
                         (int64_t)a.window, s, n_groups, a.scale, acc, (int)staged, shape.seg_len, Lq, Lr);
    else
      hipLaunchKernelGGL(tile_window_wg_kernel, grid, dim3(256), (size_t)staged * 2 * CoreF16::kBlockBytes,
                         a.stream, static_cast<const __half*>(a.Q), static_cast<const __half*>(a.K),
                         static_cast<const __half*>(a.V), static_cast<__half*>(a.O), a.lse, a.L,
                         (int64_t)a.window, s, n_groups, a.scale, acc, (int)staged, shape.seg_len, Lq, Lr);
  } else if (strip) {
    hipLaunchKernelGGL(tile_window_strip_kernel, grid, dim3(kStripWaves * kWave), 0, a.stream,
                       static_cast<const __half*>(a.Q), static_cast<const __half*>(a.K),
                       static_cast<const __half*>(a.V), static_cast<__half*>(a.O), a.lse, a.L,
                       (int64_t)a.window, s, n_groups, a.scale, acc, shape.seg_len);
  } else if (pair) {
    hipLaunchKernelGGL(tile_window_band_kernel, grid, dim3(256), 0, a.stream,
                       static_cast<const __half*>(a.Q), static_cast<const __half*>(a.K),
                       static_cast<const __half*>(a.V), static_cast<__half*>(a.O), a.lse, a.L,
                       (int64_t)a.window, s, n_groups, a.scale, acc, shape.seg_len);
  } else {
    float* parts = nullptr;
    const int nsplit = choose_window_split(a, n_wg * 4 * a.H, 2048, &parts);
    // Key blocks that the workgroups of 128 queries step through in total: from kSharedSteps on the
    // kernel that shares them (tile_window_f32_kernel) is the faster one, below it a step's latency
    // counts, which the shared form lengthens.  (One head, us, own blocks / shared: L = 32,768, +-64
    // 18 / 23, +-500 78 / 65; L = 98,304, +-32 31 / 32, +-128 63 / 54; L = 131,072, +-32 40 / 42;
    // L = 200,000, +-32 69 / 65.)
    const int64_t class_blocks = (Lc + kTile - 1) / kTile;
    const int64_t steps = n_groups * shape.n_slots * a.H * (nb_max < class_blocks ? nb_max : class_blocks);
    const bool shared = !a.split && steps >= kSharedSteps;
    const int64_t tiles = (Lc + kTile - 1) / kTile, mine = (kTile - 1 + 2 * (int64_t)a.window) / kTile + 1;
    const int64_t blocks = mine < class_blocks ? mine : class_blocks;
    const int share = a.split || shared ? 1 : window_share(tiles * shape.n_slots * a.H, blocks, nsplit);
    if (share > 1) {
      const int64_t ng = (tiles * share + 3) / 4;
      const dim3 share_grid((unsigned)((ng * shape.n_slots + 7) / 8 * 8), (unsigned)a.H);
      profile_mark_begin(a.stream, "tile_window_share_kernel");
      auto share_kernel = share == 4    ? tile_window_share_kernel<4, float>
                          : blocks == 4 ? tile_window_share_kernel<2, double>            // (see add_states)
                                        : tile_window_share_kernel<2, float>;
      hipLaunchKernelGGL(share_kernel, share_grid, dim3(256), 0, a.stream, static_cast<const float*>(a.Q), static_cast<const float*>(a.K),
                         static_cast<const float*>(a.V), static_cast<float*>(a.O), a.lse, a.L, (int64_t)a.window, s, ng,
                         a.scale, acc, shape.seg_len);
      profile_mark_end(a.stream);
      return hip_status(hipGetLastError());
    }
    if (shared) window_kernel = "tile_window_f32_kernel";
    profile_mark_begin(a.stream, window_kernel);
    auto kernel = a.split ? tile_window_kernel<float, kPipeSplit>
                  : shared ? tile_window_f32_kernel : tile_window_kernel<float, kPipeRegK>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(n_wg * nsplit), (unsigned)a.H), dim3(256), 0, a.stream,
                       static_cast<const float*>(a.Q), static_cast<const float*>(a.K),
                       static_cast<const float*>(a.V), static_cast<float*>(a.O), a.lse, a.L,
                       (int64_t)a.window, s, n_groups, a.scale, acc, shape.seg_len, nsplit, parts);
    if (nsplit > 1) {
      profile_mark_end(a.stream);
      hipLaunchKernelGGL((window_merge_kernel<float, kHeadDim>), dim3((unsigned)(n_wg * 4), (unsigned)a.H, 4),
                         dim3(kHeadDim), 0, a.stream, static_cast<float*>(a.O), a.lse, parts, a.L, s, n_groups,
                         acc, shape.seg_len, nsplit);
      return hip_status(hipGetLastError());
    }
  }
  profile_mark_end(a.stream);
  return hip_status(hipGetLastError());
}

}  // namespace

// The CSR -> tile pass is a chain of dependent loads per item: one wavefront per tile and a
// margin for the extra segments keeps every item's chain in flight at once; from the fourfold of what the chip holds on,
// wavefronts that go on to further items save the start of others (BigBird mask of 32-token blocks, L = 524,288, mask
// build and forward, us, at most 16,384 workgroups / 4,096: 425 / 405; +-300, L = 300,000 318 / 310).
void launch_tile_analyze(const AttnArgs& a) {
  const int64_t n_tiles = (a.L + kTile - 1) / kTile;
  int64_t nwg_analyze = n_tiles + 64;
  if (nwg_analyze < 2048) nwg_analyze = 2048;
  if (nwg_analyze > 4096) nwg_analyze = 4096;
  hipLaunchKernelGGL(tile_analyze_kernel, dim3((unsigned)nwg_analyze), dim3(256), 0, a.stream, a.row_ptr,
                     a.col_idx, a.L, a.H, a.dtype, a.d, a.ws, a.ws_bytes);
}

sga_status launch_tile_explicit(const AttnArgs& a) {
  if (!a.ws || a.ws_bytes < 256) return launch_gather_explicit(a, false, false);
  // (a prepared graph in which no tile qualified goes straight to the per-row kernels)
  if (!(a.prepared && a.plan_no_tiles)) {
    const sga_status st = a.dtype == SGA_F32 ? run_tile_explicit<float>(a) : run_tile_explicit<__half>(a);
    if (st != SGA_OK) return st;
  }
  if (a.prepared && a.plan_tiles_cover_all) return SGA_OK;
  // rows of tiles that did not qualify (or everything, if the workspace is too small)
  return launch_gather_explicit(a, true, true);
}

namespace {
template <typename T>
void run_tile_nonlocal(const AttnArgs& a, int64_t g, float* partials, int32_t* n_chunks) {
  constexpr int kPipe = DtypeOf<T>::code == SGA_F16 ? kPipeLdsK : kPipeRegK;
  const T* Q = static_cast<const T*>(a.Q);
  const T* K = static_cast<const T*>(a.K);
  const T* V = static_cast<const T*>(a.V);
  const int acc = a.accumulate ? 1 : 0;
  const int64_t first_tile = g / kTile, n_tiles = (a.L + kTile - 1) / kTile;
  const int64_t col_wgs = n_tiles > first_tile && a.L > g ? (n_tiles - first_tile + 3) / 4 : 0;
  int64_t ranges = 0, per = 1, row_wgs = 0;
  if (g > 0) {
    // ranges of at least 8 key blocks, as many as the partial states of the workspace allow
    // (kMaxImplicitGlobal rows x kMaxSplit ranges in all: fewer global rows, more ranges each)
    const int64_t g_tiles = (g + kTile - 1) / kTile;
    int64_t max_ranges = (int64_t)kMaxImplicitGlobal * kMaxSplit / (g_tiles * kTile);
    if (max_ranges > 256) max_ranges = 256;
    per = (n_tiles + max_ranges - 1) / max_ranges;
    if (per < 8) per = 8;
    ranges = (n_tiles + per - 1) / per;
    row_wgs = g_tiles * ranges;
  }
  *n_chunks = (int32_t)ranges;
  if (row_wgs + col_wgs == 0) return;
  profile_mark_begin(a.stream, "tile_nonlocal_kernel");
  hipLaunchKernelGGL((tile_nonlocal_kernel<T, kPipe>), dim3((unsigned)(row_wgs + col_wgs), (unsigned)a.H), dim3(256), 0,
                     a.stream, Q, K, V, static_cast<T*>(a.O), a.lse, a.L, (int64_t)a.window, g, a.scale, acc,
                     (uint32_t)row_wgs, (uint32_t)ranges, per, partials);
  profile_mark_end(a.stream);
}
}  // namespace

namespace {
template <typename T, int kD>
void run_tile_nonlocal_wide(const AttnArgs& a, int64_t g, float* partials, int32_t* n_chunks) {
  constexpr int kPipe = DtypeOf<T>::code == SGA_F16 ? kPipeLdsK : kPipeRegK;
  const T* Q = static_cast<const T*>(a.Q);
  const T* K = static_cast<const T*>(a.K);
  const T* V = static_cast<const T*>(a.V);
  const int acc = a.accumulate ? 1 : 0;
  const int64_t first_tile = g / kTile, n_tiles = (a.L + kTile - 1) / kTile;
  if (n_tiles > first_tile && a.L > g) {
    profile_mark_begin(a.stream, "tile_nonlocal_cols_wide_kernel");
    hipLaunchKernelGGL((tile_nonlocal_cols_wide_kernel<T, kD, kPipe>), dim3((unsigned)(n_tiles - first_tile), (unsigned)a.H),
                       dim3(kD), 0, a.stream, Q, K, V, static_cast<T*>(a.O), a.lse, a.L, (int64_t)a.window, g, a.scale,
                       acc);
    profile_mark_end(a.stream);
  }
  *n_chunks = 0;
  if (g > 0) {
    const int64_t g_rows = (g + kTile - 1) / kTile * kTile;
    int64_t max_ranges = (int64_t)kMaxImplicitGlobal * kMaxSplit / g_rows;
    if (max_ranges > 256) max_ranges = 256;
    int64_t per = (n_tiles + max_ranges - 1) / max_ranges;
    if (per < 8) per = 8;
    const int64_t ranges = (n_tiles + per - 1) / per;
    *n_chunks = (int32_t)ranges;
    hipLaunchKernelGGL((tile_nonlocal_rows_wide_kernel<T, kD, kPipe>),
                       dim3((unsigned)ranges, (unsigned)((g + kTile - 1) / kTile), (unsigned)a.H), dim3(kD), 0, a.stream,
                       Q, K, V, a.L, (int64_t)a.window, g, per, a.scale, partials);
  }
}
}  // namespace

void launch_tile_nonlocal(const AttnArgs& a, int64_t g, float* partials, int32_t* n_chunks) {
  if (a.d == 128) {
    if (a.dtype == SGA_F32) run_tile_nonlocal_wide<float, 128>(a, g, partials, n_chunks);
    else run_tile_nonlocal_wide<__half, 128>(a, g, partials, n_chunks);
  } else if (a.d == 256) {
    if (a.dtype == SGA_F32) run_tile_nonlocal_wide<float, 256>(a, g, partials, n_chunks);
    else run_tile_nonlocal_wide<__half, 256>(a, g, partials, n_chunks);
  } else {
    if (a.dtype == SGA_F32) run_tile_nonlocal<float>(a, g, partials, n_chunks);
    else run_tile_nonlocal<__half>(a, g, partials, n_chunks);
  }
}

sga_status launch_tile_implicit(const AttnArgs& a) {
  // (the tile kernels keep per-lane byte offsets of up to 31 keys in 32 bits, which bounds the
  // distance between consecutive keys of a class to 2^27 bytes)
  const int64_t key_bytes = (int64_t)a.stride * a.d * (a.dtype == SGA_F32 ? 4 : 2);
  if (a.H > 65535 || key_bytes > (int64_t(1) << 27)) return launch_gather_implicit(a);
  return run_tile_implicit(a);
}

}  // namespace sga
