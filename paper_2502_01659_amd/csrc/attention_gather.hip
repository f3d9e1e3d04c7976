// Gather path of Algorithm 1: one wavefront per query row, per-edge K/V row gathers.
//
// Lane layout.  A K or V row is d*4 B (fp32) or d*2 B (fp16), d in {32, 64, 128, 256}; a
// group of LPK lanes reads one row with one 16-byte load per lane (LPK = d/4 for fp32, d/8
// for fp16: 16 and 8 at d = 64), so a wavefront pulls G = 64/LPK rows per load instruction
// and every row is a fully coalesced gather.  The dot product Q_i.K_j is reduced inside the lane
// group with DPP adds (no LDS); each group keeps its own running (m, l, acc) state of
// the recurrence in Algorithm 1 for the keys it has seen, and the G group states are
// merged with wavefront shuffles once per row.  The accumulator is kept un-normalised
// and divided by l once at the end, which is the same real number as the per-step
// normalisation printed in Algorithm 1.
//
// Rows with more than kSplitThreshold neighbours (global tokens) are split into chunks
// that separate wavefronts reduce to partial (m, l, acc) states; a merge kernel combines
// the partials in chunk order, so the result is deterministic.
#include <type_traits>

#include "sga_internal.h"
#include "tile_merge.h"

namespace sga {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kMinusHuge = -1.0e30f;   // finite stand-in for m = -inf (keeps m - m finite)
constexpr int kUnroll = 4;               // keys per lane group per loop trip

template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, false));
}

// Sum over the LPK consecutive lanes of a group; every lane of the group gets the total.
template <int LPK>
__device__ __forceinline__ float group_sum(float x) {
  static_assert(LPK == 4 || LPK == 8 || LPK == 16 || LPK == 32 || LPK == 64, "lanes per row");
  x += dpp<0xB1>(x);    // quad_perm [1,0,3,2]
  x += dpp<0x4E>(x);    // quad_perm [2,3,0,1]
  if (LPK >= 8) x += dpp<0x141>(x);    // row_half_mirror: lane k <-> 7-k of each 8
  if (LPK >= 16) x += dpp<0x140>(x);   // row_mirror: lane k <-> 15-k of each 16
  if (LPK >= 32) x += __shfl_xor(x, 16, kWave);
  if (LPK >= 64) x += __shfl_xor(x, 32, kWave);
  return x;
}

template <typename T, int D>
struct Row;

template <int D>
struct Row<float, D> {
  static constexpr int VEC = 4, LPK = D / VEC;
  __device__ static void load(const float* p, float (&v)[4]) {
    const float4 t = *reinterpret_cast<const float4*>(p);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  }
  __device__ static void store(float* p, const float (&v)[4]) {
    *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
  }
};

template <int D>
struct Row<__half, D> {
  static constexpr int VEC = 8, LPK = D / VEC;
  __device__ static void load(const __half* p, float (&v)[8]) {
    const uint4 t = *reinterpret_cast<const uint4*>(p);
    const uint32_t w[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const __half2 h = __builtin_bit_cast(__half2, w[k]);
      v[2 * k] = __low2float(h);
      v[2 * k + 1] = __high2float(h);
    }
  }
  __device__ static void store(__half* p, const float (&v)[8]) {
    uint32_t w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      w[k] = __builtin_bit_cast(uint32_t, __floats2half2_rn(v[2 * k], v[2 * k + 1]));
    *reinterpret_cast<uint4*>(p) = make_uint4(w[0], w[1], w[2], w[3]);
  }
};

__device__ __forceinline__ float load_scalar(const float* p) { return *p; }
__device__ __forceinline__ float load_scalar(const __half* p) { return __half2float(*p); }
__device__ __forceinline__ void store_scalar(float* p, float v) { *p = v; }
__device__ __forceinline__ void store_scalar(__half* p, float v) { *p = __float2half_rn(v); }

struct WindowNeighbours {   // Get_Neighbors, implicit: j = first + e*step
  int64_t first, step;
  __device__ int64_t operator()(int64_t e) const { return first + e * step; }
};

// Running state of one lane group for the channels this lane owns.
template <int VEC>
struct State {
  float m, l, acc[VEC];
  __device__ void init() {
    m = kMinusHuge;
    l = 0.f;
#pragma unroll
    for (int c = 0; c < VEC; ++c) acc[c] = 0.f;
  }
};

// One step of the recurrence for kUnroll keys per lane group, K and V rows already in registers.
template <int LPK, int VEC>
__device__ __forceinline__ void attend_loaded(const float (&q)[VEC], const float (&kf)[kUnroll][VEC],
                                              const float (&vf)[kUnroll][VEC], const bool (&valid)[kUnroll],
                                              State<VEC>& st) {
  float s[kUnroll];
  float smax = st.m;
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    float part = 0.f;
#pragma unroll
    for (int c = 0; c < VEC; ++c) part = __builtin_fmaf(q[c], kf[u][c], part);
    part = group_sum<LPK>(part);
    s[u] = valid[u] ? part : -INFINITY;
    smax = fmaxf(smax, s[u]);
  }
  const float alpha = __builtin_amdgcn_exp2f(st.m - smax);
  st.l *= alpha;
#pragma unroll
  for (int c = 0; c < VEC; ++c) st.acc[c] *= alpha;
#pragma unroll
  for (int u = 0; u < kUnroll; ++u) {
    const float p = __builtin_amdgcn_exp2f(s[u] - smax);
    st.l += p;
#pragma unroll
    for (int c = 0; c < VEC; ++c) st.acc[c] = __builtin_fmaf(p, vf[u][c], st.acc[c]);
  }
  st.m = smax;
}

// Visit edges [e0, e1) of one row.  q holds this lane's channels of Q_i * scale * log2(e).
template <typename T, int D, typename Nbr>
__device__ __forceinline__ void attend_range(const T* __restrict__ Kh, const T* __restrict__ Vh,
                                             const float (&q)[Row<T, D>::VEC], const Nbr& nbr,
                                             int64_t e0, int64_t e1, int lane,
                                             State<Row<T, D>::VEC>& st) {
  constexpr int LPK = Row<T, D>::LPK, VEC = Row<T, D>::VEC, G = kWave / LPK;
  const int grp = lane / LPK;
  const int cofs = (lane % LPK) * VEC;
  for (int64_t base = e0; base < e1; base += G * kUnroll) {
    float kf[kUnroll][VEC], vf[kUnroll][VEC];
    bool valid[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int64_t e = base + u * G + grp;
      valid[u] = e < e1;
      const int64_t j = nbr(valid[u] ? e : e1 - 1);   // out-of-range lanes re-read a real neighbour
      Row<T, D>::load(Kh + j * D + cofs, kf[u]);
      Row<T, D>::load(Vh + j * D + cofs, vf[u]);
    }
    attend_loaded<LPK, VEC>(q, kf, vf, valid, st);
  }
}

// attend_range over a slice of col_idx (explicit Get_Neighbors).  The column indices are read 64
// at a time with one coalesced load (lane l holds column base + l) and handed to the lane groups
// through the LDS crossbar, and the next 64 are requested before the current ones are used: the
// K/V row gathers then no longer wait for an index load of their own each, and a third of the
// vector memory instructions go away.
// kNear: one head's K (and V) is below 4 GiB, so row offsets fit 32 bits.
template <typename T, int D, bool kNear>
__device__ __forceinline__ void attend_columns(const T* __restrict__ Kh, const T* __restrict__ Vh,
                                               const float (&q)[Row<T, D>::VEC],
                                               const int32_t* __restrict__ cols, int64_t e0, int64_t e1,
                                               int lane, State<Row<T, D>::VEC>& st) {
  constexpr int LPK = Row<T, D>::LPK, VEC = Row<T, D>::VEC, G = kWave / LPK;
  constexpr int kStep = G * kUnroll;                 // edges per step of the recurrence
  static_assert(kWave % kStep == 0, "a batch of 64 columns is a whole number of steps");
  if (e0 >= e1) return;
  const int grp = lane / LPK;
  const int cofs = (lane % LPK) * VEC;
  const int64_t last = e1 - 1;
  int32_t cur = cols[e0 + lane < last ? e0 + lane : last];
  for (int64_t base = e0; base < e1; base += kWave) {
    const int64_t nb = base + kWave;
    int32_t nxt = 0;
    if (nb < e1) nxt = cols[nb + lane < last ? nb + lane : last];
    const int n_here = e1 - base < kWave ? (int)(e1 - base) : kWave;     // columns of this batch
#pragma unroll
    for (int sub = 0; sub < kWave / kStep; ++sub) {
      if (sub * kStep >= n_here) break;
      float kf[kUnroll][VEC], vf[kUnroll][VEC];
      bool valid[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int el = sub * kStep + u * G + grp;
        valid[u] = el < n_here;
        const int32_t j = __shfl(cur, valid[u] ? el : n_here - 1, kWave);   // out-of-range lanes re-read a real neighbour
        if (kNear) {
          // one 32-bit byte offset serves the K and the V row (wave-uniform base + per-lane offset)
          const uint32_t off = (uint32_t)j * (uint32_t)(D * sizeof(T)) + (uint32_t)(cofs * sizeof(T));
          Row<T, D>::load(reinterpret_cast<const T*>(reinterpret_cast<const char*>(Kh) + off), kf[u]);
          Row<T, D>::load(reinterpret_cast<const T*>(reinterpret_cast<const char*>(Vh) + off), vf[u]);
        } else {
          Row<T, D>::load(Kh + (int64_t)j * D + cofs, kf[u]);
          Row<T, D>::load(Vh + (int64_t)j * D + cofs, vf[u]);
        }
      }
      attend_loaded<LPK, VEC>(q, kf, vf, valid, st);
    }
    cur = nxt;
  }
}

// st and another state of the same row, as one.
template <int VEC>
__device__ __forceinline__ void merge_state(State<VEC>& st, const State<VEC>& other) {
  const float mn = fmaxf(st.m, other.m);
  const float a1 = __builtin_amdgcn_exp2f(st.m - mn);
  const float a2 = __builtin_amdgcn_exp2f(other.m - mn);
  st.l = __builtin_fmaf(st.l, a1, other.l * a2);
#pragma unroll
  for (int c = 0; c < VEC; ++c) st.acc[c] = __builtin_fmaf(st.acc[c], a1, other.acc[c] * a2);
  st.m = mn;
}

// Merge the G lane-group states of a wavefront; afterwards every group holds the row's state.
template <int LPK, int VEC>
__device__ __forceinline__ void merge_groups(State<VEC>& st) {
#pragma unroll
  for (int off = LPK; off < kWave; off <<= 1) {
    State<VEC> other;
    other.m = __shfl_xor(st.m, off, kWave);
    other.l = __shfl_xor(st.l, off, kWave);
#pragma unroll
    for (int c = 0; c < VEC; ++c) other.acc[c] = __shfl_xor(st.acc[c], off, kWave);
    merge_state(st, other);
  }
}

template <typename T, int D>
__device__ __forceinline__ void load_query(const T* Qrow, float scale, int lane,
                                           float (&q)[Row<T, D>::VEC]) {
  Row<T, D>::load(Qrow + (lane % Row<T, D>::LPK) * Row<T, D>::VEC, q);
  const float c = scale * kLog2e;
#pragma unroll
  for (int k = 0; k < Row<T, D>::VEC; ++k) q[k] *= c;
}

// Normalise and store a row whose whole state the lanes of a group hold (cl: the lane's place in it; store: this
// group writes); with `accumulate` the row continues the (O, lse) state already
// in the output buffers (sequential composition on one state, Section V-F).
template <typename T, int D>
__device__ __forceinline__ void finish_merged(T* Orow, float* lse_i, int cl, bool store,
                                              const State<Row<T, D>::VEC>& st, bool accumulate) {
  constexpr int VEC = Row<T, D>::VEC;
  const bool empty = !(st.l > 0.f);
  float inv = empty ? 0.f : 1.0f / st.l;
  float lse_row = empty ? -INFINITY : (st.m + __builtin_amdgcn_logf(st.l)) * kLn2;
  float w_prev = 0.f;
  if (accumulate) {     // every lane reads the earlier lse before lane 0 replaces it
    const CarryWeights cw = carry_weights(*lse_i, lse_row);
    inv *= cw.w_now;
    w_prev = cw.w_prev;
    lse_row = cw.lse;
  }
  float o[VEC];
#pragma unroll
  for (int c = 0; c < VEC; ++c) o[c] = st.acc[c] * inv;
  if (!store) return;
  if (accumulate) {
    float old[VEC];
    Row<T, D>::load(Orow + cl * VEC, old);
#pragma unroll
    for (int c = 0; c < VEC; ++c) o[c] = __builtin_fmaf(w_prev, old[c], o[c]);
  }
  Row<T, D>::store(Orow + cl * VEC, o);
  if (lse_i && cl == 0) *lse_i = lse_row;
}

template <typename T, int D>
__device__ __forceinline__ void finish_row(T* Orow, float* lse_i, int lane,
                                           State<Row<T, D>::VEC>& st, bool accumulate) {
  constexpr int LPK = Row<T, D>::LPK;
  merge_groups<LPK, Row<T, D>::VEC>(st);
  finish_merged<T, D>(Orow, lse_i, lane % LPK, lane < LPK, st, accumulate);
}

__host__ __device__ inline void split_shape(int64_t deg, int chunk, int32_t& nchunks, int32_t& len) {
  int64_t n = (deg + chunk - 1) / chunk;
  if (n > kMaxSplit) n = kMaxSplit;
  int64_t l = (deg + n - 1) / n;
  l = (l + 31) / 32 * 32;
  len = (int32_t)l;
  nchunks = (int32_t)((deg + l - 1) / l);
}

// ---- kernels ----------------------------------------------------------------

// Zeroes the counters and (tile_flags != 0) the per-tile flags of the tile path.
__global__ __launch_bounds__(256) void clear_workspace_kernel(void* ws, size_t ws_bytes,
                                                              const int64_t* row_ptr, int64_t L,
                                                              int32_t H, int32_t dtype, int32_t d,
                                                              int tile_flags) {
  uint32_t* ctr = reinterpret_cast<uint32_t*>(ws);
  if (blockIdx.x == 0 && threadIdx.x < kNumCounters) ctr[threadIdx.x] = 0;
  if (!tile_flags) return;
  const WorkspacePlan pl = plan_workspace(L, H, row_ptr[L], dtype, d);
  if (pl.total_bytes > ws_bytes) return;
  int32_t* bad = reinterpret_cast<int32_t*>(static_cast<char*>(ws) + pl.off_tile_bad);
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < pl.n_tiles;
       t += (int64_t)gridDim.x * blockDim.x)
    bad[t] = 0;
  uint32_t* next = reinterpret_cast<uint32_t*>(static_cast<char*>(ws) + pl.off_work_next);
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < (int64_t)H;
       i += (int64_t)gridDim.x * blockDim.x)
    next[i] = 0;          // claim counters of the heads
}

// One thread per row, see record_split_rows: the rows of a call on the per-row kernels alone, or (after_tiles) the rows
// that the tile path left over where the CSR -> tile pass could not tell (tile_parts_in_doubt).
__global__ __launch_bounds__(256) void split_prepass_kernel(const int64_t* __restrict__ row_ptr,
                                                            int64_t L, int32_t H, int32_t dtype,
                                                            int32_t d, void* ws, size_t ws_bytes, int after_tiles) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  bool mine = i < L && row_ptr[i + 1] - row_ptr[i] > kSplitThreshold / 2;      // (no rule splits a shorter row)
  if (!__any(mine)) return;
  const WorkspacePlan pl = plan_workspace(L, H, row_ptr[L], dtype, d);
  if (pl.total_bytes > ws_bytes || (after_tiles && !tile_parts_in_doubt(pl))) return;
  if (mine && after_tiles) mine = !tile_handled(pl, ws, row_ptr, L, i / kTile);
  record_split_rows(row_ptr, i, mine, pl, ws);
}

// The list of long rows that this call uses.
__device__ __forceinline__ const int4* long_rows(const WorkspacePlan& pl, const void* ws, uint32_t& max_chunks) {
  const uint32_t* ctr = reinterpret_cast<const uint32_t*>(ws);
  const bool fine = split_is_fine(pl, ctr);
  max_chunks = ctr[fine ? kCtrMaxChunksFine : kCtrMaxChunks];
  return reinterpret_cast<const int4*>(static_cast<const char*>(ws) + pl.off_long) + (fine ? pl.cap_items : 0);
}

// True when the long rows of this call are handled by the chunk kernels.
__device__ __forceinline__ bool split_active(const int64_t* row_ptr, int64_t L, int32_t H,
                                             int32_t dtype, int32_t d, const void* ws,
                                             size_t ws_bytes) {
  if (!ws) return false;
  const WorkspacePlan pl = plan_workspace(L, H, row_ptr[L], dtype, d);
  if (pl.total_bytes > ws_bytes) return false;
  const uint32_t need = reinterpret_cast<const uint32_t*>(ws)[kCtrChunksNeeded];
  return (int64_t)need <= pl.cap_items;
}

// True when this call's tile path produced row i (its 32-row tile has a block list).
__device__ __forceinline__ bool row_done_by_tiles(const int64_t* row_ptr, int64_t L, int32_t H,
                                                  int32_t dtype, int32_t d, const void* ws,
                                                  size_t ws_bytes, int64_t i) {
  const WorkspacePlan pl = plan_workspace(L, H, row_ptr[L], dtype, d);
  if (pl.total_bytes > ws_bytes) return false;
  return tile_handled(pl, ws, row_ptr, L, i / kTile);
}

// (wg of n_wg: this workgroup's place among those that share the rows of a head)
template <typename T, int D>
__device__ __forceinline__ void gather_csr_body(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, T* __restrict__ O,
    float* __restrict__ lse, const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
    int64_t L, float scale, const void* ws, size_t ws_bytes, int use_split, int skip_tiled,
    int accumulate, uint32_t wg, uint32_t n_wg) {
  const int lane = threadIdx.x & (kWave - 1);
  const int waves = blockDim.x / kWave;
  const int64_t h = blockIdx.y;
  const int32_t H = (int32_t)gridDim.y;
  const int64_t hoff = h * L * D;
  // After the tile path the rows left are those of the tiles it gave up (the list the CSR -> tile
  // pass wrote) and, if the partial states of the multi-segment tiles did not fit, of those
  // tiles (the merge list): the wavefronts stride over these tiles' rows instead of testing
  // every row of the sequence (L = 262,144 with one tile left: 430 -> 10 microseconds).
  int64_t n_units = L;                  // rows, or 32 x listed tiles
  const int32_t* bad_list = nullptr;
  const int4* multi_list = nullptr;
  int64_t n_bad = 0, n_multi = 0;
  bool listed = false, parts_fit = true;
  WorkspacePlan pl{};
  if (skip_tiled) {
    pl = plan_workspace(L, H, row_ptr[L], DtypeOf<T>::code, D);
    if (pl.total_bytes <= ws_bytes) {
      if (tiles_cover_everything(pl, ws)) return;
      const uint32_t* ctr = reinterpret_cast<const uint32_t*>(ws);
      parts_fit = (int64_t)ctr[kCtrTilePartsNeeded] <= pl.cap_tparts;
      n_bad = ctr[kCtrTilesBad];
      n_multi = parts_fit ? 0 : ctr[kCtrMultiTiles];
      if (n_multi <= pl.cap_tparts) {     // (a merge list that overflowed is incomplete: test every row then)
        listed = true;
        bad_list = reinterpret_cast<const int32_t*>(static_cast<const char*>(ws) + pl.off_bad_list);
        multi_list = reinterpret_cast<const int4*>(static_cast<const char*>(ws) + pl.off_multi_tiles);
        n_units = (n_bad + n_multi) * kTile;
      }
    }
  }
  // (Every head starts its list on another XCD: n_wg is a multiple of 8, and the row of a global token, the longest,
  // often comes first.  One such token, L = 1,000, fp32, 8 heads, prepared, us: all on one XCD 63.5, so 46.8.
  // The head's first workgroups take the end of the list: where there are more rows than wavefronts the front ones have a
  // row more, and a last workgroup with the first rows ended late: 3 %, L = 6,000, fp32, d = 128, two heads 103 -> 110.)
  if (skip_tiled) {
    const uint32_t turn = (uint32_t)h & 7;
    wg = wg >= turn ? wg - turn : wg - turn + n_wg;
  }
  for (int64_t u = (int64_t)wg * waves + (threadIdx.x / kWave); u < n_units;
       u += (int64_t)n_wg * waves) {
    int64_t i = u;
    if (listed) {
      const int64_t ti = u / kTile;
      const int64_t t = ti < n_bad ? bad_list[ti] : multi_list[ti - n_bad].x;
      // (a multi-segment tile that was also given up is in both lists when the parts do not fit)
      if (ti < n_bad && !parts_fit && tile_segments(row_ptr, L, pl.seg_shift, t) > 1) continue;
      i = t * kTile + (u - ti * kTile);
      if (i >= L) continue;
    } else if (skip_tiled && row_done_by_tiles(row_ptr, L, H, DtypeOf<T>::code, D, ws, ws_bytes, i)) {
      continue;
    }
    const int64_t r0 = row_ptr[i], r1 = row_ptr[i + 1];
    if (use_split && r1 - r0 > kSplitThreshold / 2 && split_active(row_ptr, L, H, DtypeOf<T>::code, D, ws, ws_bytes) &&
        row_is_split(r1 - r0, plan_workspace(L, H, row_ptr[L], DtypeOf<T>::code, D)))
      continue;
    float q[Row<T, D>::VEC];
    load_query<T, D>(Q + hoff + i * D, scale, lane, q);
    State<Row<T, D>::VEC> st;
    st.init();
    if (L * D * (int64_t)sizeof(T) < (int64_t(1) << 32))
      attend_columns<T, D, true>(K + hoff, V + hoff, q, col_idx + r0, 0, r1 - r0, lane, st);
    else
      attend_columns<T, D, false>(K + hoff, V + hoff, q, col_idx + r0, 0, r1 - r0, lane, st);
    finish_row<T, D>(O + hoff + i * D, lse ? lse + h * L + i : nullptr, lane, st, accumulate != 0);
  }
}

template <typename T, int D>
__global__ __launch_bounds__(256) void gather_csr_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, T* __restrict__ O,
    float* __restrict__ lse, const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
    int64_t L, float scale, const void* ws, size_t ws_bytes, int use_split, int skip_tiled,
    int accumulate) {
  gather_csr_body<T, D>(Q, K, V, O, lse, row_ptr, col_idx, L, scale, ws, ws_bytes, use_split, skip_tiled,
                        accumulate, blockIdx.x, gridDim.x);
}

// Prepared graphs of short rows of about one length and no tiles, K and V beyond one L2 (even_rows): a row per group of
// LPK lanes, so that a wavefront takes G rows at once and four times (fp32, d = 64) as many rows are under way.  All
// of them read their sorted neighbours from the first key to the last at about the same pace, so a key that one row has
// brought into an L2 is still there for the others.  The arithmetic is gather_csr_body's: there group g of a wavefront
// takes every G-th edge from g on and the groups' states are merged, here one group holds those G states in turn;
// the bits are the same, and so are those of the call without a plan.  Bound by what misses the L2s (6.4 TB/s) where K and V
// are several times an L2: 35,000 rows of 35 neighbours, fp32, d = 64 77 -> 73 us; by the L2s below that: random 1 %,
// L = 24,576, fp32, d = 64 247 -> 177 us, d = 128 613 -> 571; fp16, d = 128 250 -> 178; L = 8,000, four heads, fp32, d = 64
// 92 -> 65.  Registers for four wavefronts per SIMD; with more, the G states spill (six: 277 us,
// eight: 422 of the 177).  Which of eight neighbouring workgroups takes which rows turns from eight to eight: else lengths
// that alternate every 64 rows (fp32, d = 64) leave the long rows to four of the XCDs (11 and 58 neighbours, L = 50,000
// 140 -> 112 us, a wavefront per row 111).
template <typename T, int D>
__global__ __attribute__((amdgpu_waves_per_eu(4))) __launch_bounds__(256) void gather_even_rows_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, T* __restrict__ O,
    float* __restrict__ lse, const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx, int64_t L, float scale,
    int accumulate) {
  constexpr int LPK = Row<T, D>::LPK, VEC = Row<T, D>::VEC, G = kWave / LPK;
  constexpr int kStep = G * kUnroll;
  static_assert(LPK % kStep == 0, "a group's columns are a whole number of steps");
  const int lane = threadIdx.x & (kWave - 1), cl = lane % LPK;
  const unsigned eight = blockIdx.x & ~7u;
  const unsigned wg = eight + 8 <= gridDim.x ? eight + ((blockIdx.x + (blockIdx.x >> 3)) & 7) : blockIdx.x;
  const int64_t i = ((int64_t)wg * 4 + threadIdx.x / kWave) * G + lane / LPK;
  if (i >= L) return;
  const int64_t h = blockIdx.y, hoff = h * L * D;
  const int64_t r0 = row_ptr[i];
  const int deg = (int)(row_ptr[i + 1] - r0);
  const int32_t* cols = col_idx + r0;
  const char* Kb = reinterpret_cast<const char*>(K + hoff);
  const char* Vb = reinterpret_cast<const char*>(V + hoff);
  float q[VEC];
  load_query<T, D>(Q + hoff + i * D, scale, lane, q);
  State<VEC> st[G];
#pragma unroll
  for (int g = 0; g < G; ++g) st[g].init();
  int32_t cur = deg > 0 ? cols[min(cl, deg - 1)] : 0;
  for (int base = 0; base < deg; base += LPK) {
    const int32_t nxt = cols[min(base + LPK + cl, deg - 1)];
#pragma unroll 1
    for (int sub = 0; sub < LPK; sub += kStep) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (base + sub + g < deg) {
          float kf[kUnroll][VEC], vf[kUnroll][VEC];
          bool valid[kUnroll];
#pragma unroll
          for (int u = 0; u < kUnroll; ++u) {
            const int el = sub + u * G + g;
            valid[u] = base + el < deg;
            const uint32_t off = (uint32_t)__shfl(cur, el, LPK) * (uint32_t)(D * sizeof(T)) + (uint32_t)(cl * VEC * sizeof(T));
            Row<T, D>::load(reinterpret_cast<const T*>(Kb + off), kf[u]);
            Row<T, D>::load(reinterpret_cast<const T*>(Vb + off), vf[u]);
          }
          attend_loaded<LPK, VEC>(q, kf, vf, valid, st[g]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    cur = nxt;
  }
#pragma unroll
  for (int n = 1; n < G; n <<= 1)
#pragma unroll
    for (int g = 0; g < G; g += 2 * n) merge_state(st[g], st[g + n]);
  finish_merged<T, D>(O + hoff + i * D, lse ? lse + h * L + i : nullptr, cl, true, st[0], accumulate != 0);
}

template <typename T, int D>
__global__ __launch_bounds__(256) void gather_window_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, T* __restrict__ O,
    float* __restrict__ lse, int64_t L, int64_t W, int64_t s, float scale, int accumulate) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t i = (int64_t)blockIdx.x * (blockDim.x / kWave) + (threadIdx.x / kWave);
  if (i >= L) return;
  const int64_t h = blockIdx.y;
  const int64_t hoff = h * L * D;
  const int64_t kl = min(W, i / s), kr = min(W, (L - 1 - i) / s);
  float q[Row<T, D>::VEC];
  load_query<T, D>(Q + hoff + i * D, scale, lane, q);
  State<Row<T, D>::VEC> st;
  st.init();
  WindowNeighbours nbr{i - kl * s, s};
  attend_range<T, D>(K + hoff, V + hoff, q, nbr, 0, kl + kr + 1, lane, st);
  finish_row<T, D>(O + hoff + i * D, lse ? lse + h * L + i : nullptr, lane, st, accumulate != 0);
}

// Implicit Get_Neighbors for the masks whose rows are one arithmetic run of keys that is not a
// centred window: the 2-D dilated blocks of Section II-C, and the rows below the global rows
// of the "global (non-local)" mask of Section IV-B.  One wavefront per row; a row without
// neighbours is written as the initial state (or left as it is when accumulating).
struct RowRun {
  int64_t first, step, count;
};

__device__ __forceinline__ RowRun row_run(int32_t kind, int64_t i, int64_t L, int64_t W, int64_t s,
                                          int64_t g, int64_t B) {
  if (kind == SGA_MASK_DILATED_2D) {
    const int64_t blk = i / B, r = i - blk * B;
    if (r % s != 0) return {0, 1, 0};
    const int64_t len = min(B, L - blk * B);
    return {blk * B, s, (len + s - 1) / s};
  }
  // non-local, row i >= g: global columns 0..g-1 that lie left of the window
  const int64_t n = min(g, i - W);
  return {0, 1, n > 0 ? n : 0};
}

template <typename T, int D>
__global__ __launch_bounds__(256) void gather_runs_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, T* __restrict__ O,
    float* __restrict__ lse, int64_t L, int32_t kind, int64_t W, int64_t s, int64_t g, int64_t B,
    int64_t row0, float scale, int accumulate) {
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t i = row0 + (int64_t)blockIdx.x * (blockDim.x / kWave) + (threadIdx.x / kWave);
  if (i >= L) return;
  const int64_t h = blockIdx.y;
  const int64_t hoff = h * L * D;
  const RowRun run = row_run(kind, i, L, W, s, g, B);
  float q[Row<T, D>::VEC];
  load_query<T, D>(Q + hoff + i * D, scale, lane, q);
  State<Row<T, D>::VEC> st;
  st.init();
  if (run.count > 0) {
    WindowNeighbours nbr{run.first, run.step};
    attend_range<T, D>(K + hoff, V + hoff, q, nbr, 0, run.count, lane, st);
  }
  finish_row<T, D>(O + hoff + i * D, lse ? lse + h * L + i : nullptr, lane, st, accumulate != 0);
}

// Partial states p0[c * step + ...] = {acc[D], m, l}, c < n, reduced in order to one; one wavefront, lane c
// owns channels c, c + 64, ...  The maxima are read 64 partials at a time and the states eight
// at a time, so that a row of a thousand chunks does not wait for a thousand loads one after the
// other; the sums run in chunk order all the same.  (The 256 partials of a global row of the
// non-local mask, a quarter per wavefront: 20 us one after the other.)
// Sum: what the sums are held in.
template <int D, typename Sum>
__device__ __forceinline__ void reduce_partials(const float* p0, int64_t step, int n, int lane, float& M, Sum& l,
                                                Sum (&acc)[(D + kWave - 1) / kWave]) {
  constexpr int kCh = (D + kWave - 1) / kWave;
  constexpr int kAhead = 8;
  M = kMinusHuge;
  for (int c = lane; c < n; c += kWave) M = fmaxf(M, p0[c * step + D]);
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) M = fmaxf(M, __shfl_xor(M, off, kWave));
  l = 0.f;
#pragma unroll
  for (int k = 0; k < kCh; ++k) acc[k] = 0.f;
  for (int c0 = 0; c0 < n; c0 += kAhead) {
    float mm[kAhead], ll[kAhead], aa[kAhead][kCh];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const float* p = p0 + (c0 + u < n ? c0 + u : n - 1) * step;
      mm[u] = p[D];
      ll[u] = p[D + 1];
#pragma unroll
      for (int k = 0; k < kCh; ++k) aa[u][k] = lane + k * kWave < D ? p[lane + k * kWave] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      if (c0 + u < n) {
        const Sum w = __builtin_amdgcn_exp2f(mm[u] - M);
        l = __builtin_elementwise_fma((Sum)ll[u], w, l);
#pragma unroll
        for (int k = 0; k < kCh; ++k) acc[k] = __builtin_elementwise_fma((Sum)aa[u][k], w, acc[k]);
      }
    }
  }
}
// ... and left as one partial state at `out`
template <int D, typename Sum = float>
__device__ __forceinline__ void combine_partials(const float* p0, int64_t step, int n, float* out, int lane) {
  constexpr int kCh = (D + kWave - 1) / kWave;
  float M;
  Sum l, acc[kCh];
  reduce_partials<D>(p0, step, n, lane, M, l, acc);
#pragma unroll
  for (int k = 0; k < kCh; ++k)
    if (lane + k * kWave < D) out[lane + k * kWave] = (float)acc[k];
  if (lane == 0) {
    out[D] = M;
    out[D + 1] = (float)l;
  }
}

// Combine the n partial (m, l, acc) states of one row in their stored order (deterministic) and
// write the row: one wavefront, lane c owns channels c, c + 64, ...
template <typename T, int D, typename Sum = float>
__device__ __forceinline__ void merge_row_partials(const float* p0, int64_t step, int n, T* Orow,
                                                   float* lse_i, int lane, bool accumulate) {
  constexpr int kCh = (D + kWave - 1) / kWave;
  float M;
  Sum sum, acc[kCh];
  reduce_partials<D>(p0, step, n, lane, M, sum, acc);
  const float l = (float)sum;
  const bool empty = !(l > 0.f);
  const float inv = empty ? 0.f : 1.0f / l;
  float lse_row = empty ? -INFINITY : (M + __builtin_amdgcn_logf(l)) * kLn2;
  CarryWeights cw{0.f, 1.f, lse_row};
  if (accumulate) {      // every lane reads the earlier lse before lane 0 replaces it
    cw = carry_weights(*lse_i, lse_row);
    lse_row = cw.lse;
  }
#pragma unroll
  for (int k = 0; k < kCh; ++k) {
    const int ch = lane + k * kWave;
    if (ch < D) {
      float o = (float)acc[k] * inv * cw.w_now;
      if (accumulate) o = __builtin_fmaf(cw.w_prev, load_scalar(Orow + ch), o);
      store_scalar(Orow + ch, o);
    }
  }
  if (lse_i && lane == 0) *lse_i = lse_row;
}

// Global rows i < g of the non-local mask attend every key outside their window: about L
// neighbours each.  grid = (chunks, g, H): a wavefront reduces the keys of one chunk of the
// key range (the window cut out) to a partial (m, l, acc) state ...
template <typename T, int D>
__global__ __launch_bounds__(64) void nonlocal_chunk_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, int64_t L, int64_t W,
    int64_t chunk_len, float scale, float* __restrict__ partials) {
  const int lane = threadIdx.x;
  const int64_t c = blockIdx.x, i = blockIdx.y, h = blockIdx.z;
  const int64_t H = gridDim.z, n_chunks = gridDim.x;
  const int64_t hoff = h * L * D;
  const int64_t lo = c * chunk_len, hi = min(L, lo + chunk_len);      // keys [lo, hi)
  float q[Row<T, D>::VEC];
  load_query<T, D>(Q + hoff + i * D, scale, lane, q);
  State<Row<T, D>::VEC> st;
  st.init();
  const int64_t a1 = min(hi, i - W);             // keys [lo, a1) lie left of the window
  if (a1 > lo) {
    WindowNeighbours nbr{lo, 1};
    attend_range<T, D>(K + hoff, V + hoff, q, nbr, 0, a1 - lo, lane, st);
  }
  const int64_t b0 = max(lo, i + W + 1);         // keys [b0, hi) lie right of it
  if (hi > b0) {
    WindowNeighbours nbr{b0, 1};
    attend_range<T, D>(K + hoff, V + hoff, q, nbr, 0, hi - b0, lane, st);
  }
  merge_groups<Row<T, D>::LPK, Row<T, D>::VEC>(st);
  float* p = partials + ((i * n_chunks + c) * H + h) * (D + 4);
  if (lane < Row<T, D>::LPK) {
#pragma unroll
    for (int k = 0; k < Row<T, D>::VEC; ++k) p[lane * Row<T, D>::VEC + k] = st.acc[k];
  }
  if (lane == 0) {
    p[D] = st.m;
    p[D + 1] = st.l;
  }
}

// ... and one workgroup per (global row, head) combines the row's partials: each of its four
// wavefronts reduces a quarter of the chunks, in chunk order, to one partial state in LDS, and
// the first wavefront combines the four in wavefront order and writes the row (a fixed order:
// deterministic).  fp32: in 64 bits, since a row of 20,000 keys is 79 ranges whose sums in 32 bits are half of its error, the more
// so as the wavefronts of tile_nonlocal_kernel merge four parts of each before (error of 64 global rows against 64 bits, one
// chain of blocks per range 2.74e-7, four parts 2.80e-7, so 2.66e-7; L = 3,000 1.87e-7, 1.89e-7, 1.83e-7; 0.1 us a call, 0.7 where 137 ranges are summed).
template <typename T, int D>
__global__ __launch_bounds__(256) void nonlocal_merge_kernel(T* __restrict__ O, float* __restrict__ lse,
                                                             int64_t L, int32_t n_chunks,
                                                             const float* __restrict__ partials,
                                                             int accumulate) {
  __shared__ float quarter[4][D + 4];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int64_t i = blockIdx.x, h = blockIdx.y, H = gridDim.y;
  const int64_t step = H * (D + 4);
  const int per = (n_chunks + 3) / 4;
  const int c0 = wave * per < n_chunks ? wave * per : n_chunks;
  const int c1 = c0 + per < n_chunks ? c0 + per : n_chunks;
  const float* p0 = partials + ((i * n_chunks + c0) * H + h) * (D + 4);
  using Sum = std::conditional_t<DtypeOf<T>::code == SGA_F32, double, float>;
  combine_partials<D, Sum>(p0, step, c1 - c0, &quarter[wave][0], lane);
  __syncthreads();
  if (wave == 0)
    merge_row_partials<T, D, Sum>(&quarter[0][0], D + 4, 4, O + h * L * D + i * D, lse ? lse + h * L + i : nullptr, lane,
                             accumulate != 0);
}

// One wavefront per (chunk of a long row, head): partial state of a slice of the row.  Chunk c
// of every row is computed on XCD c % 8 (workgroups go to the XCDs round-robin in launch order
// and gridDim.x is a multiple of 8): chunks are ranges of the rows' sorted neighbour lists, so
// an XCD's L2 sees the same part of the key range from every row.  Rows of a few chunks start at an XCD of
// their own instead (first_xcd).
// The work units of XCD x are the pairs (long row s, j) with chunk c = (x - first_xcd) % 8 + 8j, numbered
// j * n_long + s (rows of few chunks have no unit for the larger j) and dealt to the XCD's wavefronts in turn.
template <typename T, int D>
__device__ __forceinline__ void gather_chunk_body(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V,
    const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx, int64_t L, float scale,
    void* ws, size_t ws_bytes, int may_share, uint32_t wg, uint32_t n_wg) {
  const int32_t H = (int32_t)gridDim.y;
  constexpr int32_t dtype = DtypeOf<T>::code;
  const uint32_t n_long = reinterpret_cast<const uint32_t*>(ws)[kCtrLongRows];      // (none where the plan has no room)
  if (n_long == 0 || !split_active(row_ptr, L, H, dtype, D, ws, ws_bytes)) return;
  const WorkspacePlan pl = plan_workspace(L, H, row_ptr[L], dtype, D);
  uint32_t max_chunks;
  const int4* lr = long_rows(pl, ws, max_chunks);
  if (may_share && shared_chunks(pl, row_ptr[L], L, H, D, dtype, reinterpret_cast<const uint32_t*>(ws))) return;      // (shared_chunk_kernel)
  float* partials = reinterpret_cast<float*>(static_cast<char*>(ws) + pl.off_partials);
  const int lane = threadIdx.x & (kWave - 1);
  const int waves = blockDim.x / kWave;
  const int64_t h = blockIdx.y;
  const int64_t hoff = h * L * D;
  const uint32_t xcd = wg & 7;
  const uint64_t n_units = (uint64_t)n_long * ((max_chunks + 7) / 8);
  for (uint64_t u = (uint64_t)(wg >> 3) * waves + threadIdx.x / kWave; u < n_units;
       u += (uint64_t)(n_wg >> 3) * waves) {
    const uint32_t s = (uint32_t)(u % n_long);
    const int4 rec = lr[s];                                  // {row, first partial slot, chunks, chunk length}
    const int32_t c = (int32_t)(((xcd - first_xcd(s, rec.z)) & 7) + 8 * (u / n_long));
    if (c >= rec.z) continue;
    const int64_t i = rec.x;
    const int64_t r0 = row_ptr[i], deg = row_ptr[i + 1] - r0;
    const int64_t e0 = (int64_t)c * rec.w;
    const int64_t e1 = min(deg, e0 + rec.w);
    float q[Row<T, D>::VEC];
    load_query<T, D>(Q + hoff + i * D, scale, lane, q);
    State<Row<T, D>::VEC> st;
    st.init();
    if (L * D * (int64_t)sizeof(T) < (int64_t(1) << 32))
      attend_columns<T, D, true>(K + hoff, V + hoff, q, col_idx + r0, e0, e1, lane, st);
    else
      attend_columns<T, D, false>(K + hoff, V + hoff, q, col_idx + r0, e0, e1, lane, st);
    merge_groups<Row<T, D>::LPK, Row<T, D>::VEC>(st);
    float* p = partials + ((int64_t)(rec.y + c) * H + h) * (D + 4);
    if (lane < Row<T, D>::LPK) {
#pragma unroll
      for (int k = 0; k < Row<T, D>::VEC; ++k) p[lane * Row<T, D>::VEC + k] = st.acc[k];
    }
    if (lane == 0) {
      p[D] = st.m;
      p[D + 1] = st.l;
    }
  }
}

template <typename T, int D>
__global__ __launch_bounds__(256) void gather_chunk_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V,
    const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx, int64_t L, float scale,
    void* ws, size_t ws_bytes, int may_share) {
  gather_chunk_body<T, D>(Q, K, V, row_ptr, col_idx, L, scale, ws, ws_bytes, may_share, blockIdx.x, gridDim.x);
}

// ---- chunks of many split rows: K and V through LDS ---------------------------------------------
// Every edge of gather_chunk_kernel draws its own K and V row through the vector L1 (30.9 GB at 21.9 TB/s for a
// tenth of the pairs of L = 24,576, d = 64, fp32) and spends 8 vector instructions, most of them on sums and
// softmax steps that the 16 lanes of a group repeat.  Where many rows are split and their neighbours
// are dense enough, a workgroup takes the same chunk of kRows rows, 16 lanes each, and passes over the
// key blocks of the chunk's range: a block's K and V rows are copied to LDS once and each row's
// neighbours in it are read from there, up to 16 at a time.  The 16 partial dot products
// of a lane are summed over the lanes by halves, so that lane e ends with the score of edge e: maximum,
// exponential and sum cost one lane each, and the products with V take the numerator of
// edge e from lane e (row_newbcast).  The chunk of a row is a part of the keys here, not of its edges: by
// edges, the chunks of 64 rows spread over half as many blocks again (1,164 us).  The products of a step
// are added to the row's state at once: 24 additions per chunk at that density where a group of
// gather_chunk_kernel does 77.
// That case: 1,276 -> 835 us (880 in a loop of nothing else), error 2.2e-7 -> 1.9e-7.  Bound by the vector unit (busy 88 % of the time): a
// row has 12.8 edges in a block, but the four rows of a wavefront take 1.45 steps of 16 for them, as many as the longest
// row; of the slots in the fours that a step does not skip 72 % hold an edge.  d = 64: one buffer, two
// workgroups per CU, 64 registers (7 spill outside the steps); two buffers and one workgroup 1,061 us.
//
// A row's steps are cut at its own key blocks (multiples of kKeys) and nowhere else, so its result does not
// depend on the rows it shares a workgroup with, nor on whether the block came through LDS: where the
// rows' ranges have little in common (kKeys keys copied for fewer edges) every row reads its own.
template <typename T, int D>
struct SharedChunk {
  static constexpr int kVec = D / 16;                        // channels per lane
  static constexpr int kRowBytes = D * (int)sizeof(T);
  static constexpr int kBuffers = kVec > 4 ? 2 : 1;
  static constexpr int kThreads = 1024;
  static constexpr int kKeys = kRowBytes > 256 ? 64 : 128;   // 66 KB for K and V of a block (fp16, d = 64: 33)
  static constexpr int kRows = kThreads / 16;
  static_assert(kRows == kSharedRows, "see shared_chunks");
  static constexpr int kBatch = 4;                           // edges whose rows are read together (registers)
  static constexpr int kPlane = (kKeys + 1) * kRowBytes;     // the row of zeros behind the block stands in for edges that are not there

  // Byte offset of a lane's channels inside a row, and the channel of its element k.  (fp32, d = 128: two
  // 16-byte parts 256 bytes apart, so that every read of 16 lanes is 256 contiguous bytes.)
  __device__ static uint32_t lane_bytes(int l16) { return l16 * (sizeof(T) == 2 && kVec == 4 ? 8 : 16); }
  __device__ static int channel(int l16, int k) {
    return sizeof(T) == 4 && kVec == 8 ? (k >> 2) * 64 + 4 * l16 + (k & 3) : kVec * l16 + k;
  }
  __device__ static void load(const char* p, float (&v)[kVec]) {
    if constexpr (sizeof(T) == 4) {
#pragma unroll
      for (int i = 0; i < kVec / 4; ++i) {
        const float4 t = *reinterpret_cast<const float4*>(p + i * 256);
        v[4 * i] = t.x; v[4 * i + 1] = t.y; v[4 * i + 2] = t.z; v[4 * i + 3] = t.w;
      }
    } else {
      using half_vec = _Float16 __attribute__((ext_vector_type(kVec)));
      const half_vec t = *reinterpret_cast<const half_vec*>(p);
#pragma unroll
      for (int k = 0; k < kVec; ++k) v[k] = (float)t[k];
    }
  }
};

// the bits of a ballot that belong to this lane's 16
__device__ __forceinline__ int count16(uint64_t ballot, int lane) {
  return __popc(__builtin_amdgcn_ubfe(lane & 32 ? (uint32_t)(ballot >> 32) : (uint32_t)ballot, lane & 16, 16));
}

// lane u of each 16
template <int U>
__device__ __forceinline__ int bcast16(int x) {
  return __builtin_amdgcn_mov_dpp(x, 0x150 + U, 0xf, 0xf, true);
}
template <int N, typename F>
__device__ __forceinline__ void unrolled(const F& f) {
  if constexpr (N > 0) {
    unrolled<N - 1>(f);
    f(std::integral_constant<int, N - 1>{});
  }
}

// lo + its partner's lo in one half of every 16 lanes, hi + its partner's hi in the other: lanes l and l ^ 8 (lanes 8 to 15
// take hi), lanes l and 7 - l of every eight (lanes 4 to 7 take hi).  Two instructions in place of an addition and two
// selections; s_nop: two states lie between the write of a register and its use across lanes.  (Random 10 %, L = 24,576,
// us, fp32 824 -> 810, two heads fp16 1,518 -> 1,482.  Products with V that take the numerator across lanes
// themselves, to save the copy, lose 4 %, fp16 13 %: such an instruction takes longer than the plain one.)
__device__ __forceinline__ float add_halves8(float lo, float hi) {
  float x = lo + dpp<0x128>(lo);                                  // row_ror:8
  asm("s_nop 1\n\tv_add_f32_dpp %0, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xc" : "+v"(x) : "v"(hi));
  return x;
}
__device__ __forceinline__ float add_halves4(float lo, float hi) {
  float x = lo + dpp<0x141>(lo);                                  // row_half_mirror
  asm("s_nop 1\n\tv_add_f32_dpp %0, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xa" : "+v"(x) : "v"(hi));
  return x;
}

// One step of a row's 16 lanes: up to 16 edges, lane e holding edge e (valid), its row `off` bytes into K and
// V.  held: the valid lanes of the wavefront (a prefix of every 16).
template <typename T, int D, bool kLds>
__device__ __forceinline__ void attend_step(const char* Kb, const char* Vb, uint32_t off, bool valid, uint64_t held,
                                            int l16, const float (&q)[D / 16], float& m, float& l,
                                            float (&acc)[D / 16]) {
  using S = SharedChunk<T, D>;
  constexpr int kVec = S::kVec;
  const uint32_t own = S::lane_bytes(l16);
  auto load = [&](const char* base, uint32_t at, bool there, float (&v)[kVec]) {
    if (kLds) {
      S::load(base + at, v);
      return;
    }
#pragma unroll
    for (int k = 0; k < kVec; ++k) v[k] = 0.f;
    if (there) S::load(base + at, v);
  };
  auto product = [&](auto edge) {           // of this lane's channels
    constexpr int u = decltype(edge)::value;
    float kf[kVec];
    load(Kb, (uint32_t)bcast16<u>((int)off) + own, kLds || bcast16<u>(valid), kf);
    float part = q[0] * kf[0];
#pragma unroll
    for (int k = 1; k < kVec; ++k) part = __builtin_fmaf(q[k], kf[k], part);
    return part;
  };
  // halves: lane l and lane l ^ 8 add up edge u (lanes 0 to 7) and edge u + 8 (lanes 8 to 15), and so on
  float a[8], b[4], c[2];
#pragma unroll
  for (int u = 0; u < 8; ++u) a[u] = 0.f;
  unrolled<8 / S::kBatch>([&](auto batch) {
    constexpr int g = S::kBatch * decltype(batch)::value;
    if (g > 0 && !(held & (0x0001000100010001ull << g))) return;
    unrolled<S::kBatch>([&](auto i) { a[g + decltype(i)::value] = product(std::integral_constant<int, g + decltype(i)::value>{}); });
    if (held & (0x0100010001000100ull << g)) {
      unrolled<S::kBatch>([&](auto i) {
        constexpr int u = g + decltype(i)::value;
        a[u] = add_halves8(a[u], product(std::integral_constant<int, u + 8>{}));
      });
    } else {
      unrolled<S::kBatch>([&](auto i) { a[g + decltype(i)::value] += dpp<0x128>(a[g + decltype(i)::value]); });
    }
  });
#pragma unroll
  for (int u = 0; u < 4; ++u) b[u] = add_halves4(a[u], a[u + 4]);
#pragma unroll
  for (int u = 0; u < 2; ++u) c[u] = (l16 & 2 ? b[u + 2] : b[u]) + dpp<0x4E>(l16 & 2 ? b[u] : b[u + 2]);    // quad_perm [2,3,0,1]
  const float sum = (l16 & 1 ? c[1] : c[0]) + dpp<0xB1>(l16 & 1 ? c[0] : c[1]);                             // quad_perm [1,0,3,2]
  const float score = valid ? sum : -INFINITY;
  float most = fmaxf(score, dpp<0xB1>(score));
  most = fmaxf(most, dpp<0x4E>(most));
  most = fmaxf(most, dpp<0x141>(most));
  most = fmaxf(most, dpp<0x140>(most));
  most = fmaxf(m, most);
  const float alpha = __builtin_amdgcn_exp2f(m - most);
  const float p = __builtin_amdgcn_exp2f(score - most);
  m = most;
  l = __builtin_fmaf(l, alpha, p);
  float now[kVec];
#pragma unroll
  for (int k = 0; k < kVec; ++k) now[k] = 0.f;
  unrolled<16 / S::kBatch>([&](auto batch) {
    constexpr int g = S::kBatch * decltype(batch)::value;
    if (g > 0 && !(held & (0x0001000100010001ull << g))) return;
    unrolled<S::kBatch>([&](auto i) {
      constexpr int u = g + decltype(i)::value;
      float vf[kVec];
      load(Vb, (uint32_t)bcast16<u>((int)off) + own, kLds || bcast16<u>(valid), vf);
      const float pu = __builtin_bit_cast(float, bcast16<u>(__builtin_bit_cast(int, p)));
#pragma unroll
      for (int k = 0; k < kVec; ++k) now[k] = __builtin_fmaf(pu, vf[k], now[k]);
    });
  });
#pragma unroll
  for (int k = 0; k < kVec; ++k) acc[k] = __builtin_fmaf(acc[k], alpha, now[k]);
}

// key[i] -> the first of the ascending cols[0 .. n) that is not below it (n: none), by the 16 lanes of a row.
__device__ __forceinline__ void first_at_least(const int32_t* cols, int n, int (&key)[2], int lane) {
  const int l16 = lane & 15;
  int lo[2] = {0, 0}, hi[2] = {n, n};
  while (__builtin_amdgcn_ballot_w64(lo[0] < hi[0] || lo[1] < hi[1])) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int step = (hi[i] - lo[i] + 15) / 16, at = lo[i] + (l16 + 1) * step - 1;
      const bool below = at < hi[i] && step > 0 && cols[at] < key[i];
      const int k = count16(__builtin_amdgcn_ballot_w64(below), lane);
      hi[i] = step > 0 ? min(hi[i], lo[i] + (k + 1) * step - 1) : hi[i];
      lo[i] += k * step;
    }
  }
  key[0] = lo[0];
  key[1] = lo[1];
}

template <typename T, int D>
__global__ __attribute__((amdgpu_waves_per_eu((D == 64 ? 8 : 4), (D == 64 ? 8 : 4)))) __launch_bounds__((SharedChunk<T, D>::kThreads)) void shared_chunk_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V,
    const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx, int64_t L, float scale,
    void* ws, size_t ws_bytes) {
  using S = SharedChunk<T, D>;
  constexpr int kVec = S::kVec;
  __shared__ __attribute__((aligned(16))) char planes[2 * S::kBuffers * S::kPlane];
  __shared__ int range[3];                  // first and last key block of the unit, its edges
  const int32_t H = (int32_t)gridDim.y;
  constexpr int32_t dtype = DtypeOf<T>::code;
  const uint32_t n_long = reinterpret_cast<const uint32_t*>(ws)[kCtrLongRows];      // (none where the plan has no room)
  // (the count first: a call with nothing for this kernel launches it once per head, and every idle workgroup that worked
  // out its plan cost +-200, L = 8,192, 32 heads, fp32 294 -> 463 us; so 276)
  if (n_long < kSharedMinRows || !split_active(row_ptr, L, H, dtype, D, ws, ws_bytes)) return;
  const WorkspacePlan pl = plan_workspace(L, H, row_ptr[L], dtype, D);
  uint32_t max_chunks;
  const int4* lr = long_rows(pl, ws, max_chunks);
  if (!shared_chunks(pl, row_ptr[L], L, H, D, dtype, reinterpret_cast<const uint32_t*>(ws))) return;
  float* partials = reinterpret_cast<float*>(static_cast<char*>(ws) + pl.off_partials);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lane = threadIdx.x & (kWave - 1), l16 = lane & 15;
  const int64_t h = blockIdx.y;
  const char* Kb = reinterpret_cast<const char*>(K + h * L * D);
  const char* Vb = reinterpret_cast<const char*>(V + h * L * D);
  // (the rows of zeros stay)
  if (threadIdx.x < S::kRowBytes / 4) {
#pragma unroll
    for (int i = 0; i < 2 * S::kBuffers; ++i)
      reinterpret_cast<uint32_t*>(planes + i * S::kPlane + S::kKeys * S::kRowBytes)[threadIdx.x] = 0;
  }
  const uint32_t cohorts = (n_long + S::kRows - 1) / S::kRows;
  // All units go round all workgroups, the chunks of the 64 rows to as many of them (their numbers are an odd number
  // apart, the grid is a power of two): one row of many chunks among rows of two would keep one busy for 3 ms
  // (random 8 %, L = 32,768, fp32, us: without such a row 1,135; with one of all keys, every chunk c on XCD c % 8 4,935,
  // its chunks on one workgroup 4,270, so 1,440).  No part of the keys has an XCD of its own, as it has in
  // gather_chunk_kernel: 64 rows share each copy, and masks denser in a part of the keys would leave XCDs
  // idle (12 % of the right half only, L = 24,576, fp32 876 -> 508; uniform 10 % 821 / 827, L = 12,001 241 / 236).
  const uint32_t n_units = cohorts * max_chunks;
  for (uint32_t u = blockIdx.x; u < n_units; u += gridDim.x) {
    const uint32_t c = u / cohorts, cohort = (u + (cohorts & 1 ? 0 : c)) % cohorts;
    const uint32_t r = cohort * S::kRows + threadIdx.x / 16;
    const int4 rec = r < n_long ? lr[r] : make_int4(0, 0, 0, 0);        // {row, first partial slot, chunks, chunk length}
    const bool active = (int)c < rec.z;
    if (!__syncthreads_or(active)) continue;          // (no row of the 64 has that many chunks)
    const int64_t r0 = row_ptr[rec.x];
    const int deg = (int)(row_ptr[rec.x + 1] - r0);
    const int32_t* cols = col_idx + r0;
    // this row's edges: those of the c-th of rec.z equal parts of the key blocks, found by 16-way searches
    const int n_blocks = (int)((L + S::kKeys - 1) / S::kKeys);
    int bound[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) bound[i] = active ? (int)((int64_t)(c + i) * n_blocks / rec.z) * S::kKeys : 0;
    first_at_least(cols, active ? deg : 0, bound, lane);
    int e = bound[0];                       // the next edge
    const int e1 = bound[1];
    const int last = max(e1 - 1, 0);
    __syncthreads();                        // the previous unit's range has been read
    if (threadIdx.x == 0) {
      range[0] = INT32_MAX;
      range[1] = -1;
      range[2] = 0;
    }
    __syncthreads();
    if (l16 == 0 && e < e1) {
      atomicMin(&range[0], cols[e] / S::kKeys);
      atomicMax(&range[1], cols[last] / S::kKeys);
      atomicAdd(&range[2], e1 - e);
    }
    __syncthreads();
    const int b0 = __builtin_amdgcn_readfirstlane(range[0]), b1 = __builtin_amdgcn_readfirstlane(range[1]);
    const int edges = __builtin_amdgcn_readfirstlane(range[2]);
    float q[kVec], acc[kVec], m = kMinusHuge, l = 0.f;
    S::load(reinterpret_cast<const char*>(Q + (h * L + rec.x) * D) + S::lane_bytes(l16), q);
    const float scale2 = scale * kLog2e;
#pragma unroll
    for (int k = 0; k < kVec; ++k) {
      q[k] *= scale2;
      acc[k] = 0.f;
    }
    // (a row without edges in this unit reads no column: its loads are of the call's first, which exists)
    const int32_t* own_cols = e < e1 ? cols : col_idx;
    if (edges > 0 && (int64_t)(b1 - b0 + 1) * S::kKeys <= edges) {
      auto stage = [&](int blk) {
        char* const to = planes + ((blk - b0) & (S::kBuffers - 1)) * 2 * S::kPlane;
        const int64_t first = (int64_t)blk * S::kKeys * S::kRowBytes, left = L * S::kRowBytes - first;
        const uint32_t end = (uint32_t)min(left, (int64_t)S::kKeys * S::kRowBytes) - 16;    // (bytes past the last key are not read back)
#pragma unroll
        for (int i = 0; i < S::kKeys * S::kRowBytes / (16 * S::kThreads); ++i) {
          const int part = (i * S::kThreads + wave * kWave) * 16;       // this wavefront's 1,024 bytes
          const uint32_t at = min((uint32_t)(part + lane * 16), end);
          copy16_to_lds_untracked(Kb + first + at, to + part);
          copy16_to_lds_untracked(Vb + first + at, to + S::kPlane + part);
        }
      };
      if (S::kBuffers > 1) stage(b0);
      int32_t c0 = own_cols[min(e + l16, last)], c1 = own_cols[min(e + 16 + l16, last)];
      __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0): this wavefront's copies are there
      __syncthreads();
      for (int blk = b0; blk <= b1; ++blk) {
        if (S::kBuffers > 1) {
          if (blk < b1) stage(blk + 1);
        } else {
          stage(blk);
          __builtin_amdgcn_s_waitcnt(0x0F70);
          __syncthreads();
        }
        const char* const lds_k = planes + ((blk - b0) & (S::kBuffers - 1)) * 2 * S::kPlane;
        const int key0 = blk * S::kKeys;
        uint64_t held1;
        do {
          // the next 32 columns of the row, those of this block among them (the block's end, or the row's, ends them)
          const int k0 = c0 - key0, k1 = c1 - key0;
          const bool v0 = e + l16 < e1 && (uint32_t)k0 < (uint32_t)S::kKeys;
          const bool v1 = e + 16 + l16 < e1 && (uint32_t)k1 < (uint32_t)S::kKeys;
          const uint64_t held0 = __builtin_amdgcn_ballot_w64(v0);
          held1 = __builtin_amdgcn_ballot_w64(v1);
          e += count16(held0, lane) + count16(held1, lane);
          c0 = own_cols[min(e + l16, last)];
          c1 = own_cols[min(e + 16 + l16, last)];
          if (held0)
            attend_step<T, D, true>(lds_k, lds_k + S::kPlane, (uint32_t)((v0 ? k0 : S::kKeys) * S::kRowBytes), v0, held0, l16,
                                    q, m, l, acc);
          if (held1)
            attend_step<T, D, true>(lds_k, lds_k + S::kPlane, (uint32_t)((v1 ? k1 : S::kKeys) * S::kRowBytes), v1, held1, l16,
                                    q, m, l, acc);
        } while (held1 & 0x8000800080008000ull);      // some row may go on in this block
        __builtin_amdgcn_s_waitcnt(0x0F70);
        __syncthreads();                    // the next block is there and every wavefront has left this one
      }
    } else {
      while (true) {                        // every row at its own block
        const int at = e + l16;
        const int32_t col = own_cols[min(at, last)];
        const bool valid = at < e1 && col / S::kKeys == bcast16<0>(col) / S::kKeys;
        const uint64_t held = __builtin_amdgcn_ballot_w64(valid);
        if (held == 0) break;
        attend_step<T, D, false>(Kb, Vb, (uint32_t)col * S::kRowBytes, valid, held, l16, q, m, l, acc);
        e += count16(held, lane);
      }
    }
    l = group_sum<16>(l);
    if (active) {
      float* p = partials + ((int64_t)(rec.y + c) * H + h) * (D + 4);
#pragma unroll
      for (int k = 0; k < kVec; ++k) p[S::channel(l16, k)] = acc[k];
      if (l16 == 0) {
        p[D] = m;
        p[D + 1] = l;
      }
    }
  }
}

// What the tile path leaves over, in one launch for the call that does not know whether there is anything
// (none reads what another writes): the first n_merge workgroups of a head merge the tiles' segments,
// the next n_rows take the leftover rows, the others the chunks of the split rows.  (n_merge and
// n_rows are multiples of 8, so that the chunk workgroups keep their XCDs.)  An empty launch costs 3 to 6
// us of a small call: +-32, L = 4,096, fp32, mask build and forward, in three launches 42.0 us, in two 38.9.
// The chunks have as many workgroups as the chip holds twice (leftover_chunk_workgroups), however short the sequence:
// in a scattered mask every row is split (us, 10 %, fp16, L = 13,001, two heads: with L / 32 over the heads 949,
// with 512 a head 520, with 1,024 a head 505), and idle ones cost less than the launch they spare (+-16, fp32,
// L = 4,096, eight heads 51.9 in launches of their own, 40.7 so).  Workgroups that take rows first and chunks then
// bring keys of the whole range into the L2s that the chunks of others share (10 % below the diagonal, fp32, L = 24,576:
// 977 against 814).
// Four wavefronts per SIMD: fp32 at d = 256 has registers for five, which start on a second head's K and V
// while the first is in the L2s (11.5 %, L = 9,001, two heads 3,182 against 2,932).  At d = 128 three, as the row kernel
// has, for the same reason (6 %, L = 12,001, us: 545 with four, 504 so; 5 %, L = 20,000, two heads 3,627, 3,460).
template <typename T, int D>
__global__ __attribute__((amdgpu_waves_per_eu(1, sizeof(T) == 4 && D == 128 ? 3 : 4))) __launch_bounds__(256) void leftovers_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, T* __restrict__ O,
    float* __restrict__ lse, const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
    int64_t L, float scale, void* ws, size_t ws_bytes, int use_split, int may_share, int accumulate,
    uint32_t n_merge, uint32_t n_rows) {
  if (blockIdx.x < n_merge) {
    tile_merge_body<T, D>(O, lse, row_ptr, L, ws, ws_bytes, accumulate, blockIdx.x / kTile, n_merge / kTile,
                          blockIdx.x % kTile, kTile);
    return;
  }
  if (blockIdx.x < n_merge + n_rows)
    gather_csr_body<T, D>(Q, K, V, O, lse, row_ptr, col_idx, L, scale, ws, ws_bytes, use_split, 1, accumulate,
                          blockIdx.x - n_merge, n_rows);
  else
    gather_chunk_body<T, D>(Q, K, V, row_ptr, col_idx, L, scale, ws, ws_bytes, may_share, blockIdx.x - n_merge - n_rows,
                            gridDim.x - n_merge - n_rows);
}

// Rows of up to kMaxSplit chunks: one wavefront per (long row, head) combines the row's partials
// in chunk order.  Rows of more chunks (cut by edge count into up to kMaxSplitLong): one
// workgroup per row, each of its four wavefronts combines a quarter of the partials in chunk
// order, the first one the four results in wavefront order (a fixed order whatever the
// schedule).
template <typename T, int D>
__global__ __launch_bounds__(256) void gather_merge_kernel(T* __restrict__ O, float* __restrict__ lse,
                                                           const int64_t* __restrict__ row_ptr,
                                                           int64_t L, void* ws, size_t ws_bytes,
                                                           int accumulate) {
  __shared__ float quarter[4][D + 4];
  const int32_t H = (int32_t)gridDim.y;
  constexpr int32_t dtype = DtypeOf<T>::code;
  const uint32_t n_long = reinterpret_cast<const uint32_t*>(ws)[kCtrLongRows];      // (none where the plan has no room)
  if (n_long == 0 || !split_active(row_ptr, L, H, dtype, D, ws, ws_bytes)) return;
  const WorkspacePlan pl = plan_workspace(L, H, row_ptr[L], dtype, D);
  uint32_t max_chunks;
  const int4* lr = long_rows(pl, ws, max_chunks);
  const float* partials = reinterpret_cast<const float*>(static_cast<char*>(ws) + pl.off_partials);
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  const int64_t h = blockIdx.y;
  const int64_t step = (int64_t)H * (D + 4);
  for (uint32_t r = blockIdx.x * 4 + wave; r < n_long; r += gridDim.x * 4) {
    const int4 rec = lr[r];
    if (rec.z > kMaxSplit) continue;
    const int64_t i = rec.x;
    merge_row_partials<T, D>(partials + ((int64_t)rec.y * H + h) * (D + 4), step, rec.z, O + h * L * D + i * D,
                             lse ? lse + h * L + i : nullptr, lane, accumulate != 0);
  }
  if (max_chunks <= (uint32_t)kMaxSplit) return;
  for (uint32_t r = blockIdx.x; r < n_long; r += gridDim.x) {      // (the same trips for the whole workgroup)
    const int4 rec = lr[r];
    if (rec.z <= kMaxSplit) continue;
    const int64_t i = rec.x;
    const float* p0 = partials + ((int64_t)rec.y * H + h) * (D + 4);
    T* Orow = O + h * L * D + i * D;
    float* lse_i = lse ? lse + h * L + i : nullptr;
    const int per = (rec.z + 3) / 4;
    const int c0 = wave * per < rec.z ? wave * per : rec.z;
    const int c1 = c0 + per < rec.z ? c0 + per : rec.z;
    __syncthreads();                 // the previous row's combine has read the shared records
    combine_partials<D>(p0 + c0 * step, step, c1 - c0, &quarter[wave][0], lane);
    __syncthreads();
    if (wave == 0) merge_row_partials<T, D>(&quarter[0][0], D + 4, 4, Orow, lse_i, lane, accumulate != 0);
  }
}

template <typename T, int D>
sga_status run_explicit(const AttnArgs& a, bool allow_split, bool skip_tiled) {
  const T* Q = static_cast<const T*>(a.Q);
  const T* K = static_cast<const T*>(a.K);
  const T* V = static_cast<const T*>(a.V);
  T* O = static_cast<T*>(a.O);
  const bool split = allow_split && a.ws && a.ws_bytes >= 256 && a.L > kSplitThreshold;
  // (after the tile path the CSR -> tile pass has recorded the split rows of most calls, and a prepared graph holds them)
  if (split && !a.prepared && (!skip_tiled || tile_parts_may_be_in_doubt(a.dtype, a.ws_bytes)))
    launch_split_prepass(a, skip_tiled);
  // after the tile path only leftover rows remain: a grid of about one chip-full of wavefronts
  // over all heads strides over the rows (it returns at once when the tiles covered everything)
  const int64_t nwg = skip_tiled ? leftover_workgroups(a.prepared ? a.plan_rows_left : a.L, a.H) : (a.L + 3) / 4;
  const dim3 grid((unsigned)nwg, (unsigned)a.H);
  // the benchmark hook brackets the kernel that does the work: the row kernel, or the chunk
  // kernel where a prepared graph has found every row left to it split
  const bool mark = !skip_tiled || (a.prepared && a.plan_no_tiles);
  const bool mark_chunks = mark && a.prepared && a.plan_long_rows > 0;
  const bool fused = D >= kHeadDim && skip_tiled && !a.prepared;     // (nothing known about what is left)
  const bool may_share = split && (a.prepared ? a.plan_rows_share : shared_chunks_possible(a.L, a.H, a.d, a.dtype, a.ws_bytes));
  if constexpr (D >= kHeadDim) {
    if (fused) {
      const unsigned n_merge = merge_tiles(a) * kTile, n_chunks = split ? (unsigned)leftover_chunk_workgroups(a.H) : 0;
      hipLaunchKernelGGL((leftovers_kernel<T, D>), dim3(n_merge + (unsigned)nwg + n_chunks, (unsigned)a.H), dim3(256), 0, a.stream, Q, K, V, O,
                         a.lse, a.row_ptr, a.col_idx, a.L, a.scale, a.ws, a.ws_bytes, split ? 1 : 0, may_share ? 1 : 0,
                         a.accumulate ? 1 : 0, n_merge, (unsigned)nwg);
    }
  }
  if (!fused && !(a.prepared && a.plan_long_rows == a.L)) {       // (a prepared graph all of whose rows are split: 19 us of L = 24,576)
    if constexpr (kWave / Row<T, D>::LPK > 1 && kWave / Row<T, D>::LPK <= 4) {
      if (a.prepared && a.plan_rows_even && even_rows(a.L, a.H, D, a.dtype)) {
        constexpr int kRows = 4 * kWave / Row<T, D>::LPK;
        profile_mark_begin(a.stream, "gather_even_rows_kernel");
        hipLaunchKernelGGL((gather_even_rows_kernel<T, D>), dim3((unsigned)((a.L + kRows - 1) / kRows), (unsigned)a.H), dim3(256),
                           0, a.stream, Q, K, V, O, a.lse, a.row_ptr, a.col_idx, a.L, a.scale, a.accumulate ? 1 : 0);
        profile_mark_end(a.stream);
        return hip_status(hipGetLastError());
      }
    }
    if (mark && !mark_chunks) profile_mark_begin(a.stream, "gather_csr_kernel");
    hipLaunchKernelGGL((gather_csr_kernel<T, D>), grid, dim3(256), 0, a.stream, Q, K, V, O, a.lse,
                       a.row_ptr, a.col_idx, a.L, a.scale, a.ws, a.ws_bytes, split ? 1 : 0,
                       skip_tiled ? 1 : 0, a.accumulate ? 1 : 0);
    if (mark && !mark_chunks) profile_mark_end(a.stream);
  }
  if (split && (!a.prepared || a.plan_long_rows > 0)) {
    if (mark_chunks) profile_mark_begin(a.stream, may_share ? "shared_chunk_kernel" : "gather_chunk_kernel");
    if (!fused && !(a.prepared && may_share)) {
      const unsigned chunk_wgs = skip_tiled && a.H >= 8 ? 128 : 1024;
      hipLaunchKernelGGL((gather_chunk_kernel<T, D>), dim3(chunk_wgs, (unsigned)a.H), dim3(256), 0, a.stream, Q,
                         K, V, a.row_ptr, a.col_idx, a.L, a.scale, a.ws, a.ws_bytes, may_share ? 1 : 0);
    }
    if constexpr (D == 64 || D == 128) {
      if (may_share) {
        using S = SharedChunk<T, D>;
        hipLaunchKernelGGL((shared_chunk_kernel<T, D>), dim3(shared_places(D), (unsigned)a.H), dim3(S::kThreads), 0, a.stream, Q, K, V,
                           a.row_ptr, a.col_idx, a.L, a.scale, a.ws, a.ws_bytes);
      }
    }
    if (mark_chunks) profile_mark_end(a.stream);
    // one wavefront per long row and head, one workgroup for a row of more than kMaxSplit
    // chunks; a prepared graph knows how many rows there are
    int64_t merge_wgs = a.prepared ? (int64_t)a.plan_long_rows : (a.L + 15) / 16;
    const int64_t merge_cap = 4096 / a.H > 64 ? 4096 / a.H : 64;
    if (merge_wgs > merge_cap) merge_wgs = merge_cap;
    hipLaunchKernelGGL((gather_merge_kernel<T, D>), dim3((unsigned)merge_wgs, (unsigned)a.H), dim3(256), 0, a.stream, O,
                       a.lse, a.row_ptr, a.L, a.ws, a.ws_bytes, a.accumulate ? 1 : 0);
  }
  return hip_status(hipGetLastError());
}

}  // namespace

void clear_workspace(const AttnArgs& a, bool tile_flags) {
  const int64_t n_tiles = (a.L + kTile - 1) / kTile;
  int64_t nwg = tile_flags ? (n_tiles + 255) / 256 : 1;
  if (nwg > 1024) nwg = 1024;
  hipLaunchKernelGGL(clear_workspace_kernel, dim3((unsigned)nwg), dim3(256), 0, a.stream, a.ws,
                     a.ws_bytes, a.row_ptr, a.L, a.H, a.dtype, a.d, tile_flags ? 1 : 0);
}

void launch_split_prepass(const AttnArgs& a, bool after_tiles) {
  hipLaunchKernelGGL(split_prepass_kernel, dim3((unsigned)((a.L + 255) / 256)), dim3(256), 0, a.stream,
                     a.row_ptr, a.L, a.H, a.dtype, a.d, a.ws, a.ws_bytes, after_tiles ? 1 : 0);
}

namespace {
// The length of the longest row and the sum of the squared lengths, into counters (graph preparation only).  Two atomics on
// one line per workgroup: with two per wavefront and 512 workgroups it waits for them (L = 1,048,576 54 us, 12.5 so).
__global__ __launch_bounds__(256) void row_lengths_kernel(const int64_t* __restrict__ row_ptr, int64_t L, uint32_t* ctr) {
  int64_t most = 0;
  unsigned long long squares = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < L; i += (int64_t)gridDim.x * 256) {
    const int64_t deg = row_ptr[i + 1] - row_ptr[i];
    most = deg > most ? deg : most;
    const unsigned long long n = deg < 65535 ? deg : 65535;      // (the sum stays below 2^63; such rows are not even ones)
    squares += n * n;
  }
  int longest = (int)most;                 // (a row has at most L < 2^31 neighbours)
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    longest = max(longest, __shfl_xor(longest, off, kWave));
    squares += __shfl_xor(squares, off, kWave);
  }
  __shared__ int wave_longest[4];
  __shared__ unsigned long long wave_squares[4];
  if ((threadIdx.x & (kWave - 1)) == 0) {
    wave_longest[threadIdx.x / kWave] = longest;
    wave_squares[threadIdx.x / kWave] = squares;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) {
      longest = max(longest, wave_longest[w]);
      squares += wave_squares[w];
    }
    atomicMax(&ctr[kCtrLongestRow], (uint32_t)longest);
    atomicAdd(reinterpret_cast<unsigned long long*>(&ctr[kCtrLengthSquares]), squares);
  }
}
}  // namespace

void launch_row_lengths(const AttnArgs& a) {
  const int64_t wgs = (a.L + 255) / 256;
  hipLaunchKernelGGL(row_lengths_kernel, dim3((unsigned)(wgs < 256 ? wgs : 256)), dim3(256), 0, a.stream, a.row_ptr, a.L,
                     static_cast<uint32_t*>(a.ws));
}

sga_status launch_gather_explicit(const AttnArgs& a, bool allow_split, bool skip_tiled) {
  switch (a.d) {
    case 32:
      return a.dtype == SGA_F32 ? run_explicit<float, 32>(a, allow_split, skip_tiled)
                                : run_explicit<__half, 32>(a, allow_split, skip_tiled);
    case 64:
      return a.dtype == SGA_F32 ? run_explicit<float, 64>(a, allow_split, skip_tiled)
                                : run_explicit<__half, 64>(a, allow_split, skip_tiled);
    case 128:
      return a.dtype == SGA_F32 ? run_explicit<float, 128>(a, allow_split, skip_tiled)
                                : run_explicit<__half, 128>(a, allow_split, skip_tiled);
    case 256:
      return a.dtype == SGA_F32 ? run_explicit<float, 256>(a, allow_split, skip_tiled)
                                : run_explicit<__half, 256>(a, allow_split, skip_tiled);
    default:
      return SGA_ERR_UNSUPPORTED;
  }
}

template <typename T, int D>
static sga_status run_implicit(const AttnArgs& a) {
  const T* Q = static_cast<const T*>(a.Q);
  const T* K = static_cast<const T*>(a.K);
  const T* V = static_cast<const T*>(a.V);
  T* O = static_cast<T*>(a.O);
  const int acc = a.accumulate ? 1 : 0;
  if (a.mask_kind == SGA_MASK_SLIDING || a.mask_kind == SGA_MASK_DILATED) {
    const dim3 grid((unsigned)((a.L + 3) / 4), (unsigned)a.H);
    profile_mark_begin(a.stream, "gather_window_kernel");
    hipLaunchKernelGGL((gather_window_kernel<T, D>), grid, dim3(256), 0, a.stream, Q, K, V, O, a.lse, a.L,
                       (int64_t)a.window, (int64_t)a.stride, a.scale, acc);
    profile_mark_end(a.stream);
    return hip_status(hipGetLastError());
  }
  // rows that are one arithmetic run: all rows of the 2-D dilated mask, rows >= g of the
  // non-local mask
  const int64_t g = a.mask_kind == SGA_MASK_NONLOCAL ? (a.n_global < a.L ? a.n_global : a.L) : 0;
  if constexpr (D >= kHeadDim) {
    if (a.mask_kind == SGA_MASK_NONLOCAL && a.tiles_allowed) {
      // matrix-core tiles: 32 rows >= g at a time against the one or two key blocks that hold the
      // global tokens; the g global rows as one or two tiles over ranges of all key blocks, with
      // partial states that the merge below combines in range order
      float* partials = g > 0 ? reinterpret_cast<float*>(static_cast<char*>(a.ws) +
                                                         plan_workspace(a.L, a.H, -1, a.dtype, D).off_partials)
                              : nullptr;
      int32_t n_chunks = 0;
      launch_tile_nonlocal(a, g, partials, &n_chunks);
      if (g > 0)
        hipLaunchKernelGGL((nonlocal_merge_kernel<T, D>), dim3((unsigned)g, (unsigned)a.H), dim3(256), 0, a.stream,
                           O, a.lse, a.L, n_chunks, partials, acc);
      return hip_status(hipGetLastError());
    }
  }
  if (a.L > g) {
    const dim3 grid((unsigned)((a.L - g + 3) / 4), (unsigned)a.H);
    profile_mark_begin(a.stream, "gather_runs_kernel");
    hipLaunchKernelGGL((gather_runs_kernel<T, D>), grid, dim3(256), 0, a.stream, Q, K, V, O, a.lse, a.L,
                       a.mask_kind, (int64_t)a.window, (int64_t)a.stride, g, (int64_t)a.block, g, a.scale,
                       acc);
    profile_mark_end(a.stream);
  }
  if (g > 0) {
    // the g global rows: split over the key range, partial states in the workspace
    int32_t n_chunks, len;
    split_shape(a.L, kSplitChunk, n_chunks, len);
    float* partials = reinterpret_cast<float*>(static_cast<char*>(a.ws) +
                                               plan_workspace(a.L, a.H, -1, a.dtype, D).off_partials);
    hipLaunchKernelGGL((nonlocal_chunk_kernel<T, D>), dim3((unsigned)n_chunks, (unsigned)g, (unsigned)a.H),
                       dim3(64), 0, a.stream, Q, K, V, a.L, (int64_t)a.window, (int64_t)len, a.scale,
                       partials);
    hipLaunchKernelGGL((nonlocal_merge_kernel<T, D>), dim3((unsigned)g, (unsigned)a.H), dim3(256), 0, a.stream,
                       O, a.lse, a.L, n_chunks, partials, acc);
  }
  return hip_status(hipGetLastError());
}

sga_status launch_gather_implicit(const AttnArgs& a) {
  switch (a.d) {
    case 32: return a.dtype == SGA_F32 ? run_implicit<float, 32>(a) : run_implicit<__half, 32>(a);
    case 64: return a.dtype == SGA_F32 ? run_implicit<float, 64>(a) : run_implicit<__half, 64>(a);
    case 128: return a.dtype == SGA_F32 ? run_implicit<float, 128>(a) : run_implicit<__half, 128>(a);
    case 256: return a.dtype == SGA_F32 ? run_implicit<float, 256>(a) : run_implicit<__half, 256>(a);
    default: return SGA_ERR_UNSUPPORTED;
  }
}

}  // namespace sga
