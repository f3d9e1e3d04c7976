// The merge of multi-segment tiles, shared by its own kernel (prepared graphs, attention_tile.hip) and the launch
// that takes the leftover rows (attention_gather.hip).
#pragma once

#include "sga_internal.h"

namespace sga {
namespace {

constexpr float kMergeLn2 = 0.6931471805599453f;

__device__ __forceinline__ float load_out(const float* p) { return *p; }
__device__ __forceinline__ float load_out(const __half* p) { return __half2float(*p); }
__device__ __forceinline__ void store_out(float* p, float v) { *p = v; }
__device__ __forceinline__ void store_out(__half* p, float v) { *p = __float2half_rn(v); }

// Merge of the multi-segment tiles' partial states.  The workgroups of a head (blockIdx.y) are numbered (wg
// of n_wg, part of n_parts): wg strides over the merge list, part names the rows of a tile in
// groups of 32 / n_parts.  Per row: the running maximum M over all
// segments (every thread takes every 256th segment, so all loads are in flight together), the
// weights 2^(m_c - M), and the weighted sums of l and of the accumulators.  The 4 wavefronts of
// a workgroup take every 4th segment (lane = channel within each 64-channel slice; a partial
// of a kD-wide tile is kD / 64 records, one per slice, with the same m and l), four segments per
// trip so that their loads overlap, each in ascending segment order; the four results are added
// in wavefront order, so the summation order is fixed.
template <typename T, int kD>
__device__ __forceinline__ void tile_merge_body(T* __restrict__ O, float* __restrict__ lse,
                                                const int64_t* __restrict__ row_ptr, int64_t L, void* ws, size_t ws_bytes,
                                                int accumulate, uint32_t wg, uint32_t n_wg, uint32_t part, uint32_t n_parts) {
  constexpr int kSlices = kD / kHeadDim;
  __shared__ float sm_acc[4][kD];
  __shared__ float sm_m[4], sm_l[4];
  const int32_t H = (int32_t)gridDim.y;
  constexpr int32_t dtype = DtypeOf<T>::code;
  const WorkspacePlan pl = plan_workspace(L, H, row_ptr[L], dtype, kD);
  if (pl.total_bytes > ws_bytes) return;
  if ((int64_t)reinterpret_cast<const uint32_t*>(ws)[kCtrTilePartsNeeded] > pl.cap_tparts) return;     // (see tile_handled)
  char* base_ws = static_cast<char*>(ws);
  const uint32_t n_multi = reinterpret_cast<const uint32_t*>(ws)[kCtrMultiTiles];
  const int4* multi = reinterpret_cast<const int4*>(base_ws + pl.off_multi_tiles);     // {tile, first partial slot, segments, -}
  const int32_t* tile_bad = reinterpret_cast<const int32_t*>(base_ws + pl.off_tile_bad);
  const float* parts = reinterpret_cast<const float*>(base_ws + pl.off_tpartials);
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = threadIdx.x / kWave;
  const int64_t hd = blockIdx.y;
  for (uint32_t i = wg; i < n_multi; i += n_wg) {
    const int4 rec = multi[i];
    const int64_t t = rec.x;
    if (tile_bad[t]) continue;
    const int nseg = rec.z;
    const float* p0 = parts + ((int64_t)rec.y * H + hd) * (kSlices * kTilePartialFloats);
    const int64_t step = (int64_t)H * (kSlices * kTilePartialFloats);
    const int rows_per_wg = kTile / (int)n_parts;
    for (int r = part * rows_per_wg; r < (int)(part + 1) * rows_per_wg; ++r) {
      const int64_t row = t * kTile + r;
      const float* pm = p0 + kTile * 64 + r;       // segment c: m = pm[c * step], l = pm[c * step + kTile]
      float M = -1.0e30f;
      for (int c = threadIdx.x; c < nseg; c += 256) M = fmaxf(M, pm[c * step]);
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) M = fmaxf(M, __shfl_xor(M, off, kWave));
      __syncthreads();            // the previous row's combine has read the shared arrays
      if (lane == 0) sm_m[wave] = M;
      __syncthreads();
      M = fmaxf(fmaxf(sm_m[0], sm_m[1]), fmaxf(sm_m[2], sm_m[3]));
      float l = 0.f, acc[kSlices];
#pragma unroll
      for (int sl = 0; sl < kSlices; ++sl) acc[sl] = 0.f;
      for (int c = wave; c < nseg; c += 16) {
        float mc[4], lc[4], oc[4][kSlices];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int cc = c + 4 * u < nseg ? c + 4 * u : c;
          mc[u] = pm[cc * step];
          lc[u] = pm[cc * step + kTile];
#pragma unroll
          for (int sl = 0; sl < kSlices; ++sl) oc[u][sl] = p0[cc * step + sl * kTilePartialFloats + r * 64 + lane];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float wgt = c + 4 * u < nseg ? __builtin_amdgcn_exp2f(mc[u] - M) : 0.f;
          l = __builtin_fmaf(lc[u], wgt, l);
#pragma unroll
          for (int sl = 0; sl < kSlices; ++sl) acc[sl] = __builtin_fmaf(oc[u][sl], wgt, acc[sl]);
        }
      }
#pragma unroll
      for (int sl = 0; sl < kSlices; ++sl) sm_acc[wave][sl * 64 + lane] = acc[sl];
      if (lane == 0) sm_l[wave] = l;
      __syncthreads();
      if (wave == 0 && row < L) {
        const float lt = ((sm_l[0] + sm_l[1]) + sm_l[2]) + sm_l[3];
        const bool empty = !(lt > 0.f);
        float lse_row = empty ? -INFINITY : (M + __builtin_amdgcn_logf(lt)) * kMergeLn2;
        CarryWeights cw{0.f, 1.f, lse_row};
        if (accumulate) {
          cw = carry_weights(lse[hd * L + row], lse_row);
          lse_row = cw.lse;
        }
#pragma unroll
        for (int sl = 0; sl < kSlices; ++sl) {
          const float at = ((sm_acc[0][sl * 64 + lane] + sm_acc[1][sl * 64 + lane]) +
                            sm_acc[2][sl * 64 + lane]) + sm_acc[3][sl * 64 + lane];
          T* dst = O + hd * L * kD + row * kD + sl * 64 + lane;
          float o = empty ? 0.f : at / lt;
          if (accumulate) o = cw.w_prev * load_out(dst) + cw.w_now * o;
          store_out(dst, o);
        }
        if (lse && lane == 0) lse[hd * L + row] = lse_row;
      }
    }
  }
}

// Workgroups per row and head of the merge of multi-segment tiles, each of which walks the merge list:
// one per tile where a prepared graph knows their number, up to four rounds of the chip's 2,048
// workgroups.  (768 tiles of six segments, one head: 96 us with 16 workgroups per row.)  A call that does not
// know whether there are any has 16, and fewer where the heads alone make four rounds: the launch that also takes
// the rows left over holds four wavefronts per SIMD, and starting 512 idle workgroups of it per head cost more than a
// kernel of its own (+-16, fp32, L = 1,000, 64 heads, us: that 120.8, 127.3, with four 85.6).
inline unsigned merge_tiles(const AttnArgs& a) {
  const int64_t most = 8192 / (kTile * (int64_t)a.H);
  if (!a.prepared) return (unsigned)(most > 16 ? 16 : most < 1 ? 1 : most);
  int64_t n = (int64_t)a.plan_multi_tiles;
  if (n > most) n = most;
  return (unsigned)(n < 16 ? (a.plan_multi_tiles < 16 ? a.plan_multi_tiles : 16) : n);
}

}  // namespace
}  // namespace sga
