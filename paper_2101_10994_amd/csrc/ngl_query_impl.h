// SDF query kernels (Sec. 3.2, Eq. 2; continuous LOD, Eq. 3), finite-
// difference normals (App. A.4) and their launchers, shared by the per-width
// translation units ngl_query_m{8,16,32,64}.hip and the entry points in
// ngl_query.hip.
#pragma once

#include "ngl_common.h"
#include "ngl_device.h"
#include "ngl_mfma.h"

namespace ngl {

// Locate x at feature levels 1..Lp: vox[l-1] (or -1) and the level's cell;
// *vlast = voxel of level Lp, *vnext = voxel of level `next` (both or -1).
template <int MAXL>
__device__ inline void locate(const ngl_model& md, const float x[3], int Lp, int* vox, int* cx, int* cy, int* cz,
                              int* vlast, int next = -1, int* vnext = nullptr) {
  const int Dp = Lp + 1;
  if (!in_box(x[0], x[1], x[2])) {
#pragma unroll
    for (int l = 0; l < MAXL; ++l) vox[l] = -1;
    *cx = *cy = *cz = 0;
    *vlast = -1;
    if (vnext) *vnext = -1;
    return;
  }
  const int r = 1 << Dp;
  *cx = cell_of(x[0], r);
  *cy = cell_of(x[1], r);
  *cz = cell_of(x[2], r);
  descend<MAXL>(md, *cx, *cy, *cz, Dp, vox, vlast, next, vnext);
}

template <int M, typename FT, bool XYZ>
__global__ __launch_bounds__(kBlock) void k_query(ngl_model md, const float* __restrict__ xs, int64_t P, int lod,
                                                  float alpha, const float* __restrict__ alpha_pp,
                                                  float* __restrict__ sdf, uint8_t* __restrict__ valid,
                                                  int32_t* __restrict__ vox_out) {
  const int64_t p = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  if (p >= P) return;
  const float x[3] = {xs[p], xs[P + p], xs[2 * P + p]};
  const bool blend = alpha_pp != nullptr || alpha > 0.0f;
  const int Lp = blend ? lod + 1 : lod;
  const float a = alpha_pp ? alpha_pp[p] : alpha;
  int vox[NGL_MAX_LODS];
  int cx, cy, cz, vlast, vn;
  locate<NGL_MAX_LODS>(md, x, Lp, vox, &cx, &cy, &cz, &vlast, lod + 1, &vn);
  float z[M];
#pragma unroll
  for (int k = 0; k < M; ++k) z[k] = 0.0f;
  // Level loops are unrolled over the compile-time maximum so that the
  // per-level arrays stay in registers.
#pragma unroll
  for (int l = 1; l <= NGL_MAX_LODS; ++l)
    if (l <= lod && vox[l - 1] >= 0) interp_level<M, FT>(md, l, vox[l - 1], cx >> (Lp - l), cy >> (Lp - l), cz >> (Lp - l), x, z);
  float out = decode_f32<M, XYZ>(md, lod, x, z);
  if (blend) {
    // z_{L+1} = z_L + psi_{L+1}
    if (vn >= 0) interp_level<M, FT>(md, lod + 1, vn, cx, cy, cz, x, z);
    out = (1.0f - a) * out + a * decode_f32<M, XYZ>(md, lod + 1, x, z);
  }
  sdf[p] = out;
  if (valid) valid[p] = vlast >= 0 ? 1 : 0;
  if (vox_out) {
#pragma unroll
    for (int l = 1; l <= NGL_MAX_LODS; ++l)
      if (l <= Lp) vox_out[int64_t(l - 1) * P + p] = vox[l - 1];
  }
}

// All discrete LODs: the level sum is shared, one decoder per LOD.
template <int M, typename FT, bool XYZ>
__global__ __launch_bounds__(kBlock) void k_query_all(ngl_model md, const float* __restrict__ xs, int64_t P,
                                                      float* __restrict__ sdf_all) {
  const int64_t p = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  if (p >= P) return;
  const float x[3] = {xs[p], xs[P + p], xs[2 * P + p]};
  const int Lm = md.num_lods;
  int vox[NGL_MAX_LODS];
  int cx, cy, cz, vlast;
  locate<NGL_MAX_LODS>(md, x, Lm, vox, &cx, &cy, &cz, &vlast);
  float z[M];
#pragma unroll
  for (int k = 0; k < M; ++k) z[k] = 0.0f;
#pragma unroll
  for (int l = 1; l <= NGL_MAX_LODS; ++l) {
    if (l <= Lm) {
      const int s = Lm - l;
      if (vox[l - 1] >= 0) interp_level<M, FT>(md, l, vox[l - 1], cx >> s, cy >> s, cz >> s, x, z);
      sdf_all[int64_t(l - 1) * P + p] = decode_f32<M, XYZ>(md, l, x, z);
    }
  }
}

// Matrix-core decoder (BF16 or FP32 form): the same location and gather per
// lane, then the first decoder layer for the wavefront's 64 points on the
// matrix cores.  Grid-stride over points so each block stages the decoder
// fragments in LDS once; inside the loop only wavefront-level LDS ordering
// is needed.
template <int M, typename FT, bool XYZ, int NW, class DEC>
__global__ __launch_bounds__(64 * NW) void k_query_mfma(ngl_model md, const float* __restrict__ xs, int64_t P,
                                                        int lod, float alpha, const float* __restrict__ alpha_pp,
                                                        float* __restrict__ sdf, uint8_t* __restrict__ valid,
                                                        int32_t* __restrict__ vox_out) {
  extern __shared__ __align__(16) char smem[];
  const int H = md.hidden;
  const bool blend = alpha_pp != nullptr || alpha > 0.0f;
  DecLds<DEC> S(smem, H, blend);
  DEC::load(md, lod, S.frag0, S.w2s0);
  if (blend) DEC::load(md, lod + 1, S.frag1, S.w2s1);
  __syncthreads();
  const float b2a = md.b2[lod - 1];
  const float b2b = blend ? md.b2[lod] : 0.0f;
  const int Lp = blend ? lod + 1 : lod;
  for (int64_t base = int64_t(blockIdx.x) * (64 * NW); base < P; base += int64_t(gridDim.x) * (64 * NW)) {
    const int64_t p = base + threadIdx.x;
    const bool act = p < P;
    float x[3] = {0.0f, 0.0f, 0.0f};
    if (act) {
      x[0] = xs[p];
      x[1] = xs[P + p];
      x[2] = xs[2 * P + p];
    }
    int vox[NGL_MAX_LODS];
    int cx, cy, cz, vlast, vn;
    locate<NGL_MAX_LODS>(md, x, Lp, vox, &cx, &cy, &cz, &vlast, lod + 1, &vn);
    if (!act) {
#pragma unroll
      for (int l = 0; l < NGL_MAX_LODS; ++l) vox[l] = -1;
      vlast = vn = -1;
    }
    float z[M];
#pragma unroll
    for (int k = 0; k < M; ++k) z[k] = 0.0f;
#pragma unroll
    for (int l = 1; l <= NGL_MAX_LODS; ++l)
      if (l <= lod && vox[l - 1] >= 0)
        interp_level<M, FT>(md, l, vox[l - 1], cx >> (Lp - l), cy >> (Lp - l), cz >> (Lp - l), x, z);
    DEC::stage(S.stage, x, z);
    wave_lds_sync();
    float out = DEC::decode(S.frag0, S.w2s0, b2a, S.stage, H, __ballot(act));
    if (blend) {
      if (vn >= 0) interp_level<M, FT>(md, lod + 1, vn, cx, cy, cz, x, z);
      wave_lds_sync();
      DEC::stage(S.stage, x, z);
      wave_lds_sync();
      const float a = act ? (alpha_pp ? alpha_pp[p] : alpha) : 0.0f;
      out = (1.0f - a) * out + a * DEC::decode(S.frag1, S.w2s1, b2b, S.stage, H, __ballot(act));
    }
    wave_lds_sync();
    if (act) {
      sdf[p] = out;
      if (valid) valid[p] = vlast >= 0 ? 1 : 0;
      if (vox_out) {
#pragma unroll
        for (int l = 1; l <= NGL_MAX_LODS; ++l)
          if (l <= Lp) vox_out[int64_t(l - 1) * P + p] = vox[l - 1];
      }
    }
  }
}

// A wavefront's points by how many levels they have (voxels nest, so these are the
// coarsest ones), most first, so that points in empty space share tiles that
// skip the fine levels; lanes without a point come last.  2^20 FP32 queries, half
// of them uniform in the box (they have 2.7 of 5 levels on average): 0.209 -> 0.187
// ms; 2^22 blended queries of the 7-LOD 16-bit model 0.829 -> 0.766 ms.
__device__ __forceinline__ PointOrder order_by_depth(const int* vox, int Lp, bool act) {
  const int lane = threadIdx.x & 63;
  const uint64_t below = (1ull << lane) - 1ull;
  int depth = 0;
#pragma unroll
  for (int l = 1; l <= NGL_MAX_LODS; ++l) depth += l <= Lp && vox[l - 1] >= 0;
  if (!act) depth = -1;
  int base = 0, rank = 0;
#pragma unroll
  for (int d = NGL_MAX_LODS; d >= -1; --d) {
    if (d > Lp) continue;
    const uint64_t m = __ballot(depth == d);
    if (depth == d) rank = base + __popcll(m & below);
    base += __popcll(m);
  }
  return {rank, __builtin_amdgcn_ds_permute(4 * rank, lane)};
}

// Cooperative gather: lanes locate their own points as above, then the
// wavefront gathers and decodes its 64 points one 16-point tile at a time
// (TileShape): the 4 lanes of group r serve point r of the tile, lane g
// loading the elements [g M/4, g M/4 + M/4) of every corner row, so a row
// (32 to 256 bytes) is read by 4 lanes together where one lane per point
// reads whole rows alone.  Every element is accumulated in the same order
// as interp_level and the staged decoder rows hold the same values, so the
// results are those of k_query_mfma bit for bit.  Only one tile's
// accumulators and staging rows are live at a time.
//
// One evaluation of the wavefront's located points: features of levels
// 1..lod, the decoder lod, and with `blend` the Eq. 3 mix (weight a, this
// lane's) with decoder lod+1 on z + the level lod+1 voxel vn.  ORDERED: the points
// are taken in another order than the lanes', order.rank being this lane's place
// and order.from the lane whose point has this lane's place.  Levels that no point
// of a tile has are skipped.  Every lane must call it.
template <int M, typename FT, class DEC, bool ORDERED>
__device__ __forceinline__ float coop_eval(const ngl_model& md, const DecLds<DEC>& S, const float x[3],
                                           const int* vox, int cx, int cy, int cz, int vn, bool act, int lod, int Lp,
                                           bool blend, float a, float b2a, float b2b, const void* l1s = nullptr,
                                           bool l1 = false, PointOrder order = PointOrder{}) {
  uint64_t live = __ballot(act);  // tiles without an active point are skipped
  if (ORDERED) live = __popcll(live) == 64 ? ~0ull : (1ull << __popcll(live)) - 1ull;
  constexpr int D = TileShape<M>::D;
  const int lane = threadIdx.x & 63, r = lane >> 2, g = lane & 3;
  const int H = md.hidden;
  typename DEC::Stage* rows = S.stage;
  float mine = 0.0f;
  if (ORDERED && blend) a = __shfl(a, order.from, 64);  // the weight of the point at this lane's place
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    if (((live >> (16 * t)) & 0xffffull) == 0) continue;
    const int q = ORDERED ? __shfl(order.from, 16 * t + r, 64) : 16 * t + r;  // the group's point
    float xq[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) xq[k] = __shfl(x[k], q, 64);
    const int qx = __shfl(cx, q, 64), qy = __shfl(cy, q, 64), qz = __shfl(cz, q, 64);
    float acc[D];
#pragma unroll
    for (int i = 0; i < D; ++i) acc[i] = 0.0f;
#pragma unroll
    for (int l = 1; l <= NGL_MAX_LODS; ++l) {
      if (l > lod) break;
      const int vq = __shfl(act ? vox[l - 1] : -1, q, 64);
      if (__ballot(vq >= 0) == 0) break;
      const int sh = Lp - l;
      tile_level<M, FT>(md, l, vq, xq, qx >> sh, qy >> sh, qz >> sh, g, acc, l1s, l1);
    }
    DEC::template tile_slice<D>(rows, r, g * D, acc);
    if (g == 0) DEC::tile_rest(rows, r, xq);
    wave_lds_sync();
    const float p0 = DEC::tile(S.frag0, S.w2s0, rows, H);
    float out = b2a + p0;
    if (blend) {
      // z_{L+1} = z_L + psi_{L+1}
      wave_lds_sync();
      const int vq = __shfl(act ? vn : -1, q, 64);
      if (__ballot(vq >= 0) != 0) {
        tile_level<M, FT>(md, lod + 1, vq, xq, qx, qy, qz, g, acc);
        DEC::template tile_slice<D>(rows, r, g * D, acc);
        wave_lds_sync();
      }
      const float p1 = DEC::tile(S.frag1, S.w2s1, rows, H);
      out = (1.0f - a) * out + a * (b2b + p1);
    }
    wave_lds_sync();
    if ((lane >> 4) == t) mine = out;  // lane 16 t + j has the point at place 16 t + j
  }
  return ORDERED ? __shfl(mine, order.rank, 64) : mine;
}

// STREAMED: tile_eval instead of coop_eval.  DecF32All: the grid's row y evaluates LOD y + 1 into sdf[y][P].  Each row
// gathers its own levels again, and still 65,537 points at 5 LODs take 86 us
// against 235 with a lane per point walking the LODs (k_query_all).
template <int M, typename FT, bool XYZ, int NW, class DEC, bool STREAMED>
__global__ __launch_bounds__(64 * NW) void k_query_coop(ngl_model md, const float* __restrict__ xs, int64_t P,
                                                        int lod, float alpha, const float* __restrict__ alpha_pp,
                                                        float* __restrict__ sdf, uint8_t* __restrict__ valid,
                                                        int32_t* __restrict__ vox_out, bool l1) {
  extern __shared__ __align__(16) char smem[];
  if constexpr (std::is_same<DEC, DecF32All<M, XYZ>>::value) {
    lod = int(blockIdx.y) + 1;
    sdf += int64_t(blockIdx.y) * P;
  }
  const int H = md.hidden;
  const bool blend = alpha_pp != nullptr || alpha > 0.0f;
  const int tile_bytes = STREAMED ? tile_lds_bytes<DEC>(blend ? lod + 1 : lod) : DEC::TILE_BYTES;
  DecLds<DEC> S(smem, H, blend, tile_bytes / 4);
  // level 1's table after the staging rows (when the launch reserved it)
  char* l1s = smem + DecLds<DEC>::fixed_bytes(H, blend) + NW * size_t(tile_bytes);
  DEC::load(md, lod, S.frag0, S.w2s0);
  if (blend) DEC::load(md, lod + 1, S.frag1, S.w2s1);
  if (l1) stage_l1<M, FT>(md, l1s);
  __syncthreads();
  const float b2a = md.b2[lod - 1];
  const float b2b = blend ? md.b2[lod] : 0.0f;
  const int Lp = blend ? lod + 1 : lod;
  for (int64_t base = int64_t(blockIdx.x) * (64 * NW); base < P; base += int64_t(gridDim.x) * (64 * NW)) {
    const int64_t p = base + threadIdx.x;
    const bool act = p < P;
    float x[3] = {0.0f, 0.0f, 0.0f};
    if (act) {
      x[0] = xs[p];
      x[1] = xs[P + p];
      x[2] = xs[2 * P + p];
    }
    int vox[NGL_MAX_LODS];
    int cx, cy, cz, vlast, vn;
    locate<NGL_MAX_LODS>(md, x, Lp, vox, &cx, &cy, &cz, &vlast, lod + 1, &vn);
    if (!act) {
#pragma unroll
      for (int l = 0; l < NGL_MAX_LODS; ++l) vox[l] = -1;
      vlast = vn = -1;
    }
    const float a = act ? (alpha_pp ? alpha_pp[p] : alpha) : 0.0f;
    // 16 points are one tile in any order, and 32 gain less than the ordering takes: a
    // point of 16-bit features takes 8.9 us instead of 10.0 without it (m = 32, h =
    // 128), 32 points of a small model 7.65 instead of 7.86.  Of one or two levels
    // there is little to skip: 2^20 points in order take 1 % to 10 % more at one
    // level, at two 3 % less to 8 % more (2 % to 6 % less at m = 64), at five 0 % to
    // 15 % less.
    PointOrder order{int(threadIdx.x & 63), int(threadIdx.x & 63)};
    if (P - base > 32 && Lp >= (M >= 64 ? 2 : 3)) order = order_by_depth(vox, Lp, act);
    float out;
    if constexpr (STREAMED)
      out = tile_eval<M, FT, DEC>(md, S, x, vox, pack_cell(cx, cy, cz), act, blend, a, lod, Lp, b2a, b2b, order);
    else
      out = coop_eval<M, FT, DEC, true>(md, S, x, vox, cx, cy, cz, vn, act, lod, Lp, blend, a, b2a, b2b, l1s, l1, order);
    if (act) {
      sdf[p] = out;
      if (valid) valid[p] = vlast >= 0 ? 1 : 0;
      if (vox_out) {
#pragma unroll
        for (int l = 1; l <= NGL_MAX_LODS; ++l)
          if (l <= Lp) vox_out[int64_t(l - 1) * P + p] = vox[l - 1];
      }
    }
  }
}

template <int M, typename FT, bool XYZ, int NW, class DEC, bool STREAMED>
static int launch_query_coop_nw(const ngl_model& md, const float* x, int64_t P, int lod, float alpha,
                                const float* app, float* sdf, uint8_t* valid, int32_t* vox, hipStream_t s,
                                size_t lds, int rows) {
  // Grid-stride over the points with one round of resident blocks (each
  // stages the decoder once), or at most NGL_OPT_QUERY_BLOCKS_PER_CU per CU.
  const void* kern = reinterpret_cast<const void*>(&k_query_coop<M, FT, XYZ, NW, DEC, STREAMED>);
  const int bpc = option(NGL_OPT_QUERY_BLOCKS_PER_CU);
  int dev = 0, cus = 256;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    cus = 256;
  // level 1's rows in LDS when the table fits beside the decoder
  const bool l1 = l1_bytes<M, FT>() > 0 && l1_fits(md) && lds + l1_bytes<M, FT>() <= 65536;
  if (l1) lds += l1_bytes<M, FT>();
  int64_t grid = (P + 64 * NW - 1) / (64 * NW);
  const int64_t cap = bpc > 0 ? int64_t(cus) * bpc : resident_grid(kern, 64 * NW, lds, 0);
  if (grid > cap) grid = cap;
  k_query_coop<M, FT, XYZ, NW, DEC, STREAMED><<<dim3(unsigned(grid), unsigned(rows)), 64 * NW, lds, s>>>(
      md, x, P, lod, alpha, app, sdf, valid, vox, l1);
  NGL_LAUNCHED();
  return NGL_OK;
}

// Whether 16-bit rows are streamed (tile_eval): at m = 64, and at m = 32 from five
// levels on.  Time of 2^18 and 2^20 points over FP16 features, discrete LODs, against
// level by level: m = 64 0.91 and 0.99 at one level, 0.62 and 0.58 at five; m = 32 1.17
// and 1.14 at one, 1.13 and 1.01 at four, 1.08 and 0.96 at five (0.97 of 257 and 5,000
// points); m = 16 1.29 and 1.18 at one, 1.15 and 0.99 at five; m = 8 1.01 to 1.10.
template <int M, typename FT>
constexpr bool rows_streamed(int levels) {
  return !std::is_same<FT, F32>::value && (M >= 64 || (M == 32 && levels >= 5));
}
template <int M, typename FT, class DEC>
constexpr size_t query_tile_bytes(int levels) {
  return rows_streamed<M, FT>(levels) ? tile_lds_bytes<DEC>(levels) : DEC::TILE_BYTES;
}

template <int M, typename FT, bool XYZ, class DEC, bool STREAMED>
static int launch_query_coop_form(const ngl_model& md, const float* x, int64_t P, int lod, float alpha,
                                  const float* app, float* sdf, uint8_t* valid, int32_t* vox, hipStream_t s, int rows) {
  const bool blend = app != nullptr || alpha > 0.0f;
  const size_t fixed = DecLds<DEC>::fixed_bytes(md.hidden, blend);
  const size_t R = query_tile_bytes<M, FT, DEC>(blend ? lod + 1 : lod);
  if (fixed + 4 * R <= 65536)
    return launch_query_coop_nw<M, FT, XYZ, 4, DEC, STREAMED>(md, x, P, lod, alpha, app, sdf, valid, vox, s,
                                                              fixed + 4 * R, rows);
  if (fixed + 2 * R <= 65536)
    return launch_query_coop_nw<M, FT, XYZ, 2, DEC, STREAMED>(md, x, P, lod, alpha, app, sdf, valid, vox, s,
                                                              fixed + 2 * R, rows);
  return launch_query_coop_nw<M, FT, XYZ, 1, DEC, STREAMED>(md, x, P, lod, alpha, app, sdf, valid, vox, s, fixed + R,
                                                            rows);
}

template <int M, typename FT, bool XYZ, class DEC>
static int launch_query_coop(const ngl_model& md, const float* x, int64_t P, int lod, float alpha, const float* app,
                             float* sdf, uint8_t* valid, int32_t* vox, hipStream_t s, int rows = 1) {
  const bool streamed = rows_streamed<M, FT>(app != nullptr || alpha > 0.0f ? lod + 1 : lod);
  if constexpr (rows_streamed<M, FT>(NGL_MAX_LODS)) {
    if (streamed)
      return launch_query_coop_form<M, FT, XYZ, DEC, true>(md, x, P, lod, alpha, app, sdf, valid, vox, s, rows);
  }
  if constexpr (!rows_streamed<M, FT>(1))
    return launch_query_coop_form<M, FT, XYZ, DEC, false>(md, x, P, lod, alpha, app, sdf, valid, vox, s, rows);
  return NGL_E_INVALID;  // not reached: one of the two forms
}

template <int M, typename FT, bool XYZ, int NW, class DEC>
static int launch_query_mfma_nw(const ngl_model& md, const float* x, int64_t P, int lod, float alpha,
                                const float* app, float* sdf, uint8_t* valid, int32_t* vox, hipStream_t s,
                                size_t lds) {
  int64_t grid = (P + 64 * NW - 1) / (64 * NW);
  if (grid > 4096) grid = 4096;
  k_query_mfma<M, FT, XYZ, NW, DEC><<<unsigned(grid), 64 * NW, lds, s>>>(md, x, P, lod, alpha, app, sdf, valid, vox);
  NGL_LAUNCHED();
  return NGL_OK;
}

template <int M, typename FT, bool XYZ, class DEC>
static int launch_query_mfma(const ngl_model& md, const float* x, int64_t P, int lod, float alpha, const float* app,
                             float* sdf, uint8_t* valid, int32_t* vox, hipStream_t s) {
  if (option(NGL_OPT_COOP_GATHER) == 1)
    return launch_query_coop<M, FT, XYZ, DEC>(md, x, P, lod, alpha, app, sdf, valid, vox, s);
  const bool blend = app != nullptr || alpha > 0.0f;
  const size_t fixed = DecLds<DEC>::fixed_bytes(md.hidden, blend);
  if (fixed + 4 * DEC::STAGE_BYTES <= 65536)
    return launch_query_mfma_nw<M, FT, XYZ, 4, DEC>(md, x, P, lod, alpha, app, sdf, valid, vox, s,
                                                    fixed + 4 * DEC::STAGE_BYTES);
  if (fixed + 2 * DEC::STAGE_BYTES <= 65536)
    return launch_query_mfma_nw<M, FT, XYZ, 2, DEC>(md, x, P, lod, alpha, app, sdf, valid, vox, s,
                                                    fixed + 2 * DEC::STAGE_BYTES);
  return launch_query_mfma_nw<M, FT, XYZ, 1, DEC>(md, x, P, lod, alpha, app, sdf, valid, vox, s,
                                                  fixed + DEC::STAGE_BYTES);
}

// Central-difference normals: six queries per point.  MFMA selects the
// matrix-core decoder (every lane joins each of the six decodes).
struct NormalArgs {
  const float* x;       // points [3][P], or null with rays below
  const float* o;
  const float* d;
  const float* t_hit;
  const uint8_t* status;
  int64_t P;
  int lod;
  float alpha;
  float h;
  float* normals;       // [3][P]
  bool l1;              // level 1's table staged in LDS (k_normals_coop)
};

template <int M, typename FT, bool XYZ>
__device__ inline void query_z(const ngl_model& md, const float x[3], int lod, bool blend, float* z, float* zn) {
  const int Lp = blend ? lod + 1 : lod;
  int vox[NGL_MAX_LODS];
  int cx, cy, cz, vlast, vn;
  locate<NGL_MAX_LODS>(md, x, Lp, vox, &cx, &cy, &cz, &vlast, lod + 1, &vn);
#pragma unroll
  for (int k = 0; k < M; ++k) z[k] = 0.0f;
#pragma unroll
  for (int l = 1; l <= NGL_MAX_LODS; ++l)
    if (l <= lod && vox[l - 1] >= 0)
      interp_level<M, FT>(md, l, vox[l - 1], cx >> (Lp - l), cy >> (Lp - l), cz >> (Lp - l), x, z);
  if (blend) {
#pragma unroll
    for (int k = 0; k < M; ++k) zn[k] = z[k];
    if (vn >= 0) interp_level<M, FT>(md, lod + 1, vn, cx, cy, cz, x, zn);
  }
}

template <int M, typename FT, bool XYZ, int NW, class DEC, bool MFMA>
__global__ __launch_bounds__(64 * NW) void k_normals(ngl_model md, NormalArgs A) {
  extern __shared__ __align__(16) char smem[];
  const int H = md.hidden;
  const bool blend = A.alpha > 0.0f;
  DecLds<DEC> S(smem, H, blend && MFMA);
  if constexpr (MFMA) {
    DEC::load(md, A.lod, S.frag0, S.w2s0);
    if (blend) DEC::load(md, A.lod + 1, S.frag1, S.w2s1);
    __syncthreads();
  }
  const float b2a = md.b2[A.lod - 1];
  const float b2b = blend ? md.b2[A.lod] : 0.0f;
  const int64_t P = A.P;
  for (int64_t base = int64_t(blockIdx.x) * (64 * NW); base < P; base += int64_t(gridDim.x) * (64 * NW)) {
    const int64_t p = base + threadIdx.x;
    bool act = p < P;
    float x0[3] = {0.0f, 0.0f, 0.0f};
    if (act) {
      if (A.status) {
        act = A.status[p] == NGL_RAY_HIT;
        const float t = A.t_hit[p];
#pragma unroll
        for (int a = 0; a < 3; ++a) x0[a] = fmaf(t, A.d[a * P + p], A.o[a * P + p]);
      } else {
#pragma unroll
        for (int a = 0; a < 3; ++a) x0[a] = A.x[a * P + p];
      }
    }
    float g[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int e = 0; e < 6; ++e) {
      const int a = e >> 1;
      const float sgn = (e & 1) ? -1.0f : 1.0f;
      float x[3] = {x0[0], x0[1], x0[2]};
      x[a] = x0[a] + sgn * A.h;
      float f;
      float z[M], zn[M];
      if (act) {
        query_z<M, FT, XYZ>(md, x, A.lod, blend, z, zn);
      } else {
#pragma unroll
        for (int k = 0; k < M; ++k) z[k] = zn[k] = 0.0f;
      }
      if constexpr (MFMA) {
        DEC::stage(S.stage, x, z);
        wave_lds_sync();
        f = DEC::decode(S.frag0, S.w2s0, b2a, S.stage, H, __ballot(act));
        if (blend) {
          wave_lds_sync();
          DEC::stage(S.stage, x, zn);
          wave_lds_sync();
          f = (1.0f - A.alpha) * f + A.alpha * DEC::decode(S.frag1, S.w2s1, b2b, S.stage, H, __ballot(act));
        }
        wave_lds_sync();
      } else {
        f = 0.0f;
        if (act) {
          f = decode_f32<M, XYZ>(md, A.lod, x, z);
          if (blend) f = (1.0f - A.alpha) * f + A.alpha * decode_f32<M, XYZ>(md, A.lod + 1, x, zn);
        }
      }
      g[a] += sgn * f;
    }
    if (p < P) {
      float n[3] = {0.0f, 0.0f, 0.0f};
      if (act) {
        const float inv2h = 0.5f / A.h;
        const float gx = g[0] * inv2h, gy = g[1] * inv2h, gz = g[2] * inv2h;
        const float len = sqrtf(gx * gx + gy * gy + gz * gz);
        if (len > 0.0f) {
          n[0] = gx / len;
          n[1] = gy / len;
          n[2] = gz / len;
        }
      }
#pragma unroll
      for (int a = 0; a < 3; ++a) A.normals[a * P + p] = n[a];
    }
  }
}

// Matrix-core form: each block walks its share of the points and queues the
// active ones (rays that hit, or every point) in LDS, so its
// wavefronts only evaluate active points (a frame's misses get their zero
// normal on the way).  Each of the six probes is one cooperative,
// tile-wise evaluation (coop_eval), whose results are the bits of the
// one-lane-per-point form.  Bound by the gather as the query; what it lost
// besides was uneven shares: with contiguous ranges a wavefront was resident
// for 48 % of the launch on average.  Dealing groups and splitting the last
// pass: 1024^2 FP32 frame (452 k hits) 0.810 -> 0.659 ms, 1920x1080 frame of
// the 7-LOD 16-bit model, blended, 1.239 -> 0.970 ms.
template <int M, typename FT, bool XYZ, int NW, class DEC>
__global__ __launch_bounds__(64 * NW) void k_normals_coop(ngl_model md, NormalArgs A) {
  constexpr int NB = 64 * NW;  // points evaluated per block pass
  extern __shared__ __align__(16) char smem[];
  __shared__ int32_t queue[2 * NB];
  __shared__ int qn;
  const int H = md.hidden;
  const int lod = A.lod;
  const bool blend = A.alpha > 0.0f;
  const int Lp = blend ? lod + 1 : lod;
  DecLds<DEC> S(smem, H, blend, DEC::TILE_ELEMS);
  char* l1s = smem + DecLds<DEC>::fixed_bytes(H, blend) + NW * size_t(DEC::TILE_BYTES);
  DEC::load(md, lod, S.frag0, S.w2s0);
  if (blend) DEC::load(md, lod + 1, S.frag1, S.w2s1);
  if (A.l1) stage_l1<M, FT>(md, l1s);
  if (threadIdx.x == 0) qn = 0;
  __syncthreads();
  const float b2a = md.b2[lod - 1];
  const float b2b = blend ? md.b2[lod] : 0.0f;
  const int64_t P = A.P;
  // Groups of 64 points are dealt to the wavefronts of all blocks in turn,
  // starting seven blocks further in each round: an image's hits lie in bands
  // of rows and columns, so contiguous ranges, or the same column in every
  // round, would leave many blocks idle.  Where one round takes all points, the
  // groups that do not fill a block are the last block's: dealt too, they would
  // make it as long as the others (65,537 points, 257 blocks on 256 CUs: 184 us
  // against 157).
  const int64_t groups = (P + 63) / 64;
  const int64_t full = groups > int64_t(gridDim.x) * NW ? gridDim.x : groups < NW ? 1 : groups / NW;
  int64_t round = 0;
  for (;;) {
    // 1. queue active points until a full pass is available or the points
    // end; the count is read between two barriers, so that no wavefront
    // sees an addition of the next group
    int n = qn;
    __syncthreads();
    while (n < NB && round * int64_t(gridDim.x) * NB < P) {
      const int64_t turn = round * NW + int64_t(threadIdx.x >> 6);
      const int64_t group = blockIdx.x < full ? turn * full + (blockIdx.x + 7 * turn) % full : full * NW + turn;
      const int64_t p = group * 64 + int64_t(threadIdx.x & 63);
      bool act = false;
      if (p < P) {
        act = A.status ? A.status[p] == NGL_RAY_HIT : true;
        if (!act) {
#pragma unroll
          for (int a = 0; a < 3; ++a) A.normals[a * P + p] = 0.0f;
        }
      }
      const uint64_t m = __ballot(act);
      int base = 0;
      if ((threadIdx.x & 63) == 0 && m) base = atomicAdd(&qn, __popcll(m));
      base = __shfl(base, 0, 64);
      if (act) queue[base + __popcll(m & ((1ull << (threadIdx.x & 63)) - 1ull))] = int32_t(p);
      ++round;
      __syncthreads();
      n = qn;
      __syncthreads();
    }
    if (n == 0) break;
    const int take = n < NB ? n : NB;
    // 2. evaluate the six probes of up to NB queued points, in equal shares
    // of whole 16-point tiles: a last pass that is not full takes as long as
    // its tiles per wavefront, not as a full one
    const int share = (take + 16 * NW - 1) / (16 * NW) * 16;
    const int slot = int(threadIdx.x >> 6) * share + int(threadIdx.x & 63);
    const bool act = int(threadIdx.x & 63) < share && slot < take;
    const int64_t p = act ? queue[slot] : 0;
    float x0[3] = {0.0f, 0.0f, 0.0f};
    if (act) {
      if (A.status) {
        const float t = A.t_hit[p];
#pragma unroll
        for (int a = 0; a < 3; ++a) x0[a] = fmaf(t, A.d[a * P + p], A.o[a * P + p]);
      } else {
#pragma unroll
        for (int a = 0; a < 3; ++a) x0[a] = A.x[a * P + p];
      }
    }
    float g[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int e = 0; e < 6; ++e) {
      const int a = e >> 1;
      const float sgn = (e & 1) ? -1.0f : 1.0f;
      float x[3] = {x0[0], x0[1], x0[2]};
      x[a] = x0[a] + sgn * A.h;
      int vox[NGL_MAX_LODS];
      int cx, cy, cz, vlast, vn;
      locate<NGL_MAX_LODS>(md, x, Lp, vox, &cx, &cy, &cz, &vlast, lod + 1, &vn);
      if (!act) {
#pragma unroll
        for (int l = 0; l < NGL_MAX_LODS; ++l) vox[l] = -1;
        vn = -1;
      }
      const float f = coop_eval<M, FT, DEC, false>(md, S, x, vox, cx, cy, cz, vn, act, lod, Lp, blend, A.alpha, b2a, b2b,
                                            l1s, A.l1);
      g[a] += sgn * f;
    }
    if (act) {
      float nrm[3] = {0.0f, 0.0f, 0.0f};
      const float inv2h = 0.5f / A.h;
      const float gx = g[0] * inv2h, gy = g[1] * inv2h, gz = g[2] * inv2h;
      const float len = sqrtf(gx * gx + gy * gy + gz * gz);
      if (len > 0.0f) {
        nrm[0] = gx / len;
        nrm[1] = gy / len;
        nrm[2] = gz / len;
      }
#pragma unroll
      for (int a = 0; a < 3; ++a) A.normals[a * P + p] = nrm[a];
    }
    // 3. drop the evaluated points from the queue
    __syncthreads();
    const int rest = n - take;
    for (int i = threadIdx.x; i < rest; i += NB) queue[i] = queue[take + i];
    __syncthreads();
    if (threadIdx.x == 0) qn = rest;
    __syncthreads();
  }
}

template <int M, typename FT, bool XYZ, class DEC, bool MFMA, int NW>
static int launch_normals_nw(const ngl_model& md, const NormalArgs& A, hipStream_t s, size_t lds) {
  // one round of resident blocks looping over the points (each stages the
  // decoders once)
  const void* kern = reinterpret_cast<const void*>(&k_normals<M, FT, XYZ, NW, DEC, MFMA>);
  int64_t grid = (A.P + 64 * NW - 1) / (64 * NW);
  const int64_t cap = resident_grid(kern, 64 * NW, lds, 0);
  if (grid > cap) grid = cap;
  k_normals<M, FT, XYZ, NW, DEC, MFMA><<<unsigned(grid), 64 * NW, lds, s>>>(md, A);
  NGL_LAUNCHED();
  return NGL_OK;
}

template <int M, typename FT, bool XYZ, class DEC>
static int launch_normals_coop(const ngl_model& md, const NormalArgs& A, hipStream_t s) {
  constexpr int NW = 4;
  const bool blend = A.alpha > 0.0f;
  size_t lds = DecLds<DEC>::fixed_bytes(md.hidden, blend) + NW * size_t(DEC::TILE_BYTES);
  NormalArgs B = A;
  B.l1 = l1_bytes<M, FT>() > 0 && l1_fits(md) && lds + l1_bytes<M, FT>() <= 65536;
  if (B.l1) lds += l1_bytes<M, FT>();
  const void* kern = reinterpret_cast<const void*>(&k_normals_coop<M, FT, XYZ, NW, DEC>);
  int64_t grid = (A.P + 64 * NW - 1) / (64 * NW);
  const int64_t cap = resident_grid(kern, 64 * NW, lds, 0);
  if (grid > cap) grid = cap;
  k_normals_coop<M, FT, XYZ, NW, DEC><<<unsigned(grid), 64 * NW, lds, s>>>(md, B);
  NGL_LAUNCHED();
  return NGL_OK;
}

template <int M, typename FT, bool XYZ, class DEC, bool MFMA>
static int launch_normals(const ngl_model& md, const NormalArgs& A, hipStream_t s) {
  const bool blend = A.alpha > 0.0f;
  if constexpr (!MFMA) {
    return launch_normals_nw<M, FT, XYZ, DEC, false, 2>(md, A, s, 0);
  } else {
    if (option(NGL_OPT_COOP_GATHER) == 0) {
      // one lane per point and probe (same results as the cooperative form)
      const size_t fixed = DecLds<DEC>::fixed_bytes(md.hidden, blend);
      if (fixed + 4 * DEC::STAGE_BYTES <= 65536)
        return launch_normals_nw<M, FT, XYZ, DEC, true, 4>(md, A, s, fixed + 4 * DEC::STAGE_BYTES);
      if (fixed + 2 * DEC::STAGE_BYTES <= 65536)
        return launch_normals_nw<M, FT, XYZ, DEC, true, 2>(md, A, s, fixed + 2 * DEC::STAGE_BYTES);
      return launch_normals_nw<M, FT, XYZ, DEC, true, 1>(md, A, s, fixed + DEC::STAGE_BYTES);
    }
    return launch_normals_coop<M, FT, XYZ, DEC>(md, A, s);
  }
}

template <int M, typename FT, bool XYZ>
struct NormalOp {
  static int run(const ngl_model& md, const NormalArgs& A, hipStream_t s) {
    if (md.w_dtype == NGL_BF16) return launch_normals<M, FT, XYZ, DecBF16<M, XYZ>, true>(md, A, s);
    if (option(NGL_OPT_F32_DECODER) == 1) return launch_normals<M, FT, XYZ, DecF32<M, XYZ>, true>(md, A, s);
    return launch_normals<M, FT, XYZ, DecF32<M, XYZ>, false>(md, A, s);
  }
};

template <int M, typename FT, bool XYZ>
static int launch_query(const ngl_model& md, const float* x, int64_t P, int lod, float alpha, const float* app,
                        float* sdf, uint8_t* valid, int32_t* vox, hipStream_t s) {
  const unsigned grid = unsigned((P + kBlock - 1) / kBlock);
  k_query<M, FT, XYZ><<<grid, kBlock, 0, s>>>(md, x, P, lod, alpha, app, sdf, valid, vox);
  NGL_LAUNCHED();
  return NGL_OK;
}

template <int M, typename FT, bool XYZ>
static int launch_query_all(const ngl_model& md, const float* x, int64_t P, float* out, hipStream_t s) {
  const unsigned grid = unsigned((P + kBlock - 1) / kBlock);
  k_query_all<M, FT, XYZ><<<grid, kBlock, 0, s>>>(md, x, P, out);
  NGL_LAUNCHED();
  return NGL_OK;
}

template <int M, typename FT, bool XYZ>
struct QueryOp {
  static int run(const ngl_model& md, const float* x, int64_t P, int lod, float alpha, const float* app, float* sdf,
                 uint8_t* valid, int32_t* vox, hipStream_t s) {
    if (md.w_dtype == NGL_BF16)
      return launch_query_mfma<M, FT, XYZ, DecBF16<M, XYZ>>(md, x, P, lod, alpha, app, sdf, valid, vox, s);
    if (option(NGL_OPT_F32_DECODER) == 1)
      return launch_query_mfma<M, FT, XYZ, DecF32<M, XYZ>>(md, x, P, lod, alpha, app, sdf, valid, vox, s);
    return launch_query<M, FT, XYZ>(md, x, P, lod, alpha, app, sdf, valid, vox, s);
  }
};

// Whether query_sdf_all_lods takes a row of blocks per LOD or a lane per point.
// Rows fill the chip with few points and decode on the matrix cores, but gather
// every level again for each finer LOD.  Up to about 80,000 points rows are the
// faster form at nearly every width (65,537 points of 5 LODs, time of a lane per
// point = 1: M = 8, H = 32 0.90, 32 and 128 0.37, 64 and 256 0.94; not H = 16,
// where M = 16 takes 1.28).  Beyond, they are where the decoder outweighs the
// gather, H >= 64 and 2 M (2^18 points: 16 and 64 0.82, 32 and 64 0.80, 64 and 128
// 0.70; against 8 and 32 1.43, 64 and 64 0.99, 1.13 at 2^19), blocks of four
// wavefronts fit into the LDS (64 and 256: 1.10 to 1.33), and beyond 2^20 points,
// M >= 32 and H >= 128 (2^22 points: 32 and 128 0.96, 32 and 64 1.15, 8 and 128
// 1.17).
template <int M, typename FT, class DEC>
static bool all_lods_in_rows(const ngl_model& md, int64_t P) {
  const int H = md.hidden;
  if (P <= (H == 16 && M > 8 ? 40960 : 81920)) return true;
  const size_t R = query_tile_bytes<M, FT, DEC>(md.num_lods);
  if (H < std::max(64, 2 * M) || DecLds<DEC>::fixed_bytes(H, false) + 4 * R > 65536) return false;
  return P <= (1 << 20) || (M >= 32 && H >= 128);
}

template <int M, typename FT, bool XYZ>
struct QueryAllOp {
  static int run(const ngl_model& md, const float* x, int64_t P, float* out, hipStream_t s) {
    // on the matrix cores: the row of LOD L is the query at LOD L, bit for bit
    if (option(NGL_OPT_F32_DECODER) == 1 && option(NGL_OPT_COOP_GATHER) == 1 &&
        all_lods_in_rows<M, FT, DecF32All<M, XYZ>>(md, P))
      return launch_query_coop<M, FT, XYZ, DecF32All<M, XYZ>>(md, x, P, md.num_lods, 0.0f, nullptr, out, nullptr,
                                                              nullptr, s, md.num_lods);
    return launch_query_all<M, FT, XYZ>(md, x, P, out, s);
  }
};

// Per-width runners, defined in ngl_query_m<width>.hip.
#define NGL_QUERY_DECLARE(M_)                                                                       \
  int query_run_m##M_(const ngl_model& md, const float* x, int64_t P, int lod, float alpha,         \
                      const float* app, float* sdf, uint8_t* valid, int32_t* vox, hipStream_t s);   \
  int query_all_run_m##M_(const ngl_model& md, const float* x, int64_t P, float* out, hipStream_t s); \
  int normals_run_m##M_(const ngl_model& md, const NormalArgs& A, hipStream_t s);
NGL_QUERY_DECLARE(8)
NGL_QUERY_DECLARE(16)
NGL_QUERY_DECLARE(32)
NGL_QUERY_DECLARE(64)
#undef NGL_QUERY_DECLARE

#define NGL_QUERY_DEFINE(M_)                                                                        \
  int query_run_m##M_(const ngl_model& md, const float* x, int64_t P, int lod, float alpha,         \
                      const float* app, float* sdf, uint8_t* valid, int32_t* vox, hipStream_t s) {  \
    return dispatch_ft<QueryOp, M_>(md, x, P, lod, alpha, app, sdf, valid, vox, s);                 \
  }                                                                                                 \
  int query_all_run_m##M_(const ngl_model& md, const float* x, int64_t P, float* out, hipStream_t s) { \
    return dispatch_ft<QueryAllOp, M_>(md, x, P, out, s);                                           \
  }                                                                                                 \
  int normals_run_m##M_(const ngl_model& md, const NormalArgs& A, hipStream_t s) {                  \
    return dispatch_ft<NormalOp, M_>(md, A, s);                                                     \
  }

}  // namespace ngl
