// Training forward+backward of Eq. 4 (Sec. 3.3) on gfx950.
//
// Feature gradients are accumulated without atomics, in a fixed order, so
// results are bitwise reproducible:
//   1. k_keys / radix sort (small batches: k_rank_sort): points are sorted by
//      the Morton code of their finest cell.  Canonical voxel indices are
//      Morton ranks, so this order groups the points of every voxel of every
//      level contiguously.
//   2. per point (in sorted order) the level sum z_L, each decoder's forward
//      pass, the upstream gradient g_L, dz_L = W1_z^T (g_L w2 . 1[a>0]) and the
//      suffix sums dpsi_l = sum_{L>=l} dz_L (Eq. 2 reversed);
//   3. decoder gradients as per-block partial sums over fixed point ranges,
//      reduced in block order (k_dec_reduce).
//      From kFusedMin points on: k_point_sums, then k_dec_fused for all the rest
//      of 2 and 3.  Smaller batches, and widths that k_dec_fused does not take:
//      k_point_wave or, from kPointWaveMax points on, k_point, and k_dec_grad.
//   4. all levels in one launch each: k_rec_count / scan / k_rec_write reduce
//      fixed tiles of 64 sorted points into per-(voxel, tile) records of
//      sum_p w_j(p) dpsi_l(p); k_vox_reduce sums each voxel's records; k_corner
//      gathers, for every corner, the partials of the (voxel, slot) pairs that
//      share it.  Small batches touch few voxels: k_corner<M, true> reads the
//      records themselves.
#include "ngl_common.h"

#include <algorithm>
#include <cmath>
#include <type_traits>
#include "ngl_device.h"
#include "ngl_mfma.h"
#include "ngl_sort.h"

namespace ngl {

constexpr int kSortGrid = 256;  // most blocks of the radix-sort passes
constexpr int kDecGrid = 204;   // most blocks per LOD of the decoder-gradient pass (5 LODs fill 256 CUs x 4)
constexpr int kFusedWaves = 8;  // wavefronts per block of k_dec_fused
constexpr int kFusedGrid = 512; // most blocks of k_dec_fused
constexpr int kCUs = 256;       // of the card: grids follow the batch alone, so that sums have the same bits everywhere

// Grids sized to the batch (small batches of the fitting loop would
// otherwise pay for the full grids): at least 1024 keys per sort block and
// 64 points (one tile) per decoder-gradient block.  Deterministic for a
// given P.
inline int sort_grid(int64_t P) { return int(std::min<int64_t>(kSortGrid, std::max<int64_t>(1, (P + 1023) / 1024))); }
inline int dec_grid(int64_t P) { return int(std::min<int64_t>(kDecGrid, std::max<int64_t>(1, (P + 63) / 64))); }
constexpr int kTile = 64;       // sorted points per record tile (one wavefront)
// Batches below this many points run the per-point stage with a wavefront
// per point (k_point_wave): a lane per point would leave most of the chip
// idle and each lane's serial decoder work would set the step time.
constexpr int64_t kPointWaveMax = 16384;
// From this many points on k_dec_fused takes the decoders of the widths it is
// made for.  A step of 1,023 points with k_point_wave and of 1,024 with it: 5 LODs,
// M = 32, H = 128 78 and 79 us, M = 32, H = 32 69 and 65, M = 8, H = 32 56 and 54; one
// LOD, M = 32, H = 128 61 and 69.  Of 4,096 points (5 LODs, 32, 128) 176 and 124, of
// 16,383 403 and 166.
constexpr int64_t kFusedMin = 1024;
inline bool fused_widths(int M, int H) { return M <= 32 && (H == 32 || H == 64 || H == 128); }
// Up to this many points k_dec_fused gives each LOD a row of blocks instead of
// having every block do all LODs in turn: a block's decoder is loaded and its
// sums are added up once instead of for every LOD (14 us each time, against
// 6 us per tile of a wavefront), and k_rec_write adds the LODs' rows, which up
// to here mostly come from the caches: a step of 65,537 points took 249 us
// instead of 307, of 262,144 584 instead of 602, of 393,216 796 instead of 773
// (with dw2 formed from G; now 262,144 points take 619 with rows, 262,145 658
// without).
constexpr int64_t kFusedRowsMax = 262144;
inline bool fused_rows(int64_t P) { return P <= kFusedRowsMax; }
// Batches up to this many points are sorted by ranks in one launch
// (k_rank_sort, P^2 comparisons on all keys in LDS, against ten radix
// launches of one to four blocks), and each record tile counts the records
// before it itself: launches are what a small step spends its time on.  A
// step of 512 points with Adam took 323 us and takes 87, with the scan, the
// record and the loss launches of each level folded into one.  One LOD has keys
// of 7 bits, a single radix pass, and gains up to 2,048 points (M = 8, H = 32: 2,048
// points 56 us against 58, 3,000 67 against 62, 4,096 78 against 65).
constexpr int64_t kRankSortMax = 4096;
inline bool rank_sorted(int num_lods, int64_t P) { return P <= (num_lods == 1 ? 2048 : kRankSortMax); }

__device__ inline uint32_t spread3_10(uint32_t v) {
  v &= 0x3ffu;
  v = (v | (v << 16)) & 0x030000FFu;
  v = (v | (v << 8)) & 0x0300F00Fu;
  v = (v | (v << 4)) & 0x030C30C3u;
  v = (v | (v << 2)) & 0x09249249u;
  return v;
}

// ---------------------------------------------------------------------------
// 1. sort keys and a stable LSD radix sort (8-bit digits)
// ---------------------------------------------------------------------------
__device__ inline uint32_t point_key(const float* xs, int64_t P, int64_t p, int D) {
  const float x = xs[p], y = xs[P + p], z = xs[2 * P + p];
  if (!in_box(x, y, z)) return 1u << (3 * D);  // after every cell
  const int r = 1 << D;
  return spread3_10(cell_of(x, r)) | spread3_10(cell_of(y, r)) << 1 | spread3_10(cell_of(z, r)) << 2;
}

__global__ __launch_bounds__(kBlock) void k_keys(const float* __restrict__ xs, int64_t P, int D,
                                                 uint32_t* __restrict__ key, uint32_t* __restrict__ val) {
  const int64_t p = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  if (p >= P) return;
  key[p] = point_key(xs, P, p, D);
  val[p] = uint32_t(p);
}

// The stable order of up to kRankSortMax keys: sidx[rank] = point, the rank
// of a point being the number of points with a smaller key, or the same key
// and a smaller index.  Each block holds every key in LDS and ranks 64
// points, its four wavefronts a quarter of the comparisons each.  On the way
// clear[0, nclear) = 0 (the voxels' first records).
__global__ __launch_bounds__(kBlock) void k_rank_sort(const float* __restrict__ xs, int P, int D,
                                                      uint32_t* __restrict__ sidx, uint32_t* __restrict__ clear,
                                                      int64_t nclear) {
  __shared__ uint32_t key[kRankSortMax];
  __shared__ int part[kBlock / 64][64];
  for (int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x; i < nclear; i += int64_t(gridDim.x) * kBlock) clear[i] = 0;
  for (int p = threadIdx.x; p < P; p += kBlock) key[p] = point_key(xs, P, p, D);
  __syncthreads();
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int me = int(blockIdx.x) * 64 + lane;
  const uint32_t mine = me < P ? key[me] : 0u;
  const int quarter = (P + kBlock / 64 - 1) / (kBlock / 64);
  const int begin = w * quarter, end = min(begin + quarter, P);
  int rank = 0;
#pragma unroll 8
  for (int q = begin; q < end; ++q) {
    const uint32_t k = key[q];
    rank += (k < mine || (k == mine && q < me)) ? 1 : 0;
  }
  part[w][lane] = rank;
  __syncthreads();
  if (w == 0 && me < P) {
    for (int q = 1; q < kBlock / 64; ++q) rank += part[q][lane];
    sidx[rank] = uint32_t(me);
  }
}

// ---------------------------------------------------------------------------
// 2. per point: forward over all LODs, upstream gradient, dz, suffix sums
// ---------------------------------------------------------------------------
struct PointArgs {
  const float* xs;
  int64_t P;
  const uint32_t* sidx;     // sorted position -> point
  const float* target;      // training: [P] (original order)
  const float* grad;        // backward only: [L][P] (original order)
  float inv_p;
  float lod_w[NGL_MAX_LODS];  // training: weight of each LOD's loss term
  float* sdf_all;           // nullable [L][P] (original order)
  float* zrows;             // [L][P][M] z_L in sorted order
  float* drows;             // [L][P][M] dpsi_l in sorted order
  float* gs;                // [L][P] g_L in sorted order
  int32_t* vox_s;           // [L][P] voxel per level in sorted order
  float* loss_part;         // [grid]
  float* xsort[3];          // [P] each: the positions in sorted order (k_point_sums)
};

template <int M, bool XYZ, bool TRAIN>
__global__ __launch_bounds__(kBlock) void k_point(ngl_model md, PointArgs A) {
  const int64_t p = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  const int64_t P = A.P;
  float lossacc = 0.0f;
  if (p < P) {
    const int64_t id = A.sidx[p];
    const float x[3] = {A.xs[id], A.xs[P + id], A.xs[2 * P + id]};
    const int Lm = md.num_lods;
    int vox[NGL_MAX_LODS];
    int cx = 0, cy = 0, cz = 0;
    if (in_box(x[0], x[1], x[2])) {
      const int r = 1 << (Lm + 1);
      cx = cell_of(x[0], r);
      cy = cell_of(x[1], r);
      cz = cell_of(x[2], r);
      descend<NGL_MAX_LODS>(md, cx, cy, cz, Lm + 1, vox);
    } else {
#pragma unroll
      for (int l = 0; l < NGL_MAX_LODS; ++l) vox[l] = -1;
    }
    constexpr int OFF = XYZ ? 3 : 0;
    constexpr int DIN = M + OFF;
    const int H = md.hidden;
    float z[M];
#pragma unroll
    for (int k = 0; k < M; ++k) z[k] = 0.0f;
    const float tgt = TRAIN ? A.target[id] : 0.0f;
#pragma unroll
    for (int l = 1; l <= NGL_MAX_LODS; ++l) {
      if (l > Lm) break;
      const int s = Lm - l;
      if (vox[l - 1] >= 0) interp_level<M, F32>(md, l, vox[l - 1], cx >> s, cy >> s, cz >> s, x, z);
      A.vox_s[int64_t(l - 1) * P + p] = vox[l - 1];
      float4* zr = reinterpret_cast<float4*>(A.zrows + (int64_t(l - 1) * P + p) * M);
#pragma unroll
      for (int q = 0; q < M / 4; ++q) zr[q] = make_float4(z[4 * q], z[4 * q + 1], z[4 * q + 2], z[4 * q + 3]);
      // decoder L = l: forward, keeping the ReLU pattern
      cptr<float> W1 = as_const<float>(md.W1[l - 1]);
      cptr<float> b1 = as_const<float>(md.b1[l - 1]);
      cptr<float> w2 = as_const<float>(md.w2[l - 1]);
      float out = as_const<float>(md.b2)[l - 1];
      uint32_t mask[NGL_MAX_HIDDEN / 32];
#pragma unroll
      for (int q = 0; q < NGL_MAX_HIDDEN / 32; ++q) mask[q] = 0;
      for (int kb = 0; kb < H; kb += 32) {
        uint32_t mword = 0;
        const int nk = H - kb < 32 ? H - kb : 32;  // H is a multiple of 16
#pragma unroll 2
        for (int kk = 0; kk < nk; ++kk) {
          const int k = kb + kk;
          cptr<float> row = W1 + k * DIN;
          float a = b1[k];
          if constexpr (XYZ) {
            a = fmaf(row[0], x[0], a);
            a = fmaf(row[1], x[1], a);
            a = fmaf(row[2], x[2], a);
          }
#pragma unroll
          for (int i = 0; i < M; ++i) a = fmaf(row[OFF + i], z[i], a);
          mword |= (a > 0.0f ? 1u : 0u) << kk;
          out = fmaf(w2[k], fmaxf(a, 0.0f), out);
        }
#pragma unroll
        for (int q = 0; q < NGL_MAX_HIDDEN / 32; ++q)
          if (q == kb / 32) mask[q] = mword;
      }
      float g;
      if constexpr (TRAIN) {
        const float wres = A.lod_w[l - 1] * (out - tgt);
        lossacc = fmaf(wres, out - tgt, lossacc);
        g = 2.0f * wres * A.inv_p;
      } else {
        g = A.grad[int64_t(l - 1) * P + id];
      }
      if (A.sdf_all) A.sdf_all[int64_t(l - 1) * P + id] = out;
      A.gs[int64_t(l - 1) * P + p] = g;
      // dz = W1_z^T (g w2 . 1[a > 0])
      float dz[M];
#pragma unroll
      for (int i = 0; i < M; ++i) dz[i] = 0.0f;
      for (int kb = 0; kb < H; kb += 32) {
        uint32_t mword = 0;
#pragma unroll
        for (int q = 0; q < NGL_MAX_HIDDEN / 32; ++q)
          if (q == kb / 32) mword = mask[q];
        const int nk = H - kb < 32 ? H - kb : 32;
#pragma unroll 2
        for (int kk = 0; kk < nk; ++kk) {
          const int k = kb + kk;
          const float ga = (mword >> kk & 1u) ? g * w2[k] : 0.0f;
          cptr<float> row = W1 + k * DIN + OFF;
#pragma unroll
          for (int i = 0; i < M; ++i) dz[i] = fmaf(row[i], ga, dz[i]);
        }
      }
      float4* dr = reinterpret_cast<float4*>(A.drows + (int64_t(l - 1) * P + p) * M);
#pragma unroll
      for (int q = 0; q < M / 4; ++q) dr[q] = make_float4(dz[4 * q], dz[4 * q + 1], dz[4 * q + 2], dz[4 * q + 3]);
    }
    // dpsi_l = sum_{L >= l} dz_L, from the finest level down
    float acc[M];
    {
      const float4* dr = reinterpret_cast<const float4*>(A.drows + (int64_t(Lm - 1) * P + p) * M);
#pragma unroll
      for (int q = 0; q < M / 4; ++q) {
        const float4 v = dr[q];
        acc[4 * q] = v.x;
        acc[4 * q + 1] = v.y;
        acc[4 * q + 2] = v.z;
        acc[4 * q + 3] = v.w;
      }
    }
    for (int l = Lm - 1; l >= 1; --l) {
      float4* dr = reinterpret_cast<float4*>(A.drows + (int64_t(l - 1) * P + p) * M);
#pragma unroll
      for (int q = 0; q < M / 4; ++q) {
        const float4 v = dr[q];
        acc[4 * q] += v.x;
        acc[4 * q + 1] += v.y;
        acc[4 * q + 2] += v.z;
        acc[4 * q + 3] += v.w;
        dr[q] = make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
      }
    }
  }
  if constexpr (TRAIN) {
    // block sum of the squared residuals in a fixed order
    __shared__ float part[kBlock / 64];
    float v = lossacc;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_down(v, off, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
      float s = 0.0f;
#pragma unroll
      for (int q = 0; q < kBlock / 64; ++q) s += part[q];
      A.loss_part[blockIdx.x] = s;
    }
  }
}

// Small batches (fewer points than lanes to keep busy): one wavefront per
// sorted point and LOD (the levels' features up to it are gathered together,
// then decoder LOD runs), the same quantities as k_point except that drows
// receives dz_L (k_rec_write adds the LODs).  Lanes split each level's gather
// (lane = corner j * 8 + slice: 8 corners x M/8 features), the hidden units
// (unit k = lane + 64 u) and the adjoint (lane = output i + M * part, parts
// summing strided unit ranges); the partial sums are combined by fixed
// butterflies, so results are deterministic.  The weighted squared residual
// goes to loss_part[LOD][p].  STAGED: the block's four wavefronts share the
// decoder's first layer in LDS, read by lane without bank conflicts (an odd
// row length), where rows read from memory take a cache line per lane.
// Bound by the latency of one point's chain.
__device__ inline void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int M, bool XYZ, bool TRAIN, bool STAGED>
__global__ __launch_bounds__(kBlock) void k_point_wave(ngl_model md, PointArgs A) {
  constexpr int OFF = XYZ ? 3 : 0;
  constexpr int DIN = M + OFF;
  constexpr int WR = DIN | 1;      // staged row: odd
  constexpr int FE = M / 8;        // gather: features per lane (8 lanes per corner row)
  constexpr int KP = 64 / M;       // adjoint: lanes per output
  constexpr int UMAX = NGL_MAX_HIDDEN / 64;
  extern __shared__ float w_s[];   // STAGED: [H][WR]
  __shared__ float zsh[kBlock / 64][M];
  __shared__ float gash[kBlock / 64][NGL_MAX_HIDDEN];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t p = int64_t(blockIdx.x) * (kBlock / 64) + w;
  const int64_t P = A.P;
  const int Lm = md.num_lods;
  const int H = md.hidden;
  const int L = blockIdx.y + 1;
  const float* W1 = static_cast<const float*>(md.W1[L - 1]);
  if constexpr (STAGED) {
    for (int e = threadIdx.x; e < H * DIN; e += kBlock) w_s[e / DIN * WR + e % DIN] = W1[e];
    __syncthreads();
  }
  if (p >= P) return;  // wave-uniform: no block-wide barrier below
  const int64_t id = A.sidx[p];
  const float x[3] = {A.xs[id], A.xs[P + id], A.xs[2 * P + id]};
  int vox[NGL_MAX_LODS];
  int cx = 0, cy = 0, cz = 0;
  if (in_box(x[0], x[1], x[2])) {
    const int r = 1 << (Lm + 1);
    cx = cell_of(x[0], r);
    cy = cell_of(x[1], r);
    cz = cell_of(x[2], r);
    descend<NGL_MAX_LODS>(md, cx, cy, cz, Lm + 1, vox);
  } else {
#pragma unroll
    for (int l = 0; l < NGL_MAX_LODS; ++l) vox[l] = -1;
  }
  const float tgt = TRAIN ? A.target[id] : 0.0f;
  const int j = lane >> 3, sl = lane & 7;        // gather: corner, slice
  const int oi = lane % M, part = lane / M;      // adjoint: output, part
  // psi_1..psi_L: corner j's slices, requested for every level together (a
  // level without a voxel reads voxel 0's row and is left out of the sum)
  float row[NGL_MAX_LODS][FE];
  int corner[NGL_MAX_LODS];
#pragma unroll
  for (int l = 1; l <= NGL_MAX_LODS; ++l) {
    corner[l - 1] = 0;
    if (l <= L && md.nvox[l + 1] > 0)
      corner[l - 1] = md.corners[l - 1][int64_t(vox[l - 1] >= 0 ? vox[l - 1] : 0) * 8 + j];
  }
#pragma unroll
  for (int l = 1; l <= NGL_MAX_LODS; ++l) {
    if (l <= L && md.nvox[l + 1] > 0) {
      const float* r = static_cast<const float*>(md.feat[l - 1]) + int64_t(corner[l - 1]) * M + sl * FE;
#pragma unroll
      for (int e = 0; e < FE; ++e) row[l - 1][e] = r[e];
    }
  }
  float zl[FE];                                  // this lane's slice of z_L
#pragma unroll
  for (int e = 0; e < FE; ++e) zl[e] = 0.0f;
#pragma unroll
  for (int l = 1; l <= NGL_MAX_LODS; ++l) {
    if (l > L || vox[l - 1] < 0) continue;
    const int s = Lm - l;
    float u[3];
    cell_local(l, cx >> s, cy >> s, cz >> s, x, u);
    const float wj = corner_weight(u, j);
    float t[FE];
#pragma unroll
    for (int e = 0; e < FE; ++e) t[e] = wj * row[l - 1][e];
#pragma unroll
    for (int off = 8; off < 64; off <<= 1)
#pragma unroll
      for (int e = 0; e < FE; ++e) t[e] += __shfl_xor(t[e], off, 64);
#pragma unroll
    for (int e = 0; e < FE; ++e) zl[e] += t[e];
  }
  if (lane == 0) A.vox_s[int64_t(L - 1) * P + p] = pick<NGL_MAX_LODS>(vox, L - 1);
  if (lane < 8) {
#pragma unroll
    for (int e = 0; e < FE; ++e) zsh[w][sl * FE + e] = zl[e];
  }
  wave_sync_lds();
  float z[M];
#pragma unroll
  for (int q = 0; q < M; ++q) z[q] = zsh[w][q];
  if (lane < M) A.zrows[(int64_t(L - 1) * P + p) * M + lane] = zsh[w][lane];
  // decoder L, units k = lane + 64 u
  const float* b1 = md.b1[L - 1];
  const float* w2 = md.w2[L - 1];
  float part_out = 0.0f;
  float ga[UMAX];
#pragma unroll
  for (int uu = 0; uu < UMAX; ++uu) {
    ga[uu] = 0.0f;
    const int k = lane + 64 * uu;
    if (k < H) {
      const float* rw = STAGED ? w_s + k * WR : W1 + k * DIN;
      float a = b1[k];
      if constexpr (XYZ) {
        a = fmaf(rw[0], x[0], a);
        a = fmaf(rw[1], x[1], a);
        a = fmaf(rw[2], x[2], a);
      }
#pragma unroll
      for (int i = 0; i < M; ++i) a = fmaf(rw[OFF + i], z[i], a);
      part_out = fmaf(w2[k], fmaxf(a, 0.0f), part_out);
      ga[uu] = a > 0.0f ? w2[k] : 0.0f;  // times g below
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) part_out += __shfl_xor(part_out, off, 64);
  const float out = md.b2[L - 1] + part_out;
  float g, wres = 0.0f;
  if constexpr (TRAIN) {
    wres = A.lod_w[L - 1] * (out - tgt);
    g = 2.0f * wres * A.inv_p;
  } else {
    g = A.grad[int64_t(L - 1) * P + id];
  }
  if (lane == 0) {
    if (A.sdf_all) A.sdf_all[int64_t(L - 1) * P + id] = out;
    A.gs[int64_t(L - 1) * P + p] = g;
    if constexpr (TRAIN) A.loss_part[int64_t(L - 1) * P + p] = wres * (out - tgt);
  }
  // dz = W1_z^T (g w2 . 1[a > 0]): ga to LDS, lane (oi, part) sums units
  // part, part + KP, ...
#pragma unroll
  for (int uu = 0; uu < UMAX; ++uu) {
    const int k = lane + 64 * uu;
    if (k < H) gash[w][k] = g * ga[uu];
  }
  wave_sync_lds();
  float d = 0.0f;
#pragma unroll 4
  for (int k = part; k < H; k += KP) d = fmaf(STAGED ? w_s[k * WR + OFF + oi] : W1[k * DIN + OFF + oi], gash[w][k], d);
#pragma unroll
  for (int off = M; off < 64; off <<= 1) d += __shfl_xor(d, off, 64);
  if (lane < M) A.drows[(int64_t(L - 1) * P + p) * M + lane] = d;
}

// ---------------------------------------------------------------------------
// 2b. large batches: the point sums, then both passes of the decoders and
// their gradients in one kernel on the matrix cores
// ---------------------------------------------------------------------------
// z_l of the sorted points, M / 8 lanes per point with 8 features each (a
// row of 128 bytes is read by neighbouring lanes); also the voxels and the
// positions in sorted order.  A level's corners are added in interp_level's
// order or, PAIRS, as k_point_wave adds them, so that a batch keeps the
// pre-activations, and with them the ReLUs, of its size's per-point kernel bit
// for bit.  Bound by the random feature rows (8 per level and point).
template <int M, bool PAIRS>
__global__ __launch_bounds__(kBlock) void k_point_sums(ngl_model md, PointArgs A) {
  constexpr int G = M / 8;
  const int64_t e = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  const int64_t p = e / G, P = A.P;
  const int sl = int(e % G);
  if (p >= P) return;
  const int64_t id = A.sidx[p];
  const float x[3] = {A.xs[id], A.xs[P + id], A.xs[2 * P + id]};
  if (sl == 0) {
#pragma unroll
    for (int i = 0; i < 3; ++i) A.xsort[i][p] = x[i];
  }
  const int Lm = md.num_lods;
  int vox[NGL_MAX_LODS];
  int cx = 0, cy = 0, cz = 0;
  if (in_box(x[0], x[1], x[2])) {
    const int r = 1 << (Lm + 1);
    cx = cell_of(x[0], r);
    cy = cell_of(x[1], r);
    cz = cell_of(x[2], r);
    descend<NGL_MAX_LODS>(md, cx, cy, cz, Lm + 1, vox);
  } else {
#pragma unroll
    for (int l = 0; l < NGL_MAX_LODS; ++l) vox[l] = -1;
  }
  float z[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) z[i] = 0.0f;
#pragma unroll
  for (int l = 1; l <= NGL_MAX_LODS; ++l) {
    if (l > Lm) break;
    const int s = Lm - l, v = vox[l - 1];
    if (v >= 0) {
      float u[3];
      cell_local(l, cx >> s, cy >> s, cz >> s, x, u);
      const int4* cp = reinterpret_cast<const int4*>(md.corners[l - 1] + size_t(v) * 8);
      const int4 c0 = cp[0], c1 = cp[1];
      const int cs[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
      const float* feat = static_cast<const float*>(md.feat[l - 1]) + 8 * sl;
      float4 f[8][2];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float4* r = reinterpret_cast<const float4*>(feat + size_t(cs[j]) * M);
        f[j][0] = r[0];
        f[j][1] = r[1];
      }
      if constexpr (PAIRS) {
        float wj[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) wj[j] = corner_weight(u, j);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          auto fv = [&](int j) { return reinterpret_cast<const float*>(&f[j][i / 4])[i % 4]; };
          auto pair = [&](int j) { return fmaf(wj[j], fv(j), wj[j + 1] * fv(j + 1)); };
          z[i] += (pair(0) + pair(2)) + (pair(4) + pair(6));
        }
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float wj = corner_weight(u, j);
          const float fv[8] = {f[j][0].x, f[j][0].y, f[j][0].z, f[j][0].w, f[j][1].x, f[j][1].y, f[j][1].z, f[j][1].w};
#pragma unroll
          for (int i = 0; i < 8; ++i) z[i] = fmaf(wj, fv[i], z[i]);
        }
      }
    }
    if (sl == 0) A.vox_s[int64_t(l - 1) * P + p] = v;
    float4* zr = reinterpret_cast<float4*>(A.zrows + (int64_t(l - 1) * P + p) * M + 8 * sl);
    zr[0] = make_float4(z[0], z[1], z[2], z[3]);
    zr[1] = make_float4(z[4], z[5], z[6], z[7]);
  }
}

// Decoder passes of a wavefront's tiles of 16 points, two at a time; lane =
// (g = lane / 16, j = lane % 16):
//   forward  a[16h + 4g + r] of point j on v_mfma_f32_16x16x4f32 (a chain of
//            fmas over K) from C = b1 and the inputs [x, z] in the order of
//            the per-lane decoder: the same pre-activations bit for bit, so the
//            same ReLUs;
//   adjoint  dz = g (w2 W1_z)^T 1[a > 0];
//   G        = sum over the points of 1[a > 0] (g [x, z, 1])^T.
// In the last two one factor is a mask, which BF16 holds exactly, and the
// other is the sum of three BF16 parts (8 + 8 + 8 bits, all of FP32's; a fourth
// holds what w2 W1 has beyond them, an error that all points would share), so
// v_mfma_f32_16x16x32_bf16 forms the exact products at a fifth of the time of
// the FP32 instruction.  It rounds their sum to nearest from C = 0 (1018 of 1018
// probed), but not when C is of their size (847 of 1018, 0.24 units in the last
// place too high on average), which sums of mixed signs would gather over the
// tiles: in G the leading parts' sum d1 starts from C = 0 for every 32 points,
// only the small parts d2 go through C, and both are added by vector
// instructions.  65,537 points, upstream gradients of mixed sign, db1 of five
// LODs against FP64: median 3.7e-7 with one chain, 1.0e-7 with two, 3.0e-7 from
// k_dec_grad; 2^19 points take 984 us a step instead of 974.  The masks are kept
// as bits: of point j's units for the adjoint, and through LDS of a unit's points
// for G; their BF16 value is 2, which is one bit, against g / 2.
// dW1 = w2 G and db1 = w2 G_1 are left to k_dec_reduce.  dw2 is the plain sum
// of g relu(a), per lane in LDS (32 more registers are not there): as W1 G + b1
// G_1 it would lose what cancels between the two, and take a point's NaN to every
// unit (2^19 points 1023 us a step against 984 that way).
// Products below 2^-100 lose low parts (BF16 parts become subnormal), and weights
// are taken to be finite, w2 W1 in FP32's range too.
// A wavefront runs its range of tiles for LOD after LOD from the finest down
// and adds dpsi_{l+1}, which the same lane wrote, to dz_l.  The block shares
// the decoder's fragments in LDS; each wavefront keeps its sums in registers,
// which the block adds up in a fixed order after each LOD.
// Bound by the matrix instructions (2304 cycles per tile and LOD forward, 1088
// for the rest at M = 32, H = 128) and about as much vector work beside the
// FP32 ones, which does not overlap with them.  2^19 points, 5 LODs, M = 32,
// H = 128: 587 us (764 with FP32 matrix instructions throughout), and 138 for
// the sums before it, against 1040 us for one lane per point (k_point) and 853
// for the gradients (k_dec_grad).  Errors against FP64, median over four
// widths, six sizes and six seeds, here and of those kernels: feature gradients
// 6.4e-8 (6.5e-8), dW1 3.6e-8 (5.2e-8), dw2 2.9e-8 (4.4e-8) in training steps; 1.4e-7
// (1.7e-7), 7.0e-8 (1.8e-7), 1.7e-7 (2.6e-7) with upstream gradients of mixed sign.
template <int M, bool XYZ, int HT>
struct Fused {
  static constexpr int OFF = XYZ ? 3 : 0;
  static constexpr int DIN = M + OFF;
  static constexpr int KS = (DIN + 3) / 4;     // K-steps of the forward pass
  static constexpr int K4 = KS / 4;            // 16-byte fragments of four K-steps ...
  static constexpr int K1 = KS % 4;            // ... and single ones
  static constexpr int NT = M >= 16 ? M / 16 : 1;  // 16-wide tiles over the features
  static constexpr int MT = M < 16 ? M : 16;   // features of a tile: NT * i + n, i < MT
  static constexpr int CT = M < 16 ? 1 : NT + 1;   // tiles of G: features, and position and constant from
  static constexpr int X0 = M < 16 ? M : 0;        // column X0 of the last one on
  static constexpr int H = 16 * HT;
  static constexpr int HP = HT / 2;            // K-steps of the adjoint
  static constexpr int W = DIN + 2;            // a row of the partial sums: dW1, db1, dw2
  static constexpr int NW = kFusedWaves;
  static constexpr int WS = 160;               // scratch of a wavefront: masks [2][4][16], g [2][16]
  static constexpr int DS = HT * 256;          // and its lanes' sums of dw2: [HT][64][4]
  // LDS, in floats
  static constexpr int FW4 = 0;
  static constexpr int FW1 = FW4 + HT * K4 * 256;
  static constexpr int ADJ = FW1 + HT * K1 * 64;   // [4][NT][HP][64] fragments of 8 BF16
  static constexpr int B1 = ADJ + 4 * NT * HP * 256;
  static constexpr int W2 = B1 + H;
  static constexpr int TRB = W2 + H;           // the scratch, and the sums after a LOD
  static constexpr int ACC = HT * CT * 4;      // accumulators of G per lane
  static constexpr int SUM = (ACC + 1) * 64;   // one wavefront's sums
  // Blocks per CU that registers (and the LDS) allow: two with 128 registers a lane.
  static constexpr int PER_CU = HT * CT <= 2 ? 2 : 1;
  static constexpr int GRID = kCUs * PER_CU;
  static_assert(GRID <= kFusedGrid, "partials of db2 and of the loss");
  static constexpr int FLOATS = TRB + std::max({NW * (WS + DS), NW / 2 * SUM, H * W});
};

struct FusedArgs {
  PointArgs A;
  float* part;     // [L][slots][H][din+2]
  float* part_b2;  // [L][kFusedGrid]
  int64_t slots;   // of part per LOD
};

// base[off], off in bytes: a scalar base and a 32-bit vector offset.
template <typename T>
__device__ inline T at32(const void* base, uint32_t off) {
  return *reinterpret_cast<const T*>(static_cast<const char*>(base) + off);
}

// Bits i and i + 16 of v as a pair of BF16 values, 2 or 0 (i < 16).
__device__ inline uint32_t mask2(uint32_t v, int i) {
  return (i <= 14 ? v << (14 - i) : v >> (i - 14)) & 0x40004000u;
}

template <int M, bool XYZ, int HT>
__global__ __launch_bounds__(64 * kFusedWaves, (2 * Fused<M, XYZ, HT>::PER_CU)) void k_dec_fused(ngl_model md, FusedArgs F) {
  using S = Fused<M, XYZ, HT>;
  constexpr int NT = S::NT, CT = S::CT, NW = S::NW, DIN = S::DIN, OFF = S::OFF;
  __shared__ __align__(16) float sm[S::FLOATS];
  const float4* fw4 = reinterpret_cast<const float4*>(sm + S::FW4);
  const float* fw1 = sm + S::FW1;
  const uint4* adj = reinterpret_cast<const uint4*>(sm + S::ADJ);
  const float4* b1s = reinterpret_cast<const float4*>(sm + S::B1);
  const float4* w2s = reinterpret_cast<const float4*>(sm + S::W2);
  const PointArgs& A = F.A;
  const int64_t P = A.P;
  const int Lm = md.num_lods;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // so tiles are uniform: scalar bases
  uint32_t* mw = reinterpret_cast<uint32_t*>(sm + S::TRB + w * S::WS);
  float* gw = sm + S::TRB + w * S::WS + 128;
  float4* dw2 = reinterpret_cast<float4*>(sm + S::TRB + NW * S::WS + w * S::DS);
  const int64_t T = (P + 15) / 16, slots = int64_t(gridDim.x) * NW, me = int64_t(blockIdx.x) * NW + w;
  const int t0 = int(T * me / slots), t1 = int(T * (me + 1) / slots);
  // The three position arrays lie in one workspace.  Distances, so that a
  // lane's choice between them stays arithmetic and is not made a load of the
  // chosen pointer.
  const float* X0 = A.xsort[0];
  const int64_t dx1 = A.xsort[1] - X0, dx2 = A.xsort[2] - X0;
  float loss = 0.0f;
  // a row of blocks per LOD (which leaves the sum over the LODs to k_rec_write),
  // or all of them in turn
  const bool rows = gridDim.y > 1;
  const int first = rows ? Lm - int(blockIdx.y) : Lm, last = rows ? first : 1;
  for (int L = first; L >= last; --L) {
    const bool above = !rows && L < Lm;  // dpsi_{L+1} is there
    // the decoder's fragments
    {
      int tid = threadIdx.x;
      asm volatile("" : "+v"(tid));
      cptr<float> W1 = as_const<float>(md.W1[L - 1]);
      cptr<float> w2 = as_const<float>(md.w2[L - 1]);
      float* s4 = sm + S::FW4;
      for (int e = tid; e < HT * S::K4 * 256; e += 64 * NW) {
        const int c = e & 3, ln = e >> 2 & 63, q = (e >> 8) % (S::K4 ? S::K4 : 1), h = (e >> 8) / (S::K4 ? S::K4 : 1);
        const int k = 16 * q + 4 * c + (ln >> 4);
        s4[e] = k < DIN ? W1[(16 * h + (ln & 15)) * DIN + k] : 0.0f;
      }
      for (int e = tid; e < HT * S::K1 * 64; e += 64 * NW) {
        const int ln = e & 63, q = (e >> 6) % (S::K1 ? S::K1 : 1), h = (e >> 6) / (S::K1 ? S::K1 : 1);
        const int k = 4 * (4 * S::K4 + q) + (ln >> 4);
        sm[S::FW1 + e] = k < DIN ? W1[(16 * h + (ln & 15)) * DIN + k] : 0.0f;
      }
      for (int e = tid; e < NT * S::HP * 512; e += 64 * NW) {
        const int c = e & 7, ln = e >> 3 & 63, hp = (e >> 9) % S::HP, n = (e >> 9) / S::HP;
        const int u = 32 * hp + 16 * (c >> 2) + 4 * (ln >> 4) + (c & 3);
        const float f1 = w2[u], f2 = (ln & 15) < S::MT ? W1[u * DIN + OFF + NT * (ln & 15) + n] : 0.0f;
        float v = f1 * f2;
        uint16_t* dst = reinterpret_cast<uint16_t*>(sm + S::ADJ) + e;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t t = f32_to_bf16_bits(v);
          dst[q * NT * S::HP * 512] = uint16_t(t);
          const float part = __uint_as_float(t << 16);
          v = q == 0 ? fmaf(f1, f2, -part) : v - part;  // of the exact product
        }
      }
      for (int k = tid; k < S::H; k += 64 * NW) {
        sm[S::B1 + k] = md.b1[L - 1][k];
        sm[S::W2 + k] = md.w2[L - 1][k];
      }
    }
    __syncthreads();
    const float b2 = as_const<float>(md.b2)[L - 1];
    const float lw = A.lod_w[L - 1];
    const float* zl = A.zrows + int64_t(L - 1) * P * M;
    float* dl = A.drows + int64_t(L - 1) * P * M;
    const float* upl = A.target ? A.target : A.grad + int64_t(L - 1) * P;
    floatx4 acc[HT][CT];  // G, units 16h + 4g + r, column j of each tile
    float ab2 = 0.0f;
#pragma unroll
    for (int h = 0; h < HT; ++h)
#pragma unroll
      for (int n = 0; n < CT; ++n) acc[h][n] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    int g = lane >> 4, j = lane & 15;
#pragma unroll
    for (int h = 0; h < HT; ++h) dw2[64 * h + lane] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    // A tile's inputs 4s + g of point j and its target are requested while the
    // tile before is in its backward pass (b is free then).
    float b[2][S::KS], up[2] = {0.0f, 0.0f};
    uint32_t id[2] = {0, 0};
    // point i of tile t from the tile's first: the last one past the batch
    auto place = [&](int t, int i) {
      return uint32_t(min(i, int(min(P - 16 * int64_t(t), int64_t(16))) - 1));
    };
    auto request = [&](int t, int q) {
      const int64_t p0 = 16 * int64_t(t);
      const uint32_t jj = place(t, j);
      up[q] = upl[id[q]];
      const float* zt = zl + p0 * M;
#pragma unroll
      for (int s = 0; s < S::KS; ++s) {
        if (OFF && s == 0) {
          const int64_t dx = (g == 1 ? dx1 : 0) + (g == 2 ? dx2 : 0) + (g == 3 ? zl - X0 + (p0 + jj) * (M - 1) : 0);
          b[q][s] = (X0 + p0 + jj)[dx];
        } else {
          b[q][s] = at32<float>(zt, 4 * (jj * M + min(4 * s + g - OFF, M - 1)));
        }
      }
    };
    auto second = [&](int t) { return t + 1 < t1 ? t + 1 : t; };
    if (t0 < t1) {
      id[0] = (A.sidx + 16 * int64_t(t0))[place(t0, j)];
      id[1] = (A.sidx + 16 * int64_t(second(t0)))[place(second(t0), j)];
      request(t0, 0);
      request(second(t0), 1);
    }
#pragma unroll 1
    for (int t = t0; t < t1; t += 2) {
      // addresses are formed anew for each tile: kept, they would take the
      // registers of the sums
      int ln = lane;
      asm volatile("" : "+v"(ln));
      g = ln >> 4, j = ln & 15;
      const int tn = t + 2 < t1 ? t + 2 : t;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int tq = t + q;
        if (q == 1 && tq >= t1) {  // no second tile: no unit is on
          mw[64 + ln] = 0u;
          if (g == 0) gw[16 + j] = 0.0f;
          break;
        }
        const int64_t p0 = 16 * int64_t(tq);
        const bool live = p0 + j < P;
        const int tnq = q ? second(tn) : tn;
        const uint32_t idn = (A.sidx + 16 * int64_t(tnq))[place(tnq, j)];
        // dpsi_{L+1}, features NT * (4g + r) + n
        float u[4 * NT];
        const uint32_t zoff = 4 * g < S::MT ? 4 * NT * g : 0;
        {
          const float* ul = A.drows + (int64_t(above ? L : L - 1) * P + p0) * M;
#pragma unroll
          for (int e = 0; e < NT; ++e) {
            const float4 v = at32<float4>(ul, 4 * (place(tq, j) * M + zoff) + 16 * e);
            u[4 * e] = v.x, u[4 * e + 1] = v.y, u[4 * e + 2] = v.z, u[4 * e + 3] = v.w;
          }
        }
        if (4 * S::KS > DIN && g >= DIN % 4) b[q][S::KS - 1] = 0.0f;  // past the inputs
        // forward, two chains of units at a time; the next fragments are read
        // before the current products
        floatx4 a[HT];
        float f[2][2][S::KS];
        auto fetch = [&](int h) {
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            float* fe = f[h >> 1 & 1][e];
#pragma unroll
            for (int k = 0; k < S::K4; ++k) {
              const float4 v = fw4[((h + e) * S::K4 + k) * 64 + ln];
              fe[4 * k] = v.x, fe[4 * k + 1] = v.y, fe[4 * k + 2] = v.z, fe[4 * k + 3] = v.w;
            }
#pragma unroll
            for (int k = 0; k < S::K1; ++k) fe[4 * S::K4 + k] = fw1[((h + e) * S::K1 + k) * 64 + ln];
            const float4 c = b1s[4 * (h + e) + g];
            a[h + e] = floatx4{c.x, c.y, c.z, c.w};
          }
        };
        fetch(0);
#pragma unroll
        for (int h = 0; h < HT; h += 2) {
          if (h + 2 < HT) fetch(h + 2);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int s = 0; s < S::KS; ++s)
#pragma unroll
            for (int e = 0; e < 2; ++e)
              a[h + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[h >> 1 & 1][e][s], b[q][s], a[h + e], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
        // the output, and the ReLUs that are on: bit 2h + r / 2 + 16 (r % 2) is
        // unit 16h + 4g + r
        float4 c2[2] = {w2s[4 * (HT - 1) + g], w2s[4 * (HT - 2) + g]}, o = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        uint32_t even = 0, odd = 0;
#pragma unroll
        for (int i = 0; i < HT; ++i) {
          const int h = HT - 1 - i;
          const float4 c = c2[i & 1];
          if (h >= 2) c2[i & 1] = w2s[4 * (h - 2) + g];
          even = even + even + (a[h][2] > 0.0f ? 1u : 0u);
          odd = odd + odd + (a[h][3] > 0.0f ? 1u : 0u);
          even = even + even + (a[h][0] > 0.0f ? 1u : 0u);
          odd = odd + odd + (a[h][1] > 0.0f ? 1u : 0u);
          o.x = fmaf(c.x, fmaxf(a[h][0], 0.0f), o.x);
          o.y = fmaf(c.y, fmaxf(a[h][1], 0.0f), o.y);
          o.z = fmaf(c.z, fmaxf(a[h][2], 0.0f), o.z);
          o.w = fmaf(c.w, fmaxf(a[h][3], 0.0f), o.w);
        }
        const uint32_t on = even | odd << 16;
        float out = (o.x + o.y) + (o.z + o.w);
        out += __shfl_xor(out, 16, 64);
        out += __shfl_xor(out, 32, 64);
        out += b2;
        float gr = up[q];
        if (A.target) {
          const float wres = lw * (out - up[q]);
          loss = live && g == 0 ? fmaf(wres, out - up[q], loss) : loss;
          gr = 2.0f * wres * A.inv_p;
        }
        gr = live ? gr : 0.0f;
        ab2 += gr;
        if (live) {
#pragma unroll
          for (int h = 0; h < HT; ++h) {
            float4 d = dw2[64 * h + ln];
            d.x = fmaf(gr, fmaxf(a[h][0], 0.0f), d.x);
            d.y = fmaf(gr, fmaxf(a[h][1], 0.0f), d.y);
            d.z = fmaf(gr, fmaxf(a[h][2], 0.0f), d.z);
            d.w = fmaf(gr, fmaxf(a[h][3], 0.0f), d.w);
            dw2[64 * h + ln] = d;
          }
        }
        if (A.sdf_all && live && g == 0) (A.sdf_all + int64_t(L - 1) * P)[id[q]] = out;
        gr *= 0.5f;  // the masks' BF16 value is 2
        mw[64 * q + ln] = on;
        if (g == 0) gw[16 * q + j] = gr;
        __builtin_amdgcn_sched_barrier(0);
        id[q] = idn;
        request(tnq, q);
        // adjoint: the first parts' sum d1 is mostly exact (8-bit numbers), the
        // others' d2 small, so that dz is rounded about once
        floatx4 d1[NT], d2[NT];
#pragma unroll
        for (int n = 0; n < NT; ++n) d1[n] = d2[n] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int hp = 0; hp < S::HP; ++hp) {
          const bf16x8 m = __builtin_bit_cast(
              bf16x8, make_uint4(mask2(on, 4 * hp), mask2(on, 4 * hp + 1), mask2(on, 4 * hp + 2), mask2(on, 4 * hp + 3)));
#pragma unroll
          for (int e = 3; e >= 0; --e)
#pragma unroll
            for (int n = 0; n < NT; ++n) {
              const bf16x8 wf = __builtin_bit_cast(bf16x8, adj[((e * NT + n) * S::HP + hp) * 64 + ln]);
              floatx4& d = e ? d2[n] : d1[n];
              d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, m, d, 0, 0, 0);
            }
        }
        // a point without a unit that is on passes nothing back, also where its
        // upstream gradient is not finite
        uint32_t some = uint32_t(__ballot(on != 0u)) | uint32_t(__ballot(on != 0u) >> 32);
        some = (some | some >> 16) >> j & 1u;
        if (live && 4 * g < S::MT) {
          const float gz = some ? gr : 0.0f;
          float4* d4 = reinterpret_cast<float4*>(dl + p0 * M + j * M + zoff);
          float v[4 * NT];
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int n = 0; n < NT; ++n) v[NT * r + n] = fmaf(gz, d1[n][r], gz * d2[n][r]) + (above ? u[NT * r + n] : 0.0f);
#pragma unroll
          for (int e = 0; e < NT; ++e) d4[e] = make_float4(v[4 * e], v[4 * e + 1], v[4 * e + 2], v[4 * e + 3]);
        }
      }
      // G: the columns' values of the points 4g + e of both tiles
      float zc[2][4][CT];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int64_t p0 = 16 * int64_t(q ? second(t) : t);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t pe = place(q ? second(t) : t, 4 * g + e);
          if constexpr (M >= 16) {
#pragma unroll
            for (int n = 0; n < NT; ++n) zc[q][e][n] = at32<float>(zl + p0 * M, 4 * (pe * M + NT * j + n));
          }
          // the last tile: position and constant from column X0 on
          const int c = j - S::X0;
          if constexpr (M < 16 || XYZ) {
            const int64_t dx = (c == 1 ? dx1 : 0) + (c == 2 ? dx2 : 0) + (c < 0 ? zl - X0 + (p0 + pe) * (M - 1) + j : 0);
            zc[q][e][CT - 1] = (X0 + p0 + pe)[dx];
          }
        }
      }
      wave_sync_lds();
      uint4 y[CT][3];  // g times them, in three BF16 parts
      float spoilt = 0.0f;  // NaN where one is not finite
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const float4 gv = *reinterpret_cast<const float4*>(gw + 16 * q + 4 * g);
        const float gp[4] = {gv.x, gv.y, gv.z, gv.w};
#pragma unroll
        for (int n = 0; n < CT; ++n) {
#pragma unroll
          for (int e = 0; e < 4; e += 2) {
            float v0 = zc[q][e][n], v1 = zc[q][e + 1][n];
            if (n == CT - 1) {
              const int c = j - S::X0;
              const bool one = c == 3, none = c > 3 || (!XYZ && c >= 0 && c < 3);
              v0 = one ? 1.0f : none ? 0.0f : v0;
              v1 = one ? 1.0f : none ? 0.0f : v1;
            }
            const float z0 = v0, z1 = v1;
            v0 *= gp[e];
            v1 *= gp[e + 1];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
              const uint32_t t2 = pack_bf16(v0, v1);
              const float part0 = __uint_as_float(t2 << 16), part1 = __uint_as_float(t2 & 0xffff0000u);
              if (k == 0) spoilt = fmaf(part1, 0.0f, fmaf(part0, 0.0f, spoilt));
              v0 = k == 0 ? fmaf(z0, gp[e], -part0) : v0 - part0;  // of the exact products
              v1 = k == 0 ? fmaf(z1, gp[e + 1], -part1) : v1 - part1;
              if (q == 0 && e == 0) y[n][k].x = t2;
              if (q == 0 && e == 2) y[n][k].y = t2;
              if (q == 1 && e == 0) y[n][k].z = t2;
              if (q == 1 && e == 2) y[n][k].w = t2;
            }
          }
        }
      }
      // Products that are not finite would reach the units that are off, a mask
      // being a factor: these points are added one by one.
      if (__builtin_expect(__any(spoilt != 0.0f), 0)) {
#pragma unroll 1
        for (int i = 0; i < 32; ++i) {
          const int64_t p = 16 * int64_t(t) + i;
          if (p >= 16 * int64_t(t1) || p >= P) break;
          const uint32_t on = mw[64 * (i >> 4) + 16 * g + (i & 15)];
          const float gi = 2.0f * gw[i];
          float v[CT];
#pragma unroll
          for (int n = 0; n < CT; ++n) {
            const int c = j - S::X0;
            if (n < CT - 1 || c < 0) v[n] = zl[p * M + NT * j + n];
            else v[n] = c == 3 ? 1.0f : c < OFF ? (X0 + p)[(c == 1 ? dx1 : 0) + (c == 2 ? dx2 : 0)] : 0.0f;
          }
#pragma unroll
          for (int h = 0; h < HT; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float ga = on >> (2 * h + r / 2 + 16 * (r % 2)) & 1u ? gi : 0.0f;
#pragma unroll
              for (int n = 0; n < CT; ++n) acc[h][n][r] = fmaf(ga, v[n], acc[h][n][r]);
            }
        }
#pragma unroll
        for (int n = 0; n < CT; ++n)
#pragma unroll
          for (int k = 0; k < 3; ++k) y[n][k] = make_uint4(0u, 0u, 0u, 0u);
      }
      // unit 16h + j of the points 4g + e: bit 2h of the low half after the shift
      uint32_t mp[4];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const uint4 v = *reinterpret_cast<const uint4*>(mw + 64 * q + 16 * (j >> 2) + 4 * g);
        const int sh = (j >> 1 & 1) + 16 * (j & 1);
        mp[2 * q] = __builtin_amdgcn_perm(v.y >> sh, v.x >> sh, 0x05040100u);
        mp[2 * q + 1] = __builtin_amdgcn_perm(v.w >> sh, v.z >> sh, 0x05040100u);
      }
#pragma unroll
      for (int h = 0; h < HT; ++h) {
        const uint4 m = make_uint4(mask2(mp[0], 2 * h), mask2(mp[1], 2 * h), mask2(mp[2], 2 * h), mask2(mp[3], 2 * h));
        floatx4 d1[CT], d2[CT];
#pragma unroll
        for (int n = 0; n < CT; ++n) d1[n] = d2[n] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int e = 2; e >= 0; --e)
#pragma unroll
          for (int n = 0; n < CT; ++n) {
            floatx4& d = e ? d2[n] : d1[n];
            d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, m),
                                                        __builtin_bit_cast(bf16x8, y[n][e]), d, 0, 0, 0);
          }
#pragma unroll
        for (int n = 0; n < CT; ++n) acc[h][n] += d1[n] + d2[n];
      }
      wave_sync_lds();
    }
    // the wavefronts' sums, pairwise in a fixed order
    int ln = lane;
    asm volatile("" : "+v"(ln));
    g = ln >> 4, j = ln & 15;
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) ab2 += __shfl_xor(ab2, off, 64);
    // dw2 over the lanes' points, into a free column of G's last tile
#pragma unroll
    for (int h = 0; h < HT; ++h) {
      const float4 d = dw2[64 * h + ln];
      double v[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
      for (int off = 8; off >= 1; off >>= 1)
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] += __shfl_xor(v[r], off, 64);
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[h][CT - 1][r] = j - S::X0 == 4 ? float(v[r]) : acc[h][CT - 1][r];
    }
    float* sums = sm + S::TRB;
#pragma unroll 1
    for (int half = NW / 2; half >= 1; half >>= 1) {
      __syncthreads();  // the buffers are free
      float* q = sums + (w & (half - 1)) * S::SUM + ln;
      if (w >= half && w < 2 * half) {
#pragma unroll
        for (int h = 0; h < HT; ++h) {
#pragma unroll
          for (int n = 0; n < CT; ++n)
#pragma unroll
            for (int r = 0; r < 4; ++r) q[((h * CT + n) * 4 + r) * 64] = acc[h][n][r];
        }
        q[S::ACC * 64] = ab2;
      }
      __syncthreads();
      if (w < half) {
#pragma unroll
        for (int h = 0; h < HT; ++h) {
#pragma unroll
          for (int n = 0; n < CT; ++n)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[h][n][r] += q[((h * CT + n) * 4 + r) * 64];
          __builtin_amdgcn_sched_barrier(0);
        }
        ab2 += q[S::ACC * 64];
      }
    }
    __syncthreads();
    // wavefront 0 holds the block's sums: through LDS to whole lines
    if (w == 0) {
#pragma unroll
      for (int h = 0; h < HT; ++h) {
        float* row = sums + 16 * h * S::W;
#pragma unroll
        for (int n = 0; n < CT; ++n) {
          // the entry's column, or none
          const int c = j - S::X0;
          const int col = n < CT - 1 || c < 0 ? OFF + NT * j + n : c < OFF ? c : c == 3 ? DIN : c == 4 ? DIN + 1 : -1;
          if (col >= 0) {
#pragma unroll
            for (int r = 0; r < 4; ++r) row[(4 * g + r) * S::W + col] = acc[h][n][r];
          }
        }
      }
      if (lane == 0) F.part_b2[int64_t(L - 1) * kFusedGrid + blockIdx.x] = ab2;
    }
    __syncthreads();
    float* dst = F.part + ((L - 1) * F.slots + blockIdx.x) * (S::H * S::W);
    for (int e = threadIdx.x; e < S::H * S::W; e += 64 * NW) dst[e] = sums[e];
    __syncthreads();
  }
  if (A.target) {
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) loss += __shfl_xor(loss, off, 64);
    if (lane == 0) sm[S::TRB + w] = loss;
    __syncthreads();
    if (threadIdx.x == 0) {
      float s = 0.0f;
#pragma unroll
      for (int i = 0; i < NW; ++i) s += sm[S::TRB + i];
      A.loss_part[blockIdx.y * gridDim.x + blockIdx.x] = s;
    }
  }
}

// *loss = inv_p * sum of part[0, n) in a fixed order, by the whole block.
__device__ inline void loss_reduce(const float* part, int64_t n, float inv_p, float* loss) {
  __shared__ float sp[kBlock / 64];
  float s = 0.0f;
  for (int64_t i = threadIdx.x; i < n; i += kBlock) s += part[i];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
  if ((threadIdx.x & 63) == 0) sp[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = 0.0f;
#pragma unroll
    for (int i = 0; i < kBlock / 64; ++i) t += sp[i];
    *loss = t * inv_p;
  }
}

// ---------------------------------------------------------------------------
// 3. decoder gradients: fixed per-block partial sums, then a fixed reduction
// ---------------------------------------------------------------------------
struct DecArgs {
  const float* xs;
  int64_t P;
  const uint32_t* sidx;
  const float* zrows;
  const float* gs;
  float* part;      // [L][kDecGrid][PH][H][din+2] (the first gridDim.x blocks)
  float* part_b2;   // [L][kFusedGrid]
};

template <int M, bool XYZ>
__global__ __launch_bounds__(kBlock) void k_dec_grad(ngl_model md, DecArgs A) {
  constexpr int OFF = XYZ ? 3 : 0;
  constexpr int DIN = M + OFF;
  constexpr int DP = (DIN + 3) / 4 * 4;  // staged row, padded to whole 16-byte vectors
  __shared__ __align__(16) float in_s[kTile][DP];
  __shared__ float g_s[kTile];
  const int L = blockIdx.y + 1;
  const int H = md.hidden;
  const int PH = kBlock / H;
  const int k = threadIdx.x % H;
  const int ph = threadIdx.x / H;
  const int64_t P = A.P;
  cptr<float> W1 = as_const<float>(md.W1[L - 1]);
  float w[DP];
#pragma unroll
  for (int i = 0; i < DP; ++i) w[i] = i < DIN ? W1[k * DIN + i] : 0.0f;
  const float bk = as_const<float>(md.b1[L - 1])[k];
  const float w2k = as_const<float>(md.w2[L - 1])[k];
  float acc[DP];
#pragma unroll
  for (int i = 0; i < DP; ++i) acc[i] = 0.0f;
  float ab1 = 0.0f, aw2 = 0.0f, ab2 = 0.0f;
  int64_t chunk = (P + gridDim.x - 1) / gridDim.x;
  chunk = (chunk + kTile - 1) / kTile * kTile;
  const int64_t begin = int64_t(blockIdx.x) * chunk;
  const int64_t end = begin + chunk < P ? begin + chunk : P;
  for (int64_t base = begin; base < end; base += kTile) {
    for (int e = threadIdx.x; e < kTile * DP; e += kBlock) {
      const int pp = e / DP, i = e % DP;
      const int64_t p = base + pp;
      float v = 0.0f;
      if (p < end && i < DIN) {
        if (i < OFF) v = A.xs[int64_t(i) * P + A.sidx[p]];
        else v = A.zrows[(int64_t(L - 1) * P + p) * M + (i - OFF)];
      }
      in_s[pp][i] = v;
    }
    if (threadIdx.x < kTile) {
      const int64_t p = base + threadIdx.x;
      g_s[threadIdx.x] = p < end ? A.gs[int64_t(L - 1) * P + p] : 0.0f;
    }
    __syncthreads();
    for (int pp = ph; pp < kTile; pp += PH) {
      float in[DP];
#pragma unroll
      for (int q = 0; q < DP / 4; ++q) {
        const float4 v = reinterpret_cast<const float4*>(in_s[pp])[q];
        in[4 * q] = v.x;
        in[4 * q + 1] = v.y;
        in[4 * q + 2] = v.z;
        in[4 * q + 3] = v.w;
      }
      float a = bk;
#pragma unroll
      for (int i = 0; i < DIN; ++i) a = fmaf(w[i], in[i], a);
      const float g = g_s[pp];
      aw2 = fmaf(g, fmaxf(a, 0.0f), aw2);
      const float ga = a > 0.0f ? g * w2k : 0.0f;
      ab1 += ga;
#pragma unroll
      for (int i = 0; i < DIN; ++i) acc[i] = fmaf(ga, in[i], acc[i]);
    }
    if (threadIdx.x == 0)
      for (int pp = 0; pp < kTile; ++pp) ab2 += g_s[pp];
    __syncthreads();
  }
  float* dst = A.part + ((((int64_t(L - 1) * kDecGrid + blockIdx.x) * PH + ph) * H + k) * (DIN + 2));
#pragma unroll
  for (int i = 0; i < DIN; ++i) dst[i] = acc[i];
  dst[DIN] = ab1;
  dst[DIN + 1] = aw2;
  if (threadIdx.x == 0) A.part_b2[int64_t(L - 1) * kFusedGrid + blockIdx.x] = ab2;
}

struct DecOut {
  float* dW1[NGL_MAX_LODS];
  float* db1[NGL_MAX_LODS];
  float* dw2[NGL_MAX_LODS];
  const float* w2[NGL_MAX_LODS];  // FUSED: factor of dW1 and db1
  float* db2;
  float* loss;             // nullable: the sum of loss_part[0, nloss) times inv_p
  const float* loss_part;
  int64_t nloss;
  float inv_p;
};

// 64 entries of a LOD's sums per block, lane = entry, so that the partials are
// read in whole lines: each wavefront adds the slots w, w + 4, ... in order and
// the four are added in order (a fixed order, so the result is reproducible).
// FUSED: the partials of k_dec_fused, whose dW1 and db1 lack the factor w2, are
// added in FP64, k_dec_grad's in FP32.
// The block after the entries adds db2 and, at LOD 1, the loss.  256 slots of 5
// LODs of the 128-unit decoder (24 MB) take under 10 us; a wavefront per entry,
// its lanes a stride of 19 KB apart, took 49.
template <bool FUSED>
__global__ __launch_bounds__(kBlock) void k_dec_reduce(const float* __restrict__ part, int64_t stride, int nslots,
                                                       const float* __restrict__ part_b2, int nb2, int H, int din,
                                                       DecOut O) {
  const int L = blockIdx.y + 1;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (blockIdx.x == gridDim.x - 1) {
    if (w == 0) {
      float s = 0.0f;
      for (int b = lane; b < nb2; b += 64) s += part_b2[int64_t(L - 1) * kFusedGrid + b];
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
      if (lane == 0) O.db2[L - 1] = s;
    }
    if (L == 1 && O.loss) loss_reduce(O.loss_part, O.nloss, O.inv_p, O.loss);
    return;
  }
  typedef std::conditional_t<FUSED, double, float> Sum;
  __shared__ Sum sum[kBlock / 64][64];
  const int W = din + 2;
  const int e = blockIdx.x * 64 + lane;  // entry of [H][din+2]
  Sum s = 0;
  if (e < H * W) {  // eight sums of every 32nd slot, then pairwise: short chains
    const float* src = part + (L - 1) * stride * (H * W) + e;
    Sum q[8] = {};
    int j = w;
    for (; j + 28 < nslots; j += 32)
#pragma unroll
      for (int i = 0; i < 8; ++i) q[i] += src[int64_t(j + 4 * i) * (H * W)];
    for (; j < nslots; j += 4) q[0] += src[int64_t(j) * (H * W)];
    s = ((q[0] + q[1]) + (q[2] + q[3])) + ((q[4] + q[5]) + (q[6] + q[7]));
  }
  sum[w][lane] = s;
  __syncthreads();
  if (w == 0 && e < H * W) {
    double t = ((double(sum[0][lane]) + sum[1][lane]) + sum[2][lane]) + sum[3][lane];
    const int k = e / W, i = e % W;
    if (FUSED && i <= din) t *= O.w2[L - 1][k];
    const float v = float(t);
    if (i < din) O.dW1[L - 1][k * din + i] = v;
    else if (i == din) O.db1[L - 1][k] = v;
    else O.dw2[L - 1][k] = v;
  }
}

// ---------------------------------------------------------------------------
// 4. feature gradients: tile records, voxel sums, corner gather.  All levels in
// one launch: a level alone leaves most of the chip idle at the coarse ones
// (2^19 points, 5 levels: records 253 -> 124 us, voxel sums 90 -> 57, scans
// 113 -> 58).
// ---------------------------------------------------------------------------
struct FeatArgs {
  const float* xs;
  int64_t P;
  int Lm;
  int64_t ntiles;
  const uint32_t* sidx;
  const int32_t* vox_s;   // [L][P] sorted order
  const float* drows;     // [L][P][M] sorted order: dpsi_l, or dz_L (k_rec_write)
  uint32_t* rec_cnt;      // [L][cnt_stride] counts, then exclusive offsets
  int64_t cnt_stride;
  uint32_t* rec_total;    // [L]
  int32_t* rec_key;       // level l at rec_off[l]: voxel of each record (ascending)
  float* recs;            // level l at rec_off[l] * 8 M: [maxrec][8][M]
  int64_t rec_off[NGL_MAX_LODS + 1];
  float* vpart;           // level l at vox_off[l] * 8 M: [nv][8][M]
  uint32_t* vfirst;       // level l at vox_off[l]: index + 1 of the voxel's first record, 0 without
  int64_t vox_off[NGL_MAX_LODS + 1];
  int64_t corner_off[NGL_MAX_LODS + 1];
  const int32_t* adj_off[NGL_MAX_LODS];
  const int32_t* adj[NGL_MAX_LODS];
  float* dfeat[NGL_MAX_LODS];
};

// The level whose range of `off` holds i.
__device__ inline int level_of(const int64_t* off, int Lm, int64_t i) {
  int l = 0;
  while (l + 1 < Lm && i >= off[l + 1]) ++l;
  return l;
}

// Records of a tile: one per run of equal (existing) voxels.
__global__ __launch_bounds__(64) void k_rec_count(FeatArgs A) {
  const int32_t* vox = A.vox_s + int64_t(blockIdx.y) * A.P;
  const int64_t p = int64_t(blockIdx.x) * kTile + threadIdx.x;
  const int32_t v = p < A.P ? vox[p] : -1;
  const int32_t prev = __shfl_up(v, 1, 64);
  const uint64_t heads = __ballot(v >= 0 && (threadIdx.x == 0 || v != prev));
  if (threadIdx.x == 0) A.rec_cnt[blockIdx.y * A.cnt_stride + blockIdx.x] = uint32_t(__popcll(heads));
}

// One wavefront per tile and level.  DZ: the rows of drows are the dz_L,
// summed here from the finest LOD down (dpsi_l = sum_{L >= l} dz_L).  FEW (up
// to kRankSortMax points): the tile counts the records of the tiles before it
// itself, and the voxels' first records are noted.  Bound by the latency of
// the tile's chain, so the levels run side by side.
template <int M, bool DZ, bool FEW>
__global__ __launch_bounds__(64) void k_rec_write(ngl_model md, FeatArgs A) {
  __shared__ __align__(16) float w_s[kTile][8];
  __shared__ __align__(16) float d_s[kTile * M];
  const int lane = threadIdx.x;
  const int l = blockIdx.y, lvl = l + 1;
  const int32_t* vox = A.vox_s + int64_t(l) * A.P;
  const int64_t p0 = int64_t(blockIdx.x) * kTile, p = p0 + lane;
  const int n = int(A.P - p0 < kTile ? A.P - p0 : kTile);
  // the tile's dpsi rows, requested together
  constexpr int NQ = M / 4;  // 16-byte vectors per lane
  float4 rows[NQ];
  {
    const float4* src = reinterpret_cast<const float4*>(A.drows + (int64_t(DZ ? A.Lm - 1 : l) * A.P + p0) * M);
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int e = lane + 64 * q;
      rows[q] = e < n * NQ ? src[e] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
  }
  // phase A, lane = point: voxel, trilinear weights and record slot
  uint32_t base;
  if constexpr (FEW) {
    int before = 0;
    for (int t = 0; t < int(blockIdx.x); t += 8) {
      int32_t u[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) u[q] = t + q < int(blockIdx.x) ? vox[(t + q) * kTile + lane] : -1;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int32_t up = __shfl_up(u[q], 1, 64);
        before += __popcll(__ballot(u[q] >= 0 && (lane == 0 || u[q] != up)));
      }
    }
    base = uint32_t(before);
  } else {
    base = A.rec_cnt[l * A.cnt_stride + blockIdx.x];
  }
  const int32_t v = p < A.P ? vox[p] : -1;
  const int32_t prev = __shfl_up(v, 1, 64);
  const uint64_t valid = __ballot(v >= 0);
  const uint64_t heads = __ballot(v >= 0 && (lane == 0 || v != prev));
  // last points of the runs: the next point starts another run or has no voxel
  const uint64_t ends = valid & (heads >> 1 | ~(valid >> 1) | 1ull << 63);
  if (FEW && int64_t(blockIdx.x) == A.ntiles - 1 && lane == 0) A.rec_total[l] = base + uint32_t(__popcll(heads));
  float wj[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) wj[j] = 0.0f;
  if (v >= 0) {
    const int64_t id = A.sidx[p];
    const float x[3] = {A.xs[id], A.xs[A.P + id], A.xs[2 * A.P + id]};
    const uint32_t c = md.cell[lvl + 1][v];
    float u[3];
    cell_local(lvl, cell_x(c), cell_y(c), cell_z(c), x, u);
#pragma unroll
    for (int j = 0; j < 8; ++j) wj[j] = corner_weight(u, j);
  }
  int32_t* keys = A.rec_key + A.rec_off[l];
  const int64_t maxrec = A.rec_off[l + 1] - A.rec_off[l];
  if (heads >> lane & 1ull) {
    const int64_t r = int64_t(base) + __popcll(heads & ((1ull << lane) - 1ull));
    if (r < maxrec) keys[r] = v;
    // the voxel's first record, unless the tile before ends in the voxel
    if (FEW && (lane > 0 || p0 == 0 || vox[p0 - 1] != v)) A.vfirst[A.vox_off[l] + v] = uint32_t(r) + 1u;
  }
  if constexpr (DZ) {
    for (int k = A.Lm - 2; k >= l; --k) {
      const float4* src = reinterpret_cast<const float4*>(A.drows + (int64_t(k) * A.P + p0) * M);
      float4 t[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int e = lane + 64 * q;
        t[q] = e < n * NQ ? src[e] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      }
#pragma unroll
      for (int q = 0; q < NQ; ++q) rows[q].x += t[q].x, rows[q].y += t[q].y, rows[q].z += t[q].z, rows[q].w += t[q].w;
    }
  }
#pragma unroll
  for (int q = 0; q < NQ; ++q) reinterpret_cast<float4*>(d_s)[lane + 64 * q] = rows[q];
#pragma unroll
  for (int j = 0; j < 8; ++j) w_s[lane][j] = wj[j];
  __syncthreads();
  // phase B, lane = (channel, slot group): sequential over the tile's points
  constexpr int SG = 64 / M;      // slot groups
  constexpr int SPL = 8 / SG;     // slots per lane
  const int ch = lane % M;
  const int sg = lane / M;
  float* recs = A.recs + A.rec_off[l] * 8 * M;
  float acc[SPL];
#pragma unroll
  for (int s = 0; s < SPL; ++s) acc[s] = 0.0f;
  int64_t r = base;
  float row = d_s[ch], w[SPL];  // of the next point
#pragma unroll
  for (int s = 0; s < SPL; ++s) w[s] = w_s[0][sg * SPL + s];
  for (int i = 0; i < n; ++i) {
    const float row_i = row;
    float w_i[SPL];
#pragma unroll
    for (int s = 0; s < SPL; ++s) w_i[s] = w[s];
    const int next = i + 1 < kTile ? i + 1 : i;
    row = d_s[next * M + ch];
#pragma unroll
    for (int s = 0; s < SPL; ++s) w[s] = w_s[next][sg * SPL + s];
    if (!(valid >> i & 1ull)) continue;
#pragma unroll
    for (int s = 0; s < SPL; ++s) acc[s] = fmaf(w_i[s], row_i, acc[s]);
    if (ends >> i & 1ull) {
      if (r < maxrec) {
#pragma unroll
        for (int s = 0; s < SPL; ++s) recs[(r * 8 + sg * SPL + s) * M + ch] = acc[s];
      }
      ++r;
#pragma unroll
      for (int s = 0; s < SPL; ++s) acc[s] = 0.0f;
    }
  }
}

// Sum of each voxel's records (ascending record order), one wavefront per
// voxel of every level, from voxel g0 on.
template <int M>
__global__ __launch_bounds__(kBlock) void k_vox_reduce(FeatArgs A, int64_t g0) {
  const int64_t g = g0 + int64_t(blockIdx.x) * (kBlock / 64) + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (g >= A.vox_off[A.Lm]) return;
  const int l = level_of(A.vox_off, A.Lm, g);
  const int64_t v = g - A.vox_off[l];
  const int32_t* keys = A.rec_key + A.rec_off[l];
  const float* recs = A.recs + A.rec_off[l] * 8 * M;
  const int64_t maxrec = A.rec_off[l + 1] - A.rec_off[l];
  const int64_t nrec = A.rec_total[l] < maxrec ? A.rec_total[l] : maxrec;
  int64_t lo = 0, hi = nrec;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (keys[mid] < v) lo = mid + 1;
    else hi = mid;
  }
  constexpr int PER = 8 * M / 64;
  float acc[PER];
#pragma unroll
  for (int s = 0; s < PER; ++s) acc[s] = 0.0f;
  // the voxel's records are [lo, hi); eight are loaded at a time and added
  // in ascending order
  hi = nrec;
  {
    int64_t a = lo;
    while (a < hi) {
      const int64_t mid = (a + hi) >> 1;
      if (keys[mid] <= v) a = mid + 1;
      else hi = mid;
    }
  }
  int64_t r = lo;
  for (; r + 8 <= hi; r += 8) {
    float t[8][PER];
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
      for (int s = 0; s < PER; ++s) t[k][s] = recs[(r + k) * 8 * M + s * 64 + lane];
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
      for (int s = 0; s < PER; ++s) acc[s] += t[k][s];
  }
  for (; r < hi; ++r) {
#pragma unroll
    for (int s = 0; s < PER; ++s) acc[s] += recs[r * 8 * M + s * 64 + lane];
  }
#pragma unroll
  for (int s = 0; s < PER; ++s) A.vpart[g * 8 * M + s * 64 + lane] = acc[s];
}

// dZ_l[c][ch] = sum over (v, j) sharing corner c of the voxel sums of
// (v, j, ch), four channels per thread.  FEW: a voxel's sum is taken from
// its records here (few voxels have any), else from vpart.
template <int M, bool FEW>
__global__ __launch_bounds__(kBlock) void k_corner(FeatArgs A) {
  constexpr int Q = M / 4;
  const int64_t e = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  if (e >= A.corner_off[A.Lm] * Q) return;
  const int64_t g = e / Q;
  const int ch = int(e % Q) * 4;
  const int l = level_of(A.corner_off, A.Lm, g);
  const int64_t c = g - A.corner_off[l];
  float4 s = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  const int32_t* adj = A.adj[l];
  const int a0 = A.adj_off[l][c], a1 = A.adj_off[l][c + 1];
  if constexpr (FEW) {
    const int32_t* keys = A.rec_key + A.rec_off[l];
    const float* recs = A.recs + A.rec_off[l] * 8 * M;
    const int64_t nrec = A.rec_total[l];
    const uint32_t* vfirst = A.vfirst + A.vox_off[l];
    for (int a = a0; a < a1; ++a) {
      const int v = adj[a] >> 3, j = adj[a] & 7;
      const uint32_t first = vfirst[v];
      if (first == 0) continue;
      float4 t = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      for (int64_t r = first - 1; r < nrec && keys[r] == v; ++r) {
        const float4 x = *reinterpret_cast<const float4*>(recs + (r * 8 + j) * M + ch);
        t.x += x.x, t.y += x.y, t.z += x.z, t.w += x.w;
      }
      s.x += t.x, s.y += t.y, s.z += t.z, s.w += t.w;
    }
  } else {
    const float* vpart = A.vpart + A.vox_off[l] * 8 * M;
    for (int a = a0; a < a1; ++a) {
      const float4 x = *reinterpret_cast<const float4*>(vpart + int64_t(adj[a]) * M + ch);
      s.x += x.x, s.y += x.y, s.z += x.z, s.w += x.w;
    }
  }
  // the caller's gradient buffers need not be 16-byte aligned
  float* d = A.dfeat[l] + c * M + ch;
  d[0] = s.x, d[1] = s.y, d[2] = s.z, d[3] = s.w;
}

__global__ __launch_bounds__(kBlock) void k_zero(float* p, int64_t n) {
  const int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  if (i < n) p[i] = 0.0f;
}

// ---------------------------------------------------------------------------
// workspace
// ---------------------------------------------------------------------------
static size_t align256(size_t b) { return (b + 255) / 256 * 256; }

struct TrainWS {
  uint32_t* key[2];
  uint32_t* val[2];
  uint32_t* hist;
  float* zrows;
  float* drows;
  float* gs;
  int32_t* vox_s;
  float* loss_part;
  float* dec_part;
  float* dec_b2;
  uint32_t* rec_cnt;
  int64_t cnt_stride;
  uint32_t* rec_total;
  int32_t* rec_key;
  float* recs;
  float* vpart;
  uint32_t* vfirst;
  int64_t rec_off[NGL_MAX_LODS + 1];  // records before each level
  int64_t vox_off[NGL_MAX_LODS + 1];  // voxels before each level
  int64_t ntiles;
  size_t bytes;
};

static TrainWS carve(const ngl_model& m, int64_t P, void* base) {
  TrainWS w{};
  char* b = static_cast<char*>(base);
  size_t off = 0;
  auto take = [&](size_t n) {
    char* q = b ? b + off : nullptr;
    off += align256(n);
    return q;
  };
  const int L = m.num_lods, M = m.feat_dim, H = m.hidden, din = M + (m.with_xyz ? 3 : 0);
  const int PH = H > 0 ? kBlock / H : 1;
  w.ntiles = (P + kTile - 1) / kTile;
  // a level has at most a record per voxel and per tile boundary, and per point
  for (int l = 0; l < L; ++l) {
    w.rec_off[l + 1] = w.rec_off[l] + std::min<int64_t>(m.nvox[l + 2] + w.ntiles, P);
    w.vox_off[l + 1] = w.vox_off[l] + m.nvox[l + 2];
  }
  const bool few = rank_sorted(m.num_lods, P);
  for (int k = 0; k < 2; ++k) {
    w.key[k] = reinterpret_cast<uint32_t*>(take(4 * size_t(P)));
    w.val[k] = reinterpret_cast<uint32_t*>(take(4 * size_t(P)));
  }
  w.hist = reinterpret_cast<uint32_t*>(take(4 * 256 * size_t(kSortGrid)));
  w.zrows = reinterpret_cast<float*>(take(4 * size_t(L) * size_t(P) * size_t(M)));
  w.drows = reinterpret_cast<float*>(take(4 * size_t(L) * size_t(P) * size_t(M)));
  w.gs = reinterpret_cast<float*>(take(4 * size_t(L) * size_t(P)));
  w.vox_s = reinterpret_cast<int32_t*>(take(4 * size_t(L) * size_t(P)));
  // one per point and LOD of k_point_wave, per block of k_point or of k_dec_fused;
  // for the smaller batches too, so that a workspace serves them all
  const int64_t wave = std::min<int64_t>(P, (fused_widths(M, H) ? kFusedMin : kPointWaveMax) - 1);
  w.loss_part = reinterpret_cast<float*>(
      take(4 * size_t(std::max({L * wave, (P + kBlock - 1) / kBlock, int64_t(kFusedGrid)}))));
  w.dec_part = reinterpret_cast<float*>(take(4 * size_t(L) * kDecGrid * PH * size_t(H) * size_t(din + 2)));
  w.dec_b2 = reinterpret_cast<float*>(take(4 * size_t(L) * kFusedGrid));
  w.cnt_stride = (w.ntiles + 4) / 4 * 4;  // whole 16-byte vectors
  w.rec_cnt = reinterpret_cast<uint32_t*>(take(4 * size_t(L) * size_t(w.cnt_stride)));
  w.rec_total = reinterpret_cast<uint32_t*>(take(4 * size_t(L)));
  w.rec_key = reinterpret_cast<int32_t*>(take(4 * size_t(w.rec_off[L])));
  w.recs = reinterpret_cast<float*>(take(4 * 8 * size_t(M) * size_t(w.rec_off[L])));
  w.vpart = reinterpret_cast<float*>(take(few ? 0 : 4 * 8 * size_t(M) * size_t(w.vox_off[L])));
  w.vfirst = reinterpret_cast<uint32_t*>(take(few ? 4 * size_t(w.vox_off[L]) : 0));
  w.bytes = off;
  return w;
}

static int check_train(const ngl_model* m) {
  int rc = check_model(m, true);
  if (rc) return rc;
  if (m->feat_dtype != NGL_F32 || m->w_dtype != NGL_F32)
    NGL_FAIL(NGL_E_UNSUPPORTED, "training needs FP32 features and FP32 decoder weights");
  if (kBlock % m->hidden != 0) NGL_FAIL(NGL_E_UNSUPPORTED, "training needs hidden to divide %d", kBlock);
  if (m->feat_dim != 8 && m->feat_dim != 16 && m->feat_dim != 32 && m->feat_dim != 64)
    NGL_FAIL(NGL_E_UNSUPPORTED, "feat_dim %d not compiled", m->feat_dim);
  for (int l = 1; l <= m->num_lods; ++l)
    NGL_REQUIRE(m->ncorner[l - 1] == 0 || (m->corner_adj_off[l - 1] && (m->nvox[l + 1] == 0 || m->corner_adj[l - 1])),
                "corner adjacency of level %d is null (needed for training)", l);
  return NGL_OK;
}

// Launches k_dec_fused with one round of resident blocks of the whole card at
// most; returns the blocks per LOD.
template <int M, bool XYZ, int HT>
static int launch_fused_h(const ngl_model& md, const FusedArgs& F, hipStream_t s) {
  const int threads = 64 * kFusedWaves;
  int64_t grid = std::min<int64_t>(Fused<M, XYZ, HT>::GRID, F.slots);
  const int rows = fused_rows(F.A.P) ? md.num_lods : 1;
  grid = std::max<int64_t>(1, std::min(grid / rows, (F.A.P + 16 * kFusedWaves - 1) / (16 * kFusedWaves)));
  k_dec_fused<M, XYZ, HT><<<dim3(unsigned(grid), unsigned(rows)), threads, 0, s>>>(md, F);
  return int(grid);
}

template <int M, bool XYZ>
static int launch_fused(const ngl_model& md, const FusedArgs& F, hipStream_t s) {
  if constexpr (M <= 32) {
    switch (md.hidden) {
      case 32: return launch_fused_h<M, XYZ, 2>(md, F, s);
      case 64: return launch_fused_h<M, XYZ, 4>(md, F, s);
      default: return launch_fused_h<M, XYZ, 8>(md, F, s);
    }
  }
  return 0;
}

template <int M, bool XYZ>
static int run_train(const ngl_model& md, const float* x, const float* target, const float* grad, int64_t P,
                     const float* lod_weight, float* loss, float* sdf_all, float* const* dfeat, float* const* dW1,
                     float* const* db1, float* const* dw2, float* db2, const TrainWS& w, hipStream_t s) {
  const int Lm = md.num_lods;
  const int D = Lm + 1;
  const unsigned pgrid = unsigned((P + kBlock - 1) / kBlock);
  // 1. sort by finest-cell Morton code (3D+1 key bits)
  const bool few = rank_sorted(Lm, P);
  int cur = 0;
  if (few) {
    k_rank_sort<<<unsigned((P + 63) / 64), kBlock, 0, s>>>(x, int(P), D, w.val[0], w.vfirst, w.vox_off[Lm]);
  } else {
    k_keys<<<pgrid, kBlock, 0, s>>>(x, P, D, w.key[0], w.val[0]);
    cur = radix_sort_pairs(w.key, w.val, P, 3 * D + 1, sort_grid(P), w.hist, s);
  }
  const uint32_t* sidx = w.val[cur];
  // 2. per point
  PointArgs A{};
  A.xs = x;
  A.P = P;
  A.sidx = sidx;
  A.target = target;
  A.grad = grad;
  A.inv_p = 1.0f / float(P);
  for (int l = 0; l < NGL_MAX_LODS; ++l) A.lod_w[l] = lod_weight && l < Lm ? lod_weight[l] : 1.0f;
  A.sdf_all = sdf_all;
  A.zrows = w.zrows;
  A.drows = w.drows;
  A.gs = w.gs;
  A.vox_s = w.vox_s;
  A.loss_part = w.loss_part;
  int64_t nloss = 0;
  const int PH = kBlock / md.hidden;
  int nslots = 0, nb2 = 0;
  // one fused kernel on the matrix cores where a wavefront's registers hold a
  // decoder's gradients
  const bool fused = P >= kFusedMin && fused_widths(M, md.hidden);
  if (!fused && P < kPointWaveMax) {
    // small batches: one wavefront per point and LOD
    const dim3 wgrid(unsigned((P + kBlock / 64 - 1) / (kBlock / 64)), unsigned(Lm));
    const size_t lds = 4 * size_t(md.hidden) * size_t((M + (XYZ ? 3 : 0)) | 1);
    nloss = target ? Lm * P : 0;
    auto launch = [&](auto train) {
      constexpr bool TRAIN = decltype(train)::value;
      if (lds <= 49152) k_point_wave<M, XYZ, TRAIN, true><<<wgrid, kBlock, lds, s>>>(md, A);
      else k_point_wave<M, XYZ, TRAIN, false><<<wgrid, kBlock, 0, s>>>(md, A);
    };
    if (target) launch(std::true_type{});
    else launch(std::false_type{});
  } else if (fused) {
    // key[0], key[1] and the other index array are free after the sort
    A.xsort[0] = reinterpret_cast<float*>(w.key[0]);
    A.xsort[1] = reinterpret_cast<float*>(w.key[1]);
    A.xsort[2] = reinterpret_cast<float*>(w.val[1 - cur]);
    const unsigned sgrid = unsigned((P * (M / 8) + kBlock - 1) / kBlock);
    if (P < kPointWaveMax) k_point_sums<M, true><<<sgrid, kBlock, 0, s>>>(md, A);
    else k_point_sums<M, false><<<sgrid, kBlock, 0, s>>>(md, A);
    const FusedArgs B{A, w.dec_part, w.dec_b2, int64_t(kDecGrid) * PH};
    nslots = nb2 = launch_fused<M, XYZ>(md, B, s);
    nloss = target ? nb2 * (fused_rows(P) ? Lm : 1) : 0;
  } else if (target) {
    k_point<M, XYZ, true><<<pgrid, kBlock, 0, s>>>(md, A);
    nloss = pgrid;
  } else {
    k_point<M, XYZ, false><<<pgrid, kBlock, 0, s>>>(md, A);
  }
  // 3. decoder gradients
  if (!fused) {
    DecArgs B{x, P, sidx, w.zrows, w.gs, w.dec_part, w.dec_b2};
    nb2 = dec_grid(P);
    nslots = nb2 * PH;
    k_dec_grad<M, XYZ><<<dim3(nb2, Lm), kBlock, 0, s>>>(md, B);
  }
  DecOut O{};
  for (int l = 0; l < Lm; ++l) {
    O.dW1[l] = dW1[l];
    O.db1[l] = db1[l];
    O.dw2[l] = dw2[l];
    O.w2[l] = static_cast<const float*>(md.w2[l]);
  }
  O.db2 = db2;
  O.loss = target ? loss : nullptr;
  O.loss_part = w.loss_part;
  O.nloss = nloss;
  O.inv_p = 1.0f / float(P);
  const int din = M + (XYZ ? 3 : 0);
  const int H = md.hidden;
  (fused ? k_dec_reduce<true> : k_dec_reduce<false>)<<<dim3(unsigned((H * (din + 2) + 63) / 64) + 1, Lm), kBlock, 0, s>>>(
      w.dec_part, int64_t(kDecGrid) * PH, nslots, w.dec_b2, nb2, H, din, O);
  // 4. feature gradients
  FeatArgs C{};
  C.xs = x;
  C.P = P;
  C.Lm = Lm;
  C.ntiles = w.ntiles;
  C.sidx = sidx;
  C.vox_s = w.vox_s;
  C.drows = w.drows;
  C.rec_cnt = w.rec_cnt;
  C.cnt_stride = w.cnt_stride;
  C.rec_total = w.rec_total;
  C.rec_key = w.rec_key;
  C.recs = w.recs;
  C.vpart = w.vpart;
  C.vfirst = w.vfirst;
  for (int l = 0; l < Lm; ++l) {
    C.rec_off[l + 1] = w.rec_off[l + 1];
    C.vox_off[l + 1] = w.vox_off[l + 1];
    C.corner_off[l + 1] = C.corner_off[l] + md.ncorner[l];
    C.adj_off[l] = md.corner_adj_off[l];
    C.adj[l] = md.corner_adj[l];
    C.dfeat[l] = dfeat[l];
  }
  const dim3 tgrid(unsigned(w.ntiles), unsigned(Lm));
  const unsigned cgrid = unsigned((C.corner_off[Lm] * (M / 4) + kBlock - 1) / kBlock);
  if (cgrid == 0) {
    NGL_LAUNCHED();
    return NGL_OK;
  }
  if (few) {
    k_rec_write<M, true, true><<<tgrid, 64, 0, s>>>(md, C);
    k_corner<M, true><<<cgrid, kBlock, 0, s>>>(C);
  } else {
    k_rec_count<<<tgrid, 64, 0, s>>>(C);
    k_scan_inplace<<<Lm, 1024, 0, s>>>(w.rec_cnt, w.ntiles, w.rec_total, w.cnt_stride);
    if (P < kPointWaveMax || (fused && fused_rows(P))) k_rec_write<M, true, false><<<tgrid, 64, 0, s>>>(md, C);
    else k_rec_write<M, false, false><<<tgrid, 64, 0, s>>>(md, C);
    // a launch has fewer than 2^32 threads, 64 per voxel
    constexpr int64_t kVoxLaunch = int64_t(1) << 25;
    for (int64_t g0 = 0; g0 < C.vox_off[Lm]; g0 += kVoxLaunch) {
      const int64_t n = std::min(kVoxLaunch, C.vox_off[Lm] - g0);
      k_vox_reduce<M><<<unsigned((n + kBlock / 64 - 1) / (kBlock / 64)), kBlock, 0, s>>>(C, g0);
    }
    k_corner<M, false><<<cgrid, kBlock, 0, s>>>(C);
  }
  NGL_LAUNCHED();
  return NGL_OK;
}

static int zero_grads(const ngl_model& md, float* loss, float* const* dfeat, float* const* dW1, float* const* db1,
                      float* const* dw2, float* db2, hipStream_t s) {
  const int din = md.feat_dim + (md.with_xyz ? 3 : 0);
  auto z = [&](float* p, int64_t n) {
    if (p && n > 0) k_zero<<<unsigned((n + kBlock - 1) / kBlock), kBlock, 0, s>>>(p, n);
  };
  z(loss, 1);
  z(db2, md.num_lods);
  for (int l = 0; l < md.num_lods; ++l) {
    z(dfeat[l], md.ncorner[l] * md.feat_dim);
    z(dW1[l], int64_t(md.hidden) * din);
    z(db1[l], md.hidden);
    z(dw2[l], md.hidden);
  }
  NGL_LAUNCHED();
  return NGL_OK;
}

static int train_entry(const ngl_model* m, const float* x, const float* target, const float* grad, int64_t P,
                       const float* lod_weight, float* loss, float* sdf_all, float* const* dfeat, float* const* dW1, float* const* db1,
                       float* const* dw2, float* db2, void* ws, size_t ws_bytes, void* stream) {
  int rc = check_train(m);
  if (rc) return rc;
  NGL_REQUIRE(P >= 0 && P < (int64_t(1) << 31), "point count out of range");
  NGL_REQUIRE(dfeat && dW1 && db1 && dw2 && db2, "gradient buffers are null");
  for (int l = 0; l < m->num_lods; ++l)
    NGL_REQUIRE((dfeat[l] || m->ncorner[l] == 0) && dW1[l] && db1[l] && dw2[l], "gradient buffer of LOD %d is null",
                l + 1);
  hipStream_t s = (hipStream_t)stream;
  if (P == 0) return zero_grads(*m, loss, dfeat, dW1, db1, dw2, db2, s);
  NGL_REQUIRE(x != nullptr, "x is null");
  NGL_REQUIRE(target || grad, "target or upstream gradient is null");
  TrainWS w = carve(*m, P, ws);
  NGL_REQUIRE(ws != nullptr && ws_bytes >= w.bytes, "workspace too small: %zu < %zu bytes", ws_bytes, w.bytes);
  const ngl_model& md = *m;
#define NGL_TRAIN_CALL(M_, X_) \
  return run_train<M_, X_>(md, x, target, grad, P, lod_weight, loss, sdf_all, dfeat, dW1, db1, dw2, db2, w, s)
#define NGL_TRAIN_M(M_)          \
  if (md.with_xyz) NGL_TRAIN_CALL(M_, true); \
  else NGL_TRAIN_CALL(M_, false);
  switch (md.feat_dim) {
    case 8: NGL_TRAIN_M(8);
    case 16: NGL_TRAIN_M(16);
    case 32: NGL_TRAIN_M(32);
    default: NGL_TRAIN_M(64);
  }
#undef NGL_TRAIN_M
#undef NGL_TRAIN_CALL
}

}  // namespace ngl

extern "C" {

int ngl_train_workspace(const ngl_model* m, int64_t P, size_t* bytes) {
  int rc = ngl::check_train(m);
  if (rc) return rc;
  NGL_REQUIRE(bytes && P >= 0, "invalid workspace query");
  *bytes = ngl::carve(*m, P, nullptr).bytes;
  return NGL_OK;
}

int ngl_backward_all_lods(const ngl_model* m, const float* x, int64_t P, const float* grad_sdf, float* const* dfeat,
                          float* const* dW1, float* const* db1, float* const* dw2, float* db2, void* ws,
                          size_t ws_bytes, void* stream) {
  NGL_REQUIRE(P == 0 || grad_sdf != nullptr, "grad_sdf is null");
  return ngl::train_entry(m, x, nullptr, grad_sdf, P, nullptr, nullptr, nullptr, dfeat, dW1, db1, dw2, db2, ws,
                          ws_bytes, stream);
}

int ngl_train_fwd_bwd(const ngl_model* m, const float* x, const float* target, int64_t P, float* loss,
                      float* sdf_all, float* const* dfeat, float* const* dW1, float* const* db1, float* const* dw2,
                      float* db2, void* ws, size_t ws_bytes, void* stream) {
  NGL_REQUIRE(P == 0 || target != nullptr, "target is null");
  NGL_REQUIRE(loss != nullptr, "loss is null");
  return ngl::train_entry(m, x, target, nullptr, P, nullptr, loss, sdf_all, dfeat, dW1, db1, dw2, db2, ws, ws_bytes,
                          stream);
}

int ngl_train_fwd_bwd_lods(const ngl_model* m, const float* x, const float* target, int64_t P,
                           const float* lod_weight, float* loss, float* sdf_all, float* const* dfeat,
                           float* const* dW1, float* const* db1, float* const* dw2, float* db2, void* ws,
                           size_t ws_bytes, void* stream) {
  NGL_REQUIRE(P == 0 || target != nullptr, "target is null");
  NGL_REQUIRE(loss != nullptr && lod_weight != nullptr, "loss or lod_weight is null");
  NGL_REQUIRE(m != nullptr, "model is null");
  for (int l = 0; l < m->num_lods && l < NGL_MAX_LODS; ++l)
    NGL_REQUIRE(std::isfinite(lod_weight[l]) && lod_weight[l] >= 0.0f, "lod_weight[%d] must be finite and >= 0", l);
  return ngl::train_entry(m, x, target, nullptr, P, lod_weight, loss, sdf_all, dfeat, dW1, db1, dw2, db2, ws,
                          ws_bytes, stream);
}

}  // extern "C"
