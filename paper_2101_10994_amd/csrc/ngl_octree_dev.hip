// Sparse voxel octree from finest-level occupancy on the device (Sec. 3.2;
// App. A.1): the same canonical layout as the host build, bit for bit.
//
// Canonical indices are Morton ranks, so the tree is held as bitmaps in
// Morton order, one bit per cell of every depth and per lattice point of
// every feature level, and an index is the number of set bits before a bit:
//   1. k_oct_mark: every occupied cell sets its bit and climbs, setting its
//      ancestors' bits until it meets one that is set.  k_oct_lattice: a
//      level's lattice points are the voxels' bits grown by one cell, 32
//      points at a time.
//   2. k_oct_sums, k_oct_prefix: set bits before every word (block sums, then
//      each block adds those before it in its bitmap), and the totals.
//   3. k_oct_emit: per voxel its cell, its child mask (the byte of its eight
//      children in the next bitmap), first child and parent (ranks); per
//      corner bitmap block the number of (voxel, slot) pairs at its corners.
//   4. k_oct_corners: per corner the up to eight voxels around it give its
//      entries of the corner table and, in ascending order, its adjacency.
// No sort, and seven launches whatever the number of levels.  The bitmaps of a
// 7-level tree take 2.4 MB per array (they stay in L2), of an 8-level one 38 MB.
// Sizes stay on the device; arrays are caller-allocated to upper bounds.
//
// 641,375 cells, 7 levels (784,817 voxels, 1,145,279 corners), allocations and
// the read of the sizes included: 6.41 -> 0.54 ms (radix sorts of the cells
// and of eight corner pairs per voxel, with one-block scans, before).  The
// marking kernel's atomics (0.17 ms) and the corner tables' scattered writes
// (0.10 ms) take most of what is left on the device.
#include "ngl_common.h"
#include "ngl_device.h"

#include <algorithm>

namespace ngl {

__device__ inline uint32_t spread3_u32(uint32_t v) {
  v &= 0x3ffu;
  v = (v | (v << 16)) & 0x030000FFu;
  v = (v | (v << 8)) & 0x0300F00Fu;
  v = (v | (v << 4)) & 0x030C30C3u;
  v = (v | (v << 2)) & 0x09249249u;
  return v;
}

__device__ inline uint32_t compact3_u32(uint32_t v) {
  v &= 0x09249249u;
  v = (v ^ (v >> 2)) & 0x030C30C3u;
  v = (v ^ (v >> 4)) & 0x0300F00Fu;
  v = (v ^ (v >> 8)) & 0x030000FFu;
  v = (v ^ (v >> 16)) & 0x000003FFu;
  return v;
}

__device__ inline uint32_t morton3_u32(uint32_t x, uint32_t y, uint32_t z) {
  return spread3_u32(x) | spread3_u32(y) << 1 | spread3_u32(z) << 2;
}

// Two coordinates interleaved (a in the even bits).
__device__ inline uint32_t spread2_u32(uint32_t v) {
  v &= 0xffffu;
  v = (v | (v << 8)) & 0x00FF00FFu;
  v = (v | (v << 4)) & 0x0F0F0F0Fu;
  v = (v | (v << 2)) & 0x33333333u;
  v = (v | (v << 1)) & 0x55555555u;
  return v;
}

__device__ inline uint32_t compact2_u32(uint32_t v) {
  v &= 0x55555555u;
  v = (v | (v >> 1)) & 0x33333333u;
  v = (v | (v >> 2)) & 0x0F0F0F0Fu;
  v = (v | (v >> 4)) & 0x00FF00FFu;
  v = (v | (v >> 8)) & 0x0000FFFFu;
  return v;
}

__device__ inline uint32_t morton2_u32(uint32_t a, uint32_t b) { return spread2_u32(a) | spread2_u32(b) << 1; }

// Bit of the lattice point (x, y, z), coordinates 0..r, r = 2^b, in the order
// of its Morton code.  A coordinate equal to r has only the code's top bit of
// its axis, so the codes sort by which axes are at r first and by the
// interleaved other coordinates then: the r^3 points below r on every axis,
// and after them the faces, edges and the corner at r, without gaps
// ((r + 1)^3 bits instead of 8 r^3).
__device__ inline uint32_t lattice_bit(int b, uint32_t x, uint32_t y, uint32_t z) {
  const uint32_t r1 = 1u << b, r2 = 1u << (2 * b), r3 = 1u << (3 * b);
  switch (x >> b | y >> b << 1 | z >> b << 2) {
    case 0: return morton3_u32(x, y, z);
    case 1: return r3 + morton2_u32(y, z);
    case 2: return r3 + r2 + morton2_u32(x, z);
    case 3: return r3 + 2 * r2 + z;
    case 4: return r3 + 2 * r2 + r1 + morton2_u32(x, y);
    case 5: return r3 + 3 * r2 + r1 + y;
    case 6: return r3 + 3 * r2 + 2 * r1 + x;
    default: return r3 + 3 * r2 + 3 * r1;
  }
}

__device__ inline void lattice_point(int b, uint32_t bit, uint32_t p[3]) {
  const uint32_t r1 = 1u << b, r2 = 1u << (2 * b), r3 = 1u << (3 * b);
  if (bit < r3) {
    p[0] = compact3_u32(bit), p[1] = compact3_u32(bit >> 1), p[2] = compact3_u32(bit >> 2);
    return;
  }
  bit -= r3;
  p[0] = p[1] = p[2] = r1;
  if (bit < r2) {
    p[1] = compact2_u32(bit), p[2] = compact2_u32(bit >> 1);
  } else if (bit < 2 * r2) {
    bit -= r2, p[0] = compact2_u32(bit), p[2] = compact2_u32(bit >> 1);
  } else if (bit < 2 * r2 + r1) {
    p[2] = bit - 2 * r2;
  } else if (bit < 3 * r2 + r1) {
    bit -= 2 * r2 + r1, p[0] = compact2_u32(bit), p[1] = compact2_u32(bit >> 1);
  } else if (bit < 3 * r2 + 2 * r1) {
    p[1] = bit - (3 * r2 + r1);
  } else if (bit < 3 * r2 + 3 * r1) {
    p[0] = bit - (3 * r2 + 2 * r1);
  }
}

constexpr int kOctWords = 1024;  // words of a bitmap per block of the sums
constexpr int kOctSegs = NGL_MAX_DEPTH + NGL_MAX_LODS;

// Bitmaps one after another, each padded to whole blocks: depths 0..D, then
// levels 1..L (segment D + l).
struct OctMaps {
  int D, L;
  uint32_t off[kOctSegs + 1];  // first word of each segment (and the end)
  uint32_t* words;
  uint32_t* pre;   // set bits of the segment before each word
  uint32_t* bsum;  // [blocks] set bits
  uint32_t* dsum;  // [words / kBlock] (voxel, slot) pairs at the corners (corner segments)
  // segment of block b
  __device__ int segment(uint32_t b) const {
    int s = 0;
    while (b * kOctWords >= off[s + 1]) ++s;
    return s;
  }
  // set bits before `bit` in segment s
  __device__ uint32_t rank(int s, uint32_t bit) const {
    const uint32_t w = off[s] + (bit >> 5);
    return pre[w] + uint32_t(__popc(words[w] & ((1u << (bit & 31u)) - 1u)));
  }
};

static __global__ __launch_bounds__(kBlock) void k_oct_clear(uint4* words, uint32_t n4, int64_t* bad, int32_t* parent0) {
  const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
  if (i < n4) words[i] = make_uint4(0u, 0u, 0u, 0u);
  if (i == 0) {
    *bad = 0;
    parent0[0] = -1;
  }
}

// Sets a bit; true if this call was the one that did.  Bits that are set are
// mostly found by the load, which saves the atomic.
__device__ inline bool set_bit(uint32_t* words, uint32_t bit) {
  uint32_t* w = words + (bit >> 5);
  const uint32_t m = 1u << (bit & 31u);
  if (__hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & m) return false;
  return !(atomicOr(w, m) & m);
}

// Bound by the scattered atomics (about one per voxel).
static __global__ __launch_bounds__(kBlock) void k_oct_mark(const int32_t* __restrict__ ijk, int64_t n, OctMaps M,
                                                            int64_t* bad) {
  const int64_t k = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  if (k >= n) return;
  const int32_t res = 1 << M.D;
  const int32_t x = ijk[3 * k], y = ijk[3 * k + 1], z = ijk[3 * k + 2];
  if (x < 0 || y < 0 || z < 0 || x >= res || y >= res || z >= res) {
    atomicAdd(reinterpret_cast<unsigned long long*>(bad), 1ull);
    return;
  }
  const uint32_t code = morton3_u32(uint32_t(x), uint32_t(y), uint32_t(z));
  for (int d = M.D; d >= 0; --d) {
    const int s = M.D - d;
    if (!set_bit(M.words + M.off[d], code >> (3 * s))) return;  // its ancestors are someone else's
    // lattice points at the far faces (the others come from k_oct_lattice)
    const uint32_t r = 1u << d, c[3] = {uint32_t(x >> s), uint32_t(y >> s), uint32_t(z >> s)};
    if (d >= 2 && (c[0] == r - 1 || c[1] == r - 1 || c[2] == r - 1)) {
      for (uint32_t j = 1; j < 8; ++j) {
        const uint32_t px = c[0] + (j & 1), py = c[1] + (j >> 1 & 1), pz = c[2] + (j >> 2);
        if (px == r || py == r || pz == r) set_bit(M.words + M.off[M.D + d - 1], lattice_bit(d, px, py, pz));
      }
    }
  }
}

// Lattice points below r on every axis: bit p of level l is set when one of
// the voxels p, p - (1,0,0), .. p - (1,1,1) of depth l + 1 is.  A word holds
// a block of 4 x 4 x 2 points (bits x0 y0 z0 x1 y1 of the index), the same
// block of voxels has the same word of the depth's bitmap, and along an axis
// the OR with the block moved up by one takes the block before it.
__device__ inline uint32_t grow_x(uint32_t w, uint32_t before) {
  return w | (w & 0x55555555u) << 1 | (w & 0x00aa00aau) << 7 | (before & 0xaa00aa00u) >> 9;
}
__device__ inline uint32_t grow_y(uint32_t w, uint32_t before) {
  return w | (w & 0x33333333u) << 2 | (w & 0x0000ccccu) << 14 | (before & 0xcccc0000u) >> 18;
}
__device__ inline uint32_t grow_z(uint32_t w, uint32_t before) {
  return w | (w & 0x0f0f0f0fu) << 4 | (before & 0xf0f0f0f0u) >> 4;
}

// Blocks of the corner segments, a thread per word; bound by its eight reads
// (in cache: neighbouring words are near in Morton order).
static __global__ __launch_bounds__(kBlock) void k_oct_lattice(OctMaps M) {
  const uint32_t w = M.off[M.D + 1] + blockIdx.x * kBlock + threadIdx.x;
  const int s = M.segment(w / kOctWords);
  const int d = s - M.D + 1;  // depth of the level's voxels
  const uint32_t at = w - M.off[s];
  if (at >= 1u << (3 * d - 5)) return;
  const uint32_t x = compact3_u32(at << 5), y = compact3_u32(at << 4), z = compact3_u32(at << 3);
  const uint32_t* vox = M.words + M.off[d];
  uint32_t n[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const bool in = (!(j & 1) || x >= 4) && (!(j & 2) || y >= 4) && (!(j & 4) || z >= 2);
    n[j] = in ? vox[morton3_u32(x - 4 * (j & 1), y - 4 * (j >> 1 & 1), z - 2 * (j >> 2)) >> 5] : 0u;
  }
  const uint32_t a0 = grow_y(grow_x(n[0], n[1]), grow_x(n[2], n[3])), a1 = grow_y(grow_x(n[4], n[5]), grow_x(n[6], n[7]));
  M.words[w] = grow_z(a0, a1);
}

// Sum of v over the block's threads, in every thread.  `part`: 4 words.
__device__ inline uint32_t block_sum(uint32_t v, uint32_t* part) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
  __syncthreads();
  return part[0] + part[1] + part[2] + part[3];
}

// Exclusive sum of v over the block's threads in order; *total = the sum.
__device__ inline uint32_t block_scan(uint32_t v, uint32_t* part, uint32_t* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  __syncthreads();
  if (lane == 63) part[w] = x;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int q = 0; q < kBlock / 64; ++q) {
    if (q < w) before += part[q];
    all += part[q];
  }
  *total = all;
  return before + x - v;
}

// Sum of a[first, end) by the whole block.
__device__ inline uint32_t block_range_sum(const uint32_t* a, uint32_t first, uint32_t end, uint32_t* part) {
  uint32_t v = 0;
  for (uint32_t i = first + threadIdx.x; i < end; i += kBlock) v += a[i];
  return block_sum(v, part);
}

static __global__ __launch_bounds__(kBlock) void k_oct_sums(OctMaps M) {
  __shared__ uint32_t part[kBlock / 64];
  const uint4 v = reinterpret_cast<const uint4*>(M.words + blockIdx.x * kOctWords)[threadIdx.x];
  const uint32_t s = block_sum(uint32_t(__popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w)), part);
  if (threadIdx.x == 0) M.bsum[blockIdx.x] = s;
}

static __global__ __launch_bounds__(kBlock) void k_oct_prefix(OctMaps M, int64_t* nvox, int64_t* ncorner) {
  __shared__ uint32_t part[kBlock / 64];
  const uint32_t b = blockIdx.x;
  const int s = M.segment(b);
  const uint32_t base = block_range_sum(M.bsum, M.off[s] / kOctWords, b, part);
  const uint4 v = reinterpret_cast<const uint4*>(M.words + b * kOctWords)[threadIdx.x];
  const uint32_t c[4] = {uint32_t(__popc(v.x)), uint32_t(__popc(v.y)), uint32_t(__popc(v.z)), uint32_t(__popc(v.w))};
  uint32_t total;
  const uint32_t p = base + block_scan(c[0] + c[1] + c[2] + c[3], part, &total);
  reinterpret_cast<uint4*>(M.pre + b * kOctWords)[threadIdx.x] =
      make_uint4(p, p + c[0], p + c[0] + c[1], p + c[0] + c[1] + c[2]);
  if (threadIdx.x == 0 && (b + 1) * kOctWords == M.off[s + 1]) {
    if (s <= M.D) nvox[s] = int64_t(base + total);
    else ncorner[s - M.D - 1] = int64_t(base + total);
  }
}

// The set bits of kBlock words from `words` as word << 5 | bit, in order;
// returns their number.
__device__ inline uint32_t expand_bits(const uint32_t* words, uint16_t* list, uint32_t* part) {
  uint32_t w = words[threadIdx.x], n;
  uint32_t at = block_scan(uint32_t(__popc(w)), part, &n);
  while (w) {
    list[at++] = uint16_t(threadIdx.x << 5 | uint32_t(__ffs(w) - 1));
    w &= w - 1u;
  }
  __syncthreads();
  return n;
}

// The voxels around the lattice point p (coordinates 0..r) of level l, depth
// l + 1: bit j of the result is set when the voxel that has p as its corner
// slot j exists.
__device__ inline uint32_t voxels_around(const OctMaps& M, int depth, const uint32_t p[3], uint32_t code[8]) {
  const uint32_t r = 1u << depth;
  uint32_t w[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const uint32_t x = p[0] - (j & 1), y = p[1] - (j >> 1 & 1), z = p[2] - (j >> 2);
    const bool in = x < r && y < r && z < r;  // below 0 wraps above r
    code[j] = in ? morton3_u32(x, y, z) : 0u;
    w[j] = in ? M.words[M.off[depth] + (code[j] >> 5)] : 0u;
  }
  uint32_t mask = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) mask |= (w[j] >> (code[j] & 31u) & 1u) << j;
  return mask;
}

// A block takes kBlock words.
static __global__ __launch_bounds__(kBlock) void k_oct_emit(OctMaps M, ngl_octree_device O) {
  __shared__ uint32_t part[kBlock / 64];
  __shared__ uint16_t list[kBlock * 32];
  const uint32_t w0 = blockIdx.x * kBlock;
  const int s = M.segment(w0 / kOctWords);
  const uint32_t n = expand_bits(M.words + w0, list, part);
  const uint32_t first = M.pre[w0], bit0 = (w0 - M.off[s]) << 5;
  uint32_t pairs = 0;
  for (uint32_t i = threadIdx.x; i < n; i += kBlock) {
    const uint32_t c = bit0 + list[i];
    if (s > M.D) {
      uint32_t p[3], code[8];
      lattice_point(s - M.D + 1, c, p);
      pairs += uint32_t(__popc(voxels_around(M, s - M.D + 1, p, code)));
      continue;
    }
    const uint32_t v = first + i;
    O.cell[s][v] = compact3_u32(c) | compact3_u32(c >> 1) << 10 | compact3_u32(c >> 2) << 20;
    if (s > 0) O.parent[s][v] = int32_t(M.rank(s - 1, c >> 3));
    if (s < M.D) {
      O.child_mask[s][v] = uint8_t(M.words[M.off[s + 1] + (c >> 2)] >> (8u * (c & 3u)));
      O.first_child[s][v] = int32_t(M.rank(s + 1, 8u * c));
    } else {
      if (O.child_mask[s]) O.child_mask[s][v] = 0;
      if (O.first_child[s]) O.first_child[s][v] = -1;
    }
  }
  if (s <= M.D) return;
  const uint32_t all = block_sum(pairs, part);
  if (threadIdx.x == 0) M.dsum[blockIdx.x] = all;
}

// Blocks of the corner segments.
static __global__ __launch_bounds__(kBlock) void k_oct_corners(OctMaps M, ngl_octree_device O) {
  __shared__ uint32_t part[kBlock / 64];
  __shared__ uint16_t list[kBlock * 32];
  const uint32_t b = M.off[M.D + 1] / kBlock + blockIdx.x, w0 = b * kBlock;
  const int s = M.segment(w0 / kOctWords);
  const int l = s - M.D, depth = l + 1;
  int32_t* adj_off = O.corner_adj_off[l - 1];
  int32_t* adj = O.corner_adj[l - 1];
  if (w0 == M.off[s] && threadIdx.x == 0 && adj_off) adj_off[O.ncorner[l - 1]] = int32_t(8 * O.nvox[depth]);
  const uint32_t n = expand_bits(M.words + w0, list, part);
  if (n == 0) return;
  uint32_t at = block_range_sum(M.dsum, M.off[s] / kBlock, b, part);  // pairs at the corners before
  const uint32_t first = M.pre[w0], bit0 = (w0 - M.off[s]) << 5;
  for (uint32_t i0 = 0; i0 < n; i0 += kBlock) {
    const uint32_t i = i0 + threadIdx.x;
    uint32_t e[8], deg = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) e[j] = 0xffffffffu;
    if (i < n) {
      const uint32_t c = first + i;
      uint32_t p[3], code[8];
      lattice_point(depth, bit0 + list[i], p);
      const uint32_t mask = voxels_around(M, depth, p, code);
      deg = uint32_t(__popc(mask));
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (mask >> j & 1u) {
          e[j] = 8u * M.rank(depth, code[j]) + uint32_t(j);
          O.corners[l - 1][e[j]] = int32_t(c);
        }
      if (O.corner_cell[l - 1]) {
#pragma unroll
        for (int a = 0; a < 3; ++a) O.corner_cell[l - 1][3 * size_t(c) + a] = int32_t(p[a]);
      }
    }
    uint32_t chunk;
    const uint32_t o = at + block_scan(deg, part, &chunk);
    if (adj && i < n) {
      adj_off[first + i] = int32_t(o);
      // ascending: odd-even transposition of the eight
#pragma unroll
      for (int round = 0; round < 8; ++round)
#pragma unroll
        for (int j = round & 1; j + 1 < 8; j += 2) {
          const uint32_t lo = min(e[j], e[j + 1]), hi = max(e[j], e[j + 1]);
          e[j] = lo, e[j + 1] = hi;
        }
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (uint32_t(j) < deg) adj[o + j] = int32_t(e[j]);
    }
    at += chunk;
  }
}

// Bitmaps and sums in the workspace (sizes depend on the levels alone).
static size_t oct_carve(void* base, int L, OctMaps* M) {
  const int D = L + 1;
  M->D = D;
  M->L = L;
  uint64_t w = 0;
  auto add = [&](int s, uint64_t bits) {
    M->off[s] = uint32_t(w);
    w += (bits + 32 * kOctWords - 1) / (32 * kOctWords) * kOctWords;
  };
  for (int d = 0; d <= D; ++d) add(d, uint64_t(1) << (3 * d));
  for (int l = 1; l <= L; ++l) {
    const uint64_t r = (uint64_t(1) << (l + 1)) + 1;
    add(D + l, r * r * r);
  }
  M->off[D + L + 1] = uint32_t(w);
  char* p = static_cast<char*>(base);
  size_t off = 0;
  auto take = [&](size_t b) {
    char* r = p ? p + off : nullptr;
    off += (b + 255) & ~size_t(255);
    return reinterpret_cast<uint32_t*>(r);
  };
  M->words = take(4 * size_t(w));
  M->pre = take(4 * size_t(w));
  M->bsum = take(4 * size_t(w / kOctWords));
  M->dsum = take(4 * size_t(w / kBlock));
  return off;
}

}  // namespace ngl

extern "C" {

int ngl_octree_build_device_workspace(int64_t n, int32_t num_lods, size_t* bytes) {
  NGL_REQUIRE(bytes != nullptr && n >= 0 && n < (int64_t(1) << 28), "bad arguments");
  NGL_REQUIRE(num_lods >= 1 && num_lods <= NGL_MAX_LODS, "num_lods %d outside 1..%d", num_lods, NGL_MAX_LODS);
  ngl::OctMaps M;
  *bytes = ngl::oct_carve(nullptr, num_lods, &M);
  return NGL_OK;
}

int ngl_octree_build_device(const int32_t* ijk, int64_t n, int32_t num_lods, const ngl_octree_device* out,
                            void* ws, size_t ws_bytes, void* stream) {
  using namespace ngl;
  NGL_REQUIRE(out != nullptr, "output struct is null");
  NGL_REQUIRE(n >= 0 && n < (int64_t(1) << 28), "cell count out of range");
  NGL_REQUIRE(num_lods >= 1 && num_lods <= NGL_MAX_LODS, "num_lods %d outside 1..%d", num_lods, NGL_MAX_LODS);
  NGL_REQUIRE(n == 0 || ijk != nullptr, "ijk is null");
  const int L = num_lods, D = L + 1;
  OctMaps M;
  const size_t need = oct_carve(ws, L, &M);
  NGL_REQUIRE(ws != nullptr && ws_bytes >= need, "workspace too small: %zu < %zu bytes", ws_bytes, need);
  NGL_REQUIRE(out->nvox && out->ncorner && out->bad, "count arrays are null");
  for (int d = 0; d <= D; ++d) {
    NGL_REQUIRE(out->cell[d] && out->parent[d], "cell or parent array of depth %d is null", d);
    if (d < D) NGL_REQUIRE(out->child_mask[d] && out->first_child[d], "child arrays of depth %d are null", d);
  }
  for (int l = 1; l <= L; ++l)
    NGL_REQUIRE((out->corner_adj_off[l - 1] == nullptr) == (out->corner_adj[l - 1] == nullptr),
                "corner adjacency of level %d needs both arrays or neither", l);
  for (int l = 1; l <= L; ++l) NGL_REQUIRE(out->corners[l - 1], "corners of level %d are null", l);
  hipStream_t s = (hipStream_t)stream;
  const uint32_t words = M.off[D + L + 1], blocks = words / kOctWords;
  k_oct_clear<<<(words / 4 + kBlock - 1) / kBlock, kBlock, 0, s>>>(reinterpret_cast<uint4*>(M.words), words / 4,
                                                                   out->bad, out->parent[0]);
  if (n > 0) k_oct_mark<<<unsigned((n + kBlock - 1) / kBlock), kBlock, 0, s>>>(ijk, n, M, out->bad);
  const uint32_t corner_words = words - M.off[D + 1];
  k_oct_lattice<<<corner_words / kBlock, kBlock, 0, s>>>(M);
  k_oct_sums<<<blocks, kBlock, 0, s>>>(M);
  k_oct_prefix<<<blocks, kBlock, 0, s>>>(M, out->nvox, out->ncorner);
  k_oct_emit<<<words / kBlock, kBlock, 0, s>>>(M, *out);
  k_oct_corners<<<corner_words / kBlock, kBlock, 0, s>>>(M, *out);
  NGL_LAUNCHED();
  return NGL_OK;
}

}  // extern "C"
