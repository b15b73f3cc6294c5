// Octree construction on the GPU (the host build of Sec. 2.1 moved to the
// device), bit-identical to the host build: the same 63-bit Morton keys from
// the same FP64 grid arithmetic, a stable radix sort (ties by input index),
// the same breadth-first cell order, and FP64 boxes and
// moments bottom-up with the host's operation order (no contraction, the
// host's min / max), so every exported array matches bitwise.
//
// Subdivision: which cells start at a particle follows from the sorted keys
// around it (level_range), so all levels are numbered by one scan and written
// by one kernel.  Boxes and moments: one thread per leaf, then eight lanes per
// inner cell, deepest level first.  Then the FP32 images, the walk records, the
// learned criterion's cell features, the groups (scattered to their first
// particle and compacted, which orders them by first particle) and the work
// chunks.
#include <hip/hip_runtime.h>

#include <cstddef>
#include <hipcub/hipcub.hpp>

#include <cmath>
#include <cstring>
#include <type_traits>
#include <vector>

#include "cell_numbers.h"
#include "device_common.h"
#include "octgrav_internal.h"

namespace octgrav {
namespace {

constexpr uint32_t kGridMax = (1u << kMaxDepth) - 1;
constexpr int kT = 256;

inline int blocks(int64_t n) { return (int)((n + kT - 1) / kT); }

// Bounding box: per-block min / max of each coordinate (FP32 values are
// exact in FP64, so the order of the reduction does not matter).
// With mass != nullptr (inputs already on the device) it also checks them in
// the same pass: bit 1 of *bad = a position not finite or |x| >= 2^60, bit 2
// = a mass not finite or not > 0.
__global__ void bbox_kernel(const float* __restrict__ pos, const float* __restrict__ mass,
                            int64_t n, float* __restrict__ part, int32_t* __restrict__ bad) {
  __shared__ float sh[6][kT];
  // min / max with the host's tie rule (keeps the earlier of equal values,
  // so +0 / -0 resolve as they do on the host)
  float v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
  int bd = 0;
  for (int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kT) {
    for (int k = 0; k < 3; ++k) {
      const float x = pos[3 * i + k];
      v[k] = x < v[k] ? x : v[k];
      v[3 + k] = v[3 + k] < x ? x : v[3 + k];
      if (!(fabsf(x) < 0x1p60f)) bd |= 1;  // also catches NaN
    }
    if (mass) {
      const float m = mass[i];
      if (!(m > 0.0f) || !(m < INFINITY)) bd |= 2;
    }
  }
  if (mass) {
    if (__any(bd & 1) && (threadIdx.x & 63) == 0) atomicOr(bad, 1);
    if (__any(bd & 2) && (threadIdx.x & 63) == 0) atomicOr(bad, 2);
  }
  for (int k = 0; k < 6; ++k) sh[k][threadIdx.x] = v[k];
  __syncthreads();
  for (int o = kT / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o)
      for (int k = 0; k < 6; ++k) {
        const float a = sh[k][threadIdx.x], b = sh[k][threadIdx.x + o];
        sh[k][threadIdx.x] = k < 3 ? (b < a ? b : a) : (a < b ? b : a);
      }
    __syncthreads();
  }
  if (threadIdx.x < 6) part[6 * blockIdx.x + threadIdx.x] = sh[threadIdx.x][0];
}

// The host's root cube of a bounding box (FP64, the same operations): cube =
// corner xyz, side, grid step, 1 / step.
__device__ void root_cube_of(const double lo[3], const double hi[3], double* __restrict__ cube) {
#pragma clang fp contract(off)
  const double e1 = hi[1] - lo[1], e2 = hi[2] - lo[2], e0 = hi[0] - lo[0];
  const double e12 = e1 < e2 ? e2 : e1;
  const double ext = e0 < e12 ? e12 : e0;
  int e = 1;
  if (ext > 0) (void)frexp(ext, &e);
  const double side = ext > 0 ? ldexp(1.0, e) : 1.0;
  for (int k = 0; k < 3; ++k) cube[k] = (lo[k] + hi[k]) * 0.5 - 0.5 * side;
  cube[3] = side;
  cube[4] = ldexp(side, -kMaxDepth);
  cube[5] = ldexp(1.0 / side, kMaxDepth);
}

// Root cube from the bounding-box partials with the host's rules (min / max
// keeping the earlier of equal values, combined over contiguous ranges in
// index order; the cube of the largest extent rounded up to a power of two,
// centred on the box; FP64, the same operations): cube = corner xyz, side,
// grid step, 1 / step.  One block of kT threads.
__global__ __launch_bounds__(kT) void root_kernel(const float* __restrict__ part, int nbb,
                                                  double* __restrict__ cube) {
#pragma clang fp contract(off)
  __shared__ float sh[6][kT];
  const int t = threadIdx.x, per = (nbb + kT - 1) / kT;
  float v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
  for (int i = t * per; i < min(nbb, (t + 1) * per); ++i)
    for (int k = 0; k < 3; ++k) {
      const float x = part[6 * i + k], y = part[6 * i + 3 + k];
      v[k] = x < v[k] ? x : v[k];
      v[3 + k] = v[3 + k] < y ? y : v[3 + k];
    }
  for (int k = 0; k < 6; ++k) sh[k][t] = v[k];
  __syncthreads();
  for (int w = 1; w < kT; w <<= 1) {  // thread t holds [t, t + 2w) after this step
    if ((t & (2 * w - 1)) == 0)
      for (int k = 0; k < 6; ++k) {
        const float a = sh[k][t], b = sh[k][t + w];
        sh[k][t] = k < 3 ? (b < a ? b : a) : (a < b ? b : a);
      }
    __syncthreads();
  }
  if (t != 0) return;
  double lo[3], hi[3];
  for (int k = 0; k < 3; ++k) {
    lo[k] = sh[k][0];
    hi[k] = sh[3 + k][0];
  }
  root_cube_of(lo, hi, cube);
}

// The host's grid coordinate: floor, then exact against the grid planes.
__device__ __forceinline__ uint32_t grid_coord(double x, double corner, double step,
                                               double inv_step) {
#pragma clang fp contract(off)
  const double f = floor((x - corner) * inv_step);
  int64_t u = f < 0 ? 0 : (f > (double)kGridMax ? (int64_t)kGridMax : (int64_t)f);
  while (u > 0 && corner + (double)u * step > x) --u;
  while (u < (int64_t)kGridMax && corner + (double)(u + 1) * step <= x) ++u;
  return (uint32_t)u;
}

__device__ __forceinline__ uint64_t spread3(uint32_t v) {
  uint64_t x = v & 0x1fffff;
  x = (x | x << 32) & 0x1f00000000ffffull;
  x = (x | x << 16) & 0x1f0000ff0000ffull;
  x = (x | x << 8) & 0x100f00f00f00f00full;
  x = (x | x << 4) & 0x10c30c30c30c30c3ull;
  x = (x | x << 2) & 0x1249249249249249ull;
  return x;
}

// cube: corner xyz, side, grid step, 1 / step (root_cube_of).
__device__ __forceinline__ uint64_t particle_key(float x, float y, float z, const double* cube) {
  const double step = cube[4], inv = cube[5];
  const uint32_t u0 = grid_coord((double)x, cube[0], step, inv);
  const uint32_t u1 = grid_coord((double)y, cube[1], step, inv);
  const uint32_t u2 = grid_coord((double)z, cube[2], step, inv);
  return spread3(u0) | spread3(u1) << 1 | spread3(u2) << 2;
}

// Also packs each particle as (x, y, z, m) in input order, so that the gather
// after the sort reads one aligned 16-byte record per particle.
__global__ void keys_kernel(const float* __restrict__ pos, const float* __restrict__ mass,
                            int64_t n, const double* __restrict__ cube,
                            uint64_t* __restrict__ key, int32_t* __restrict__ idx,
                            float4* __restrict__ packed) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i >= n) return;
  const float x = pos[3 * i], y = pos[3 * i + 1], z = pos[3 * i + 2];
  key[i] = particle_key(x, y, z, cube);
  idx[i] = (int32_t)i;
  packed[i] = make_float4(x, y, z, mass[i]);
}

struct Cells {
  int32_t* first;   // first particle
  int32_t* n;       // particles
  int32_t* depth;
  int32_t* parent;
  int32_t* fc;      // first child (-1)
  int32_t* nc;      // children
};

// ---- subdivision.  A cell of level L (the particles that share L octant
// digits) exists if its parent holds more than n_leaf particles.  For particle
// i let lcp be the number of digits it shares with particle i - 1, and D the
// deepest level at which the cell around it holds more than n_leaf: n_leaf + 1
// consecutive keys share D digits, so D is the maximum, over the windows of
// n_leaf + 1 keys that contain i, of the digits shared by the window's ends.
// Then the cells that start at i are those of levels lcp + 1 ... D + 1, the
// last of them a leaf.  Counting starts level by level in particle order is
// the breadth-first numbering; the parent of a cell is the last start of the
// level above, and the first child of a split cell the next level's cell that
// starts with it.  (Level by level, two launches each, this was 125 us of a
// rebuild of 262144 particles; count, scan and write are 20, with fewer gaps.
// Whole rebuild, before and now, us: 16384 263 / 173, 65536 297 / 214, 262144
// 394 / 300, 1M 655 / 527.)
constexpr int kMaxLeaf = 64;            // largest n_leaf
constexpr int kLevels = kMaxDepth + 1;  // levels 0 ... kMaxDepth
constexpr int kST = 1024;               // particles, and threads, per block
constexpr int kSW = kST / 64;

// Octant digits shared by two keys (63 bits: the top bit is clear).
__device__ __forceinline__ int shared_digits(uint64_t a, uint64_t b) {
  const uint64_t x = a ^ b;
  return x == 0 ? kMaxDepth : (__clzll((long long)x) - 1) / 3;
}

// Digits shared by the ends of the window of n_leaf + 1 keys that starts at j
// (-1: no such window).
__device__ __forceinline__ int8_t window_digits(const uint64_t* key, int64_t n, int n_leaf,
                                                int64_t j) {
  return j >= 0 && j + n_leaf < n ? (int8_t)shared_digits(key[j], key[j + n_leaf]) : (int8_t)-1;
}

// out[e]: the maximum of the 2 run windows from e on, from those of run windows
// (len entries, a block of kST threads).
__device__ __forceinline__ void join_windows(const int8_t* in, int8_t* out, int len, int run) {
  for (int e = threadIdx.x; e < len; e += kST) out[e] = max(in[e], in[e + run < len ? e + run : e]);
}

// The levels of the cells that start at a particle: lo ... hi (none if lo > hi).
struct LevelRange {
  int lo, hi;
};
__device__ __forceinline__ LevelRange level_range(const uint64_t* key, int64_t i, int D) {
  return LevelRange{i > 0 ? shared_digits(key[i - 1], key[i]) + 1 : 0, min(D + 1, kMaxDepth)};
}

// Starts of each level among the wave's particles, to row[L * stride].
__device__ __forceinline__ void count_starts(LevelRange r, int* row, int stride) {
  const int lane = threadIdx.x & 63;
  int v = 0;
  const int hi = r.lo <= r.hi ? r.hi : -1;
  for (int L = 0; L < kLevels && __any(L <= hi); ++L) {
    const int k = __popcll(__ballot(r.lo <= L && L <= hi));
    if (lane == L) v = k;
  }
  if (lane < kLevels) row[lane * stride] = v;
}

// Writes the cells that start at the wave's particles (this lane's: i), as
// far as they fit cap <= kMaxCells cells; row[L * stride]: the number of the
// wave's first cell of level L.  Particle and child counts of split cells follow later
// (close_parent, inner_moments).
__device__ __forceinline__ void write_cells(const Cells& C, const uint64_t* key, int32_t n,
                                            int32_t i, LevelRange r, int n_leaf, int64_t cap,
                                            const int* row, int stride) {
  int32_t up = 0, up_end = 0;  // of the level above: this lane's cell, cells up to and with it
  int32_t leaf = -1;
  for (int L = 0; L < kLevels; ++L) {
    if (!__any(r.lo <= r.hi && L <= r.hi)) break;
    const bool m = r.lo <= L && L <= r.hi;
    const uint64_t b = __ballot(m);
    const int32_t c = row[L * stride] +
                      (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0));
    if (m && c < cap) {
      C.first[c] = i;
      C.depth[c] = L;
      C.parent[c] = up_end - 1;
      if (L == r.hi) leaf = c;
    }
    if (m && L > r.lo && up < cap) C.fc[up] = c;
    up = c;
    up_end = c + m;
  }
  if (leaf < 0) return;
  int32_t l = i + 1, h = r.hi == kMaxDepth || n - i <= n_leaf ? n : i + n_leaf;
  const int sh = 3 * (kMaxDepth - r.hi);
  const uint64_t k = key[i] >> sh;
  while (l < h) {
    const int32_t mid = l + ((h - l) >> 1);
    if (key[mid] >> sh == k) l = mid + 1;
    else h = mid;
  }
  C.n[leaf] = l - i;
  C.fc[leaf] = -1;
  C.nc[leaf] = 0;
}

// Number of children of the parent of cell c (of nc), written by the last child.
__device__ __forceinline__ void close_parent(const Cells& C, int64_t c, int64_t nc) {
  const int32_t p = C.parent[c];
  if (p >= 0 && (c + 1 == nc || C.parent[c + 1] != p)) C.nc[p] = (int32_t)(c + 1) - C.fc[p];
}

// Level ranges of the particles and each block's starts per level (cnt[L *
// gridDim.x + block]; a 0 behind the last).  Also clears the group marks.
template <typename Count>
__global__ __launch_bounds__(kST) void starts_kernel(const uint64_t* __restrict__ key, int64_t n,
                                                     int n_leaf, uchar2* __restrict__ range,
                                                     Count* __restrict__ cnt,
                                                     int32_t* __restrict__ group_at) {
  __shared__ int8_t sw[2][kST + kMaxLeaf];
  __shared__ int rows[kLevels][kSW];
  const int t = threadIdx.x;
  const int64_t i0 = (int64_t)blockIdx.x * kST, i = i0 + t;
  const int len = kST + n_leaf;
  for (int e = t; e < len; e += kST) sw[0][e] = window_digits(key, n, n_leaf, i0 - n_leaf + e);
  __syncthreads();
  int at = 0, run = 1;
  for (; 2 * run <= n_leaf + 1; run *= 2, at ^= 1) {
    join_windows(sw[at], sw[at ^ 1], len, run);
    __syncthreads();
  }
  const int D = max(sw[at][t], sw[at][t + n_leaf - run + 1]);
  LevelRange r{1, 0};
  if (i < n) {
    r = level_range(key, i, D);
    range[i] = make_uchar2((unsigned char)r.lo, (unsigned char)r.hi);
    group_at[i] = -1;
  }
  count_starts(r, &rows[0][t >> 6], kSW);
  __syncthreads();
  if (t < kLevels) {
    int k = 0;
    for (int v = 0; v < kSW; ++v) k += rows[t][v];
    cnt[(int64_t)t * gridDim.x + blockIdx.x] = k;
  }
  if (t == 0 && blockIdx.x == 0) cnt[(int64_t)kLevels * gridDim.x] = 0;
}

// The cells, numbered by the counts; block 0 records where each level begins.
// SCANNED: sums holds the scan of the counts (CellSum); otherwise the counts, of
// which every block adds up those before its own, a wave per level (at most
// kOwnScan blocks, so 22 * 2^20 cells: two launches less, rebuilds of 16384 and
// 262144 particles 153 -> 136 and 222 -> 193 us together with the groups' two
// launches below).
constexpr int kOwnScan = 1024;
template <bool SCANNED>
using StartCount = std::conditional_t<SCANNED, CellSum, int32_t>;
template <bool SCANNED>
__global__ __launch_bounds__(kST) void cells_kernel(Cells C, const uint64_t* __restrict__ key,
                                                    int32_t n, int n_leaf,
                                                    const uchar2* __restrict__ range,
                                                    const StartCount<SCANNED>* __restrict__ sums,
                                                    int64_t cap, int64_t* __restrict__ level) {
  __shared__ int rows[kLevels][kSW];
  __shared__ int all[kLevels + 1], before[kLevels];
  const int t = threadIdx.x, nb = (int)gridDim.x, blk = (int)blockIdx.x;
  const int64_t i = (int64_t)blk * kST + t;
  LevelRange r{1, 0};
  if (i < n) {
    const uchar2 v = range[i];
    r = LevelRange{v.x, v.y};
  }
  count_starts(r, &rows[0][t >> 6], kSW);
  if constexpr (!SCANNED) {
    for (int L = t >> 6; L < kLevels; L += kSW) {
      int a = 0, b = 0;
      for (int k = t & 63; k < nb; k += 64) {
        const int v = sums[L * nb + k];
        a += v;
        b += k < blk ? v : 0;
      }
      for (int o = 32; o > 0; o >>= 1) {
        a += __shfl_xor(a, o);
        b += __shfl_xor(b, o);
      }
      if ((t & 63) == 0) {
        all[L] = a;
        before[L] = b;
      }
    }
  }
  __syncthreads();
  if (t <= kLevels) {
    StartCount<SCANNED> begin = 0;  // the level's first cell
    if constexpr (SCANNED) begin = sums[(int64_t)t * nb];
    else
      for (int L = 0; L < t; ++L) begin += all[L];
    if (blk == 0) level[t] = begin;
    if (t < kLevels) {
      int at;
      if constexpr (SCANNED) at = cell_number(sums[(int64_t)t * nb + blk]);
      else at = begin + before[t];
      for (int v = 0; v < kSW; ++v) {
        const int k = rows[t][v];
        rows[t][v] = at;
        at += k;
      }
    }
  }
  __syncthreads();
  write_cells(C, key, n, (int32_t)i, r, n_leaf, cap, &rows[0][t >> 6], kSW);
}

// Sum of v over the block (kT threads); every thread gets it.
__device__ int block_sum(int v, int* sh) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  int t = 0;
  for (int k = 0; k < kT / 64; ++k) t += sh[k];
  __syncthreads();
  return t;
}

__global__ void gather_kernel(const float4* __restrict__ packed, const int32_t* __restrict__ perm,
                              int64_t n, float4* __restrict__ part, int32_t* __restrict__ iperm) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i >= n) return;
  const int32_t p = perm[i];
  part[i] = packed[p];
  iperm[p] = (int32_t)i;
}

// The host's std::min / std::max on doubles.
__device__ __forceinline__ double hmin(double a, double b) { return b < a ? b : a; }
__device__ __forceinline__ double hmax(double a, double b) { return a < b ? b : a; }

// Box and FP64 moments of leaf c (nothing if it has children), as the host
// computes them.  The loads of its particles (kMomChunk at a time) are issued
// before their sums, so a leaf costs a few memory round trips instead of one
// per particle.  The sums keep the host's order; a slot past the end repeats
// the last particle with weight +0, which leaves every sum and the box
// unchanged bit for bit (the sums start at +0 and the inputs are finite).
constexpr int kMomChunk = 16;
__device__ __forceinline__ void leaf_moments(const Cells& C, const float4* __restrict__ part,
                                             int64_t c, double* __restrict__ box,
                                             double* __restrict__ mp64) {
#pragma clang fp contract(off)
  if (C.fc[c] >= 0) return;
  double bx[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
  double M = 0, sx = 0, sy = 0, sz = 0;
  double Q[6] = {0, 0, 0, 0, 0, 0};
  const int32_t f = C.first[c], e = f + C.n[c];
  for (int32_t i0 = f; i0 < e; i0 += kMomChunk) {
    float4 pb[kMomChunk];
#pragma unroll
    for (int k = 0; k < kMomChunk; ++k) pb[k] = part[i0 + k < e ? i0 + k : e - 1];
#pragma unroll
    for (int k = 0; k < kMomChunk; ++k) {
      const double x[3] = {pb[k].x, pb[k].y, pb[k].z};
      for (int d = 0; d < 3; ++d) {
        bx[d] = hmin(bx[d], x[d]);
        bx[3 + d] = hmax(bx[3 + d], x[d]);
      }
      const double w = i0 + k < e ? (double)pb[k].w : 0.0;
      M += w;
      sx += w * x[0];
      sy += w * x[1];
      sz += w * x[2];
    }
  }
  const double com[3] = {sx / M, sy / M, sz / M};
  for (int32_t i0 = f; i0 < e; i0 += kMomChunk) {
    float4 pb[kMomChunk];
#pragma unroll
    for (int k = 0; k < kMomChunk; ++k) pb[k] = part[i0 + k < e ? i0 + k : e - 1];
#pragma unroll
    for (int k = 0; k < kMomChunk; ++k) {
      const float4 p = pb[k];
      const double d0 = p.x - com[0], d1 = p.y - com[1], d2 = p.z - com[2];
      const double w = i0 + k < e ? (double)p.w : 0.0;
      const double r2 = d0 * d0 + d1 * d1 + d2 * d2;
      Q[0] += w * (3 * d0 * d0 - r2);
      Q[1] += w * (3 * d1 * d1 - r2);
      Q[2] += w * (3 * d2 * d2 - r2);
      Q[3] += w * 3 * d0 * d1;
      Q[4] += w * 3 * d0 * d2;
      Q[5] += w * 3 * d1 * d2;
    }
  }
  double* o = box + 6 * c;
  for (int k = 0; k < 6; ++k) o[k] = bx[k];
  double* q = mp64 + 10 * c;
  q[0] = M;
  for (int k = 0; k < 3; ++k) q[1 + k] = com[k];
  for (int k = 0; k < 6; ++k) q[4 + k] = Q[k];
}

// Every leaf (leaves need only their particles) and every parent's number of
// children, one thread per cell.
__global__ __launch_bounds__(kT) void leaf_moments_kernel(Cells C, const float4* __restrict__ part,
                                                          int64_t nc, double* __restrict__ box,
                                                          double* __restrict__ mp64) {
  const int64_t c = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (c >= nc) return;
  close_parent(C, c, nc);
  leaf_moments(C, part, c, box, mp64);
}

// Lane K of each group of eight lanes (the LDS crossbar's bit-mask mode).
template <int K>
__device__ __forceinline__ double of_lane8(double v) {
  constexpr int m = K << 5 | 0x18;
  return __hiloint2double(__builtin_amdgcn_ds_swizzle(__double2hiint(v), m),
                          __builtin_amdgcn_ds_swizzle(__double2loint(v), m));
}

// Box, FP64 moments and particle count of cell c from its children's (nothing
// if it is a leaf, or !valid), by the eight lanes of a group, which all come
// here with the same c.  Lane d loads child d, so the children arrive in one
// memory latency, and forms its terms; the terms change places through LDS so
// that lane d then folds quantity d over the children in their order, as the
// host does (a box's upper side as the minimum of the negated sides, which
// picks the same values).  A lane without a child has terms +0 and infinity,
// which leave every sum and side unchanged bit for bit.  One thread per cell, four children at
// a time, took four latencies and the serial chains of ten quantities: 6.9 us a
// level of 262144 particles' tree, now 4.1, and 5003 particles in one block
// 121 -> 106 us a rebuild.  (With the terms exchanged by ds_swizzle, 176 a
// wave, the block was slower than one thread per cell.)
constexpr int kFoldRow = 66;  // 64 terms a quantity; rows start four banks apart
struct FoldBuf {
  double t[8][kFoldRow];
};
__device__ __forceinline__ double fold8(const FoldBuf& F, bool sum) {
#pragma clang fp contract(off)
  const double* t = &F.t[threadIdx.x & 7][threadIdx.x & 56];
  double v[8], s = sum ? 0.0 : (double)INFINITY;
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = t[k];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const double a = s + v[k], m = v[k] < s ? v[k] : s;
    s = sum ? a : m;
  }
  return s;
}
// The wave's LDS accesses before come before those after.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
__device__ __forceinline__ void inner_moments(const Cells& C, int64_t c, bool valid, FoldBuf& F,
                                              double* __restrict__ box,
                                              double* __restrict__ mp64) {
#pragma clang fp contract(off)
  const int d = threadIdx.x & 7, lane = threadIdx.x & 63;
  const int32_t f = valid ? C.fc[c] : -1;
  if (!__any(f >= 0)) return;
  const int nk = f >= 0 ? C.nc[c] : 0;
  const bool live = d < nk;
  const int64_t ch = live ? (int64_t)f + d : 0;
  double bx[6], q[10];
  for (int k = 0; k < 6; ++k) bx[k] = box[6 * ch + k];
  for (int k = 0; k < 10; ++k) q[k] = mp64[10 * ch + k];
  if (d == nk - 1) C.n[c] = C.first[ch] + C.n[ch] - C.first[c];
  const double w = live ? q[0] : 0.0;
  for (int k = 0; k < 6; ++k) bx[k] = live ? (k < 3 ? bx[k] : -bx[k]) : (double)INFINITY;
  F.t[0][lane] = w;
  for (int k = 1; k < 4; ++k) F.t[k][lane] = live ? w * q[k] : 0.0;
  for (int k = 0; k < 4; ++k) F.t[4 + k][lane] = bx[k];
  wave_lds_order();
  // M, the sums of m x, the lower sides and the first upper side
  double s = fold8(F, d < 4);
  const double M = of_lane8<0>(s);
  if (d > 0 && d < 4) s = s / M;
  const double com[3] = {of_lane8<1>(s), of_lane8<2>(s), of_lane8<3>(s)};
  if (nk > 0) *(d < 4 ? mp64 + 10 * c + d : box + 6 * c + (d - 4)) = d == 7 ? -s : s;
  const double d0 = q[1] - com[0], d1 = q[2] - com[1], d2 = q[3] - com[2];
  const double r2 = d0 * d0 + d1 * d1 + d2 * d2;
  const double Q[6] = {q[4] + w * (3 * d0 * d0 - r2), q[5] + w * (3 * d1 * d1 - r2),
                       q[6] + w * (3 * d2 * d2 - r2), q[7] + w * 3 * d0 * d1,
                       q[8] + w * 3 * d0 * d2,        q[9] + w * 3 * d1 * d2};
  wave_lds_order();
  for (int k = 0; k < 6; ++k) F.t[k][lane] = live ? Q[k] : 0.0;
  for (int k = 6; k < 8; ++k) F.t[k][lane] = bx[k - 2];
  wave_lds_order();
  s = fold8(F, d < 6);
  if (nk > 0) *(d < 6 ? mp64 + 10 * c + 4 + d : box + 6 * c + (d - 2)) = d < 6 ? s : -s;
  wave_lds_order();
}

// Cells [a, b) of one level, after the levels below it.
__global__ __launch_bounds__(kT) void inner_moments_kernel(Cells C, int64_t a, int64_t b,
                                                           double* __restrict__ box,
                                                           double* __restrict__ mp64) {
  __shared__ FoldBuf F[kT / 64];
  const int64_t c = a + ((int64_t)blockIdx.x * kT + threadIdx.x) / 8;
  inner_moments(C, c, c < b, F[threadIdx.x >> 6], box, mp64);
}

// Levels L ... 0, of at most kTopCells cells each, by one block: B.at[L] ...
// B.at[L + 1] are level L's cells.  (16384 and 262144 particles: 151 and 273 us
// a rebuild, without it 157 and 281, with levels of up to 1024 cells 163 and 281.)
constexpr int kTopCells = 128, kTopT = 1024;
struct LevelBegin {
  int32_t at[kLevels + 1];
};
__global__ __launch_bounds__(kTopT) void top_moments_kernel(Cells C, LevelBegin B, int L,
                                                            double* box, double* mp64) {
  __shared__ FoldBuf F[kTopT / 64];
  for (; L >= 0; --L) {
    for (int base = B.at[L]; base < B.at[L + 1]; base += kTopT / 8) {
      const int c = base + (int)threadIdx.x / 8;
      inner_moments(C, c, c < B.at[L + 1], F[threadIdx.x >> 6], box, mp64);
    }
    __syncthreads();
  }
}

// Arrays of FP32 images per cell (images_kernel).
struct Images {
  int4* topo;
  float4 *geo_host, *geo, *wrec, *mp, *fcell;
  int32_t* depth;
};

// FP32 images of one cell: topology, boundary (centre of the tight box, side =
// largest extent; the device copy carries the leaf flag in the side's sign
// bit), walk record, moments, depth, and the learned criterion's cell
// features with the host's FP32 expressions.
__device__ __forceinline__ void cell_image(const Cells& C, int64_t c, const double* __restrict__ box,
                                           const double* __restrict__ mp64, const Images& I) {
#pragma clang fp contract(off)
  const int4 tp = make_int4(C.fc[c], C.nc[c], C.first[c], C.n[c]);
  I.topo[c] = tp;
  const int32_t dc = C.depth[c];
  I.depth[c] = dc;
  const double* bx = box + 6 * c;
  double l = 0;
  float g[3];
  for (int k = 0; k < 3; ++k) {
    g[k] = (float)((bx[k] + bx[3 + k]) * 0.5);
    l = hmax(l, bx[3 + k] - bx[k]);
  }
  const float lf = (float)l;
  I.geo_host[c] = make_float4(g[0], g[1], g[2], lf);
  const float4 gd = make_float4(g[0], g[1], g[2], tp.y == 0 ? -lf : lf);
  I.geo[c] = gd;
  I.wrec[2 * c] = gd;
  I.wrec[2 * c + 1] = make_float4(__int_as_float(tp.x), __int_as_float(tp.y), __int_as_float(tp.z),
                                  __int_as_float(tp.w));
  const double* q = mp64 + 10 * c;
  const float m[10] = {(float)q[1], (float)q[2], (float)q[3], (float)q[0], (float)q[4],
                       (float)q[5], (float)q[6], (float)q[7], (float)q[8], (float)q[9]};
  I.mp[3 * c] = make_float4(m[0], m[1], m[2], m[3]);
  I.mp[3 * c + 1] = make_float4(m[4], m[5], m[6], m[7]);
  I.mp[3 * c + 2] = make_float4(m[8], m[9], 0.0f, 0.0f);
  const float mtot = (float)mp64[0];
  const float M = m[3];
  const float qn = sqrtf((m[4] * m[4] + m[5] * m[5] + m[6] * m[6]) +
                         2.0f * (m[7] * m[7] + m[8] * m[8] + m[9] * m[9]));
  float s2 = 0.0f;
  for (int k = 0; k < 3; ++k) {
    const float d = m[k] - g[k];
    s2 += d * d;
  }
  I.fcell[2 * c] = make_float4(log10f(M / mtot) / 3.0f, qn / (M * lf * lf),
                               (float)(bx[3] - bx[0]) / lf, (float)(bx[4] - bx[1]) / lf);
  I.fcell[2 * c + 1] = make_float4((float)(bx[5] - bx[2]) / lf,
                                   log2f(1.0f + (float)dc) / log2f(22.0f), sqrtf(s2) / lf, 0.0f);
}

__device__ __forceinline__ bool is_group(const Cells& C, int64_t c, int n_group) {
  const bool cand = C.n[c] <= n_group || C.nc[c] == 0;
  const bool top = c == 0 || C.n[C.parent[c]] > n_group;
  return cand && top;
}

// cell_image of every cell, the leaves of each block's cells, and the groups
// (the maximal cells with at most n_group particles, or leaves): their
// particle ranges partition the particles, so each is marked at its first
// particle, which orders them.
__global__ void images_kernel(Cells C, int64_t nc, const double* __restrict__ box,
                              const double* __restrict__ mp64, Images I,
                              int32_t* __restrict__ leaf_part, int n_group,
                              int32_t* __restrict__ group_at) {
  __shared__ int sh[kT / 64];
  const int64_t c = (int64_t)blockIdx.x * kT + threadIdx.x;
  // the block's leaf count (one store per block: same-address atomics
  // from every wave serialise)
  const int nl = block_sum(c < nc && C.nc[c < nc ? c : 0] == 0 ? 1 : 0, sh);
  if (threadIdx.x == 0) leaf_part[blockIdx.x] = nl;
  if (c < nc) {
    cell_image(C, c, box, mp64, I);
    if (is_group(C, c, n_group)) group_at[C.first[c]] = (int32_t)c;
  }
}

// Arrays per group.
struct Groups {
  int32_t* cell;
  int4* info;
  float4* box;
};

// Chunks of each item class of a group of n particles.
__device__ __forceinline__ int4 group_chunks(int32_t n) {
  const int32_t rest = n % kChunk;
  int32_t k[kItemClasses] = {0, 0, 0, 0};
  k[item_class(kChunk)] = n / kChunk;
  for (int q = 0; q < kItemClasses; ++q) k[q] += rest > 0 && item_class(rest) == q;
  return make_int4(k[0], k[1], k[2], k[3]);
}

// Writes group g, cell c; returns its chunks per item class.
__device__ __forceinline__ int4 write_group(const Cells& C, int64_t g, int32_t c,
                                            const double* __restrict__ box, const Groups& G) {
  G.cell[g] = c;
  G.info[g] = make_int4(C.first[c], C.n[c], c, 0);
  const double* bx = box + 6 * (int64_t)c;
  G.box[2 * g] = make_float4((float)bx[0], (float)bx[1], (float)bx[2], 0.0f);
  G.box[2 * g + 1] = make_float4((float)bx[3], (float)bx[4], (float)bx[5], 0.0f);
  return group_chunks(C.n[c]);
}

// Work items of group g of n particles, in group order (work) and class by
// class (wwork); p and t: chunks of each class in the groups before, and in all.
__device__ __forceinline__ void write_items(int64_t g, int32_t n, int4 p, int4 t,
                                            int2* __restrict__ work, int2* __restrict__ wwork) {
  const int32_t at = p.x + p.y + p.z + p.w;
  const int32_t begin[kItemClasses] = {p.x, t.x + p.y, t.x + t.y + p.z, t.x + t.y + t.z + p.w};
  for (int32_t k = 0, off = 0; off < n; ++k, off += kChunk) {
    const int2 w = make_int2((int32_t)g, off);
    const int c = item_class(n - off < kChunk ? n - off : kChunk);
    work[at + k] = w;
    // a group's full chunks come before its rest, which may be of the same class
    for (int q = 0; q < kItemClasses; ++q)
      if (c == q) wwork[begin[q] + (q == item_class(kChunk) ? k : 0)] = w;
  }
}

struct Int4Sum {
  __host__ __device__ int4 operator()(const int4& a, const int4& b) const {
    return make_int4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
  }
};

// The build's scalars the host needs, gathered in one place on the device so
// that one copy fetches them.
struct BuildInfo {
  int64_t level[kLevels + 1];  // where each level's cells begin; all cells
  double cube[6];  // root_kernel
  int32_t bad;       // input check (bbox_kernel)
  int32_t unsorted;  // a bucket was too large (bucket_sort_kernel)
  int32_t ng, nw, leaves;
};

// ---- small trees: three launches (keys, order, and one block for all the
// rest) do what the kernels above and below do in about 25, which for a few
// thousand particles are all launch and latency.  The same functions and orders, so the
// same tree.  The one block's time goes with its cells, hence with the particles
// per leaf as well.  Rebuild of a Plummer sphere, many launches / three, in us:
//   particles  n_leaf 1    2          4          8          16
//   1000       120 / 95    110 / 79   103 / 67   99 / 59    95 / 57
//   2000       140 / 149   124 / 113  110 / 89   110 / 77   106 / 69
//   3000       136 / 196   134 / 144  121 / 113  116 / 91   113 / 78
//   5003       137 / 291   130 / 209  125 / 156  126 / 124  128 / 102
//   7168       143 / 389   136 / 276  136 / 200  134 / 155  130 / 124
// The line runs through the crossings; at 8192 and n_leaf 16 it is 129 / 140.
constexpr int kOneBlock = 7168;  // particles above which it is never one block
constexpr bool one_block(int64_t n, int n_leaf) {
  return n <= std::min<int64_t>(kOneBlock, 1400 + 470 * (int64_t)n_leaf);
}
constexpr int kSmallN = 8192;    // what they hold (sorted keys in LDS: 64 KB)
constexpr int kSmallT = 1024;

// Exclusive prefixes of the N values over the block in thread order, and the
// block totals.
template <int N>
__device__ __forceinline__ void block_exclusives(int (&v)[N], int (&total)[N], int (*sh)[N]) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr int kW = kSmallT / 64;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const int incl = dev::wave_inclusive_sum(v[k]);
    if (lane == 63) sh[w][k] = incl;
    v[k] = incl - v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const int incl = dev::wave_inclusive_sum(lane < kW ? sh[lane][k] : 0);
    total[k] = __builtin_amdgcn_readlane(incl, kW - 1);
    v[k] += w == 0 ? 0 : __builtin_amdgcn_readlane(incl, max(w - 1, 0));
  }
  __syncthreads();
}

// Input check, root cube and keys: kSmallKeys keys a block, each block after a
// pass of its own over all positions (block 0 writes what it found).  The key
// arithmetic in FP64 is the longer part: one block for all keys took 23 us for
// 5003 particles, these take 9.
constexpr int kSmallKeys = 256;
__global__ __launch_bounds__(kSmallT) void small_keys_kernel(const float* __restrict__ pos,
                                                             const float* __restrict__ mass, int n,
                                                             BuildInfo* __restrict__ info,
                                                             uint64_t* __restrict__ key) {
  __shared__ float sh[kSmallT / 64][6];
  __shared__ int bad[kSmallT / 64];
  __shared__ double cube[6];
  const int t = threadIdx.x;
  float v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
  int bd = 0;
  for (int i = t; i < n; i += kSmallT) {
    for (int k = 0; k < 3; ++k) {
      const float x = pos[3 * i + k];
      v[k] = x < v[k] ? x : v[k];
      v[3 + k] = v[3 + k] < x ? x : v[3 + k];
      if (!(fabsf(x) < 0x1p60f)) bd |= 1;  // also catches NaN
    }
    const float m = mass[i];
    if (!(m > 0.0f) || !(m < INFINITY)) bd |= 2;
  }
  for (int o = 32; o > 0; o >>= 1)
    for (int k = 0; k < 6; ++k) {
      const float b = __shfl_xor(v[k], o);
      v[k] = k < 3 ? (b < v[k] ? b : v[k]) : (v[k] < b ? b : v[k]);
    }
  for (int o = 32; o > 0; o >>= 1) bd |= __shfl_xor(bd, o);
  if ((t & 63) == 0) {
    for (int k = 0; k < 6; ++k) sh[t >> 6][k] = v[k];
    bad[t >> 6] = bd;
  }
  __syncthreads();
  if (t == 0) {
    double lo[3], hi[3];
    int b = 0;
    for (int k = 0; k < 3; ++k) {
      float a = sh[0][k], c = sh[0][3 + k];
      for (int w = 1; w < kSmallT / 64; ++w) {
        a = sh[w][k] < a ? sh[w][k] : a;
        c = c < sh[w][3 + k] ? sh[w][3 + k] : c;
      }
      lo[k] = a;
      hi[k] = c;
    }
    for (int w = 0; w < kSmallT / 64; ++w) b |= bad[w];
    root_cube_of(lo, hi, cube);
    if (blockIdx.x == 0) {
      for (int k = 0; k < 6; ++k) info->cube[k] = cube[k];
      info->bad = b;
    }
  }
  __syncthreads();
  const int i = blockIdx.x * kSmallKeys + t;
  if (t < kSmallKeys && i < n) key[i] = particle_key(pos[3 * i], pos[3 * i + 1], pos[3 * i + 2], cube);
}

// The stable sort by counting: a key's place is the number of keys before it
// in (key, index) order.  A block places kRankKeys of the n keys at(0) ...
// at(n - 1), n <= kSmallN: its threads hold all keys between them and each compare's lane
// mask is counted by the scalar unit.  n^2 compares over the whole device take 12 us for
// 5003 keys (16 for 8000), where rocPRIM's block sort and merge passes took 35
// in six launches.  Returns the place of key kRankKeys * block + t in thread t <
// kRankKeys, -1 in others.
constexpr int kRankKeys = 32;
template <typename At>
__device__ __forceinline__ int rank_by_counting(const At& at, int n) {
  constexpr int kHeld = kSmallN / kSmallT;
  static_assert(64 % kRankKeys == 0, "a block's keys lie in one run of 64");
  __shared__ int cnt[kSmallT / 64][kRankKeys];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int e0 = blockIdx.x * kRankKeys;
  uint64_t kj[kHeld];  // of keys q * kSmallT + t; past the end larger than any key
#pragma unroll
  for (int q = 0; q < kHeld; ++q) {
    const int j = q * kSmallT + t;
    kj[q] = j < n ? at(j) : ~0ull;
  }
  const int jw = __builtin_amdgcn_readfirstlane(w) * 64;
  const int run = e0 & ~63;  // the block's keys lie in run ... run + 63
  // (the block's keys from a lane each: loaded one by one they cost a memory
  // latency per key)
  const uint64_t ke = at(min(e0 + (lane & (kRankKeys - 1)), n - 1));
  constexpr int kU = 8;
#pragma unroll 1
  for (int g = 0; g < kRankKeys; g += kU) {
    uint64_t ki[kU];
    int c[kU] = {};
#pragma unroll
    for (int u = 0; u < kU; ++u)
      ki[u] = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(ke >> 32), g + u) << 32 |
              (uint32_t)__builtin_amdgcn_readlane((int)ke, g + u);
#pragma unroll
    for (int q = 0; q < kHeld; ++q) {
      if (q * kSmallT >= n) break;
      const int jb = q * kSmallT + jw;  // keys jb ... jb + 63 are this wave's
      const uint64_t tie = jb < run ? 1 : 0;
#pragma unroll
      for (int u = 0; u < kU; ++u) c[u] += __popcll(__ballot(kj[q] < ki[u] + tie));
      if (jb == run)
#pragma unroll
        for (int u = 0; u < kU; ++u)
          c[u] += __popcll(__ballot(kj[q] == ki[u]) & ((1ull << (e0 + g + u - run)) - 1));
    }
#pragma unroll
    for (int u = 0; u < kU; ++u)
      if (lane == u) cnt[w][g + u] = c[u];
  }
  __syncthreads();
  if (t >= kRankKeys || e0 + t >= n) return -1;
  int r = 0;
  for (int k = 0; k < kSmallT / 64; ++k) r += cnt[k][t];
  return r;
}

// The order of all particles, and the particles in it.
__global__ __launch_bounds__(kSmallT) void small_rank_kernel(const uint64_t* __restrict__ key,
                                                             const float* __restrict__ pos,
                                                             const float* __restrict__ mass, int n,
                                                             uint64_t* __restrict__ sorted,
                                                             int32_t* __restrict__ perm,
                                                             float4* __restrict__ part,
                                                             int32_t* __restrict__ iperm) {
  const int r = rank_by_counting([&](int j) { return key[j]; }, n);
  if (r < 0) return;
  const int i = blockIdx.x * kRankKeys + threadIdx.x;
  sorted[r] = key[i];
  perm[r] = i;
  iperm[i] = r;
  part[r] = make_float4(pos[3 * i], pos[3 * i + 1], pos[3 * i + 2], mass[i]);
}

// ---- the sort of up to kSampleMax particles, by (key, index): buckets of
// about kBucket particles between splitters taken from a sorted sample, each
// sorted by one block in LDS.  262144 particles: sample 13 us, count 7, scan 8,
// scatter 10, buckets 23, where rocPRIM's block sort and sixteen launches of
// merge passes took 115.  Whole rebuild with the library's sort and with this, in us:
// 16384 176 / 174, 65536 200 / 187, 262144 268 / 222, 2^20 474 / 412.  A bucket of more than kBucketMax
// particles (input whose keys at regular places tell nothing of the others)
// is reported, and the host sorts with the library.
constexpr int kSampleMax = 1 << 20;
constexpr int kBucket = 1024, kBucketMax = 4096, kBuckets = kSampleMax / kBucket;
constexpr int kSplitN = 4096;  // particles per block of the count and the scatter
// Buckets: a block for each compute unit, of up to kBucket particles on average.
inline int bucket_count(int64_t n) { return (int)std::max<int64_t>(256, (n + kBucket - 1) / kBucket); }
// Samples: 8 per bucket while kBucketMax is at least 16 times the mean, 16 up
// to 2^18 particles, 8 to 16 up to 2^20 (a bucket of four times the mean is then less
// likely than one in 10^4 trees).
inline int sample_size(int64_t n) { return n <= (1 << 16) ? 2048 : n <= (1 << 18) ? 4096 : 8192; }

// Splitter q (1 ... nb - 1) is the sample of rank floor(q S / nb).
__global__ __launch_bounds__(kSmallT) void splitters_kernel(const uint64_t* __restrict__ key,
                                                            int64_t n, int S, int nb,
                                                            uint64_t* __restrict__ skey,
                                                            int32_t* __restrict__ sidx) {
  auto index = [&](int j) { return (int64_t)j * n / S; };
  const int r = rank_by_counting([&](int j) { return key[index(j)]; }, S);
  if (r < 0) return;
  const int q = (r * nb + S - 1) / S;
  if (q < 1 || q >= nb || q * S / nb != r) return;
  const int64_t i = index(blockIdx.x * kRankKeys + threadIdx.x);
  skey[q - 1] = key[i];
  sidx[q - 1] = (int32_t)i;
}

// Bucket of every particle (splitters at or before it) and each block's
// particles per bucket, cnt[bucket * gridDim.x + block]; a 0 behind the last.
__global__ __launch_bounds__(kSmallT) void bucket_count_kernel(const uint64_t* __restrict__ key,
                                                               int64_t n, int nb,
                                                               const uint64_t* __restrict__ skey,
                                                               const int32_t* __restrict__ sidx,
                                                               uint16_t* __restrict__ bucket,
                                                               int32_t* __restrict__ cnt) {
  __shared__ uint64_t sk[kBuckets];
  __shared__ int32_t si[kBuckets], hist[kBuckets];
  const int t = threadIdx.x;
  if (t < nb) hist[t] = 0;
  if (t < nb - 1) {
    sk[t] = skey[t];
    si[t] = sidx[t];
  }
  __syncthreads();
  static_assert(kBuckets <= kSmallT, "one bucket per thread");
  for (int u = 0; u < kSplitN / kSmallT; ++u) {
    const int64_t i = (int64_t)blockIdx.x * kSplitN + u * kSmallT + t;
    if (i >= n) break;
    const uint64_t k = key[i];
    int l = 0, h = nb - 1;
    while (l < h) {
      const int mid = (l + h) >> 1;
      if (sk[mid] < k || (sk[mid] == k && si[mid] <= (int32_t)i)) l = mid + 1;
      else h = mid;
    }
    bucket[i] = (uint16_t)l;
    atomicAdd(&hist[l], 1);
  }
  __syncthreads();
  if (t < nb) cnt[(int64_t)t * gridDim.x + blockIdx.x] = hist[t];
  if (t == 0 && blockIdx.x == 0) cnt[(int64_t)nb * gridDim.x] = 0;
}

// Particles to their buckets, in any order within one.
__global__ __launch_bounds__(kSmallT) void bucket_scatter_kernel(const uint64_t* __restrict__ key,
                                                                 int64_t n, int nb,
                                                                 const uint16_t* __restrict__ bucket,
                                                                 const int32_t* __restrict__ before,
                                                                 uint64_t* __restrict__ key_out,
                                                                 int32_t* __restrict__ idx_out) {
  __shared__ int32_t next[kBuckets];
  const int t = threadIdx.x;
  if (t < nb) next[t] = before[(int64_t)t * gridDim.x + blockIdx.x];
  __syncthreads();
  for (int u = 0; u < kSplitN / kSmallT; ++u) {
    const int64_t i = (int64_t)blockIdx.x * kSplitN + u * kSmallT + t;
    if (i >= n) break;
    const int32_t p = atomicAdd(&next[bucket[i]], 1);
    key_out[p] = key[i];
    idx_out[p] = (int32_t)i;
  }
}

// Bucket blockIdx.x (of nblk counts each): a merge sort in LDS in which every
// element finds its place by a binary search in the run its own is merged with
// (keys first, indices only between equal keys; every step lies within the
// two runs).  (A bitonic network of the next power of two: 26 us at 16384
// particles in 16 buckets, this 23 at 262144 in 256.)  Also writes the particles
// in order (a launch of 8 us of its own before, 5 more here).
__global__ __launch_bounds__(kSmallT) void bucket_sort_kernel(const int32_t* __restrict__ before,
                                                              int nblk,
                                                              const uint64_t* __restrict__ key_in,
                                                              const int32_t* __restrict__ idx_in,
                                                              const float4* __restrict__ packed,
                                                              uint64_t* __restrict__ sorted,
                                                              int32_t* __restrict__ perm,
                                                              float4* __restrict__ part,
                                                              int32_t* __restrict__ iperm,
                                                              int32_t* __restrict__ unsorted) {
  __shared__ uint64_t key[2][kBucketMax];
  __shared__ int32_t idx[2][kBucketMax];
  const int t = threadIdx.x;
  const int32_t lo = before[(int64_t)blockIdx.x * nblk];
  const int m = before[(int64_t)(blockIdx.x + 1) * nblk] - lo;
  if (m > kBucketMax) {  // uniform
    if (t == 0) *unsorted = 1;
    return;
  }
  for (int i = t; i < m; i += kSmallT) {
    key[0][i] = key_in[lo + i];
    idx[0][i] = idx_in[lo + i];
  }
  __syncthreads();
  int cur = 0;
  for (int run = 1; run < m; run *= 2, cur ^= 1) {
    for (int i = t; i < m; i += kSmallT) {
      const uint64_t k = key[cur][i];
      const int32_t v = idx[cur][i];
      const int mine = i & ~(run - 1), other = mine ^ run;
      int l = min(m, other), h = min(m, other + run);
      const int from = l;
      while (l < h) {
        const int mid = (l + h) >> 1;
        const uint64_t km = key[cur][mid];
        if (km < k || (km == k && idx[cur][mid] < v)) l = mid + 1;
        else h = mid;
      }
      const int to = min(mine, other) + (i - mine) + (l - from);
      key[cur ^ 1][to] = k;
      idx[cur ^ 1][to] = v;
    }
    __syncthreads();
  }
  for (int i = t; i < m; i += kSmallT) {
    const int32_t v = idx[cur][i];
    sorted[lo + i] = key[cur][i];
    perm[lo + i] = v;
    part[lo + i] = packed[v];
    iperm[v] = lo + i;
  }
}

// Everything after the sort.  Cell, image, group and item arrays hold cap
// cells and n groups; for more cells it only counts them, and the host calls
// it again with larger arrays.
__global__ __launch_bounds__(kSmallT) void small_tree_kernel(
    Cells C, const uint64_t* __restrict__ key, const float4* __restrict__ part, int n, int n_leaf,
    int n_group, int cap, double* box, double* mp64, Images I, Groups G, int32_t* at, int4* nchunk,
    int2* __restrict__ work, int2* __restrict__ wwork, BuildInfo* __restrict__ info) {
  constexpr int kHeld = kSmallN / kSmallT, kRows = kSmallN / 64;
  struct Split {
    uint64_t key[kSmallN];
    int8_t sw[2][kSmallN + kMaxLeaf];
  };
  __shared__ union {
    Split split;
    FoldBuf fold[kSmallT / 64];
  } u;  // one after the other
  uint64_t* skey = u.split.key;
  auto& sw = u.split.sw;
  __shared__ int rows[kLevels * kRows];
  __shared__ int sh[kSmallT / 64][4];
  auto* sh1 = reinterpret_cast<int(*)[1]>(&sh[0][0]);
  __shared__ int lbegs[kLevels + 1];
  const int t = threadIdx.x, w = t >> 6;
  for (int i = t; i < n; i += kSmallT) {
    skey[i] = key[i];
    at[i] = -1;
  }
  __syncthreads();

  // Subdivision.
  const int len = n + n_leaf;
  for (int e = t; e < len; e += kSmallT) sw[0][e] = window_digits(skey, n, n_leaf, e - n_leaf);
  __syncthreads();
  int cur = 0, run = 1;
  static_assert(kSmallT == kST, "join_windows");
  for (; 2 * run <= n_leaf + 1; run *= 2, cur ^= 1) {
    join_windows(sw[cur], sw[cur ^ 1], len, run);
    __syncthreads();
  }
  LevelRange r[kHeld];
#pragma unroll
  for (int q = 0; q < kHeld; ++q) {
    const int i = q * kSmallT + t;
    r[q] = LevelRange{1, 0};
    if (i < n) r[q] = level_range(skey, i, max(sw[cur][i], sw[cur][i + n_leaf - run + 1]));
    if (q * kSmallT < n) count_starts(r[q], rows + q * (kSmallT / 64) + w, kRows);
    else if ((t & 63) < kLevels) rows[(t & 63) * kRows + q * (kSmallT / 64) + w] = 0;
  }
  __syncthreads();
  constexpr int kPer = (kLevels * kRows + kSmallT - 1) / kSmallT;
  int mine[kPer], sum[1] = {0}, cells[1];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int e = t * kPer + k;
    mine[k] = e < kLevels * kRows ? rows[e] : 0;
    sum[0] += mine[k];
  }
  block_exclusives(sum, cells, sh1);
  const int nc = cells[0];
  int before = sum[0];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int e = t * kPer + k;
    if (e < kLevels * kRows) rows[e] = before;
    before += mine[k];
  }
  __syncthreads();
  if (t <= kLevels) {
    lbegs[t] = t < kLevels ? rows[t * kRows] : nc;
    info->level[t] = lbegs[t];
  }
  if (nc > cap) return;  // uniform
#pragma unroll
  for (int q = 0; q < kHeld; ++q)
    if (q * kSmallT < n)
      write_cells(C, skey, n, q * kSmallT + t, r[q], n_leaf, cap, rows + q * (kSmallT / 64) + w,
                  kRows);
  __syncthreads();
  int levels = 0;
  while (levels < kLevels && lbegs[levels] < nc) ++levels;

  // Boxes and moments: the leaves, then level by level upwards (the deepest
  // level holds only leaves).
  for (int c = t; c < nc; c += kSmallT) {
    close_parent(C, c, nc);
    leaf_moments(C, part, c, box, mp64);
  }
  __syncthreads();
  for (int L = levels - 2; L >= 0; --L) {
    for (int base = lbegs[L]; base < lbegs[L + 1]; base += kSmallT / 8) {
      const int c = base + t / 8;
      inner_moments(C, c, c < lbegs[L + 1], u.fold[w], box, mp64);
    }
    __syncthreads();
  }

  // Images, leaves and group marks.
  int nl[1] = {0}, leaves[1];
  for (int c = t; c < nc; c += kSmallT) {
    cell_image(C, c, box, mp64, I);
    nl[0] += C.nc[c] == 0;
    if (is_group(C, c, n_group)) at[C.first[c]] = c;
  }
  block_exclusives(nl, leaves, sh1);  // (its barriers also order the marks)

  // Groups in particle order, then their work items.
  const int per = (n + kSmallT - 1) / kSmallT;
  const int i0 = min(n, t * per), i1 = min(n, i0 + per);
  int k[1] = {0}, groups[1];
  for (int i = i0; i < i1; ++i) k[0] += at[i] >= 0;
  block_exclusives(k, groups, sh1);
  const int ng = groups[0];
  int g = k[0];
  for (int i = i0; i < i1; ++i)
    if (at[i] >= 0) {
      nchunk[g] = write_group(C, g, at[i], box, G);
      ++g;
    }
  __syncthreads();
  const int gper = (ng + kSmallT - 1) / kSmallT;
  const int g0 = min(ng, t * gper), g1 = min(ng, g0 + gper);
  int4 s = make_int4(0, 0, 0, 0), p, tot;
  const Int4Sum add;
  for (int i = g0; i < g1; ++i) s = add(s, nchunk[i]);
  int v[4] = {s.x, s.y, s.z, s.w}, all[4];
  block_exclusives(v, all, sh);
  p = make_int4(v[0], v[1], v[2], v[3]);
  tot = make_int4(all[0], all[1], all[2], all[3]);
  for (int i = g0; i < g1; ++i) {
    write_items(i, G.info[i].y, p, tot, work, wwork);
    p = add(p, nchunk[i]);
  }
  if (t == 0) {
    info->ng = ng;
    info->nw = tot.x + tot.y + tot.z + tot.w;
    info->leaves = leaves[0];
  }
}

// ---- groups and work items from the marks, in two launches: the groups and
// chunks of each block's per particles, then every block adds up those of the
// blocks before it and writes its own.  (Marks, flags, two library scans, groups, items and
// counts were ten launches, 43 us at 262144 particles; these two are 10.)
constexpr int kGroupBlocks = 1024;  // at most

constexpr int kGroupSums = 5;       // chunks of each class, groups

__global__ __launch_bounds__(kSmallT) void group_count_kernel(Cells C,
                                                              const int32_t* __restrict__ at,
                                                              int64_t n, int64_t per,
                                                              int32_t* __restrict__ sums) {
  __shared__ int sh[kSmallT / 64][kGroupSums];
  const int64_t i0 = blockIdx.x * per, i1 = i0 + per < n ? i0 + per : n;
  int v[kGroupSums] = {0, 0, 0, 0, 0}, total[kGroupSums];
  for (int64_t i = i0 + threadIdx.x; i < i1; i += kSmallT) {
    const int32_t c = at[i];
    if (c < 0) continue;
    const int4 k = group_chunks(C.n[c]);
    v[0] += k.x;
    v[1] += k.y;
    v[2] += k.z;
    v[3] += k.w;
    ++v[4];
  }
  block_exclusives(v, total, sh);
  if (threadIdx.x == 0)
    for (int k = 0; k < kGroupSums; ++k) sums[k * gridDim.x + blockIdx.x] = total[k];
}

// Block 0 also records the counts, with the leaves (nl counts of the images kernel).
__global__ __launch_bounds__(kSmallT) void group_write_kernel(
    Cells C, const int32_t* __restrict__ at, int64_t n, int64_t per,
    const int32_t* __restrict__ sums, const double* __restrict__ box, Groups G,
    int2* __restrict__ work, int2* __restrict__ wwork, const int32_t* __restrict__ leaf_part,
    int64_t nl, BuildInfo* __restrict__ info) {
  __shared__ int all[kGroupSums + 1], before[kGroupSums];
  __shared__ int sh[kSmallT / 64][3];
  const int t = threadIdx.x, blk = (int)blockIdx.x, nb = (int)gridDim.x, w = t >> 6;
  // a wave per quantity; one wave of block 0 adds up the leaves
  if (w < kGroupSums || (w == kGroupSums && blk == 0)) {
    int a = 0, b = 0;
    if (w < kGroupSums) {
      for (int k = t & 63; k < nb; k += 64) {
        const int v = sums[w * nb + k];
        a += v;
        b += k < blk ? v : 0;
      }
    } else {
      for (int64_t k = t & 63; k < nl; k += 64) a += leaf_part[k];
    }
    a = dev::wave_inclusive_sum(a);
    b = dev::wave_inclusive_sum(b);
    if ((t & 63) == 63) {
      all[w] = a;
      if (w < kGroupSums) before[w] = b;
    }
  }
  __syncthreads();
  const int4 tot = make_int4(all[0], all[1], all[2], all[3]);
  int4 p = make_int4(before[0], before[1], before[2], before[3]);
  int g = before[4];
  const Int4Sum add;
  const int64_t i0 = blk * per, i1 = i0 + per < n ? i0 + per : n;
  for (int64_t base = i0; base < i1; base += kSmallT) {
    const int64_t i = base + t;
    const int32_t c = i < i1 ? at[i] : -1;
    const int4 k = c >= 0 ? group_chunks(C.n[c]) : make_int4(0, 0, 0, 0);
    // a group has at most one chunk of the classes after the first
    int v[3] = {(c >= 0) | k.y << 16, k.z | k.w << 16, k.x}, all3[3];
    block_exclusives(v, all3, sh);
    if (c >= 0) {
      const int64_t q = g + (v[0] & 0xffff);
      write_group(C, q, c, box, G);
      write_items(q, C.n[c], add(p, make_int4(v[2], v[0] >> 16, v[1] & 0xffff, v[1] >> 16)), tot,
                  work, wwork);
    }
    g += all3[0] & 0xffff;
    p = add(p, make_int4(all3[2], all3[0] >> 16, all3[1] & 0xffff, all3[1] >> 16));
  }
  if (blk == 0 && t == 0) {
    info->ng = all[4];
    info->nw = tot.x + tot.y + tot.z + tot.w;
    info->leaves = all[kGroupSums];
  }
}

// Scratch allocations of one build: cut from an arena freed on every exit, or
// slots of a pool kept for the next build.
struct Scratch {
  SeqPool* pool = nullptr;
  Arena arena;
  explicit Scratch(SeqPool* sp, size_t expect = 0) : pool(sp) { arena.expect(expect); }
  template <typename T>
  T* get(int64_t count) {
    const size_t bytes = (size_t)count * sizeof(T);
    return static_cast<T*>(pool ? pool->take(bytes) : arena.take(bytes));
  }
};

template <typename T>
int exclusive_sum(const T* in, T* out, int64_t n, Scratch& S, hipStream_t s) {
  size_t bytes = 0;
  if (hipcub::DeviceScan::ExclusiveSum(nullptr, bytes, in, out, (int)n, s) != hipSuccess) return -1;
  void* tmp = S.get<char>((int64_t)bytes);
  if (!tmp) return -2;
  return hipcub::DeviceScan::ExclusiveSum(tmp, bytes, in, out, (int)n, s) == hipSuccess ? 0 : -1;
}

}  // namespace

void* Arena::take(size_t bytes) {
  bytes = (std::max<size_t>(bytes, 1) + 255) & ~size_t(255);
  if (bytes > left) {
    // A chunk for all that is expected or, where the device has no room for it in
    // one piece, for this array alone.
    size_t want = std::max(bytes, next);
    void* q = nullptr;
    if (device_malloc(&q, want) != hipSuccess) {
      (void)hipGetLastError();
      want = bytes;
      if (want >= next || device_malloc(&q, want) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
      }
    }
    chunks.push_back(q);
    at = static_cast<char*>(q);
    left = want;
    next = 0;
  }
  void* p = at;
  at += bytes;
  left -= bytes;
  return p;
}

Arena::~Arena() {
  for (void* q : chunks) hipFree(q);
}

void* SeqPool::take(size_t bytes) {
  bytes = std::max<size_t>(bytes, 256);
  if (next < ptr.size() && cap[next] >= bytes) return ptr[next++];
  // Grown slots get a quarter of headroom so that the small changes of a
  // tree from one step to the next do not reallocate them.
  const size_t want = ((bytes + bytes / 4) + 255) & ~size_t(255);
  void* q = nullptr;
  if (next < ptr.size()) {
    hipFree(ptr[next]);
    ptr[next] = nullptr;
    cap[next] = 0;
  }
  if (hipMalloc(&q, want) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  if (next == ptr.size()) {
    ptr.push_back(q);
    cap.push_back(want);
  } else {
    ptr[next] = q;
    cap[next] = want;
  }
  return ptr[next++];
}

SeqPool::~SeqPool() {
  for (void* q : ptr)
    if (q) hipFree(q);
}

BuildPools::~BuildPools() {
  if (pinned) hipHostFree(pinned);
}

int build_device_tree(const float* pos_in, const float* mass_in, bool inputs_on_device, int64_t n,
                      int n_leaf, int n_group, HostTree& h, DevTree& dt, DeviceArrays& out,
                      DevAlloc& alloc, void* stream, std::string& err, BuildPools* pools) {
  hipStream_t s = (hipStream_t)stream;
  if (n_leaf < 1 || n_leaf > kMaxLeaf) {  // (the callers have checked it)
    err = "n_leaf out of range";
    return -1;
  }
  if (pools) {
    pools->outer.rewind();
    pools->cells.rewind();
  }
  // What the arrays below add up to (the sort's and the scans' scratch included:
  // 72 to 76 bytes per particle, 16 of them the inputs); what a build needs beyond
  // that is allocated on its own.
  Scratch S(pools ? &pools->outer : nullptr, (size_t)n * (inputs_on_device ? 60 : 76) + (1 << 20));
  Scratch CS(pools ? &pools->cells : nullptr, (size_t)n * 48 + (1 << 13));
  auto fail = [&](const char* what) {
    err = what;
    return -1;
  };
  h = HostTree();
  h.n = n;
  h.n_leaf = n_leaf;
  h.n_group = n_group;

  // The scalars the host needs come back in two copies (after the levels,
  // after the groups), into page-locked memory kept with the pools.
  BuildInfo* info = S.get<BuildInfo>(1);
  if (!info) return fail("device allocation failed");
  BuildInfo local;
  BuildInfo* hinfo = &local;
  if (pools) {
    if (!pools->pinned && hipHostMalloc(&pools->pinned, sizeof(BuildInfo)) != hipSuccess) {
      (void)hipGetLastError();
      pools->pinned = nullptr;
    }
    if (pools->pinned) hinfo = static_cast<BuildInfo*>(pools->pinned);
  }
  auto fetch = [&](size_t off, size_t bytes) {
    return hipMemcpyAsync(reinterpret_cast<char*>(hinfo) + off, reinterpret_cast<char*>(info) + off,
                          bytes, hipMemcpyDeviceToHost, s) == hipSuccess &&
           hipStreamSynchronize(s) == hipSuccess;
  };

  // Inputs on the device (copied there, or checked there: finite positions
  // with |x| < 2^60 and finite masses > 0, as the host build requires; the
  // verdict comes back with the level counts, and every kernel before that
  // is safe on any input values).
  const float* pos = pos_in;
  const float* mass = mass_in;
  if (!inputs_on_device) {
    float* p = S.get<float>(3 * n);
    float* q = S.get<float>(n);
    if (!p || !q) return fail("device allocation failed");
    if (hipMemcpyAsync(p, pos_in, (size_t)n * 12, hipMemcpyHostToDevice, s) != hipSuccess ||
        hipMemcpyAsync(q, mass_in, (size_t)n * 4, hipMemcpyHostToDevice, s) != hipSuccess)
      return fail("input upload failed");
    pos = p;
    mass = q;
  }
  const bool check = inputs_on_device;  // then bbox_kernel checks them
  static_assert(kOneBlock <= kSmallN, "the one block's arrays");
  const bool small = one_block(n, n_leaf);

  // Root cube (the host's rule on the device's bounding box).
  if (!small) {
    if (hipMemsetAsync(&info->bad, 0, 8, s) != hipSuccess) return fail("memset failed");
    const int nbb = (int)std::min<int64_t>(1024, blocks(n));
    float* bbp = S.get<float>(6 * nbb);
    if (!bbp) return fail("device allocation failed");
    bbox_kernel<<<nbb, kT, 0, s>>>(pos, check ? mass : nullptr, n, bbp, &info->bad);
    root_kernel<<<1, kT, 0, s>>>(bbp, nbb, info->cube);
  }

  // Keys and the stable sort (ties keep the input order).
  uint64_t* key = S.get<uint64_t>(n);
  uint64_t* key2 = S.get<uint64_t>(n);
  float4* part = nullptr;
  int32_t *perm = nullptr, *iperm = nullptr, *idx = nullptr;
  float4* packed = nullptr;
  auto A = [&](auto** p, int64_t count) {
    return alloc.alloc((void**)p, (size_t)count * sizeof(**p)) == 0;
  };
  alloc.expect((size_t)n * 24 + 3 * 256);
  if (!key || !key2 || !A(&perm, n) || !A(&part, n) || !A(&iperm, n))
    return fail("device allocation failed");
  auto library_sort = [&]() {
    size_t sbytes = 0;
    if (hipcub::DeviceRadixSort::SortPairs(nullptr, sbytes, key, key2, idx, perm, (int)n, 0, 63,
                                           s) != hipSuccess)
      return false;
    void* stmp = S.get<char>((int64_t)sbytes);
    return stmp && hipcub::DeviceRadixSort::SortPairs(stmp, sbytes, key, key2, idx, perm, (int)n, 0,
                                                      63, s) == hipSuccess;
  };
  const bool sampled = !small && n <= kSampleMax;
  if (!small) {
    idx = S.get<int32_t>(n);
    packed = S.get<float4>(n);
    if (!idx || !packed) return fail("device allocation failed");
    keys_kernel<<<blocks(n), kT, 0, s>>>(pos, mass, n, info->cube, key, idx, packed);
  }
  if (sampled) {
    const int ns = sample_size(n), nb = bucket_count(n);
    const int nblk = (int)((n + kSplitN - 1) / kSplitN);
    const int64_t nc = (int64_t)nb * nblk + 1;
    uint64_t* skey = S.get<uint64_t>(kBuckets);
    int32_t* sidx = S.get<int32_t>(kBuckets);
    uint16_t* bucket = S.get<uint16_t>(n);
    int32_t* cnt = S.get<int32_t>(nc);
    int32_t* before = S.get<int32_t>(nc);
    uint64_t* bkey = S.get<uint64_t>(n);
    int32_t* bidx = S.get<int32_t>(n);
    if (!skey || !sidx || !bucket || !cnt || !before || !bkey || !bidx)
      return fail("device allocation failed");
    splitters_kernel<<<ns / kRankKeys, kSmallT, 0, s>>>(key, n, ns, nb, skey, sidx);
    bucket_count_kernel<<<nblk, kSmallT, 0, s>>>(key, n, nb, skey, sidx, bucket, cnt);
    if (exclusive_sum(cnt, before, nc, S, s)) return fail("scan failed");
    bucket_scatter_kernel<<<nblk, kSmallT, 0, s>>>(key, n, nb, bucket, before, bkey, bidx);
    bucket_sort_kernel<<<nb, kSmallT, 0, s>>>(before, nblk, bkey, bidx, packed, key2, perm, part, iperm,
                                              &info->unsorted);
  } else if (!small && !library_sort()) {
    return fail("sort failed");
  }

  // Cell arrays, for twice the particles at first; a tree of more cells has
  // them written again into larger ones.
  const int64_t most = max_cells();
  int64_t cap = std::min(2 * n + 64, most);
  Cells C{};
  auto cell_arrays = [&]() {
    C = Cells{CS.get<int32_t>(cap), CS.get<int32_t>(cap), CS.get<int32_t>(cap),
              CS.get<int32_t>(cap), CS.get<int32_t>(cap), CS.get<int32_t>(cap)};
    return C.first && C.n && C.depth && C.parent && C.fc && C.nc;
  };
  if (!cell_arrays()) return fail("device allocation failed");
  // The scalars of the levels, once fetched: the verdict on the inputs, the
  // root cube, and the level ranges.  False, with err, where the call is refused.
  int64_t nc = 0;
  auto read_levels = [&]() {
    if (hinfo->bad) {
      err = hinfo->bad & 1 ? "positions must be finite with |x| < 2^60" : "masses must be finite and > 0";
      return false;
    }
    for (int k = 0; k < 3; ++k) h.corner[k] = hinfo->cube[k];
    h.side = hinfo->cube[3];
    nc = hinfo->level[kLevels];
    h.max_level_cells = 0;
    h.max_depth = 0;
    for (int L = 0; L < kLevels && hinfo->level[L] < nc; ++L) {
      h.max_level_cells = std::max(h.max_level_cells, hinfo->level[L + 1] - hinfo->level[L]);
      h.max_depth = L;
    }
    return true;
  };
  auto too_many = [&]() {  // (not of keys that are still to be sorted)
    if (nc <= most) return false;
    err = too_many_cells(nc);
    return true;
  };

  // Persistent device arrays of the tree, for up to ncb cells and ngb groups.
  float4 *geo_host = nullptr, *geo = nullptr, *wrec = nullptr, *mp = nullptr,
         *fcell = nullptr, *gbox = nullptr;
  int32_t *depth = nullptr, *groups = nullptr;
  double *box = nullptr, *mp64 = nullptr;
  int4 *topo = nullptr, *ginfo = nullptr;
  int2 *work = nullptr, *wwork = nullptr;
  auto persistent = [&](int64_t ncb, int64_t ngb) {
    const int64_t nwb = ngb + n / kChunk + 1;  // a rest per group and the full chunks
    alloc.expect((size_t)ncb * 308 + (size_t)ngb * 52 + (size_t)nwb * 16 + 14 * 256);
    return A(&box, 6 * ncb) && A(&mp64, 10 * ncb) && A(&topo, ncb) &&
           A(&geo_host, ncb) && A(&geo, ncb) && A(&wrec, 2 * ncb) && A(&mp, 3 * ncb) &&
           A(&fcell, 2 * ncb) && A(&depth, ncb) && A(&groups, ngb) && A(&ginfo, ngb) &&
           A(&gbox, 2 * ngb) && A(&work, nwb) && A(&wwork, nwb);
  };
  if (small) {
    const int64_t ngb = std::min(cap, n);
    int32_t* at = S.get<int32_t>(n);
    int4* nchunk = S.get<int4>(ngb);
    if (!persistent(cap, ngb) || !at || !nchunk) return fail("device allocation failed");
    small_keys_kernel<<<((int)n + kSmallKeys - 1) / kSmallKeys, kSmallT, 0, s>>>(
        pos, mass, (int)n, info, key);
    small_rank_kernel<<<((int)n + kRankKeys - 1) / kRankKeys, kSmallT, 0, s>>>(
        key, pos, mass, (int)n, key2, perm, part, iperm);
    for (;;) {
      small_tree_kernel<<<1, kSmallT, 0, s>>>(
          C, key2, part, (int)n, n_leaf, n_group, (int)cap, box, mp64,
          Images{topo, geo_host, geo, wrec, mp, fcell, depth}, Groups{groups, ginfo, gbox}, at,
          nchunk, work, wwork, info);
      if (!fetch(0, sizeof(BuildInfo))) return fail("build failed");
      if (!read_levels() || too_many()) return kBuildRefused;
      if (nc <= cap) break;
      cap = nc;
      if (!cell_arrays() || !persistent(cap, n)) return fail("device allocation failed");
    }
  } else {
    // Cells of all levels.
    const int nb = (int)((n + kST - 1) / kST);
    uchar2* range = S.get<uchar2>(n);
    const bool scan = nb > kOwnScan;
    const int64_t ncnt = (int64_t)kLevels * nb + 1;
    int32_t* cnt = scan ? nullptr : S.get<int32_t>(ncnt);
    CellSum* cnt64 = scan ? S.get<CellSum>(ncnt) : nullptr;
    CellSum* before = scan ? S.get<CellSum>(ncnt) : nullptr;
    int32_t* at = S.get<int32_t>(n);
    if (!range || (scan ? !cnt64 || !before : !cnt) || !at) return fail("device allocation failed");
    auto write = [&]() {
      if (scan)
        cells_kernel<true><<<nb, kST, 0, s>>>(C, key2, (int32_t)n, n_leaf, range, before, cap, info->level);
      else
        cells_kernel<false><<<nb, kST, 0, s>>>(C, key2, (int32_t)n, n_leaf, range, cnt, cap, info->level);
    };
    bool gathered = sampled;
    for (bool sorted = !sampled;; sorted = true) {
      if (scan) {
        starts_kernel<<<nb, kST, 0, s>>>(key2, n, n_leaf, range, cnt64, at);
        if (exclusive_sum(cnt64, before, ncnt, S, s)) return fail("scan failed");
      } else {
        starts_kernel<<<nb, kST, 0, s>>>(key2, n, n_leaf, range, cnt, at);
      }
      write();
      if (!fetch(0, offsetof(BuildInfo, ng))) return fail("subdivision failed");
      if (!read_levels()) return kBuildRefused;
      if (sorted || !hinfo->unsorted) break;
      // (what was made of the unsorted keys stays within its arrays)
      if (!library_sort()) return fail("sort failed");
      gathered = false;
    }
    if (too_many()) return kBuildRefused;
    if (nc > cap) {
      cap = nc;
      if (!cell_arrays()) return fail("device allocation failed");
      write();
    }
    // Groups <= cells, so that the group and item counts come back in one copy at
    // the end.
    if (!persistent(nc, nc)) return fail("device allocation failed");
    if (!gathered) gather_kernel<<<blocks(n), kT, 0, s>>>(packed, perm, n, part, iperm);
    leaf_moments_kernel<<<blocks(nc), kT, 0, s>>>(C, part, nc, box, mp64);
    LevelBegin B{};
    int top = 0;  // levels 0 ... top - 1 go to one block
    while (top < h.max_depth && hinfo->level[top + 1] - hinfo->level[top] <= kTopCells) ++top;
    for (int L = 0; L <= top; ++L) B.at[L] = (int32_t)hinfo->level[L];
    for (int L = h.max_depth - 1; L >= top; --L) {  // the deepest level holds only leaves
      const int64_t a = hinfo->level[L], b = hinfo->level[L + 1];
      inner_moments_kernel<<<blocks(8 * (b - a)), kT, 0, s>>>(C, a, b, box, mp64);
    }
    if (top > 0) top_moments_kernel<<<1, kTopT, 0, s>>>(C, B, top - 1, box, mp64);
    const int64_t nbi = blocks(nc);
    int32_t* nleaf = S.get<int32_t>(nbi);
    if (!nleaf) return fail("device allocation failed");
    images_kernel<<<blocks(nc), kT, 0, s>>>(
        C, nc, box, mp64, Images{topo, geo_host, geo, wrec, mp, fcell, depth}, nleaf, n_group, at);

    // Groups and work chunks.
    const int64_t per = (n + (int64_t)kGroupBlocks * kSmallT - 1) / ((int64_t)kGroupBlocks * kSmallT) * kSmallT;
    const int gb = (int)((n + per - 1) / per);
    int32_t* gsum = S.get<int32_t>(kGroupSums * gb);
    if (!gsum) return fail("device allocation failed");
    group_count_kernel<<<gb, kSmallT, 0, s>>>(C, at, n, per, gsum);
    group_write_kernel<<<gb, kSmallT, 0, s>>>(C, at, n, per, gsum, box,
                                              Groups{groups, ginfo, gbox}, work, wwork, nleaf, nbi,
                                              info);
    if (!fetch(offsetof(BuildInfo, ng), sizeof(BuildInfo) - offsetof(BuildInfo, ng)))
      return fail("group and work counts failed");
  }
  const int64_t ng = hinfo->ng, nw = hinfo->nw;
  h.nc_dev = nc;
  h.ng_dev = ng;
  h.nw_dev = nw;
  h.n_leaves = hinfo->leaves;

  dt.part = reinterpret_cast<const float*>(part);
  dt.perm = perm;
  dt.topo = reinterpret_cast<const int32_t*>(topo);
  dt.geo = reinterpret_cast<const float*>(geo);
  dt.wrec = reinterpret_cast<const float*>(wrec);
  dt.fcell = reinterpret_cast<const float*>(fcell);
  dt.iperm = iperm;
  dt.mp = reinterpret_cast<const float*>(mp);
  dt.ginfo = reinterpret_cast<const int32_t*>(ginfo);
  dt.gbox = reinterpret_cast<const float*>(gbox);
  dt.work = reinterpret_cast<const int32_t*>(work);
  dt.wwork = reinterpret_cast<const int32_t*>(wwork);
  dt.n = n;
  dt.nc = nc;
  dt.ng = ng;
  dt.nw = nw;
  out.box = box;
  out.mp64 = mp64;
  out.geo_host = reinterpret_cast<const float*>(geo_host);
  out.depth = depth;
  out.groups = groups;
  return 0;
}

}  // namespace octgrav
