// Support kernels of the acceptance criteria: FP32 compensated direct
// summation (the accuracy reference of Sec. 3.1, and the learned criterion's
// label normalization), the features + labels of band candidates, and the
// walk records of the centre-of-mass offset opening test.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_common.h"
#include "octgrav_internal.h"

namespace octgrav {
namespace {

using namespace dev;

constexpr int kThreads = 256;
constexpr int kDTile = 256;

// Direct sum.  One wave per block takes 64 * TPL targets, TPL per lane, and
// one of the contiguous ranges of the particles, streamed through LDS in
// tiles of kDTile; plain FP32 per tile folded into compensated pairs.  The
// target itself contributes -m_i/eps to the potential and nothing to the
// acceleration; that same FP32 value is removed at the end.
//
// Bound: VALU issue, 13 FP32 instructions and one v_rsq_f32 per pair.  Measured
// issue costs (cycles per wave instruction and SIMD): 2.4 for FP32 arithmetic on
// vector registers or constants, 4.2 as soon as one operand is a scalar
// register, 8.3 for v_rsq_f32.  So eps^2 sits in a vector register, one LDS
// read serves two targets (TPL = 2; one where the chip is idle anyway, see
// direct_plan), and the tile loop is unrolled with the reads at constant
// offsets.  The ranges fill the chip for any number of targets: 4096 targets of
// 2^20 particles made 16 blocks of four waves before (39.6 ms, now 1.4).
template <int TPL>
__global__ __launch_bounds__(64) void direct_kernel(DevTree T, const int32_t* __restrict__ targets,
                                                    int64_t nt, float eps2, int64_t range,
                                                    float4* __restrict__ part_out,
                                                    float* __restrict__ acc,
                                                    float* __restrict__ pot) {
  __shared__ float4 src[kDTile];
  const float4* part = reinterpret_cast<const float4*>(T.part);
  const int lane = threadIdx.x;
  const int64_t u0 = (int64_t)blockIdx.x * (TPL * 64) + lane;
  const int64_t beg = (int64_t)blockIdx.y * range, end = min(T.n, beg + range);
  float4 xi[TPL];
  Sum4 s[TPL];
#pragma unroll
  for (int q = 0; q < TPL; ++q) {
    const int64_t u = min(u0 + 64 * q, nt - 1);  // lanes past the end repeat the last target
    xi[q] = part[T.iperm[targets ? targets[u] : u]];
    s[q].zero();
  }
  const float e2 = in_vgpr(eps2);
  for (int64_t base = beg; base < end; base += kDTile) {
#pragma unroll
    for (int k = 0; k < kDTile / 64; ++k) {
      const int64_t j = base + 64 * k + lane;
      // entries past the range carry no mass
      src[64 * k + lane] = j < end ? part[j] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __syncthreads();
    const int cnt = ((int)min((int64_t)kDTile, end - base) + 3) & ~3;
    float a[TPL][4];
#pragma unroll
    for (int q = 0; q < TPL; ++q) a[q][0] = a[q][1] = a[q][2] = a[q][3] = 0.f;
    for (int j = 0; j < cnt; j += 4) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float4 sj = src[j + k];
#pragma unroll
        for (int q = 0; q < TPL; ++q) pp_term(xi[q], sj, e2, a[q][0], a[q][1], a[q][2], a[q][3]);
      }
    }
#pragma unroll
    for (int q = 0; q < TPL; ++q) s[q].template fold<false>(a[q][0], a[q][1], a[q][2], a[q][3]);
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < TPL; ++q) {
    const int64_t u = u0 + 64 * q;
    if (u >= nt) continue;
    if (part_out) {
      float4* o = part_out + 2 * ((int64_t)blockIdx.y * nt + u);
      o[0] = make_float4(s[q].s[0], s[q].s[1], s[q].s[2], s[q].s[3]);
      o[1] = make_float4(s[q].c[0], s[q].c[1], s[q].c[2], s[q].c[3]);
      continue;
    }
    neu_add(s[q].s[3], s[q].c[3], self_term(xi[q].w, eps2));
    acc[3 * u + 0] = s[q].s[0] + s[q].c[0];
    acc[3 * u + 1] = s[q].s[1] + s[q].c[1];
    acc[3 * u + 2] = s[q].s[2] + s[q].c[2];
    if (pot) pot[u] = s[q].s[3] + s[q].c[3];
  }
}

// Adds the ranges' compensated sums of each target, sixteen lanes per target:
// every lane a contiguous run of ranges, then the lanes in order.
constexpr int kDLanes = 16;
__global__ __launch_bounds__(kThreads) void direct_combine_kernel(
    DevTree T, const int32_t* __restrict__ targets, int64_t nt, float eps2, int splits,
    const float4* __restrict__ part_in, float* __restrict__ acc, float* __restrict__ pot) {
  constexpr int kPer = kThreads / kDLanes;  // targets per block
  __shared__ float4 sh[2][kDLanes][kPer];
  const int t = threadIdx.x % kPer, l = threadIdx.x / kPer;
  const int64_t u = (int64_t)blockIdx.x * kPer + t;
  Sum4 s;
  s.zero();
  const int per = (splits + kDLanes - 1) / kDLanes;
  const int k1 = min(splits, (l + 1) * per);
  if (u < nt)
    for (int k = l * per; k < k1; ++k) {
      const float4 a = part_in[2 * ((int64_t)k * nt + u)], b = part_in[2 * ((int64_t)k * nt + u) + 1];
      s.fold<false>(a.x, a.y, a.z, a.w);
      s.fold<false>(b.x, b.y, b.z, b.w);
    }
  sh[0][l][t] = make_float4(s.s[0], s.s[1], s.s[2], s.s[3]);
  sh[1][l][t] = make_float4(s.c[0], s.c[1], s.c[2], s.c[3]);
  __syncthreads();
  if (l != 0 || u >= nt) return;
  for (int k = 1; k < kDLanes; ++k) {
    const float4 a = sh[0][k][t], b = sh[1][k][t];
    s.fold<false>(a.x, a.y, a.z, a.w);
    s.fold<false>(b.x, b.y, b.z, b.w);
  }
  const float m = reinterpret_cast<const float4*>(T.part)[T.iperm[targets ? targets[u] : u]].w;
  neu_add(s.s[3], s.c[3], self_term(m, eps2));
  acc[3 * u + 0] = s.s[0] + s.c[0];
  acc[3 * u + 1] = s.s[1] + s.c[1];
  acc[3 * u + 2] = s.s[2] + s.c[2];
  if (pot) pot[u] = s.s[3] + s.c[3];
}

// One block per band pair (group g, cell c): for every target i of g, the
// cell's monopole + quadrupole acceleration against the exact sum over its
// particles, relative to |a_i(direct)|; the label is the largest of them.
// Thread 0 also writes the pair's 12 features.
__global__ __launch_bounds__(kThreads) void mac_label_kernel(DevTree T, WalkBufs B,
                                                             const int32_t* groups, int64_t ngs,
                                                             const int64_t* out_off,
                                                             const float* acc_direct, float eps2,
                                                             float* feat, float* label,
                                                             int32_t* gout, int32_t* cout) {
  __shared__ float red[kThreads * 4];
  __shared__ float emax[kThreads];
  const int64_t p = blockIdx.x;
  // the sampled group this pair belongs to
  int64_t lo = 0, hi = ngs;
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (out_off[mid] <= p) lo = mid;
    else hi = mid;
  }
  const int64_t g = groups[lo];
  const int c = B.c_ids[B.c_off[g] + (p - out_off[lo])];
  const int4 gi = reinterpret_cast<const int4*>(T.ginfo)[g];
  const int4 tc = reinterpret_cast<const int4*>(T.topo)[c];
  const float4* part = reinterpret_cast<const float4*>(T.part);
  const float4* mp = reinterpret_cast<const float4*>(T.mp);
  const float4 m0 = mp[3 * (int64_t)c], m1 = mp[3 * (int64_t)c + 1], m2 = mp[3 * (int64_t)c + 2];
  const int tid = threadIdx.x;
  float e_blk = 0.0f;
  for (int off = 0; off < gi.y; off += kChunk) {
    const int nt = min(kChunk, gi.y - off);
    const int S = kThreads / nt, t = tid % nt, slice = tid / nt;
    const float4 xi = part[gi.x + off + t];
    Sum4 s;
    s.zero();
    if (slice < S) {
      float ax = 0.f, ay = 0.f, az = 0.f, ph = 0.f;
      int k = 0;
      for (int j = slice; j < tc.w; j += S) {
        pp_term(xi, part[tc.z + j], eps2, ax, ay, az, ph);
        if (++k == 64) {
          s.fold<false>(ax, ay, az, ph);
          ax = ay = az = ph = 0.f;
          k = 0;
        }
      }
      s.fold<false>(ax, ay, az, ph);
      for (int q = 0; q < 3; ++q) red[4 * tid + q] = s.s[q] + s.c[q];
    }
    __syncthreads();
    if (tid < nt) {
      float sx = 0.f, sy = 0.f, sz = 0.f, cx = 0.f, cy = 0.f, cz = 0.f;
      for (int sl = 0; sl < S; ++sl) {
        const float* r = red + 4 * (sl * nt + tid);
        neu_add(sx, cx, r[0]);
        neu_add(sy, cy, r[1]);
        neu_add(sz, cz, r[2]);
      }
      float px = 0.f, py = 0.f, pz = 0.f, pp = 0.f;
      pc_term(xi, m0, m1, m2, eps2, px, py, pz, pp);
      const float dx = px - (sx + cx), dy = py - (sy + cy), dz = pz - (sz + cz);
      const int64_t o = T.perm[gi.x + off + tid];
      const float ax = acc_direct[3 * o], ay = acc_direct[3 * o + 1], az = acc_direct[3 * o + 2];
      const float e = sqrtf(dx * dx + dy * dy + dz * dz) / sqrtf(ax * ax + ay * ay + az * az);
      e_blk = fmaxf(e_blk, e);
    }
    __syncthreads();
  }
  emax[tid] = e_blk;
  __syncthreads();
  for (int o = kThreads / 2; o > 0; o >>= 1) {
    if (tid < o) emax[tid] = fmaxf(emax[tid], emax[tid + o]);
    __syncthreads();
  }
  if (tid == 0) {
    label[p] = emax[0];
    const float4* gbox = reinterpret_cast<const float4*>(T.gbox);
    const float4 geo = reinterpret_cast<const float4*>(T.geo)[c];
    const float4* fc = reinterpret_cast<const float4*>(T.fcell);
    if (gout) gout[p] = (int32_t)g;
    if (cout) cout[p] = c;
    mac_features(mac_group(gbox[2 * g], gbox[2 * g + 1]), geo, fc[2 * (int64_t)c],
                 fc[2 * (int64_t)c + 1], feat + 12 * p);
  }
}

// Walk records of the offset opening test at one theta: the boundary of
// each record becomes (com, l + theta |com - cb|) with the leaf sign bit kept,
// the topology is copied, so the walk kernels' own test (d2 == 0 or
// d2 theta^2 < w^2) evaluates the offset criterion unchanged.
__global__ void com_record_kernel(const float4* __restrict__ wrec, const float4* __restrict__ mp,
                                  int64_t nc, float theta, float4* __restrict__ out) {
#pragma clang fp contract(off)
  const int64_t c = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (c >= nc) return;
  const float4 g = wrec[2 * c];
  const float4 m0 = mp[3 * c];
  const float dx = m0.x - g.x, dy = m0.y - g.y, dz = m0.z - g.z;
  const float px = dx * dx, py = dy * dy, pz = dz * dz;
  const float delta = sqrtf((px + py) + pz);  // correctly rounded (HIP default)
  const float td = theta * delta;
  const float lp = fabsf(g.w) + td;
  out[2 * c] = make_float4(m0.x, m0.y, m0.z, copysignf(lp, g.w));
  out[2 * c + 1] = wrec[2 * c + 1];
}

}  // namespace

int launch_com_records(const DevTree& T, float theta, float* out, void* stream) {
  if (T.nc <= 0) return 0;
  com_record_kernel<<<(T.nc + kThreads - 1) / kThreads, kThreads, 0, (hipStream_t)stream>>>(
      reinterpret_cast<const float4*>(T.wrec), reinterpret_cast<const float4*>(T.mp), T.nc, theta,
      reinterpret_cast<float4*>(out));
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Split of a direct sum: targets per lane, and the particle ranges, whole tiles.
// Ranges: enough waves for eight per SIMD (256 CUs x 4 SIMDs; below about four the
// issue rate falls).  The cost of a range is 32 bytes per target written and
// read again.  A sum too small for four waves per SIMD even so is bound by the
// chain of pairs in a wave, and has one target per lane: us for all of 256 / 512 /
// 1000 / 8000 particles with one target per lane 32 / 37 / 38 / 61, with two and
// ranges of two tiles 38 / 55 / 60 / 70, in one range by waves of one target per
// lane 32 / 42 / 60 / 322.  (Ranges of 128: 33 / 33 / 33 / 65, but 32 instead of 30
// at 200, where the second launch costs what they save.)
struct DirectPlan {
  int tpl, splits;
  int64_t range;
};
static DirectPlan direct_plan(int64_t n, int64_t nt) {
  auto blocks = [&](int tpl) { return (nt + 64 * tpl - 1) / (64 * tpl); };
  const int64_t tiles = (n + kDTile - 1) / kDTile;
  const int tpl = blocks(2) * tiles >= 4 * 1024 ? 2 : 1;
  const int64_t want = (8 * 1024 + blocks(tpl) - 1) / blocks(tpl);
  const int64_t k = std::max<int64_t>(1, std::min<int64_t>({want, tiles, 1024}));
  const int64_t per = (tiles + k - 1) / k;
  return {tpl, (int)((tiles + per - 1) / per), per * kDTile};  // no empty range
}

int64_t direct_scratch_bytes(int64_t n, int64_t nt) {
  if (nt <= 0) return 0;
  const int splits = direct_plan(n, nt).splits;
  return splits > 1 ? 32 * (int64_t)splits * nt : 0;
}

int launch_direct(const DevTree& T, const int32_t* targets, int64_t nt, float eps, float* acc,
                  float* pot, void* scratch, void* stream) {
  if (nt <= 0) return 0;
  hipStream_t s = (hipStream_t)stream;
  DirectPlan d = direct_plan(T.n, nt);
  if (d.splits > 1 && !scratch) d = {d.tpl, 1, T.n};
  const dim3 grid((nt + 64 * d.tpl - 1) / (64 * d.tpl), d.splits);
  float4* p = d.splits > 1 ? (float4*)scratch : nullptr;
  auto* k = d.tpl == 2 ? direct_kernel<2> : direct_kernel<1>;
  k<<<grid, 64, 0, s>>>(T, targets, nt, eps * eps, d.range, p, acc, pot);
  if (p)
    direct_combine_kernel<<<(nt + kThreads / kDLanes - 1) / (kThreads / kDLanes), kThreads, 0, s>>>(
        T, targets, nt, eps * eps, d.splits, p, acc, pot);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_mac_labels(const DevTree& T, const WalkBufs& B, const int32_t* groups, int64_t ngs,
                      const int64_t* out_off, const float* acc_direct, float eps, float* feat,
                      float* label, int32_t* gout, int32_t* cout, int64_t npairs, void* stream) {
  if (npairs <= 0) return 0;
  mac_label_kernel<<<npairs, kThreads, 0, (hipStream_t)stream>>>(
      T, B, groups, ngs, out_off, acc_direct, eps * eps, feat, label, gout, cout);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace octgrav
