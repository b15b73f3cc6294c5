// Time integration around the force call: kick-drift-kick leapfrog on
// device-resident FP32 positions and velocities, and the FP64 kinetic energy
// and momentum of the state (energy-conservation runs, Sec. 3).
#include <hip/hip_runtime.h>

#include "octgrav_internal.h"

namespace octgrav {
namespace {

constexpr int kT = 256;
constexpr int kKinBlocks = 512;

// v += h a (n x 3 FP32)
__global__ void kick_kernel(float* __restrict__ vel, const float* __restrict__ acc, int64_t n3,
                            float h) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i < n3) vel[i] = fmaf(h, acc[i], vel[i]);
}

// The start of a step: v += h a, x += dt v; BOTH: after the half-kick that ends
// the step before, v += h a with the same a.  Bound by launches up to about 10^5
// particles, then by HBM.  Two kicks and a drift of their own were 3 x 2.1 us
// of a 155 us step of 5000 particles and 3 x 3.2 us of 790 at 262144; this is one
// launch of 2.4 and 4.2 us, each velocity rounded after each kick as before.
template <bool BOTH>
__global__ void kick_drift_kernel(float* __restrict__ pos, float* __restrict__ vel,
                                  const float* __restrict__ acc, int64_t n3, float h, float dt) {
  const int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (i >= n3) return;
  const float a = acc[i];
  float v = vel[i];
  if (BOTH) v = fmaf(h, a, v);
  v = fmaf(h, a, v);
  vel[i] = v;
  pos[i] = fmaf(dt, v, pos[i]);
}

// Per-block FP64 sums of (1/2 m v^2, m vx, m vy, m vz), then one block adds
// the block sums in a fixed order (deterministic).
__global__ __launch_bounds__(kT) void kin_partial_kernel(const float* __restrict__ mass,
                                                         const float* __restrict__ vel, int64_t n,
                                                         double* __restrict__ part) {
  __shared__ double sh[4][kT];
  double s[4] = {0, 0, 0, 0};
  for (int64_t i = (int64_t)blockIdx.x * kT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kT) {
    const double m = mass[i], vx = vel[3 * i], vy = vel[3 * i + 1], vz = vel[3 * i + 2];
    s[0] += 0.5 * m * (vx * vx + vy * vy + vz * vz);
    s[1] += m * vx;
    s[2] += m * vy;
    s[3] += m * vz;
  }
  for (int k = 0; k < 4; ++k) sh[k][threadIdx.x] = s[k];
  __syncthreads();
  for (int o = kT / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o)
      for (int k = 0; k < 4; ++k) sh[k][threadIdx.x] += sh[k][threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x < 4) part[4 * blockIdx.x + threadIdx.x] = sh[threadIdx.x][0];
}

// (A block, two block sums per thread: with four threads running through the
// 512 sums one dependent load at a time this took 62 us.)
__global__ __launch_bounds__(kT) void kin_final_kernel(const double* __restrict__ part,
                                                       double* __restrict__ out) {
  static_assert(kKinBlocks == 2 * kT, "two block sums per thread");
  __shared__ double sh[4][kT];
  const int t = threadIdx.x;
  for (int k = 0; k < 4; ++k) sh[k][t] = part[4 * t + k] + part[4 * (t + kT) + k];
  __syncthreads();
  for (int o = kT / 2; o > 0; o >>= 1) {
    if (t < o)
      for (int k = 0; k < 4; ++k) sh[k][t] += sh[k][t + o];
    __syncthreads();
  }
  if (t < 4) out[t] = sh[t][0];
}

}  // namespace

int launch_kick(float* vel, const float* acc, int64_t n, float h, void* stream) {
  if (n <= 0) return 0;
  kick_kernel<<<(3 * n + kT - 1) / kT, kT, 0, (hipStream_t)stream>>>(vel, acc, 3 * n, h);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_kick_drift(float* pos, float* vel, const float* acc, int64_t n, float h, float dt,
                      bool both, void* stream) {
  if (n <= 0) return 0;
  auto* k = both ? kick_drift_kernel<true> : kick_drift_kernel<false>;
  k<<<(3 * n + kT - 1) / kT, kT, 0, (hipStream_t)stream>>>(pos, vel, acc, 3 * n, h, dt);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int64_t kinetic_scratch_entries() { return 4 * kKinBlocks; }

int launch_kinetic(const float* mass, const float* vel, int64_t n, double* part, double* out4,
                   void* stream) {
  hipStream_t s = (hipStream_t)stream;
  kin_partial_kernel<<<kKinBlocks, kT, 0, s>>>(mass, vel, n, part);
  kin_final_kernel<<<1, kT, 0, s>>>(part, out4);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace octgrav
