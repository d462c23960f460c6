// k_misc.hip -- direct summation (Eq. 1) and the leapfrog kick / drift.
#include <algorithm>

#include "nbody_internal.h"

namespace nb {

// Eq. 1 by direct summation, FP32: the interaction arithmetic of the walk's
// flush, so it calibrates the walk's arithmetic rate. The j == i term
// contributes exactly zero because eps > 0. A workgroup takes kTg targets and
// all particles, staged in LDS; its 256 / kTg streams of kTg lanes take every
// (256 / kTg)-th particle and their sums are added in a fixed order. With one
// target per lane (kTg = 256) a few thousand particles filled 16 CUs of 256:
// 4096 particles 131 us, 10.6 us with 4 targets per workgroup.
template <int kTg>
__global__ __launch_bounds__(256) void k_direct(int64_t n, const float *__restrict__ x,
                                                const float *__restrict__ y,
                                                const float *__restrict__ z,
                                                const float *__restrict__ m, float G,
                                                float eps2, float *__restrict__ ax,
                                                float *__restrict__ ay,
                                                float *__restrict__ az) {
  constexpr int kStreams = 256 / kTg;
  constexpr int kTile = kTg == 256 ? 256 : 1024;
  __shared__ float4 tile[kTile];
  const int t = threadIdx.x % kTg, stream = threadIdx.x / kTg;
  const int64_t i = blockIdx.x * (int64_t)kTg + t;
  float4 pi = make_float4(0.f, 0.f, 0.f, 0.f);
  if (i < n) pi = make_float4(x[i], y[i], z[i], m[i]);
  float sx = 0.f, sy = 0.f, sz = 0.f;
  for (int64_t j0 = 0; j0 < n; j0 += kTile) {
#pragma unroll
    for (int q = 0; q < kTile; q += 256) {
      const int64_t j = j0 + q + threadIdx.x;
      tile[q + threadIdx.x] =
          j < n ? make_float4(x[j], y[j], z[j], m[j]) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __syncthreads();
    const int cnt = (int)min((int64_t)kTile, n - j0);
    float ux = 0.f, uy = 0.f, uz = 0.f;  // the tile's sum (shorter chains of roundings)
#pragma unroll 8
    for (int k = stream; k < cnt; k += kStreams) {
      const float4 e = tile[k];
      const float dx = e.x - pi.x, dy = e.y - pi.y, dz = e.z - pi.z;
      const float r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, __builtin_fmaf(dx, dx, eps2)));
      const float rinv = __builtin_amdgcn_rsqf(r2);
      const float mr = e.w * rinv;
      const float f = mr * (rinv * rinv);
      ux = __builtin_fmaf(f, dx, ux);
      uy = __builtin_fmaf(f, dy, uy);
      uz = __builtin_fmaf(f, dz, uz);
    }
    sx += ux;
    sy += uy;
    sz += uz;
    __syncthreads();
  }
  if constexpr (kTg < 256) {
    for (int d = kTg; d < 64; d <<= 1) {
      sx += __shfl_xor(sx, d, 64);
      sy += __shfl_xor(sy, d, 64);
      sz += __shfl_xor(sz, d, 64);
    }
    // (the tile is free: one sum per wavefront and target)
    if (lane_id() < kTg) tile[(threadIdx.x >> 6) * kTg + lane_id()] = make_float4(sx, sy, sz, 0.f);
    __syncthreads();
    if (threadIdx.x >= kTg) return;
    sx = ((tile[t].x + tile[kTg + t].x) + tile[2 * kTg + t].x) + tile[3 * kTg + t].x;
    sy = ((tile[t].y + tile[kTg + t].y) + tile[2 * kTg + t].y) + tile[3 * kTg + t].y;
    sz = ((tile[t].z + tile[kTg + t].z) + tile[2 * kTg + t].z) + tile[3 * kTg + t].z;
  }
  if (i < n) {
    ax[i] = G * sx;
    ay[i] = G * sy;
    az[i] = G * sz;
  }
}

// Eq. 1 in FP64 for a subset of targets (the accuracy reference of the tree
// walk): inputs are FP32 positions and masses promoted to FP64; every pair
// j != i (by index) adds G m_j dx / (r^2 + eps^2)^(3/2) to a_i, G m_j |dx| /
// (r^2 + eps^2)^(3/2) to the scale A_i and -G m_j / (r^2 + eps^2)^(1/2) to
// phi_i. Bound by FP64 VALU issue: about 45 FP64 instructions per pair. A
// workgroup takes kD64Targets targets and a slice of the particles, each
// thread every 256th (kThreads-th) particle of the slice for all the targets (a load serves
// four pairs, no LDS); sums over the workgroup's threads in a fixed order.
// Slices fill the chip when there are few targets; their sums are added in
// slice order, by k_direct64_fold or (without scratch) in the workgroup, to
// the same bits. 2048 targets of 2^20 particles: 64 workgroups of 32 targets
// took 37.3 ms (a quarter of the CUs, IEEE square roots and divisions), this
// form 2.9 ms.
constexpr int kD64Targets = 4;
constexpr int kD64Out = 5 * kD64Targets;  // sums of a workgroup: [target][5]

// 1 / sqrt(x) for finite x > 0: the hardware's estimate and one third-order
// step, within about 1 ulp.
__device__ __forceinline__ double rsqrt_refined(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = __builtin_fma(-x * y, y, 1.0);
  return __builtin_fma(y * e, __builtin_fma(0.375, e, 0.5), y);
}

// Adds the pair (target, particle j) to the target's five sums.
__device__ __forceinline__ void pair64(double (&a)[5], double dx, double dy, double dz,
                                       double mj, double eps2) {
  const double d2 = __builtin_fma(dz, dz, __builtin_fma(dy, dy, dx * dx));
  const double r2 = d2 + eps2;
  const double rinv = r2 < INFINITY ? rsqrt_refined(r2) : __builtin_amdgcn_rsq(r2);
  // |dx|: squares of FP32 differences are 0 or over 1e-90
  const double d = d2 * rsqrt_refined(d2 + 1e-300);
  const double mr = mj * rinv;
  const double w = mr * (rinv * rinv);
  a[0] = __builtin_fma(w, dx, a[0]);
  a[1] = __builtin_fma(w, dy, a[1]);
  a[2] = __builtin_fma(w, dz, a[2]);
  a[3] = __builtin_fma(w, d, a[3]);
  a[4] -= mr;
}

template <int kThreads>
__global__ __launch_bounds__(kThreads) void k_direct64(
    int64_t n, const float *__restrict__ x, const float *__restrict__ y,
    const float *__restrict__ z, const float *__restrict__ m, int64_t nt,
    const int64_t *__restrict__ tgt, double G, double eps2, int slices, int64_t slice_len,
    double *__restrict__ part, double *__restrict__ ax, double *__restrict__ ay,
    double *__restrict__ az, double *__restrict__ aabs, double *__restrict__ phi) {
  __shared__ double s_sum[kThreads / 64][kD64Out];
  const int64_t k0 = (int64_t)blockIdx.x * kD64Targets;
  double xi[kD64Targets], yi[kD64Targets], zi[kD64Targets];
  int64_t it[kD64Targets];
#pragma unroll
  for (int t = 0; t < kD64Targets; ++t) {
    int64_t i = k0 + t < nt ? tgt[k0 + t] : -1;
    if (i >= n || i < 0) i = -1;  // a target outside [0, n) sums nothing
    it[t] = i;
    const int64_t ii = i < 0 ? 0 : i;
    xi[t] = x[ii];
    yi[t] = y[ii];
    zi[t] = z[ii];
  }
  double total = 0.0;  // thread q < kD64Out: sum q over the slices
  const int s0 = part ? (int)blockIdx.y : 0, s1 = part ? s0 + 1 : slices;
  for (int sl = s0; sl < s1; ++sl) {
    const int64_t j0 = sl * slice_len, j1 = min(n, j0 + slice_len);
    double a[kD64Targets][5];
#pragma unroll
    for (int t = 0; t < kD64Targets; ++t)
#pragma unroll
      for (int c = 0; c < 5; ++c) a[t][c] = 0.0;
    for (int64_t jb = j0; jb < j1; jb += kThreads) {
      const int64_t j = jb + threadIdx.x;
      bool self = false;  // (uniform) some target is among these particles
#pragma unroll
      for (int t = 0; t < kD64Targets; ++t) self |= it[t] >= jb && it[t] < jb + kThreads;
      if (j >= j1) continue;
      const double xj = x[j], yj = y[j], zj = z[j], mj = m[j];
      if (self) {
#pragma unroll
        for (int t = 0; t < kD64Targets; ++t)
          if (j != it[t]) pair64(a[t], xj - xi[t], yj - yi[t], zj - zi[t], mj, eps2);
      } else {
#pragma unroll
        for (int t = 0; t < kD64Targets; ++t)
          pair64(a[t], xj - xi[t], yj - yi[t], zj - zi[t], mj, eps2);
      }
    }
    __syncthreads();  // s_sum's last use
#pragma unroll
    for (int t = 0; t < kD64Targets; ++t)
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        double v = a[t][c];
        for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
        if (lane_id() == 0) s_sum[threadIdx.x >> 6][5 * t + c] = v;
      }
    __syncthreads();
    if (threadIdx.x < kD64Out) {
      const int q = threadIdx.x;
      double v = s_sum[0][q];
#pragma unroll
      for (int w = 1; w < kThreads / 64; ++w) v += s_sum[w][q];
      if (part)
        part[((int64_t)blockIdx.x * slices + sl) * kD64Out + q] = v;
      else
        total += v;
    }
  }
  if (part || threadIdx.x >= kD64Out) return;
  const int64_t k = k0 + threadIdx.x / 5;
  if (k >= nt) return;
  int64_t i = tgt[k];
  if (i >= n || i < 0) total = 0.0;
  double *const out[5] = {ax, ay, az, aabs, phi};
  double *o = out[threadIdx.x % 5];
  if (o) o[k] = G * total;
}

// The slices' sums of each target, in slice order.
__global__ __launch_bounds__(256) void k_direct64_fold(
    int64_t n, int64_t nt, const int64_t *__restrict__ tgt, double G, int slices,
    const double *__restrict__ part, double *__restrict__ ax, double *__restrict__ ay,
    double *__restrict__ az, double *__restrict__ aabs, double *__restrict__ phi) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;  // (target, sum)
  const int64_t k = e / 5, b = k / kD64Targets;
  if (k >= nt) return;
  const int q = (int)(e - b * kD64Out);
  double total = 0.0;
  for (int sl = 0; sl < slices; ++sl) total += part[(b * slices + sl) * kD64Out + q];
  const int64_t i = tgt[k];
  if (i >= n || i < 0) total = 0.0;
  double *const out[5] = {ax, ay, az, aabs, phi};
  double *o = out[e % 5];
  if (o) o[k] = G * total;
}

// v += a * (dt/2), FP32, one rounding per operation.
__global__ __launch_bounds__(256) void k_kick(int64_t n, float *__restrict__ vx,
                                              float *__restrict__ vy, float *__restrict__ vz,
                                              const float *__restrict__ ax,
                                              const float *__restrict__ ay,
                                              const float *__restrict__ az, float hdt) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float kx = ax[i] * hdt, ky = ay[i] * hdt, kz = az[i] * hdt;
    vx[i] = vx[i] + kx;
    vy[i] = vy[i] + ky;
    vz[i] = vz[i] + kz;
  }
}

// x += v * dt in FP64 and the FP32 image of x for the tree.
__global__ __launch_bounds__(256) void k_drift(int64_t n, double *__restrict__ x,
                                               double *__restrict__ y,
                                               double *__restrict__ z,
                                               const float *__restrict__ vx,
                                               const float *__restrict__ vy,
                                               const float *__restrict__ vz, double dt,
                                               float *__restrict__ x32, SortedOut so) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const double dx = (double)vx[i] * dt, dy = (double)vy[i] * dt, dz = (double)vz[i] * dt;
    const double nx = x[i] + dx, ny = y[i] + dy, nz = z[i] + dz;
    x[i] = nx;
    y[i] = ny;
    z[i] = nz;
    store_position(i, n, (float)nx, (float)ny, (float)nz, x32, so);
  }
}

// Second-order Runge-Kutta (Heun) step, predict: x_p = x + v dt in FP64.
// Only the FP32 image of x_p is stored (for the tree and the walk); the state
// keeps x, v for the correction.
__global__ __launch_bounds__(256) void k_rk2_predict(int64_t n, const double *__restrict__ x,
                                                     const double *__restrict__ y,
                                                     const double *__restrict__ z,
                                                     const float *__restrict__ vx,
                                                     const float *__restrict__ vy,
                                                     const float *__restrict__ vz, double dt,
                                                     float *__restrict__ x32, SortedOut so) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const double px = x[i] + (double)vx[i] * dt, py = y[i] + (double)vy[i] * dt,
                 pz = z[i] + (double)vz[i] * dt;
    store_position(i, n, (float)px, (float)py, (float)pz, x32, so);
  }
}

// Correct: with v_p = v + a dt (FP32), x += (v + v_p) dt/2 (FP64, the sum in
// FP64) and v += (a + a_p) dt/2 (FP32), one rounding per operation; the FP32
// image of the new x for the tree.
__global__ __launch_bounds__(256) void k_rk2_correct(
    int64_t n, double *__restrict__ x, double *__restrict__ y, double *__restrict__ z,
    float *__restrict__ vx, float *__restrict__ vy, float *__restrict__ vz,
    const float *__restrict__ ax, const float *__restrict__ ay, const float *__restrict__ az,
    const float *__restrict__ apx, const float *__restrict__ apy,
    const float *__restrict__ apz, double dt, float dt32, float hdt32,
    float *__restrict__ x32, SortedOut so) {
  const double hdt = 0.5 * dt;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float v0x = vx[i], v0y = vy[i], v0z = vz[i];
    const float a0x = ax[i], a0y = ay[i], a0z = az[i];
    const float kx = a0x * dt32, ky = a0y * dt32, kz = a0z * dt32;
    const float vpx = v0x + kx, vpy = v0y + ky, vpz = v0z + kz;
    const double sx = (double)v0x + (double)vpx, sy = (double)v0y + (double)vpy,
                 sz = (double)v0z + (double)vpz;
    const double nx = x[i] + sx * hdt, ny = y[i] + sy * hdt, nz = z[i] + sz * hdt;
    const float bx = a0x + apx[i], by = a0y + apy[i], bz = a0z + apz[i];
    const float hx = bx * hdt32, hy = by * hdt32, hz = bz * hdt32;
    x[i] = nx;
    y[i] = ny;
    z[i] = nz;
    vx[i] = v0x + hx;
    vy[i] = v0y + hy;
    vz[i] = v0z + hz;
    store_position(i, n, (float)nx, (float)ny, (float)nz, x32, so);
  }
}

static int grid_1d(int64_t n) {
  int64_t g = cdiv(n, 256 * 4);
  if (g > 8192) g = 8192;
  if (g < 1) g = 1;
  return (int)g;
}

void launch_direct(int64_t n, const float *x, const float *y, const float *z,
                   const float *m, float G, float eps, float *ax, float *ay, float *az,
                   hipStream_t st) {
  // the most targets per workgroup that still make four workgroups per CU
  auto go = [&](auto kernel, int64_t tg) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)cdiv(n, tg)), dim3(256), 0, st, n, x, y, z, m, G,
                       eps * eps, ax, ay, az);
  };
  if (n >= 256 * 1024)
    go(k_direct<256>, 256);
  else if (n >= 64 * 1024)
    go(k_direct<64>, 64);
  else if (n >= 16 * 1024)
    go(k_direct<16>, 16);
  else
    go(k_direct<4>, 4);
}

void launch_direct64(int64_t n, const float *x, const float *y, const float *z,
                     const float *m, int64_t nt, const int64_t *tgt, double G, double eps,
                     double *ax, double *ay, double *az, double *aabs, double *phi,
                     double *part, int64_t part_words, hipStream_t st) {
  // about 2048 workgroups (eight per CU; five are resident), each thread with
  // two particles at least; the same slices with and without scratch
  const int64_t groups = cdiv(nt, kD64Targets);
  const int slices = (int)std::max<int64_t>(1, std::min<int64_t>(2048 / groups, cdiv(n, 512)));
  const int64_t slice_len = cdiv(n, slices);
  if (slices == 1 || groups * slices * kD64Out > part_words) part = nullptr;
  const auto go = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)groups, part ? slices : 1), dim3(threads), 0, st, n,
                       x, y, z, m, nt, tgt, G, eps * eps, slices, slice_len, part, ax, ay, az,
                       aabs, phi);
  };
  // targets by the thousand over a few hundred particles: the sums over the
  // workgroup's threads are the work (a call of 9000 targets, 257 particles: 53 us with 256
  // threads, 36 with 64; 34 with 32 targets per workgroup)
  if (n <= 512 && groups >= 1024)
    go(k_direct64<64>, 64);
  else
    go(k_direct64<256>, 256);
  if (part)
    hipLaunchKernelGGL(k_direct64_fold, dim3((unsigned)cdiv(5 * nt, 256)), dim3(256), 0, st, n,
                       nt, tgt, G, slices, part, ax, ay, az, aabs, phi);
}

void launch_kick(int64_t n, float *vx, float *vy, float *vz, const float *ax,
                 const float *ay, const float *az, float hdt, hipStream_t st) {
  hipLaunchKernelGGL(k_kick, dim3(grid_1d(n)), dim3(256), 0, st, n, vx, vy, vz, ax, ay, az,
                     hdt);
}

void launch_drift(int64_t n, double *x, double *y, double *z, const float *vx,
                  const float *vy, const float *vz, double dt, float *x32, SortedOut so,
                  hipStream_t st) {
  hipLaunchKernelGGL(k_drift, dim3(grid_1d(n)), dim3(256), 0, st, n, x, y, z, vx, vy, vz,
                     dt, x32, so);
}

void launch_rk2_predict(int64_t n, const double *x, const double *y, const double *z,
                        const float *vx, const float *vy, const float *vz, double dt,
                        float *x32, SortedOut so, hipStream_t st) {
  hipLaunchKernelGGL(k_rk2_predict, dim3(grid_1d(n)), dim3(256), 0, st, n, x, y, z, vx, vy, vz,
                     dt, x32, so);
}

void launch_rk2_correct(int64_t n, double *x, double *y, double *z, float *vx, float *vy,
                        float *vz, const float *ax, const float *ay, const float *az,
                        const float *apx, const float *apy, const float *apz, double dt,
                        float *x32, SortedOut so, hipStream_t st) {
  hipLaunchKernelGGL(k_rk2_correct, dim3(grid_1d(n)), dim3(256), 0, st, n, x, y, z, vx, vy, vz,
                     ax, ay, az, apx, apy, apz, dt, (float)dt, (float)(0.5 * dt), x32, so);
}

// asort[s] = (a, |a|) of caller index perm[s]; |a| rounded as in the MAC.
__global__ __launch_bounds__(256) void k_asort_gather(const uint32_t *__restrict__ perm,
                                                      int64_t n, const float *__restrict__ ax,
                                                      const float *__restrict__ ay,
                                                      const float *__restrict__ az,
                                                      float4 *__restrict__ asort) {
  for (int64_t s = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; s < n;
       s += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t o = perm[s];
    const float x = ax[o], y = ay[o], z = az[o];
    asort[s] = make_float4(x, y, z, sqrt_rn(__builtin_fmaf(z, z, __builtin_fmaf(y, y, x * x))));
  }
}

void launch_asort_gather(const uint32_t *perm, int64_t n, const float *ax, const float *ay,
                         const float *az, float4 *asort, hipStream_t st) {
  int64_t g = cdiv(n, 256 * 4);
  if (g > 8192) g = 8192;
  if (g < 1) g = 1;
  hipLaunchKernelGGL(k_asort_gather, dim3(g), dim3(256), 0, st, perm, n, ax, ay, az, asort);
}

// After a rebuild: the mirror in the new key order from the mirror in the
// old one, tmp[s] = asort[inv_old[perm_new[s]]], then copied back. Particles
// move little between builds, so the reads of the old mirror are nearly in
// order (one random 4-byte read of inv_old instead of three of a_old).
__global__ __launch_bounds__(256) void k_asort_remap(const uint32_t *__restrict__ perm,
                                                     const uint32_t *__restrict__ inv_old,
                                                     int64_t n, const float4 *__restrict__ asort,
                                                     float4 *__restrict__ tmp) {
  for (int64_t s = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; s < n;
       s += (int64_t)gridDim.x * blockDim.x)
    tmp[s] = asort[inv_old[perm[s]]];
}

__global__ __launch_bounds__(256) void k_copy_f4(const float4 *__restrict__ src, int64_t n,
                                                 float4 *__restrict__ dst) {
  for (int64_t s = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; s < n;
       s += (int64_t)gridDim.x * blockDim.x)
    dst[s] = src[s];
}

void launch_asort_remap(const uint32_t *perm, const uint32_t *inv_old, int64_t n,
                        float4 *asort, float4 *tmp, hipStream_t st) {
  int64_t g = cdiv(n, 256 * 4);
  if (g > 8192) g = 8192;
  if (g < 1) g = 1;
  hipLaunchKernelGGL(k_asort_remap, dim3(g), dim3(256), 0, st, perm, inv_old, n, asort, tmp);
  hipLaunchKernelGGL(k_copy_f4, dim3(g), dim3(256), 0, st, tmp, n, asort);
}

}  // namespace nb
