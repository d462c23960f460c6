// k_cost.hip -- cost model of the walk's work queue: per-group features, a
// small tanh MLP (inference, backward pass, Adam) and the queue order by
// predicted cost.
//
// Features of group g (all FP32): log2 of its particle count; log2(h +
// 2^-40) with h half the diagonal of the members' box; log2 of its mass minus
// three times the previous feature (a density); log2(1 + the members' mean
// list length from their last walk). The last one is kept per particle in
// caller order and cleared at every rebuild (0 = not walked on the current
// tree): a length measured on an aged tree overstates the work on a fresh
// one. The target is log2 of the group's interactions (members x list
// entries).
//
// The order never changes the results: a group's list and its summation
// order depend on the group alone.
#include "nbody_internal.h"

namespace nb {

constexpr float kDensityFloor = 0x1p-40f;

__device__ __forceinline__ float wave_sum_f(float v) {
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}

__device__ __forceinline__ uint32_t wave_sum_u(uint32_t v) {
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}

// One wavefront per group (wave-uniform loop; all lanes store the result).
__global__ __launch_bounds__(256) void k_cost_features(
    const DevScalars *__restrict__ sc, const uint32_t *__restrict__ queue,
    const uint32_t *__restrict__ gbegin, const uint32_t *__restrict__ gcount,
    const float4 *__restrict__ xyzm, const uint32_t *__restrict__ perm,
    const uint32_t *__restrict__ plast, float4 *__restrict__ feat) {
  const uint32_t nq = queue ? sc->nqueue : sc->ngroup;
  const uint32_t wstride = gridDim.x * (blockDim.x >> 6);
  const uint32_t q0 = __builtin_amdgcn_readfirstlane(blockIdx.x * (blockDim.x >> 6) +
                                                     (threadIdx.x >> 6));
  for (uint32_t q = q0; q < nq; q += wstride) {
    const uint32_t g = queue ? queue[q] : q;
    const uint32_t b = gbegin[g], c = gcount[g];
    const uint32_t k = lane_id();
    const bool ok = k < c;
    const float4 p = xyzm[b + (ok ? k : 0u)];
    const uint32_t pl = ok ? plast[perm[b + k]] : 0u;
    const float ex = wave_max(p.x) - wave_min(p.x);
    const float ey = wave_max(p.y) - wave_min(p.y);
    const float ez = wave_max(p.z) - wave_min(p.z);
    const float mass = wave_sum_f(ok ? p.w : 0.0f);
    const uint32_t psum = wave_sum_u(pl);
    const float h = 0.5f * sqrtf(__builtin_fmaf(ez, ez, __builtin_fmaf(ey, ey, ex * ex)));
    const float f1 = log2f(h + kDensityFloor);
    float4 f;
    f.x = log2f((float)c);
    f.y = f1;
    f.z = log2f(mass) - 3.0f * f1;
    f.w = log2f(1.0f + (float)psum / (float)c);
    feat[g] = f;
  }
}

// After a walk: each walked group's list length to its members, and the
// training target. queue == nullptr: every group was walked.
__global__ __launch_bounds__(256) void k_cost_after(
    const DevScalars *__restrict__ sc, const uint32_t *__restrict__ queue,
    const uint32_t *__restrict__ gbegin, const uint32_t *__restrict__ gcount,
    const uint32_t *__restrict__ gent, const uint32_t *__restrict__ perm,
    uint32_t *__restrict__ plast, float *__restrict__ target) {
  const uint32_t nq = queue ? sc->nqueue : sc->ngroup;
  const uint32_t wstride = gridDim.x * (blockDim.x >> 6);
  const uint32_t q0 = __builtin_amdgcn_readfirstlane(blockIdx.x * (blockDim.x >> 6) +
                                                     (threadIdx.x >> 6));
  for (uint32_t q = q0; q < nq; q += wstride) {
    const uint32_t g = queue ? queue[q] : q;
    const uint32_t b = gbegin[g], c = gcount[g], e = gent[g];
    const uint32_t k = lane_id();
    if (k < c && e != 0xffffffffu) plast[perm[b + k]] = e;
    target[g] = log2f(fmaxf(1.0f, (float)c * (float)e));
  }
}

// ---------------------------------------------------------------- MLP
// Weight layout (row-major, output-major): mu[4] is[4] W1[H][4] b1[H]
// W2[H][H] b2[H] W3[H] b3. The inputs are standardised first, z = (f - mu)
// * is; mu and is are constants of the model (set from the training data),
// not trained. The network's output is a correction to the size-based
// estimate f.x + f.w (log2 of the group size times one plus the members' mean
// previous list length): prediction = net(z) + (f.x + f.w).
__host__ __device__ constexpr int mlp_np(int H) { return 8 + 7 * H + H * H + 1; }

// The network on the matrix cores, FP32 in and FP32 accumulated. A wavefront
// takes tiles of 32 rows; a unit block is 32 hidden units (H < 32 is padded
// with zero weights). In the accumulator layout of the 32x32x2 instruction
// (lane l, register r: row rho(r) + 4 (l / 32), column l mod 32) a lane owns
// one unit of each block and 16 rows, so biases, W1 and W3 are per-lane
// registers and the elementwise parts need no exchange. Two of the three
// products read the rows along the other axis and go through a padded LDS tile
// (Z2 = H1 W2^T, D1 = D2 W2); the third (grad W2 = D2^T H1, summed over rows)
// takes both operands straight from the registers: any order of the rows is a
// valid order of the sum, if both use the same.
// 30000 rows, 32 units: one row at a time with a lane per unit (shuffles for
// every product, 256 wavefronts) took 176 us per gradient, this form 15 us.
typedef float f32x16 __attribute__((ext_vector_type(16)));
constexpr int kMlpTile = 32;
__device__ __forceinline__ int mlp_row(int r, uint32_t lane) {
  return (r & 3) + 8 * (r >> 2) + 4 * (int)(lane >> 5);
}

template <int H>
struct MlpShape {
  static constexpr int HB = H > 32 ? H / 32 : 1;  // unit blocks
  static constexpr int HP = 32 * HB;              // padded units
  static constexpr int LD = HP + 1;               // row stride in LDS (odd: no conflicts)
};

// LDS of one wavefront: the tile's inputs and targets and one row-major
// exchange tile.
template <int H>
struct MlpTile {
  float4 z[kMlpTile];    // standardised inputs
  float base[kMlpTile];  // f.x + f.w
  float tgt[kMlpTile];
  float x[kMlpTile * MlpShape<H>::LD];
};

// Per-lane weights of the lane's unit of each block.
template <int H>
struct MlpLane {
  static constexpr int HB = MlpShape<H>::HB;
  float4 w1[HB];
  float b1[HB], b2[HB], w3[HB], b3;
  __device__ __forceinline__ void load(const float *__restrict__ w, uint32_t lane) {
    const float *W1 = w + 8, *B1 = W1 + 4 * H, *B2 = B1 + H + H * H, *W3 = B2 + H;
#pragma unroll
    for (int ub = 0; ub < HB; ++ub) {
      const int u = 32 * ub + (int)(lane & 31u);
      const bool on = u < H;
      w1[ub] = on ? make_float4(W1[4 * u], W1[4 * u + 1], W1[4 * u + 2], W1[4 * u + 3])
                  : make_float4(0.f, 0.f, 0.f, 0.f);
      b1[ub] = on ? B1[u] : 0.f;
      b2[ub] = on ? B2[u] : 0.f;
      w3[ub] = on ? W3[u] : 0.f;
    }
    b3 = W3[H];
  }
};

// W2 into LDS, row stride LD, padded with zeros (whole workgroup).
template <int H>
__device__ __forceinline__ void mlp_stage_w2(const float *__restrict__ w, float *sW2) {
  constexpr int HP = MlpShape<H>::HP, LD = MlpShape<H>::LD;
  const float *W2 = w + 8 + 5 * H;
  for (int i = threadIdx.x; i < HP * HP; i += blockDim.x) {
    const int u = i / HP, k = i % HP;
    sW2[u * LD + k] = u < H && k < H ? W2[u * H + k] : 0.f;
  }
}

__device__ __forceinline__ void mlp_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Sum over the 32 lanes of each half wavefront, in every lane.
__device__ __forceinline__ float half_sum(float v) {
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xf, 0xf, true));   // xor 1
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xf, 0xf, true));   // xor 2
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xf, 0xf, true));  // half mirror
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x140, 0xf, 0xf, true));  // mirror
  return v + __shfl_xor(v, 16, 64);
}

// Forward pass of rows [r0, r0 + 32): h1, h2 per block and the 16 outputs of
// the lane's rows (network plus f.x + f.w). Rows past the end repeat the last.
template <int H>
__device__ __forceinline__ void mlp_tile_forward(const float *__restrict__ w, const float *sW2,
                                                 const MlpLane<H> &L, MlpTile<H> &t,
                                                 const float4 *__restrict__ feat, int64_t r0,
                                                 int64_t rows, uint32_t lane,
                                                 f32x16 (&h1)[MlpShape<H>::HB],
                                                 f32x16 (&h2)[MlpShape<H>::HB], f32x16 &y) {
  constexpr int HB = MlpShape<H>::HB, HP = MlpShape<H>::HP, LD = MlpShape<H>::LD;
  const int col = (int)(lane & 31u), half = (int)(lane >> 5);
  mlp_wave_sync();  // the tile's last use
  if (lane < 32u) {
    const int64_t r = min(r0 + lane, rows - 1);
    const float4 f = feat[r];
    t.z[lane] = make_float4((f.x - w[0]) * w[4], (f.y - w[1]) * w[5], (f.z - w[2]) * w[6],
                            (f.w - w[3]) * w[7]);
    t.base[lane] = f.x + f.w;
  }
  mlp_wave_sync();
#pragma unroll
  for (int ub = 0; ub < HB; ++ub)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float4 z = t.z[mlp_row(r, lane)];
      float s = L.b1[ub];
      s = __builtin_fmaf(L.w1[ub].x, z.x, s);
      s = __builtin_fmaf(L.w1[ub].y, z.y, s);
      s = __builtin_fmaf(L.w1[ub].z, z.z, s);
      s = __builtin_fmaf(L.w1[ub].w, z.w, s);
      // (a padded unit is 0 whatever the inputs: with zero weights alone an
      // infinite feature, a group without mass, would make it NaN)
      const float h = 32 * ub + col < H ? tanhf(s) : 0.f;
      h1[ub][r] = h;
      t.x[mlp_row(r, lane) * LD + 32 * ub + col] = h;
    }
  mlp_wave_sync();
#pragma unroll
  for (int ub = 0; ub < HB; ++ub)
#pragma unroll
    for (int r = 0; r < 16; ++r) h2[ub][r] = L.b2[ub];
#pragma unroll
  for (int k = 0; k < HP; k += 2) {
    const float a = t.x[col * LD + k + half];
#pragma unroll
    for (int ub = 0; ub < HB; ++ub)
      h2[ub] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, sW2[(32 * ub + col) * LD + k + half],
                                                    h2[ub], 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    float p = 0.f;
#pragma unroll
    for (int ub = 0; ub < HB; ++ub) {
      h2[ub][r] = tanhf(h2[ub][r]);
      p = __builtin_fmaf(L.w3[ub], h2[ub][r], p);
    }
    y[r] = (L.b3 + half_sum(p)) + t.base[mlp_row(r, lane)];
  }
}

// Forward pass of few hidden units (H < 32): one thread per row, the weights
// in LDS. Padded to 32 units the tiles below do 4 or 16 times the work
// (200000 rows, 8 units: 31 us a call, this form 19; 30000 rows: 20.7 and 18.3;
// with 32 and more units the tiles are the faster form).
template <int H>
__global__ __launch_bounds__(256) void k_mlp_forward_rows(const float *__restrict__ w,
                                                          int64_t rows,
                                                          const uint32_t *__restrict__ rows_dev,
                                                          const float4 *__restrict__ feat,
                                                          float *__restrict__ y) {
  __shared__ float sw[mlp_np(H)];
  const int64_t nr = rows_dev ? min(rows, (int64_t)*rows_dev) : rows;
  if ((int64_t)blockIdx.x * blockDim.x >= nr) return;  // whole workgroup: no rows
  for (int i = threadIdx.x; i < mlp_np(H); i += blockDim.x) sw[i] = w[i];
  __syncthreads();
  const float *mu = sw, *is = sw + 4, *W1 = sw + 8, *b1 = W1 + 4 * H, *W2 = b1 + H,
              *b2 = W2 + H * H, *W3 = b2 + H, *b3 = W3 + H;
  for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < nr;
       r += (int64_t)gridDim.x * blockDim.x) {
    const float4 fr = feat[r];
    const float4 f = make_float4((fr.x - mu[0]) * is[0], (fr.y - mu[1]) * is[1],
                                 (fr.z - mu[2]) * is[2], (fr.w - mu[3]) * is[3]);
    float h1[H];
#pragma unroll
    for (int u = 0; u < H; ++u) {
      float s = b1[u];
      s = __builtin_fmaf(W1[4 * u + 0], f.x, s);
      s = __builtin_fmaf(W1[4 * u + 1], f.y, s);
      s = __builtin_fmaf(W1[4 * u + 2], f.z, s);
      s = __builtin_fmaf(W1[4 * u + 3], f.w, s);
      h1[u] = tanhf(s);
    }
    float out = b3[0];
#pragma unroll
    for (int u = 0; u < H; ++u) {
      float s = b2[u];
#pragma unroll
      for (int k = 0; k < H; ++k) s = __builtin_fmaf(W2[u * H + k], h1[k], s);
      out = __builtin_fmaf(W3[u], tanhf(s), out);
    }
    y[r] = out + (fr.x + fr.w);
  }
}

// Forward pass only. rows_dev (optional) bounds the rows on the device.
template <int H>
__global__ __launch_bounds__(256) void k_mlp_forward(const float *__restrict__ w, int64_t rows,
                                                     const uint32_t *__restrict__ rows_dev,
                                                     const float4 *__restrict__ feat,
                                                     float *__restrict__ out) {
  __shared__ float sW2[MlpShape<H>::HP * MlpShape<H>::LD];
  __shared__ MlpTile<H> tiles[4];
  const int64_t nr = rows_dev ? min(rows, (int64_t)*rows_dev) : rows;
  if ((int64_t)blockIdx.x * 4 * kMlpTile >= nr) return;  // whole workgroup: no rows
  mlp_stage_w2<H>(w, sW2);
  __syncthreads();
  const uint32_t lane = lane_id(), wv = threadIdx.x >> 6;
  MlpLane<H> L;
  L.load(w, lane);
  for (int64_t r0 = ((int64_t)blockIdx.x * 4 + wv) * kMlpTile; r0 < nr;
       r0 += (int64_t)gridDim.x * 4 * kMlpTile) {
    f32x16 h1[MlpShape<H>::HB], h2[MlpShape<H>::HB], y;
    mlp_tile_forward<H>(w, sW2, L, tiles[wv], feat, r0, nr, lane, h1, h2, y);
    // lanes 0 and 32 hold all 32 outputs: through LDS for one coalesced store
    mlp_wave_sync();
    if ((lane & 31u) == 0u)
#pragma unroll
      for (int r = 0; r < 16; ++r) tiles[wv].tgt[mlp_row(r, lane)] = y[r];
    mlp_wave_sync();
    if (lane < 32u && r0 + lane < nr) out[r0 + lane] = tiles[wv].tgt[lane];
  }
}

// Gradient of the mean squared error: every wavefront sums its tiles' shares in
// registers, the workgroup adds its wavefronts' in order, and share g goes to
// partial[g][0 .. np] (np = loss); the shares are added in order afterwards,
// so the result is deterministic.
template <int H>
__global__ __launch_bounds__(256) void k_mlp_grad(const float *__restrict__ w, int64_t rows,
                                                  const float4 *__restrict__ feat,
                                                  const float *__restrict__ target,
                                                  float *__restrict__ partial) {
  constexpr int HB = MlpShape<H>::HB, HP = MlpShape<H>::HP, LD = MlpShape<H>::LD;
  constexpr int np = mlp_np(H);
  __shared__ float sW2[HP * LD];
  __shared__ MlpTile<H> tiles[4];
  __shared__ float share[np + 1];
  mlp_stage_w2<H>(w, sW2);
  __syncthreads();
  const uint32_t lane = lane_id(), wv = threadIdx.x >> 6;
  const int col = (int)(lane & 31u), half = (int)(lane >> 5);
  MlpTile<H> &t = tiles[wv];
  MlpLane<H> L;
  L.load(w, lane);
  const float inv_rows = 1.0f / (float)rows;
  f32x16 gW2[HB][HB];
  float4 gW1[HB];
  float gb1[HB], gb2[HB], gW3[HB], gb3 = 0.f, loss = 0.f;
#pragma unroll
  for (int ub = 0; ub < HB; ++ub) {
    gW1[ub] = make_float4(0.f, 0.f, 0.f, 0.f);
    gb1[ub] = gb2[ub] = gW3[ub] = 0.f;
#pragma unroll
    for (int kb = 0; kb < HB; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) gW2[ub][kb][r] = 0.f;
  }
  for (int64_t r0 = ((int64_t)blockIdx.x * 4 + wv) * kMlpTile; r0 < rows;
       r0 += (int64_t)gridDim.x * 4 * kMlpTile) {
    f32x16 h1[HB], h2[HB], y;
    if (lane < 32u) t.tgt[lane] = target[min(r0 + lane, rows - 1)];
    mlp_tile_forward<H>(w, sW2, L, t, feat, r0, rows, lane, h1, h2, y);
    f32x16 d2[HB];
    mlp_wave_sync();  // every lane has read h1 from the exchange tile
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = mlp_row(r, lane);
      const float e = r0 + row < rows ? y[r] - t.tgt[row] : 0.f;
      const float dy = 2.0f * e * inv_rows;
      loss = __builtin_fmaf(e, e, loss);
      gb3 += dy;
#pragma unroll
      for (int ub = 0; ub < HB; ++ub) {
        const float h = h2[ub][r];
        gW3[ub] = __builtin_fmaf(dy, h, gW3[ub]);
        const float d = dy * L.w3[ub] * (1.0f - h * h);
        gb2[ub] += d;
        d2[ub][r] = d;
        t.x[row * LD + 32 * ub + col] = d;
      }
    }
    mlp_wave_sync();
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
      for (int ub = 0; ub < HB; ++ub)
#pragma unroll
        for (int kb = 0; kb < HB; ++kb)
          gW2[ub][kb] = __builtin_amdgcn_mfma_f32_32x32x2f32(d2[ub][r], h1[kb][r], gW2[ub][kb],
                                                             0, 0, 0);
    f32x16 d1[HB];
#pragma unroll
    for (int kb = 0; kb < HB; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) d1[kb][r] = 0.f;
#pragma unroll
    for (int u = 0; u < HP; u += 2) {
      const float a = t.x[col * LD + u + half];
#pragma unroll
      for (int kb = 0; kb < HB; ++kb)
        d1[kb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, sW2[(u + half) * LD + 32 * kb + col],
                                                      d1[kb], 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float4 z = t.z[mlp_row(r, lane)];
#pragma unroll
      for (int kb = 0; kb < HB; ++kb) {
        const float h = h1[kb][r];
        const float d = d1[kb][r] * (1.0f - h * h);
        gb1[kb] += d;
        gW1[kb].x = __builtin_fmaf(d, z.x, gW1[kb].x);
        gW1[kb].y = __builtin_fmaf(d, z.y, gW1[kb].y);
        gW1[kb].z = __builtin_fmaf(d, z.z, gW1[kb].z);
        gW1[kb].w = __builtin_fmaf(d, z.w, gW1[kb].w);
      }
    }
  }
  // the two halves of a wavefront hold different rows of the same units
  gb3 += __shfl_xor(gb3, 32, 64);
  loss += __shfl_xor(loss, 32, 64);
  for (int q = 0; q < 4; ++q) {
    if (wv == (uint32_t)q) {
      // add to what the wavefronts before stored
      auto put = [&](int i, float v) { share[i] = q == 0 ? v : share[i] + v; };
      if (lane < 8u) put((int)lane, 0.0f);  // the standardisation is not trained
#pragma unroll
      for (int ub = 0; ub < HB; ++ub) {
        const int u = 32 * ub + col;
        const float4 g1 = make_float4(gW1[ub].x + __shfl_xor(gW1[ub].x, 32, 64),
                                      gW1[ub].y + __shfl_xor(gW1[ub].y, 32, 64),
                                      gW1[ub].z + __shfl_xor(gW1[ub].z, 32, 64),
                                      gW1[ub].w + __shfl_xor(gW1[ub].w, 32, 64));
        const float s1 = gb1[ub] + __shfl_xor(gb1[ub], 32, 64);
        const float s2 = gb2[ub] + __shfl_xor(gb2[ub], 32, 64);
        const float s3 = gW3[ub] + __shfl_xor(gW3[ub], 32, 64);
        if (half == 0 && u < H) {
          put(8 + 4 * u + 0, g1.x);
          put(8 + 4 * u + 1, g1.y);
          put(8 + 4 * u + 2, g1.z);
          put(8 + 4 * u + 3, g1.w);
          put(8 + 4 * H + u, s1);
          put(8 + 5 * H + H * H + u, s2);
          put(8 + 6 * H + H * H + u, s3);
        }
#pragma unroll
        for (int kb = 0; kb < HB; ++kb)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int uu = 32 * ub + mlp_row(r, lane), k = 32 * kb + col;
            if (uu < H && k < H) put(8 + 5 * H + uu * H + k, gW2[ub][kb][r]);
          }
      }
      if (lane == 0) {
        put(np - 1, gb3);
        put(np, loss * inv_rows);
      }
    }
    __syncthreads();
  }
  float *out = partial + (int64_t)blockIdx.x * (np + 1);
  for (int i = threadIdx.x; i <= np; i += 256) out[i] = share[i];
}

// Adam (Kingma and Ba 2015) in FP32; c1 = 1/(1 - b1^t), c2 = 1/(1 - b2^t).
struct AdamArgs {
  float *w, *m, *v;
  float lr, b1, b2, eps, c1, c2;
};
__device__ __forceinline__ void adam_update(const AdamArgs &a, int64_t i, float gi) {
  const float mi = a.b1 * a.m[i] + (1.0f - a.b1) * gi;
  const float vi = a.b2 * a.v[i] + (1.0f - a.b2) * gi * gi;
  a.m[i] = mi;
  a.v[i] = vi;
  a.w[i] -= a.lr * (mi * a.c1) / (sqrtf(vi * a.c2) + a.eps);
}

// Adds the gradient shares in a fixed order (16 threads per entry, each every
// 16th share with all its loads in flight, then their sums in order): to
// out[0 .. np], or (kAdam) straight into an Adam step of entries [0, np), with
// the loss to *loss. One thread per entry over 256 dependent adds took 58 us.
template <bool kAdam>
__global__ __launch_bounds__(256) void k_mlp_reduce(const float *__restrict__ partial, int ns,
                                                    int np1, float *__restrict__ out,
                                                    AdamArgs ad, float *__restrict__ loss) {
  __shared__ float s[16][17];
  const int e = threadIdx.x & 15, q0 = threadIdx.x >> 4;
  const int i = blockIdx.x * 16 + e;
  float v = 0.f;
  if (i < np1) {
#pragma unroll 16
    for (int q = q0; q < ns; q += 16) v += partial[(int64_t)q * np1 + i];
  }
  s[q0][e] = v;
  __syncthreads();
  if (threadIdx.x >= 16 || i >= np1) return;
  float g = s[0][e];
#pragma unroll
  for (int q = 1; q < 16; ++q) g += s[q][e];
  if constexpr (kAdam) {
    if (i == np1 - 1)
      *loss = g;
    else
      adam_update(ad, i, g);
  } else {
    out[i] = g;
  }
}

// The model's input standardisation from training rows (FP64 sums per
// workgroup, added in order by the second kernel): mu = mean, is = 1 /
// max(standard deviation, 1e-6).
constexpr int kStdBlocks = 64;
__global__ __launch_bounds__(256) void k_mlp_moments(const float4 *__restrict__ feat,
                                                     int64_t rows, double *__restrict__ part) {
  __shared__ double s[4][8];
  double a[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int64_t r = blockIdx.x * 256 + threadIdx.x; r < rows; r += (int64_t)gridDim.x * 256) {
    const float4 f = feat[r];
    const double v[4] = {f.x, f.y, f.z, f.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      a[k] += v[k];
      a[4 + k] += v[k] * v[k];
    }
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    for (int d = 32; d >= 1; d >>= 1) a[k] += __shfl_xor(a[k], d, 64);
    if (lane_id() == 0) s[threadIdx.x >> 6][k] = a[k];
  }
  __syncthreads();
  if (threadIdx.x < 8)
    part[blockIdx.x * 8 + threadIdx.x] = ((s[0][threadIdx.x] + s[1][threadIdx.x]) +
                                          s[2][threadIdx.x]) + s[3][threadIdx.x];
}
// Also clears the n words of zero (Adam's moments).
__global__ __launch_bounds__(256) void k_mlp_standardize(const double *__restrict__ part,
                                                         int64_t rows, float *__restrict__ w,
                                                         float *__restrict__ m,
                                                         float *__restrict__ v, int np) {
  for (int i = threadIdx.x; i < np; i += 256) m[i] = v[i] = 0.f;
  __shared__ double s[8];
  if (threadIdx.x < 8) {
    double t = 0;
#pragma unroll 16
    for (int q = 0; q < kStdBlocks; ++q) t += part[q * 8 + threadIdx.x];
    s[threadIdx.x] = t;
  }
  __syncthreads();
  if (threadIdx.x < 4) {
    const int k = threadIdx.x;
    const double mean = s[k] / (double)rows;
    const double var = fmax(s[4 + k] / (double)rows - mean * mean, 0.0);
    w[k] = (float)mean;
    w[4 + k] = (float)(1.0 / fmax(sqrt(var), 1e-6));
  }
}

__global__ __launch_bounds__(256) void k_adam(int64_t np, const float *__restrict__ g,
                                              AdamArgs ad) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < np;
       i += (int64_t)gridDim.x * blockDim.x)
    adam_update(ad, i, g[i]);
}

// Queue sort keys: one 8-bit digit, larger predicted cost first; equal digits
// keep group order in the stable digit sort, which covers the queue's entries
// only (the count is read on the device). Modes 1 and 2 take whole octaves of
// the predicted interactions: the tail only needs the costs in rough order, and
// in group order neighbours share cells in the caches. Below 2^14.5 no group
// decides when the walk ends: one bucket. (2^23 galaxy, block steps, rebuild
// every 2nd step, per walk over 16 steps: quarter octaves 2.44 ms, quarter octaves
// with one bucket below 2^18 2.31, octaves 2.21, plain 2.60; over 20 steps, where
// the rebuilds fall on other steps, octaves 2.18, plain 2.20.) Mode 3 keeps quarter
// octaves.
constexpr float kBulkLog2 = 14.0f;
__global__ __launch_bounds__(256) void k_cost_keys(
    const DevScalars *__restrict__ sc, const uint32_t *__restrict__ queue, int mode,
    const float4 *__restrict__ feat, const float *__restrict__ pred,
    const float *__restrict__ target, int64_t n_upper, uint64_t *__restrict__ keys,
    uint32_t *__restrict__ vals) {
  const uint32_t nq = queue ? sc->nqueue : sc->ngroup;
  (void)n_upper;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < nq;
       i += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t g = queue ? queue[i] : (uint32_t)i;
    const float4 f = feat[g];
    // mode 1: log2(count) + log2(1 + previous list length); mode 2: the
    // model; mode 3: the log2 interactions the last ordered walk recorded
    const float c = mode == 2 ? pred[g] : mode == 3 ? target[g] : f.x + f.w;
    const float q = mode == 3 ? fminf(fmaxf(c * 4.0f, 0.0f), 254.0f)  // NaN -> 0
                              : fminf(fmaxf(c + 0.5f, kBulkLog2), 254.0f);
    keys[i] = 254u - (uint32_t)q;
    vals[i] = g;
  }
}

__global__ void k_cost_qtotal(DevScalars *sc, int queued) {
  if (threadIdx.x == 0 && !queued) sc->nqueue = sc->ngroup;
}

namespace {
unsigned grid_for(int64_t n, int per_block, int cap) {
  int64_t g = cdiv(n, per_block);
  if (g > cap) g = cap;
  if (g < 1) g = 1;
  return (unsigned)g;
}

template <int H>
void forward_h(const float *w, int64_t rows, const uint32_t *rows_dev, const float4 *feat,
               float *y, hipStream_t st) {
  if constexpr (H < 32)
    hipLaunchKernelGGL(k_mlp_forward_rows<H>, dim3(grid_for(rows, 256, 4096)), dim3(256), 0, st,
                       w, rows, rows_dev, feat, y);
  else
    hipLaunchKernelGGL(k_mlp_forward<H>, dim3(grid_for(rows, 4 * kMlpTile, 1024)), dim3(256), 0,
                       st, w, rows, rows_dev, feat, y);
}

// gradient shares: one per workgroup, a tile per wavefront up to kMlpShares
template <int H>
int grad_h(const float *w, int64_t rows, const float4 *feat, const float *target,
           float *partial, hipStream_t st) {
  const unsigned shares = grid_for(rows, 4 * kMlpTile, kMlpShares);
  hipLaunchKernelGGL(k_mlp_grad<H>, dim3(shares), dim3(256), 0, st, w, rows, feat, target,
                     partial);
  return (int)shares;
}

int launch_grad(int H, const float *w, int64_t rows, const float4 *feat, const float *target,
                float *partial, hipStream_t st) {
  switch (H) {
    case 8: return grad_h<8>(w, rows, feat, target, partial, st);
    case 16: return grad_h<16>(w, rows, feat, target, partial, st);
    case 32: return grad_h<32>(w, rows, feat, target, partial, st);
    default: return grad_h<64>(w, rows, feat, target, partial, st);
  }
}

AdamArgs adam_args(float *w, float *m, float *v, int step, float lr, float b1, float b2,
                   float eps) {
  return AdamArgs{w, m, v, lr, b1, b2, eps, (float)(1.0 / (1.0 - pow((double)b1, (double)step))),
                  (float)(1.0 / (1.0 - pow((double)b2, (double)step)))};
}
}  // namespace

bool mlp_hidden_ok(int H) { return H == 8 || H == 16 || H == 32 || H == 64; }
int64_t mlp_nparams(int H) { return mlp_np(H); }

void launch_mlp_forward(int H, const float *w, int64_t rows, const uint32_t *rows_dev,
                        const float4 *feat, float *y, hipStream_t st) {
  switch (H) {
    case 8: forward_h<8>(w, rows, rows_dev, feat, y, st); break;
    case 16: forward_h<16>(w, rows, rows_dev, feat, y, st); break;
    case 32: forward_h<32>(w, rows, rows_dev, feat, y, st); break;
    case 64: forward_h<64>(w, rows, rows_dev, feat, y, st); break;
    default: break;
  }
}

void launch_mlp_grad(int H, const float *w, int64_t rows, const float4 *feat,
                     const float *target, float *partial, float *grad_loss, hipStream_t st) {
  const int shares = launch_grad(H, w, rows, feat, target, partial, st);
  const int np1 = mlp_np(H) + 1;
  hipLaunchKernelGGL(k_mlp_reduce<false>, dim3(grid_for(np1, 16, 4096)), dim3(256), 0, st,
                     partial, shares, np1, grad_loss, AdamArgs{}, nullptr);
}

void launch_mlp_train_step(int H, float *w, int64_t rows, const float4 *feat,
                           const float *target, float *partial, float *m, float *v, int step,
                           float lr, float b1, float b2, float eps, float *loss,
                           hipStream_t st) {
  const int shares = launch_grad(H, w, rows, feat, target, partial, st);
  const int np1 = mlp_np(H) + 1;
  hipLaunchKernelGGL(k_mlp_reduce<true>, dim3(grid_for(np1, 16, 4096)), dim3(256), 0, st,
                     partial, shares, np1, nullptr, adam_args(w, m, v, step, lr, b1, b2, eps),
                     loss);
}

void launch_adam(int64_t np, float *w, const float *g, float *m, float *v, int step, float lr,
                 float b1, float b2, float eps, hipStream_t st) {
  hipLaunchKernelGGL(k_adam, dim3(grid_for(np, 256, 64)), dim3(256), 0, st, np, g,
                     adam_args(w, m, v, step, lr, b1, b2, eps));
}

void launch_mlp_standardize(int H, const float4 *feat, int64_t rows, float *w, float *m,
                            float *v, float *scratch, hipStream_t st) {
  double *part = reinterpret_cast<double *>(scratch);
  hipLaunchKernelGGL(k_mlp_moments, dim3(kStdBlocks), dim3(256), 0, st, feat, rows, part);
  hipLaunchKernelGGL(k_mlp_standardize, dim3(1), dim3(256), 0, st, part, rows, w, m, v,
                     mlp_np(H));
}

void launch_cost_features(int64_t n, bool queued, const uint32_t *perm, const Ptrs &P,
                          hipStream_t st) {
  hipLaunchKernelGGL(k_cost_features, dim3(grid_for(n, 4 * 8, 8192)), dim3(256), 0, st, P.sc,
                     queued ? P.order : nullptr, P.gbegin, P.gcount, P.xyzm, perm, P.plast,
                     P.feat);
}

void launch_cost_after(int64_t n, bool queued, const uint32_t *perm, const Ptrs &P,
                       hipStream_t st) {
  hipLaunchKernelGGL(k_cost_after, dim3(grid_for(n, 4 * 8, 8192)), dim3(256), 0, st, P.sc,
                     queued ? P.order : nullptr, P.gbegin, P.gcount, P.gent, perm, P.plast,
                     P.target);
}

void launch_cost_order(int64_t n, bool queued, int mode, int H, const Ptrs &P,
                       hipStream_t st) {
  if (mode == 2)
    launch_mlp_forward(H, P.mlpw, n, &P.sc->ngroup, P.feat, P.pred, st);
  hipLaunchKernelGGL(k_cost_keys, dim3(grid_for(n, 256 * 8, 8192)), dim3(256), 0, st, P.sc,
                     queued ? P.order : nullptr, mode, P.feat, P.pred, P.target, n, P.okeys,
                     P.qtmp);
  launch_digit_sort(n, queued ? &P.sc->nqueue : &P.sc->ngroup, 0, P.okeys, P.qtmp, P.okeys + n,
                    P.order, P.hist, st);
  hipLaunchKernelGGL(k_cost_qtotal, dim3(1), dim3(64), 0, st, P.sc, queued ? 1 : 0);
}

}  // namespace nb
