// k_walk.hip -- group bounds and the group-wise tree walk (Sec. 1).
//
// One wavefront serves one i-group at a time, taking groups from a global
// work queue until the queue is empty (persistent kernel). For its group it
// traverses the tree from the root, depth first in chunks: the top 64 (or
// fewer) candidate cells of the wave's stack in global memory (the paper's
// per-SM cell buffer, Sec. 3) are popped and tested against the acceleration
// MAC of Eq. 2, one lane per cell; accepted cells enter the interaction list
// as pseudo-particles (centre of mass, mass), opened leaves contribute their
// particles, opened internal cells push their children (lane order). Each
// chunk pushes at most 512 cells, so the stack never holds more than 512 per
// tree level (under 11K cells), unlike a breadth-first frontier, which can
// hold a whole level. Offsets come from wave prefix sums. The list lives in
// LDS; whenever it holds `list_tile` entries it is flushed: every lane adds
// Eq. 1 over the tile for its particle, in FP32.
//
// Canonical order: list entries appear in the order of this traversal (a
// function of the tree and the group alone). Entry j belongs to block j / 64;
// each lane keeps four FP32 running sums and adds the entries of block b, in
// list order, to sum b mod 4; the four sums are added in that order at the
// end. A flush only cuts the sequence at block boundaries (tiles are
// multiples of 64 entries), so each lane's summation order is fixed by the
// group alone: it does not depend on the tile size, the stack capacity, the
// queue order, which wave runs the group, or the split below. Results are
// bit-identical across all of them. (The compensated sum keeps two running
// sums, b mod 2, each with its correction, and is split in two at most. With one
// it was a single wavefront's chain of up to 4096 entries: potential of 130003
// particles 1050 us, 874 in two; of 10007 609 and 437.)
//
// Split walk: when few groups are queued (block steps often walk a few
// thousand heavy groups, fewer than the resident wavefronts), K = 2 or 4
// wavefronts take the same group: each traverses the whole tree (the MAC
// decisions are the same in each) but adds only the blocks b with
// b mod K == its part, i.e. the running sums r with r mod K == its part, and
// stores them; k_walk_mid adds the four sums per lane in order and writes the
// results. This turns a queue of q heavy groups into
// K q tasks of a quarter or half the arithmetic each.
//
// Heavy groups: a few groups meet far longer lists than the rest (members
// scattered over a sparse outskirt: their box spans the dense centre, and
// nearly every particle is an entry). One group's walk is a serial chain, so
// such a group decided the walk's time (sphere of 2*10^5 particles: mean list
// 1840, longest 199938; 3.2 ms, of which all other groups needed 0.4). A group
// with more entries in its reach (k_group_bounds) than heavy_limit() of its walk
// root's particles is therefore left by the main pass and walked in parts:
// k_walk_mid cuts the part of the tree that the group meets into an ordered front
// of cells (breadth first, the group's own MAC) and the front into parts of about
// equal particle counts; k_heavy_walk walks each part like a group of its own (its
// stack starts with the part's cells), and k_heavy_end adds the parts' sums in
// order. Reach, front, parts and sums depend on the tree, the group and its a_old
// alone.
// Where all lists are long (a small delta_acc, large leaves, a_old far too small)
// nothing is gained by parts: the groups keep the chip busy, and every one is
// walked up to the limit first. With a limit on the whole list a sphere of 300007
// particles at 2^-12 took 17.3 ms instead of 5.7 without parts, a galaxy of 200000
// with 64-particle leaves at 2^-11 2.4 instead of 0.62; by the entries in reach 1.1
// and 0.61. Over-full leaves (particles that the keys do not tell apart) do not
// count: every group that lies in one meets it (half of 200000 particles at one
// point: 13.0 ms with them, 4.6 without, 3.8 before there were parts).
//
// Lane layout: groups of at most 8, 16 or 32 members use S = 8, 4 or 2
// "streams": lane = stream * (64 / S) + member, stream s adds the entries
// whose list index is s mod S, and the S partial sums are combined at the
// end by a fixed butterfly. S depends only on the group size.
//
// Group-wise MAC (a reading of Eq. 2 for a shared list): d is the distance
// from the cell's centre of mass to the group's bounding box (no larger than
// any member's distance) and |a_old| the smallest previous acceleration in
// the group; accept iff d^2 > b^2 and delta_acc*|a_old|*d^4 >= G m b^2, all in
// FP32. Without a_old (bootstrap) accept iff d^2 > 4 b^2.
#include <algorithm>

#include "nbody_internal.h"

namespace nb {

struct WalkArgs {
  const float4 *nodeA;
  const float4 *nodeB;
  const float4 *xyzm;
  const uint32_t *gbegin;
  const uint32_t *gcount;
  const float4 *gbox;
  const float *greach;
  const uint32_t *perm;
  const uint32_t *order;   // queue -> group (nullptr: identity)
  const uint32_t *qcount;  // queue length (device)
  const uint32_t *groot;   // per group root cell (nullptr: the root, cell 0)
  float4 *asort;           // key-ordered copy of the outputs with |a| (nullptr: none)
  const uint32_t *cpcount;
  uint32_t *retry;         // the groups left to the retry pass
  uint32_t *nretry;
  uint32_t *heavy;         // the groups over heavy_limit()
  uint4 *hparts;           // parts of heavy groups: (group, front begin, cells, -)
  uint2 *hrec;             // per heavy group: first part, parts (0: no room)
  uint32_t *hfront;        // the fronts' cells
  float *hsum;             // per part: partial sums per lane
  uint32_t hslots, hfront_cap, hwords;  // capacities of hparts / hfront; words per part
  uint32_t *head;          // the work queue's claim counter
  uint32_t *frontier;
  uint32_t *gent;
  unsigned long long *ghash;
  DevScalars *sc;
  float *ax, *ay, *az;
  float *phi;              // potential output (the potential variant only)
  float *split;            // partial sums of split groups, per queue position
  float G, eps2;
  uint32_t n;
  uint32_t tile;
  uint32_t fmask;
  int bootstrap;
  int may_retry;           // overflowing groups are walked again (else reported)
  int split_mode;          // -1 never (retry pass), 0 by queue length, else 1, 2, 4
  uint32_t split_slots, slot_words, split_waves;
};

// Longest list that one wavefront walks, for a walk root holding n particles.
// At 2*10^5 particles 1.3 % of the particles have lists of over 4096 entries;
// the limit bounds the main pass's longest chain. In larger trees lists grow and
// thousands of groups keep the chip busy while a long one is walked: the limit
// grows with them (in the 2^23 galaxy, 32768 instead of 2^17 made the block
// steps' walks 4 % shorter in group order and 1 % longer in the learned order).
__host__ __device__ __forceinline__ uint32_t heavy_limit(uint32_t n) {
  const uint32_t q = n / 64u;
  return q < 4096u ? 4096u : q;
}
// Wavefronts per group for a queue of ng groups walked by `waves` wavefronts.
// Each of them repeats the group's traversal: four pay while they still find a
// chip with room (galaxies, us per walk of 65536, 90000, 200003 and 400000
// particles, ng = 1490, 2050, 4500 and 9000: K = 4 135, 176, 331, 649; K = 2
// 163, 155, 250, 523), two until the queue is several times the chip (10^6
// particles, ng = 22154: 851 against 1026 with K = 1; 1.5 million: the same).
// Where longer lists stay in the main pass, four pay for as much longer queues
// (block steps of the 2^23 galaxy, 16 steps: 50.3 ms, 52.9 with K = 2 from
// ng = waves / 4 on); `limit` is heavy_limit() of the tree.
__device__ __forceinline__ uint32_t split_factor(uint32_t ng, uint32_t waves, uint32_t slots,
                                                 int mode, uint32_t limit) {
  if (mode < 0 || ng > slots || ng > 4u * waves) return 1u;
  if (mode > 0) return (uint32_t)mode;
  return ng < min(waves / 4u * (limit / 4096u), 2u * waves) ? 4u : 2u;
}
// Particles under a part's cells, about. A part is a chain of its own and ends the
// walk of a small tree; many parts cost room and repeat the descent from the
// group's front (10007 particles, two walks a step, 4 steps: 1850 us with 1024,
// 1665 with 512, 1579 with 256; 65536, 8 steps: 2729, 2599, 2590 with 384; a batch
// of 64 systems: 15.8 ms, 15.8, 16.0 with 384 for all).
__host__ __device__ __forceinline__ uint32_t part_work(uint32_t n) {
  return n <= 32768u ? 256u : 512u;
}
constexpr uint32_t kMaxParts = 128;
constexpr uint32_t kPartSlice = 1u << 31;  // a part of particles, not of cells
// a front cell holding more particles is opened further
__device__ __forceinline__ uint32_t front_cell_max(uint32_t n) {
  const uint32_t q = n / 256u;
  return q < 64u ? 64u : q > 2048u ? 2048u : q;
}

// Group-wise MAC (see above): the cell with node words A = (com, b^2) and mass m
// against the group's box, dA = delta_acc |a_old|. G m b^2 is made here: as a word
// of the node it cost every tree a launch of its own, 4 to 5 us.
// The squared distance comes back in d2.
__device__ __forceinline__ bool mac_accept(float4 A, float m, float G, float4 glo, float4 ghi,
                                           float dA, int bootstrap, float &d2) {
  const float tx = fmaxf(fmaxf(glo.x - A.x, A.x - ghi.x), 0.0f);
  const float ty = fmaxf(fmaxf(glo.y - A.y, A.y - ghi.y), 0.0f);
  const float tz = fmaxf(fmaxf(glo.z - A.z, A.z - ghi.z), 0.0f);
  d2 = __builtin_fmaf(tz, tz, __builtin_fmaf(ty, ty, tx * tx));
  bool accept = false;
  if (d2 > A.w) {
    if (bootstrap) {
      const float four_b2 = 4.0f * A.w;
      accept = d2 > four_b2;
    } else {
      const float d4 = d2 * d2;
      const float lhs = dA * d4;
      const float gm = G * m;
      const float q = gm * A.w;
      accept = lhs >= q;
    }
  }
  return accept;
}

__device__ __forceinline__ uint64_t mix64(uint64_t v) {
  v += 0x9E3779B97F4A7C15ull;
  v = (v ^ (v >> 30)) * 0xBF58476D1CE4E5B9ull;
  v = (v ^ (v >> 27)) * 0x94D049BB133111EBull;
  return v ^ (v >> 31);
}

// One lane's running sums of the acceleration components and, in the
// potential variant (kPot), of the potential: sum of -m_j / r_j.
template <bool kComp, bool kPot>
struct Acc3 {
  float x = 0.f, y = 0.f, z = 0.f, w = 0.f;
  __device__ __forceinline__ void add(float dx, float dy, float dz, float f, float mr) {
    x = __builtin_fmaf(f, dx, x);
    y = __builtin_fmaf(f, dy, y);
    z = __builtin_fmaf(f, dz, z);
    if constexpr (kPot) w = w - mr;
  }
  __device__ __forceinline__ void total(float &ox, float &oy, float &oz, float &ow) const {
    ox = x;
    oy = y;
    oz = z;
    ow = w;
  }
};

// Neumaier's compensated summation (Neumaier 1974) per component.
template <bool kPot>
struct Acc3<true, kPot> {
  float x = 0.f, y = 0.f, z = 0.f, w = 0.f, cx = 0.f, cy = 0.f, cz = 0.f, cw = 0.f;
  __device__ __forceinline__ static void nadd(float &s, float &c, float v) {
    const float t = s + v;
    c += (fabsf(s) >= fabsf(v)) ? ((s - t) + v) : ((v - t) + s);
    s = t;
  }
  __device__ __forceinline__ void add(float dx, float dy, float dz, float f, float mr) {
    nadd(x, cx, f * dx);
    nadd(y, cy, f * dy);
    nadd(z, cz, f * dz);
    if constexpr (kPot) nadd(w, cw, -mr);
  }
  __device__ __forceinline__ void merge(const Acc3 &o) {
    nadd(x, cx, o.x);
    nadd(y, cy, o.y);
    nadd(z, cz, o.z);
    cx += o.cx;
    cy += o.cy;
    cz += o.cz;
    if constexpr (kPot) {
      nadd(w, cw, o.w);
      cw += o.cw;
    }
  }
  __device__ __forceinline__ void total(float &ox, float &oy, float &oz, float &ow) const {
    ox = x + cx;
    oy = y + cy;
    oz = z + cz;
    ow = w + cw;
  }
};

// The running sums of a lane: four for the plain FP32 sum (block b of the
// list adds into sum b mod 4), two compensated ones (b mod 2). The sum of the
// block being added is always u0: after each block the sums rotate, so that
// no register is ever selected by a run-time index. A wavefront taking every
// K-th block (part p of K) holds the 4 / K sums p, p + K, ... in u0, u1, ...
// (rotating among those); after a whole number of rotation periods u_k holds
// sum p + K k.
constexpr uint32_t kBlk = 64;  // list entries per block
constexpr uint32_t kFullLeaf = 64;  // the largest leaf_max: bigger leaves are over-full
template <bool kComp, bool kPot>
struct RunSums;
template <bool kPot>
struct RunSums<false, kPot> {
  static constexpr uint32_t kNum = 4;
  Acc3<false, kPot> u0, u1, u2, u3;
  __device__ __forceinline__ void advance(uint32_t K) {
    if (K == 1u) {
      const Acc3<false, kPot> t = u0;
      u0 = u1;
      u1 = u2;
      u2 = u3;
      u3 = t;
    } else if (K == 2u) {
      const Acc3<false, kPot> t = u0;
      u0 = u1;
      u1 = t;
    }
  }
  __device__ __forceinline__ void total(float &ox, float &oy, float &oz, float &ow) const {
    ox = ((u0.x + u1.x) + u2.x) + u3.x;
    oy = ((u0.y + u1.y) + u2.y) + u3.y;
    oz = ((u0.z + u1.z) + u2.z) + u3.z;
    ow = ((u0.w + u1.w) + u2.w) + u3.w;
  }
};
template <bool kPot>
struct RunSums<true, kPot> {
  static constexpr uint32_t kNum = 2;
  Acc3<true, kPot> u0, u1;
  __device__ __forceinline__ void advance(uint32_t K) {
    if (K == 1u) {
      const Acc3<true, kPot> t = u0;
      u0 = u1;
      u1 = t;
    }
  }
  // both as one compensated sum
  __device__ __forceinline__ Acc3<true, kPot> merged() const {
    Acc3<true, kPot> m = u0;
    m.merge(u1);
    return m;
  }
  __device__ __forceinline__ void total(float &ox, float &oy, float &oz, float &ow) const {
    merged().total(ox, oy, oz, ow);
  }
};

// Entries of zero mass pad a flushed block to a multiple of S * kFlushUnroll,
// so every lane runs the same trip count and the loads of one trip are
// issued together. A padding entry adds exactly +0 to each sum (r^2 >= eps^2
// keeps it finite), and each lane still adds its entries in list order.
constexpr uint32_t kFlushUnroll = 4;
constexpr uint32_t kListPad = 8 * kFlushUnroll;  // largest S times the unroll

__device__ __forceinline__ void eq1_term(const float4 e, float4 pi, float eps2, float &dx,
                                         float &dy, float &dz, float &f, float &mr) {
  dx = e.x - pi.x;
  dy = e.y - pi.y;
  dz = e.z - pi.z;
  const float r2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, __builtin_fmaf(dx, dx, eps2)));
  const float rinv = __builtin_amdgcn_rsqf(r2);
  mr = e.w * rinv;
  const float rinv2 = rinv * rinv;
  f = mr * rinv2;
}

// The stream count S is a template constant: the trip count and the LDS
// offsets of one trip (u * S entries past the trip's base) are then uniform
// and immediate.
template <bool kComp, bool kPot, uint32_t S>
__device__ __forceinline__ void flush_run_s(const float4 *__restrict__ list, uint32_t padded,
                                            uint32_t stream, float4 pi, float eps2,
                                            Acc3<kComp, kPot> &acc) {
  constexpr uint32_t step = S * kFlushUnroll;
  const float4 *p = list + stream;
  for (uint32_t j0 = 0; j0 < padded; j0 += step) {
    float4 e[kFlushUnroll];
#pragma unroll
    for (uint32_t u = 0; u < kFlushUnroll; ++u) e[u] = p[j0 + u * S];
#pragma unroll
    for (uint32_t u = 0; u < kFlushUnroll; ++u) {
      float dx, dy, dz, f, mr;
      eq1_term(e[u], pi, eps2, dx, dy, dz, f, mr);
      acc.add(dx, dy, dz, f, mr);
    }
  }
}

template <bool kComp, bool kPot>
__device__ __forceinline__ void flush_run(const float4 *__restrict__ list, uint32_t cnt,
                                          uint32_t stream, uint32_t S, float4 pi, float eps2,
                                          Acc3<kComp, kPot> &acc) {
  const uint32_t step = S * kFlushUnroll;
  const uint32_t padded = (cnt + step - 1) / step * step;
  // S is wave-uniform: these branches are not lane-predicated
  if (S == 1)
    flush_run_s<kComp, kPot, 1>(list, padded, stream, pi, eps2, acc);
  else if (S == 2)
    flush_run_s<kComp, kPot, 2>(list, padded, stream, pi, eps2, acc);
  else if (S == 4)
    flush_run_s<kComp, kPot, 4>(list, padded, stream, pi, eps2, acc);
  else
    flush_run_s<kComp, kPot, 8>(list, padded, stream, pi, eps2, acc);
}

// Flush the tile's cnt entries: whole blocks of 64 entries (the last one
// possibly short), each into u0 followed by a rotation of the sums. nblk counts
// the blocks added.
template <bool kComp, bool kPot, uint32_t K>
__device__ __forceinline__ void flush_tile(float4 *__restrict__ list, uint32_t cnt,
                                           uint32_t lane, uint32_t stream, uint32_t S,
                                           float4 pi, float eps2, RunSums<kComp, kPot> &R,
                                           uint32_t &nblk) {
  // every lane stores (two lanes per slot, same value): no lane-predicated
  // region; slots [cnt, cnt + kListPad) are free
  list[cnt + (lane & (kListPad - 1))] = make_float4(0.f, 0.f, 0.f, 0.f);
  __builtin_amdgcn_wave_barrier();
  for (uint32_t off = 0; off < cnt; off += kBlk) {
    flush_run<kComp, kPot>(list + off, min(kBlk, cnt - off), stream, S, pi, eps2, R.u0);
    R.advance(K);
    ++nblk;
  }
}

// Per lane: the group member, the list stream, and (after adding the running
// sums) the butterfly over the streams; every lane ends with its member's sum.
__device__ __forceinline__ uint32_t stream_count(uint32_t gc) {
  return gc <= 8 ? 8u : gc <= 16 ? 4u : gc <= 32 ? 2u : 1u;
}

__device__ __forceinline__ void stream_reduce(uint32_t Wd, float &sx, float &sy, float &sz) {
  for (uint32_t d = Wd; d < 64u; d <<= 1) {
    sx += __shfl_xor(sx, (int)d, 64);
    sy += __shfl_xor(sy, (int)d, 64);
    sz += __shfl_xor(sz, (int)d, 64);
  }
}

__device__ __forceinline__ void stream_reduce1(uint32_t Wd, float &sw) {
  for (uint32_t d = Wd; d < 64u; d <<= 1) sw += __shfl_xor(sw, (int)d, 64);
}

// The results of member `lane` (< gc) of group (gb, gc): G times the sum, in
// caller order (in key order without perm), and with |a| into the
// key-ordered mirror when there is one.
__device__ __forceinline__ void store_group_result(const WalkArgs &a, uint32_t gb, uint32_t gc,
                                                   uint32_t lane, float sx, float sy,
                                                   float sz) {
  if (lane < gc) {  // lane == member here (stream 0)
    const uint32_t o = a.perm ? a.perm[gb + lane] : gb + lane;
    const float gx = a.G * sx, gy = a.G * sy, gz = a.G * sz;
    a.ax[o] = gx;
    a.ay[o] = gy;
    a.az[o] = gz;
    if (a.asort)
      a.asort[gb + lane] =
          make_float4(gx, gy, gz, sqrt_rn(__builtin_fmaf(gz, gz, __builtin_fmaf(gy, gy, gx * gx))));
  }
}

// One wavefront's LDS: the chunk's owner table, then a list tile with its
// padding (one base register: the parts are at fixed offsets).
struct WaveLds {
  float4 *base;
  __device__ __forceinline__ float4 *ent() const { return base; }
  __device__ __forceinline__ uint32_t *mark() const {
    return reinterpret_cast<uint32_t *>(base + 64);
  }
  __device__ __forceinline__ uint32_t *src() const { return mark() + 64; }
  __device__ __forceinline__ float4 *list() const { return base + 96; }
};
__device__ __forceinline__ WaveLds wave_lds(float4 *lds, uint32_t wv, uint32_t tile) {
  return WaveLds{lds + wv * (tile + kListPad + 96u)};
}

// Wavefronts per SIMD asked of the compiler: the plain walk keeps the next
// chunk's nodes in registers while it adds, and left alone takes 84 of them
// (5 wavefronts; 557, 49.1 ms and 15.4 ms where 6 took 550 us, 48.0 and 14.9 for
// 200003 particles, the 2^23 block steps and a batch of 64 systems). The plain sums
// with the potential keep 5 (left alone 4: 1.1 million particles with hashes 1146
// us, 1073 with 5), the compensated ones without hashes 5. The other forms would
// spill.
constexpr int walk_occupancy(bool comp, bool hash, bool pot) {
  return comp ? (hash || pot ? 1 : 5) : pot ? 5 : hash ? 1 : 6;
}

// The group a wavefront walks for, per lane.
struct WalkGroup {
  float4 glo, ghi, pi;
  uint32_t gb, gc, S, Wd, stream;
};
__device__ __forceinline__ WalkGroup load_group(const WalkArgs &a, uint32_t g, uint32_t lane) {
  WalkGroup w;
  w.gb = a.gbegin[g];
  w.gc = a.gcount[g];
  w.glo = a.gbox[2 * g];
  w.ghi = a.gbox[2 * g + 1];
  w.S = stream_count(w.gc);
  w.Wd = 64u / w.S;
  const uint32_t member = lane & (w.Wd - 1);
  w.stream = lane / w.Wd;
  w.pi = a.xyzm[w.gb + (member < w.gc ? member : 0u)];
  return w;
}

// v, v + 1, ... to p[0], p[1], ... (p need not be aligned to the vector).
__device__ __forceinline__ void store_run2(uint32_t *p, uint32_t v) {
  typedef uint32_t u2 __attribute__((ext_vector_type(2), aligned(4)));
  *reinterpret_cast<u2 *>(p) = u2{v, v + 1u};
}
__device__ __forceinline__ void store_run4(uint32_t *p, uint32_t v) {
  typedef uint32_t u4 __attribute__((ext_vector_type(4), aligned(4)));
  *reinterpret_cast<u4 *>(p) = u4{v, v + 1u, v + 2u, v + 3u};
}

// p[i] by a global load: next to an LDS load of the same value, a plain one is
// merged with it into a flat load, which waits for both memories.
__device__ __forceinline__ float4 load_global(const float4 *p, uint32_t i) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  typedef const __attribute__((address_space(1))) f4 *gp;
  const f4 v = reinterpret_cast<gp>(reinterpret_cast<uintptr_t>(p))[i];
  return make_float4(v.x, v.y, v.z, v.w);
}

// Entry counts of groups without results yet.
constexpr uint32_t kEntNone = 0xffffffffu;   // failed
constexpr uint32_t kEntHeavy = 0xfffffffeu;  // left to the parts' walk
constexpr uint32_t kEntRetry = 0xfffffffdu;  // left to the retry pass
// How a walk ended (wave-uniform).
constexpr uint32_t kEndOverflow = 1, kEndCorrupt = 2, kEndHeavy = 4;

// Traverse the subtrees of the `top` cells on the stack and add their list
// (with K > 1 the blocks of this part) into R; entries counts the list.
// Stops when the list holds more than `limit` entries in `reach`.
// A few wavefronts per SIMD are bound by this loop's chain (stack, nodes, scan,
// push, copy, sums), a full chip by the vector instructions of the sums and of
// the rest. So the next chunk's loads go out before this one's entries are
// copied, children are pushed by at most four stores, and entries find their
// owners by marks and a scan (a binary search was six dependent LDS reads):
// 10007 particles, two walks a step, 4 steps 1586 -> 1509 us; 65536, 8 steps
// 2593 -> 2491; 200003, a call 567 -> 550; the 2^23 block steps 50.1 -> 48.0 ms.
template <bool kComp, bool kHash, bool kPot, uint32_t K>
__device__ __forceinline__ uint32_t walk_list(const WalkArgs &a, const WaveLds &l,
                                              const WalkGroup &w, uint32_t *stk, uint32_t F,
                                              uint32_t top, uint32_t part, uint32_t limit,
                                              float reach, uint32_t ncell, uint32_t lane,
                                              RunSums<kComp, kPot> &R, uint32_t &entries,
                                              uint64_t &hsum) {
  float4 *list = l.list();
  float4 *s_ent = l.ent();
  uint32_t *s_mark = l.mark(), *s_src = l.src();
  const float dA = w.glo.w;
  const uint32_t npart = a.n;
  uint32_t visited = 0, cnt = 0;
  uint32_t nblk = 0;  // list blocks this wavefront has added
  uint32_t end = 0;
  uint32_t nnear = 0;  // per lane: entries in reach, over-full leaves aside
  uint32_t check = limit;
  // the chunk of up to 64 cells from the stack's top, and their nodes
  uint32_t nc, c;
  bool bad_c;
  float4 A, B;
  auto pop = [&]() {
    nc = min(64u, top);
    top -= nc;
    const uint32_t cc = lane < nc ? stk[top + lane] : 0u;
    bad_c = cc >= ncell;
    c = bad_c ? 0u : cc;
    A = a.nodeA[c];
    B = a.nodeB[c];
  };
  if (top > 0) pop();
  else nc = 0u;
  while (nc > 0) {
    visited += nc;
    if (visited > ncell) {  // a tree visits each cell at most once
      end = kEndCorrupt;
      break;
    }
    const bool has = lane < nc && !bad_c;
    const uint32_t w0 = __float_as_uint(B.z), w1 = __float_as_uint(B.w);
    {
      const bool lf = (w1 & kLeafBit) != 0u;
      const uint32_t k = w1 & ~kLeafBit;
      const bool bad_n = has && (lf ? (w0 > npart || k > npart - w0)
                                    : (k > 8u || w0 > ncell || k > ncell - w0));
      if (__ballot(bad_c || bad_n)) {
        end = kEndCorrupt;
        break;
      }
    }
    float d2;
    const bool accept = mac_accept(A, B.x, a.G, w.glo, w.ghi, dA, a.bootstrap, d2) && has;
    const bool leaf = (w1 & kLeafBit) != 0u;
    const uint32_t ne = !has ? 0u : accept ? 1u : leaf ? (w1 & ~kLeafBit) : 0u;
    const uint32_t nch = (has && !accept && !leaf) ? w1 : 0u;
    // children -> stack (over the popped chunk, in lane order) and entries
    // -> list: one scan of both counts (children <= 8 per lane, so at most
    // 512 per chunk: 10 bits; entries in the 22 bits above), or two scans
    // with an over-full leaf, whose entries might not fit and are not counted
    // as near
    uint32_t chi, chtot, ei, etot;
    nnear += !(d2 > A.w && d2 > reach) ? ne : 0u;
    if (__ballot(ne > kFullLeaf) == 0ull) {  // (wave-uniform)
      const uint32_t both = wave_incl_scan_dpp((ne << 10) | nch);
      const uint32_t btot = wave_last(both);
      chi = both & 1023u;
      chtot = btot & 1023u;
      ei = both >> 10;
      etot = btot >> 10;
    } else {
      chi = wave_incl_scan_dpp(nch);
      chtot = wave_last(chi);
      ei = wave_incl_scan_dpp(ne);
      etot = wave_last(ei);
      nnear -= ne > kFullLeaf && !(d2 > A.w && d2 > reach) ? ne : 0u;
    }
    if (top + chtot > F) {
      end = kEndOverflow;
      break;
    }
    // every lane has read its candidate before any lane overwrites it
    __builtin_amdgcn_wave_barrier();
    {  // at most four stores (a loop over the children took 8 rounds)
      uint32_t *d = stk + (top + chi - nch);
      uint32_t v = w0;
      if (nch & 8u) {
        store_run4(d, v);
        store_run4(d + 4, v + 4u);
      }
      if (nch & 4u) {
        store_run4(d, v);
        d += 4;
        v += 4u;
      }
      if (nch & 2u) {
        store_run2(d, v);
        d += 2;
        v += 2u;
      }
      if (nch & 1u) *d = v;
    }
    top += chtot;
    // entries -> LDS list (flushing full tiles). Lane k owns entries
    // [ef_k, ei_k); the copy is cooperative: lane r of the wave fetches entry
    // done + r of the chunk. With K > 1 only this part's blocks are copied.
    if (kHash) {
      if (accept) hsum += mix64((uint64_t)c);
      else if (ne)
        for (uint32_t k = 0; k < ne; ++k) hsum += mix64((1ull << 40) + w0 + k);
    }
    const uint32_t ef = ei - ne;  // this lane's first entry
    const uint64_t cells = __ballot(accept);
    s_src[lane] = w0 - ef;
    if (accept) s_ent[lane] = make_float4(A.x, A.y, A.z, B.x);
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // the next chunk's loads are on their way while this one's entries are added
    if (top > 0) pop();
    else nc = 0u;
    uint32_t done = 0;
    while (done < etot) {
      const uint32_t J = entries + done;  // list index of the next entry
      uint32_t seg;
      if (K == 1u) {
        seg = min(a.tile - cnt, etot - done);
      } else {
        // the rest of block J / 64 within this chunk; the tile (a multiple
        // of 64 entries) holds whole blocks, so it always has room
        seg = min(kBlk - (J & (kBlk - 1u)), etot - done);
        if (((J / kBlk) & (K - 1u)) != part) {
          done += seg;
          continue;
        }
      }
      for (uint32_t r0 = 0; r0 < seg; r0 += 64u) {
        // owners of entries j0 .. j0 + 63: each marks its first one there, and a
        // maximum over the lanes before gives every entry its owner
        const uint32_t j0 = done + r0;
        s_mark[lane] = 0u;
        __builtin_amdgcn_wave_barrier();
        if (ei > max(j0, ef) && ef < j0 + 64u) s_mark[ef > j0 ? ef - j0 : 0u] = lane;
        __builtin_amdgcn_wave_barrier();
        const uint32_t k = wave_incl_max_dpp(s_mark[lane]);
        if (r0 + lane < seg) {
          float4 e = s_ent[k];
          const uint32_t src = s_src[k];
          if (!((cells >> k) & 1ull)) e = load_global(a.xyzm, src + j0 + lane);
          list[cnt + r0 + lane] = e;
        }
        __builtin_amdgcn_wave_barrier();
      }
      cnt += seg;
      done += seg;
      if (cnt == a.tile) {
        __builtin_amdgcn_wave_barrier();
        flush_tile<kComp, kPot, K>(list, cnt, lane, w.stream, w.S, w.pi, a.eps2, R, nblk);
        __builtin_amdgcn_wave_barrier();
        cnt = 0;
      }
    }
    __builtin_amdgcn_wave_barrier();  // owner table is rewritten next chunk
    entries += etot;
    if (entries > check) {  // (wave-uniform)
      const uint32_t m = wave_last(wave_incl_scan_dpp(nnear));
      if (m > limit) {
        end = kEndHeavy;
        break;
      }
      check = entries + (limit - m);  // (not passed before)
    }
  }
  if (end) cnt = 0;
  __builtin_amdgcn_wave_barrier();
  flush_tile<kComp, kPot, K>(list, cnt, lane, w.stream, w.S, w.pi, a.eps2, R, nblk);
  __builtin_amdgcn_wave_barrier();
  // complete the rotation period (kNum / K blocks): then u_k is sum part + K k
  for (; nblk & (RunSums<kComp, kPot>::kNum / K - 1u); ++nblk) R.advance(K);
  return end;
}

// Adds the particles [p0, p0 + m) as a list of their own into R.
template <bool kComp, bool kHash, bool kPot>
__device__ __forceinline__ void add_range(const WalkArgs &a, const WaveLds &l,
                                          const WalkGroup &w, uint32_t p0, uint32_t m,
                                          uint32_t lane, RunSums<kComp, kPot> &R,
                                          uint64_t &hsum) {
  float4 *list = l.list();
  uint32_t nblk = 0;
  for (uint32_t t = 0; t < m; t += a.tile) {
    const uint32_t cnt = min(a.tile, m - t);
    for (uint32_t k = 0; k < cnt; k += 64u) {  // (every lane stores; past the end the last again)
      const uint32_t q = min(k + lane, cnt - 1u);
      list[q] = load_global(a.xyzm, p0 + t + q);
      if (kHash && k + lane < cnt) hsum += mix64((1ull << 40) + p0 + t + q);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    flush_tile<kComp, kPot, 1>(list, cnt, lane, w.stream, w.S, w.pi, a.eps2, R, nblk);
    __builtin_amdgcn_wave_barrier();
  }
  for (; nblk & (RunSums<kComp, kPot>::kNum - 1u); ++nblk) R.advance(1u);
}

// 64-bit sum over the wavefront, in every lane.
__device__ __forceinline__ uint64_t wave_sum64(uint64_t v) {
  uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  for (int d = 32; d >= 1; d >>= 1) {  // by 32-bit halves with carries
    const uint32_t olo = __shfl_xor(lo, d, 64), ohi = __shfl_xor(hi, d, 64);
    const uint32_t nlo = lo + olo;
    hi = hi + ohi + (nlo < lo ? 1u : 0u);
    lo = nlo;
  }
  return ((uint64_t)hi << 32) | lo;
}

// Results of a whole group from each lane's sums.
template <bool kPot>
__device__ __forceinline__ void finish_group(const WalkArgs &a, const WalkGroup &w,
                                             uint32_t lane, float sx, float sy, float sz,
                                             float sw) {
  stream_reduce(w.Wd, sx, sy, sz);
  store_group_result(a, w.gb, w.gc, lane, sx, sy, sz);
  if constexpr (kPot) {
    // the member's own entry (r = eps exactly) is in its list: add its
    // term back, phi_i = G (sum_j -m_j / r_j + m_i / eps)
    stream_reduce1(w.Wd, sw);
    if (lane < w.gc) {
      const float self = w.pi.w * __builtin_amdgcn_rsqf(a.eps2);
      a.phi[a.perm ? a.perm[w.gb + lane] : w.gb + lane] = a.G * (sw + self);
    }
  }
}

// Claims the next task beyond the nw first ones. The empty asm pins the
// wave-uniform result here, before the loop's back edge.
__device__ __forceinline__ uint32_t next_task(const WalkArgs &a, uint32_t nw, uint32_t lane) {
  // (the first empty asm keeps a spilled pointer's reload out of the claim)
  typedef __attribute__((address_space(1))) uint32_t *gp;
  gp head = reinterpret_cast<gp>(reinterpret_cast<uintptr_t>(a.head));
  asm volatile("" : "+s"(head));
  const uint32_t claim = __hip_atomic_fetch_add(head, lane == 0 ? 1u : 0u, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
  uint32_t t = __builtin_amdgcn_readfirstlane(claim);
  asm volatile("" : "+s"(t));
  return nw + t;
}

// Running sum r of a split group: its components, per lane, in the queue slot.
template <bool kPot>
__device__ __forceinline__ void store_sums(float *slot, uint32_t r, uint32_t lane,
                                           const Acc3<false, kPot> &u) {
  constexpr uint32_t kW = kPot ? 4 : 3;
  slot[(r * kW + 0) * 64 + lane] = u.x;
  slot[(r * kW + 1) * 64 + lane] = u.y;
  slot[(r * kW + 2) * 64 + lane] = u.z;
  if constexpr (kPot) slot[(r * kW + 3) * 64 + lane] = u.w;
}
template <bool kPot>
__device__ __forceinline__ void store_sums(float *slot, uint32_t r, uint32_t lane,
                                           const Acc3<true, kPot> &u) {
  const float v[8] = {u.x, u.y, u.z, u.w, u.cx, u.cy, u.cz, u.cw};
#pragma unroll
  for (uint32_t k = 0; k < 8; ++k) slot[(r * 8 + k) * 64 + lane] = v[k];
}

// The persistent loop with K wavefronts per group (a power of two): task t is
// part t mod K of queue position t / K. K is a constant here: as a run-time
// value it cost the loop 3 vector registers (75 against 72), one resident
// wavefront per SIMD, and spilled scalars.
template <bool kComp, bool kHash, bool kPot, uint32_t K>
__device__ __forceinline__ void walk_loop(const WalkArgs &a, const WaveLds &l, uint32_t ng,
                                          uint32_t wv, uint32_t lane) {
  uint32_t *stk =
      a.frontier + (size_t)(blockIdx.x * kWalkWavesPerWG + wv) * (size_t)(a.fmask + 1);
  const uint32_t ncell = a.sc->ncell;
  constexpr uint32_t kshift = K == 4u ? 2u : K == 2u ? 1u : 0u;
  // A wavefront's first task is its own number; it claims further ones only
  // while there are more tasks than wavefronts. (When every wavefront made a
  // first claim, 8192 atomics on one word, about 13 ns each, took 105 us of a
  // walk of 132 tasks that needed 40.)
  // No lane-predicated region may sit in this loop: the compiler threads such
  // regions across the back-edge, and a wave that re-enters with lane 0 masked
  // off reads a stale queue index. Every lane joins the queue atomic (lane 0
  // adds 1, the rest 0) and the per-group results below are stored by every
  // lane (same value, same address).
  const uint32_t nw = gridDim.x * kWalkWavesPerWG;
  const uint32_t ntask = ng << kshift;
  uint32_t task = __builtin_amdgcn_readfirstlane(blockIdx.x * kWalkWavesPerWG + wv);
  for (bool first = true; first || ntask > nw; first = false) {
    if (!first) task = next_task(a, nw, lane);
    if (task >= ntask) break;
    const uint32_t qi = task >> kshift;
    const uint32_t part = task & (K - 1u);
    const uint32_t g = a.order ? a.order[qi] : qi;
    const WalkGroup w = load_group(a, g, lane);
    const uint32_t root = a.groot ? a.groot[g] : 0u;
    const uint32_t limit = heavy_limit(a.groot ? a.cpcount[root] : a.n);
    const float reach = a.greach[g];
    stk[0] = root;  // (same value in every lane)
    RunSums<kComp, kPot> R;
    uint64_t hsum = 0;
    uint32_t entries = 0;
    const uint32_t end = walk_list<kComp, kHash, kPot, K>(
        a, l, w, stk, a.fmask + 1u, 1u, part, limit, reach, ncell, lane, R, entries, hsum);
    // `end` is wave-uniform: these branches are not lane-predicated; every
    // lane joins the atomics and stores. Every part of a split group ends the
    // same way (same traversal); a group without results is handed on to the
    // later passes by its entry count.
    if (end == kEndCorrupt || (end == kEndOverflow && !a.may_retry))
      atomicOr(&a.sc->status, end == kEndOverflow ? kStOverflow : kStCorrupt);
    if constexpr (K == 1u) {
      // (of no consequence for a group handed on: a later pass writes again)
      float sx, sy, sz, sw;
      R.total(sx, sy, sz, sw);
      finish_group<kPot>(a, w, lane, sx, sy, sz, sw);
    } else {
      // this part's running sums into the queue slot: [sum][component][lane]
      float *slot = a.split + (size_t)qi * a.slot_words;
      store_sums(slot, part, lane, R.u0);
      if constexpr (!kComp && K == 2u) store_sums(slot, part + 2u, lane, R.u1);
    }
    if (part == 0u) {
      if (kHash) a.ghash[g] = wave_sum64(hsum);
      a.gent[g] = end == 0u             ? entries
                  : end == kEndHeavy    ? kEntHeavy
                  : end == kEndOverflow ? kEntRetry
                                        : kEntNone;
    }
  }
}

template <bool kComp, bool kHash, bool kPot>
__device__ __forceinline__ void walk_body(const WalkArgs &a, float4 *lds_list) {
  const uint32_t wv = threadIdx.x >> 6;
  const uint32_t lane = lane_id();
  const WaveLds l = wave_lds(lds_list, wv, a.tile);
  const uint32_t ng = *a.qcount;
  const uint32_t K =
      split_factor(ng, a.split_waves, a.split_slots, a.split_mode,
                   heavy_limit(a.groot ? 0u : a.n));
  if (K == 1u)
    walk_loop<kComp, kHash, kPot, 1>(a, l, ng, wv, lane);
  else if (kComp || K == 2u)  // (two compensated sums)
    walk_loop<kComp, kHash, kPot, 2>(a, l, ng, wv, lane);
  else if constexpr (!kComp)
    walk_loop<kComp, kHash, kPot, 4>(a, l, ng, wv, lane);
}

// ---------------------------------------------------------------- heavy groups
// Front of a heavy group: starting from its walk root, cells that fail the MAC
// and hold more than `big` particles are replaced by their children, in order,
// round by round, until none is left or the front would not fit in kFrontCap
// cells. NT threads of one workgroup; cur and nxt hold kFrontCap cells each.
// Returns the front's length, with cur pointing at it (uniform) and nxt at the
// cells' weights: 1 for an accepted cell, another's particles, with kWeightFull for
// an over-full leaf.
constexpr uint32_t kWeightFull = 1u << 31;
template <int NT>
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t *wsum, uint32_t *total) {
  const uint32_t inc = wave_incl_scan_dpp(v);
  if constexpr (NT == 64) {
    *total = wave_last(inc);
    return inc - v;
  } else {
    const uint32_t w = threadIdx.x >> 6;
    __syncthreads();  // wsum's last use
    if (lane_id() == 63) wsum[w] = inc;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (uint32_t q = 0; q < NT / 64; ++q) {
      off += q < w ? wsum[q] : 0u;
      tot += wsum[q];
    }
    *total = tot;
    return off + inc - v;
  }
}

template <int NT>
__device__ __forceinline__ uint32_t heavy_front(const WalkArgs &a, uint32_t root, float4 glo,
                                                float4 ghi, uint32_t ncell, uint32_t big,
                                                uint32_t *&cur, uint32_t *&nxt,
                                                uint32_t *wsum, bool &any_full) {
  const uint32_t tid = threadIdx.x;
  // w: the cell's weight, nout, first: what it is replaced by (itself, or its
  // children)
  auto look = [&](uint32_t c, uint32_t &nout, uint32_t &first) -> uint32_t {
    nout = 1u;
    first = c;
    if (c >= ncell) return 1u;
    const float4 A = a.nodeA[c], B = a.nodeB[c];
    const uint32_t w0 = __float_as_uint(B.z), w1 = __float_as_uint(B.w), np = a.cpcount[c];
    float d2;
    if (mac_accept(A, B.x, a.G, glo, ghi, glo.w, a.bootstrap, d2)) return 1u;
    if (!(w1 & kLeafBit) && w1 >= 1u && w1 <= 8u && w0 > c && w0 < ncell && w1 <= ncell - w0 &&
        np > big) {
      nout = w1;
      first = w0;
    }
    return max(np, 1u) | ((w1 & kLeafBit) && np > kFullLeaf ? kWeightFull : 0u);
  };
  if (tid == 0) cur[0] = root;
  __syncthreads();
  uint32_t m = 1;
  for (int round = 0; round <= kMaxLevel; ++round) {
    // a round that cannot outgrow nxt leaves the weights in cur, in place of the
    // cells: if it opens none, it was the last, and nxt holds the same cells
    const bool fits = m <= kFrontCap / 8u;
    uint32_t out = 0, opened = 0;
    any_full = false;
    for (uint32_t k0 = 0; k0 < m; k0 += NT) {
      const bool has = k0 + tid < m;
      const uint32_t c = has ? cur[k0 + tid] : 0u;
      uint32_t nout = 0, first = c, wt = 0;
      if (has) {
        wt = look(c, nout, first);
        if (fits) cur[k0 + tid] = wt;
      }
      const bool open = first != c;  // (a child's index is never its parent's)
      // one scan: cells put out (12 bits: 8 per thread), opened and over-full ones
      static_assert(8 * NT < 4096 && NT < 512, "fields of the scan");
      uint32_t tot;
      const uint32_t v = nout | (open ? 1u << 12 : 0u) | ((wt & kWeightFull) ? 1u << 21 : 0u);
      const uint32_t ex = block_scan<NT>(v, wsum, &tot) & 0xfffu;
      if (out + (tot & 0xfffu) <= kFrontCap)
        for (uint32_t q = 0; q < nout; ++q) nxt[out + ex + q] = first + q;
      out += tot & 0xfffu;
      opened += (tot >> 12) & 0x1ffu;
      any_full = any_full || (tot >> 21) != 0u;
    }
    __syncthreads();
    if (opened == 0u || out > kFrontCap) {  // (uniform)
      if (!fits) {
        for (uint32_t k = tid; k < m; k += NT) {
          uint32_t nout, first;
          nxt[k] = look(cur[k], nout, first);
        }
        __syncthreads();
        return m;
      }
      break;
    }
    uint32_t *t = cur;
    cur = nxt;
    nxt = t;
    m = out;
  }
  uint32_t *t = cur;
  cur = nxt;
  nxt = t;
  return m;
}

// Cuts a front of m cells into parts of about equal weight: part r takes the
// cells [pb[r], pb[r + 1]), or, where any_full and ps[r] is not 0, slice ps[r] % 256 of
// ps[r] / 256 % 256 of the over-full leaf at front position ps[r] / 65536 - 1 (half
// of 40000 particles at one point: as one part a leaf of 20000 was a chain of 511
// us, 554 us for the whole walk before there were parts).
// Returns the number of parts (uniform); pb and ps are in LDS.
template <int NT>
__device__ __forceinline__ uint32_t heavy_parts(const uint32_t *weights, uint32_t work,
                                                uint32_t m, bool any_full, uint32_t *pb,
                                                uint32_t *ps, uint32_t *wsum) {
  const uint32_t tid = threadIdx.x;
  auto weight = [&](uint32_t k) -> uint32_t { return k < m ? weights[k] & ~kWeightFull : 0u; };
  auto full = [&](uint32_t k) -> bool { return k < m && (weights[k] & kWeightFull) != 0u; };
  uint32_t W = 0, tot, nfull = 0;  // (particles of over-full leaves)
  for (uint32_t k0 = 0; k0 < m; k0 += NT) {
    (void)block_scan<NT>(weight(k0 + tid), wsum, &tot);
    W += tot;
    if (any_full) {  // (uniform)
      (void)block_scan<NT>(full(k0 + tid) ? weight(k0 + tid) : 0u, wsum, &tot);
      nfull += tot;
    }
  }
  const uint32_t P = min(min((W + work - 1u) / work, kMaxParts), m + nfull / work);
  if (any_full) {
    for (uint32_t r = tid; r < P; r += NT) ps[r] = 0u;
    __syncthreads();
  }
  uint32_t base = 0;
  for (uint32_t k0 = 0; k0 < m; k0 += NT) {
    const uint32_t k = k0 + tid, wt = weight(k);
    const uint32_t pre = base + block_scan<NT>(wt, wsum, &tot);
    if (k < m) {
      const uint32_t p0 = (uint32_t)((uint64_t)pre * P / W);
      const uint32_t p1 = (uint32_t)((uint64_t)(pre + wt) * P / W);
      // an over-full leaf fills the parts after the one it starts in, up to the
      // one it ends in
      const uint32_t ns = any_full && full(k) && p1 > p0 + 1u ? p1 - p0 - 1u : 0u;
      for (uint32_t r = p0 + 1u; r <= p1; ++r) {
        pb[r] = ns != 0u && r == p0 + 1u ? k : k + 1u;
        if (r <= p0 + ns) ps[r] = ((k + 1u) << 16) | (ns << 8) | (r - p0 - 1u);
      }
      if (k == 0u) pb[0] = 0u;
    }
    base += tot;
  }
  __syncthreads();
  return P;
}

// Slice ps (see heavy_parts) of the over-full leaf c: its particles [x, x + y).
__device__ __forceinline__ uint2 leaf_slice(const WalkArgs &a, uint32_t c, uint32_t ps) {
  const float4 B = a.nodeB[c];
  const uint32_t b = __float_as_uint(B.z), i = ps & 255u, of = (ps >> 8) & 255u;
  const uint32_t n = b < a.n ? min(__float_as_uint(B.w) & ~kLeafBit, a.n - b) : 0u;
  const uint32_t lo = (uint32_t)((uint64_t)n * i / of);
  return make_uint2(b + lo, (uint32_t)((uint64_t)n * (i + 1u) / of) - lo);
}

// Results of a split group from its running sums.
template <bool kComp>
__device__ __forceinline__ void join_group(const WalkArgs &a, const WalkGroup &w,
                                           const float *slot, uint32_t lane) {
  float sx, sy, sz, sw = 0.f;
  if constexpr (kComp) {
    Acc3<true, true> u[2];
#pragma unroll
    for (uint32_t r = 0; r < 2; ++r) {
      float v[8];
#pragma unroll
      for (uint32_t k = 0; k < 8; ++k) v[k] = slot[(r * 8 + k) * 64 + lane];
      u[r].x = v[0], u[r].y = v[1], u[r].z = v[2], u[r].w = v[3];
      u[r].cx = v[4], u[r].cy = v[5], u[r].cz = v[6], u[r].cw = v[7];
    }
    u[0].merge(u[1]);  // (without the potential its sums are zero)
    u[0].total(sx, sy, sz, sw);
  } else {
    const uint32_t W = a.phi ? 4u : 3u;
    float v[4][4];
#pragma unroll
    for (uint32_t r = 0; r < 4; ++r)
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k)
        v[r][k] = k < W ? slot[(r * W + k) * 64 + lane] : 0.f;
    sx = ((v[0][0] + v[1][0]) + v[2][0]) + v[3][0];
    sy = ((v[0][1] + v[1][1]) + v[2][1]) + v[3][1];
    sz = ((v[0][2] + v[1][2]) + v[2][2]) + v[3][2];
    sw = ((v[0][3] + v[1][3]) + v[2][3]) + v[3][3];
  }
  if (a.phi)
    finish_group<true>(a, w, lane, sx, sy, sz, sw);
  else
    finish_group<false>(a, w, lane, sx, sy, sz, sw);
}

// After the main pass. Blocks [0, front_blocks): fronts and parts of the
// heavy groups (one workgroup per group; a group that finds no room in the
// part or front buffers is left to k_heavy_end). The other blocks, when the
// walk was split: per queue position, the four running sums of each lane
// added in order, then the stream butterfly and the results, as an unsplit
// walk ends; groups handed on (by their entry count) are left out. With no
// front blocks (the launch before the retry pass) they also collect that
// pass's queue.
// (Bound by a group's chain of rounds and by the requests on the counters. Heavy
// groups of a batch of 64 systems, 3.1 million particles: 214 us with 256
// workgroups, 130 with 1024, four per CU, and 104 with the weights taken in the
// front's last round and one atomic per group instead of three.)
constexpr uint32_t kFrontBlocks = 1024, kJoinBlocks = 512;
__global__ __launch_bounds__(256) void k_walk_mid(WalkArgs a, int hash, uint32_t front_blocks,
                                                  int join) {
  __shared__ uint32_t s_front[2 * kFrontCap];
  __shared__ uint32_t s_pb[kMaxParts + 1], s_ps[kMaxParts], s_wsum[4], s_at[5], s_list[256];
  const uint32_t ng = *a.qcount;
  if (blockIdx.x < front_blocks) {
    // the heavy ones among queue positions b, b + front_blocks, ...: consecutive
    // positions go to different workgroups
    const uint32_t ncell = a.sc->ncell;
    bool full = false;  // (uniform) no part slots are left
    for (uint32_t q0 = blockIdx.x; q0 < ng; q0 += 256u * front_blocks) {
      const uint64_t qi = (uint64_t)q0 + (uint64_t)threadIdx.x * front_blocks;
      if (threadIdx.x == 0) s_at[2] = 0u;
      __syncthreads();
      if (qi < ng) {
        const uint32_t gq = a.order ? a.order[qi] : (uint32_t)qi;
        if (a.gent[gq] == kEntHeavy) s_list[atomicAdd(&s_at[2], 1u)] = gq;
      }
      __syncthreads();
      const uint32_t nl = s_at[2];
      if (threadIdx.x == 0 && nl > 0u) s_at[3] = atomicAdd(&a.sc->nheavy, nl);
      for (uint32_t j = 0; j < nl; ++j) {
        const uint32_t g = s_list[j];
        if (full) {  // (uniform) left to k_heavy_end
          if (threadIdx.x == 0) {
            const uint32_t h = s_at[3] + j;
            a.heavy[h] = g;
            if (h < a.hslots) a.hrec[h] = make_uint2(0u, 0u);
            a.gent[g] = 0u;
            if (hash) a.ghash[g] = 0ull;
          }
          continue;
        }
        const uint32_t root = a.groot ? a.groot[g] : 0u;
        const float4 glo = a.gbox[2 * g], ghi = a.gbox[2 * g + 1];
        const uint32_t nr = a.groot ? a.cpcount[root] : a.n;
        uint32_t *cur = s_front, *nxt = s_front + kFrontCap;
        bool any_full;
        const uint32_t m = heavy_front<256>(a, root, glo, ghi, ncell, front_cell_max(nr), cur, nxt,
                                            s_wsum, any_full);
        const uint32_t P = heavy_parts<256>(nxt, part_work(nr), m, any_full, s_pb, s_ps,
                                              s_wsum);
        if (threadIdx.x == 0) {
          const uint32_t h = s_at[3] + j;
          // one request for parts (low word) and front cells
          const unsigned long long at =
              atomicAdd(&a.sc->nhpart, ((unsigned long long)m << 32) | P);
          const uint32_t s0 = (uint32_t)at, f0 = (uint32_t)(at >> 32);
          const bool room = s0 < a.hslots && h < a.hslots && P <= a.hslots - s0 &&
                            f0 < a.hfront_cap && m <= a.hfront_cap - f0;
          a.heavy[h] = g;
          if (h < a.hslots) a.hrec[h] = room ? make_uint2(s0, P) : make_uint2(0u, 0u);
          a.gent[g] = 0u;
          if (hash) a.ghash[g] = 0ull;
          s_at[0] = s0;
          s_at[1] = room ? f0 : kEntNone;
          s_at[4] = h;
        }
        __syncthreads();
        const uint32_t s0 = s_at[0], f0 = s_at[1], h = s_at[4];
        const bool room = f0 != kEntNone;
        full = s0 >= a.hslots;
        for (uint32_t r = threadIdx.x; r < P; r += 256u)
          if (s0 + r < a.hslots && s0 + r >= s0) {
            uint4 part = make_uint4(g, 0u, 0u, h);  // nothing to walk
            if (room && any_full && s_ps[r] != 0u) {
              const uint2 sl = leaf_slice(a, cur[(s_ps[r] >> 16) - 1u], s_ps[r]);
              part = make_uint4(g, sl.x, sl.y | kPartSlice, h);
            } else if (room) {
              part = make_uint4(g, f0 + s_pb[r], s_pb[r + 1] - s_pb[r], h);
            }
            a.hparts[s0 + r] = part;
          }
        if (room)
          for (uint32_t k = threadIdx.x; k < m; k += 256u) a.hfront[f0 + k] = cur[k];
        __syncthreads();  // LDS is reused by the next group
      }
    }
    return;
  }
  if (front_blocks == 0u) {
    // before the retry pass: collect its queue
    for (uint64_t qi = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; qi < ng;
         qi += (uint64_t)gridDim.x * blockDim.x) {
      const uint32_t g = a.order ? a.order[qi] : (uint32_t)qi;
      if (a.gent[g] == kEntRetry) a.retry[atomicAdd(&a.sc->nretry, 1u)] = g;
    }
  }
  if (!join || split_factor(ng, a.split_waves, a.split_slots, a.split_mode, 4096u) == 1u) return;
  const uint32_t lane = lane_id();
  const uint32_t nw = (gridDim.x - front_blocks) * (blockDim.x >> 6);
  for (uint32_t qi = __builtin_amdgcn_readfirstlane(
           (blockIdx.x - front_blocks) * (blockDim.x >> 6) + (threadIdx.x >> 6));
       qi < ng; qi += nw) {
    const uint32_t g = a.order ? a.order[qi] : qi;
    // (the front blocks may already have reset a heavy group's count: its
    // results are written again by k_heavy_end)
    if (a.gent[g] >= kEntRetry) continue;
    const float *slot = a.split + (size_t)qi * a.slot_words;
    const WalkGroup w = load_group(a, g, lane);
    if (a.hwords == heavy_part_words(1))
      join_group<true>(a, w, slot, lane);
    else
      join_group<false>(a, w, slot, lane);
  }
}

// A lane's sums over the parts of a heavy group, added in part order. The
// compensated form carries each part's sum and correction.
template <bool kComp, bool kPot>
struct PartSums {
  static constexpr uint32_t kWords = kPot ? 4 : 3;
  float v[4] = {0.f, 0.f, 0.f, 0.f};
  __device__ __forceinline__ static void store(float *slot, uint32_t lane,
                                               const RunSums<kComp, kPot> &R) {
    float x, y, z, w;
    R.total(x, y, z, w);
    slot[0 * 64 + lane] = x;
    slot[1 * 64 + lane] = y;
    slot[2 * 64 + lane] = z;
    if constexpr (kPot) slot[3 * 64 + lane] = w;
  }
  __device__ __forceinline__ void add(const float (&p)[8]) {
#pragma unroll
    for (uint32_t k = 0; k < kWords; ++k) v[k] += p[k];
  }
  __device__ __forceinline__ void add(const RunSums<kComp, kPot> &R) {
    float x, y, z, w;
    R.total(x, y, z, w);
    v[0] += x;
    v[1] += y;
    v[2] += z;
    if constexpr (kPot) v[3] += w;
  }
  __device__ __forceinline__ float total(uint32_t k) const { return v[k]; }
};
template <bool kPot>
struct PartSums<true, kPot> {
  static constexpr uint32_t kWords = 8;
  float v[4] = {0.f, 0.f, 0.f, 0.f}, c[4] = {0.f, 0.f, 0.f, 0.f};
  __device__ __forceinline__ static void store(float *slot, uint32_t lane,
                                               const RunSums<true, kPot> &R) {
    store_sums(slot, 0u, lane, R.merged());
  }
  __device__ __forceinline__ void add(const float (&p)[8]) {
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
      Acc3<true, kPot>::nadd(v[k], c[k], p[k]);
      c[k] += p[4 + k];
    }
  }
  __device__ __forceinline__ void add(const RunSums<true, kPot> &R) {
    const Acc3<true, kPot> u = R.merged();
    const float p[8] = {u.x, u.y, u.z, u.w, u.cx, u.cy, u.cz, u.cw};
    add(p);
  }
  __device__ __forceinline__ float total(uint32_t k) const { return v[k] + c[k]; }
};

// The parts of the heavy groups: each wavefront walks the subtrees of one
// part's cells and stores its lanes' sums in the part's slot. The parts are
// about equal, so wavefront w takes parts w, w + nw, ...; taken from a queue,
// 44000 parts of a batch of 64 systems were 44000 atomics on one word: 572 us,
// 241 without, and no wavefronts more helped before. A part's stack stays under
// kFrontCap cells but for trees far from any in use; a part that outgrows it
// leaves its group to k_heavy_end, whose stacks hold every cell.
template <bool kComp, bool kHash, bool kPot>
__global__ __launch_bounds__(64 * kWalkWavesPerWG,
                             walk_occupancy(kComp, kHash, kPot)) void k_heavy_walk(WalkArgs a) {
  HIP_DYNAMIC_SHARED(float4, lds_list)
  const uint32_t wv = threadIdx.x >> 6;
  const uint32_t lane = lane_id();
  const WaveLds l = wave_lds(lds_list, wv, a.tile);
  uint32_t *stk =
      a.frontier + (size_t)(blockIdx.x * kWalkWavesPerWG + wv) * (size_t)(a.fmask + 1);
  const uint32_t np = min((uint32_t)a.sc->nhpart, a.hslots);
  const uint32_t ncell = a.sc->ncell;
  const uint32_t nw = gridDim.x * kWalkWavesPerWG;
  for (uint32_t t = __builtin_amdgcn_readfirstlane(blockIdx.x * kWalkWavesPerWG + wv); t < np;
       t += nw) {
    const uint4 part = a.hparts[t];
    const uint32_t g = __builtin_amdgcn_readfirstlane(part.x);
    const uint32_t f0 = __builtin_amdgcn_readfirstlane(part.y);
    const uint32_t m = __builtin_amdgcn_readfirstlane(part.z);
    const WalkGroup w = load_group(a, g, lane);
    RunSums<kComp, kPot> R;
    uint64_t hsum = 0;
    uint32_t entries = 0, end = 0;
    if (m & kPartSlice) {  // (uniform)
      entries = m & ~kPartSlice;
      add_range<kComp, kHash, kPot>(a, l, w, f0, entries, lane, R, hsum);
    } else {
      // (every lane stores; past the end the last cell again)
      for (uint32_t k = 0; k < m; k += 64u) {
        const uint32_t q = min(k + lane, m - 1u);
        stk[q] = a.hfront[f0 + q];
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      end = walk_list<kComp, kHash, kPot, 1>(a, l, w, stk, a.fmask + 1u, m, 0u, 0xffffffffu,
                                             0.f, ncell, lane, R, entries, hsum);
    }
    if (end == kEndOverflow) a.hrec[part.w] = make_uint2(0u, 0u);  // left to k_heavy_end
    if (end == kEndCorrupt) atomicOr(&a.sc->status, kStCorrupt);
    PartSums<kComp, kPot>::store(a.hsum + (size_t)t * a.hwords, lane, R);
    atomicAdd(&a.gent[g], lane == 0 ? entries : 0u);
    if (kHash) {
      const unsigned long long hs = wave_sum64(hsum);
      atomicAdd(&a.ghash[g], lane == 0 ? hs : 0ull);
    }
  }
}

// Results of the heavy groups: one wavefront (workgroup) per group adds its
// parts' sums in order. A group that found no room for its parts is walked
// here, part after part, with the same sums. Each workgroup's region of the
// stack buffer holds a stack of `cap` cells and two fronts.
template <bool kComp, bool kHash, bool kPot>
__global__ __launch_bounds__(64) void k_heavy_end(WalkArgs a) {
  HIP_DYNAMIC_SHARED(float4, lds_list)
  __shared__ uint32_t s_pb[kMaxParts + 1], s_ps[kMaxParts];
  using Sums = PartSums<kComp, kPot>;
  const uint32_t lane = lane_id();
  const WaveLds l = wave_lds(lds_list, 0u, a.tile);
  uint32_t *stk = a.frontier + (size_t)blockIdx.x * (size_t)(a.fmask + 1u + 2u * kFrontCap);
  const uint32_t nh = a.sc->nheavy, ncell = a.sc->ncell;
  for (uint32_t h = blockIdx.x; h < nh; h += gridDim.x) {
    const uint32_t g = __builtin_amdgcn_readfirstlane(a.heavy[h]);
    const WalkGroup w = load_group(a, g, lane);
    const uint2 rec = h < a.hslots ? a.hrec[h] : make_uint2(0u, 0u);
    const uint32_t s0 = __builtin_amdgcn_readfirstlane(rec.x);
    const uint32_t P = __builtin_amdgcn_readfirstlane(rec.y);
    Sums T;
    if (P > 0u) {
      // eight parts' loads in flight (P is at most kMaxParts)
      for (uint32_t r = 0; r < P; r += 8u) {
        float p[8][8];
#pragma unroll
        for (uint32_t j = 0; j < 8; ++j) {
          const float *slot = a.hsum + (size_t)(s0 + min(r + j, P - 1u)) * a.hwords;
#pragma unroll
          for (uint32_t k = 0; k < 8; ++k) p[j][k] = k < Sums::kWords ? slot[k * 64 + lane] : 0.f;
        }
#pragma unroll
        for (uint32_t j = 0; j < 8; ++j)
          if (r + j < P) T.add(p[j]);
      }
    } else {
      uint32_t *cur = stk + a.fmask + 1u, *nxt = cur + kFrontCap;
      const uint32_t root = a.groot ? a.groot[g] : 0u;
      const uint32_t nr = a.groot ? a.cpcount[root] : a.n;
      bool any_full;
      const uint32_t m = heavy_front<64>(a, root, w.glo, w.ghi, ncell, front_cell_max(nr), cur, nxt,
                                         nullptr, any_full);
      const uint32_t Q = heavy_parts<64>(nxt, part_work(nr), m, any_full, s_pb, s_ps, nullptr);
      uint64_t hsum = 0;
      uint32_t entries = 0, end = 0;
      for (uint32_t r = 0; r < Q && end == 0u; ++r) {
        const uint32_t sl = any_full ? __builtin_amdgcn_readfirstlane(s_ps[r]) : 0u;
        RunSums<kComp, kPot> R;
        if (sl != 0u) {
          const uint2 range = leaf_slice(a, cur[(sl >> 16) - 1u], sl);
          const uint32_t n = __builtin_amdgcn_readfirstlane(range.y);
          add_range<kComp, kHash, kPot>(a, l, w, __builtin_amdgcn_readfirstlane(range.x), n, lane,
                                        R, hsum);
          entries += n;
          T.add(R);
          continue;
        }
        const uint32_t k0 = __builtin_amdgcn_readfirstlane(s_pb[r]);
        const uint32_t c = __builtin_amdgcn_readfirstlane(s_pb[r + 1]) - k0;
        for (uint32_t k = 0; k < c; k += 64u) {
          const uint32_t q = min(k + lane, c - 1u);
          stk[q] = cur[k0 + q];
        }
        __syncthreads();
        uint32_t ent = 0;
        end = walk_list<kComp, kHash, kPot, 1>(a, l, w, stk, a.fmask + 1u, c, 0u, 0xffffffffu,
                                               0.f, ncell, lane, R, ent, hsum);
        entries += ent;
        T.add(R);
      }
      if (end && lane == 0)
        atomicOr(&a.sc->status, end == kEndOverflow ? kStOverflow : kStCorrupt);
      if (lane == 0) a.gent[g] = entries;
      if (kHash) {
        const uint64_t hs = wave_sum64(hsum);
        if (lane == 0) a.ghash[g] = hs;
      }
      __syncthreads();
    }
    finish_group<kPot>(a, w, lane, T.total(0), T.total(1), T.total(2), T.total(3));
  }
}

// Interactions of the walked groups, and of those the tree's reference walk
// also took, now and then (the reference walk records them here): integer
// sums per workgroup into part[4 * blockIdx.x ..] (same-address atomics from
// every workgroup would serialise), added up by k_walk_stat_fold. A small
// set's walk (kOne) takes one workgroup, which finishes the statistics itself.
__device__ __forceinline__ void store_walk_stat(DevScalars *__restrict__ sc, bool queued,
                                                const unsigned long long (&t)[4],
                                                unsigned long long t1, uint32_t seq,
                                                WalkStat *__restrict__ host) {
  WalkStat w;
  w.ngroup = sc->ngroup;
  w.queued = queued ? sc->nqueue : sc->ngroup;
  w.inter = t[0];
  w.inter_a = t[1];
  w.inter_ref = t[2];
  w.entries = t[3];
  w.tick = sc->tick;
  w.kmax = sc->kmax;
  w.t0 = sc->walk_t0;
  w.t1 = t1;
  w.seq = 0u;
  *host = w;  // page-locked host memory: no copy after the kernel
  // (the host reads the rest once it sees the number)
  __hip_atomic_store(&host->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

constexpr int kStatThreads = 1024;  // of the single workgroup
template <bool kOne>
__global__ __launch_bounds__(kOne ? kStatThreads : 256) void k_walk_stat(
    DevScalars *__restrict__ sc, const uint32_t *__restrict__ order,
    const uint32_t *__restrict__ gcount, const uint32_t *__restrict__ gent,
    uint32_t *__restrict__ gref, int record, unsigned long long *__restrict__ part,
    uint32_t seq, WalkStat *__restrict__ host) {
  const unsigned long long t1 = wall_clock64();  // the walk has ended
  constexpr int kWaves = (kOne ? kStatThreads : 256) / 64;
  __shared__ unsigned long long s_sum[kWaves][4];
  const uint32_t nq = order ? sc->nqueue : sc->ngroup;
  unsigned long long v[4] = {0, 0, 0, 0};  // interactions: all, of reference groups now, then
  for (uint32_t q = blockIdx.x * blockDim.x + threadIdx.x; q < nq;
       q += gridDim.x * blockDim.x) {
    const uint32_t g = order ? order[q] : q;
    const uint32_t e = gent[g], c = gcount[g];
    if (e == 0xffffffffu) continue;
    const unsigned long long ec = (unsigned long long)e * c;
    v[0] += ec;
    v[3] += e;
    uint32_t r = gref[g];
    if (record && r == 0) {
      r = e;
      gref[g] = e;
    }
    if (r != 0) {
      v[1] += ec;
      v[2] += (unsigned long long)r * c;
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    for (int d = 32; d >= 1; d >>= 1) v[k] += __shfl_xor(v[k], d, 64);
    if (lane_id() == 0) s_sum[threadIdx.x >> 6][k] = v[k];
  }
  __syncthreads();
  if constexpr (kOne) {
    if (threadIdx.x == 0) {
      unsigned long long t[4] = {0, 0, 0, 0};
      for (int w = 0; w < kWaves; ++w)
        for (int k = 0; k < 4; ++k) t[k] += s_sum[w][k];
      store_walk_stat(sc, order != nullptr, t, t1, seq, host);
    }
  } else if (threadIdx.x < 4) {
    part[4 * blockIdx.x + threadIdx.x] = s_sum[0][threadIdx.x] + s_sum[1][threadIdx.x] +
                                         s_sum[2][threadIdx.x] + s_sum[3][threadIdx.x];
    if (blockIdx.x == 0 && threadIdx.x == 0) sc->walk_t1 = t1;
  }
}

// The walk statistics: the partials' sums and the step's scalars (one
// workgroup of kStatBlocks threads).
__global__ __launch_bounds__(kStatBlocks) void k_walk_stat_fold(
    DevScalars *__restrict__ sc, const unsigned long long *__restrict__ part, int queued,
    uint32_t seq, WalkStat *__restrict__ host) {
  __shared__ unsigned long long s_sum[kStatBlocks / 64][4];
  unsigned long long v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    v[k] = part[4 * threadIdx.x + k];
    for (int d = 32; d >= 1; d >>= 1) v[k] += __shfl_xor(v[k], d, 64);
  }
  if (lane_id() == 0)
    for (int k = 0; k < 4; ++k) s_sum[threadIdx.x >> 6][k] = v[k];
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long t[4] = {0, 0, 0, 0};
    for (int w = 0; w < kStatBlocks / 64; ++w)
      for (int k = 0; k < 4; ++k) t[k] += s_sum[w][k];
    store_walk_stat(sc, queued != 0, t, sc->walk_t1, seq, host);
  }
}

// The walk, and its retry pass as a kernel of its own (so that profiles and
// the walk timing see the main pass alone).
template <bool kComp, bool kHash>
__global__ __launch_bounds__(64 * kWalkWavesPerWG,
                             walk_occupancy(kComp, kHash, false)) void k_walk(WalkArgs a) {
  HIP_DYNAMIC_SHARED(float4, lds_list)
  walk_body<kComp, kHash, false>(a, lds_list);
}

template <bool kComp, bool kHash>
__global__ __launch_bounds__(64 * kWalkWavesPerWG,
                             walk_occupancy(kComp, kHash, false)) void k_walk_retry(WalkArgs a) {
  HIP_DYNAMIC_SHARED(float4, lds_list)
  walk_body<kComp, kHash, false>(a, lds_list);
}

// The potential variant (also writes phi), main and retry pass.
template <bool kComp, bool kHash>
__global__ __launch_bounds__(64 * kWalkWavesPerWG,
                             walk_occupancy(kComp, kHash, true)) void k_walk_pot(WalkArgs a) {
  HIP_DYNAMIC_SHARED(float4, lds_list)
  walk_body<kComp, kHash, true>(a, lds_list);
}

__global__ void k_fill_u32(uint32_t *p, uint32_t v, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

void launch_fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t st) {
  int64_t g = cdiv(n, 256);
  if (g > 1024) g = 1024;
  if (g < 1) g = 1;
  hipLaunchKernelGGL(k_fill_u32, dim3(g), dim3(256), 0, st, p, v, n);
}

// Up to this many particles (so, at some ten and more per group, a few
// thousand groups) the statistics take one workgroup.
constexpr int64_t kStatOne = 128 * 1024;

void launch_walk_stat(int64_t n, bool queued, bool record, const Ptrs &P, WalkStat *host,
                      hipStream_t st, uint32_t seq) {
  const uint32_t *order = queued ? P.order : nullptr;
  if (n <= kStatOne) {
    hipLaunchKernelGGL(k_walk_stat<true>, dim3(1), dim3(kStatThreads), 0, st, P.sc, order,
                       P.gcount, P.gent, P.gref, record ? 1 : 0, P.wpart, seq, host);
    return;
  }
  hipLaunchKernelGGL(k_walk_stat<false>, dim3(kStatBlocks), dim3(256), 0, st, P.sc, order,
                     P.gcount, P.gent, P.gref, record ? 1 : 0, P.wpart, seq, host);
  hipLaunchKernelGGL(k_walk_stat_fold, dim3(1), dim3(kStatBlocks), 0, st, P.sc, P.wpart,
                     queued ? 1 : 0, seq, host);
}


namespace {
WalkArgs walk_args(const WalkCfg &c, const uint32_t *perm, int64_t n, float *ax, float *ay,
                   float *az, const Ptrs &P) {
  WalkArgs a;
  a.nodeA = P.nodeA;
  a.nodeB = P.nodeB;
  a.xyzm = P.xyzm;
  a.gbegin = P.gbegin;
  a.gcount = P.gcount;
  a.gbox = P.gbox;
  a.greach = P.greach;
  a.perm = perm;
  a.order = c.use_order ? P.order : nullptr;
  a.qcount = c.use_order ? &P.sc->nqueue : &P.sc->ngroup;
  a.groot = c.batch ? P.groot : nullptr;
  a.asort = c.asort_out ? P.asort : nullptr;
  a.cpcount = P.cpcount;
  // a stack that holds every cell of the tree cannot overflow: no retry pass
  a.may_retry = c.frontier_cap < c.heavy_cap ? 1 : 0;
  a.retry = P.retry;
  a.nretry = &P.sc->nretry;
  a.heavy = P.heavy;
  a.hparts = P.hparts;
  a.hrec = P.hrec;
  a.hfront = P.hfront;
  a.hsum = P.hsum;
  a.hslots = (uint32_t)c.heavy_slots;
  a.hfront_cap = (uint32_t)c.heavy_slots * kHeavyFrontPerSlot;
  a.hwords = heavy_part_words(c.compensated);
  a.head = &P.sc->queue_head;
  a.frontier = P.frontier;
  a.gent = P.gent;
  a.ghash = P.ghash;
  a.sc = P.sc;
  a.ax = ax;
  a.ay = ay;
  a.az = az;
  a.phi = c.phi;
  a.G = c.G;
  a.eps2 = c.eps * c.eps;
  a.n = (uint32_t)n;
  a.tile = (uint32_t)c.list_tile;
  a.fmask = (uint32_t)c.frontier_cap - 1u;
  a.bootstrap = c.bootstrap;
  a.split = P.split;
  a.split_mode = c.split;
  // (room for the plain sums only, on the allocation-free call's scratch: its
  // compensated sums are not split)
  const bool fits = c.slot_bytes >= (c.compensated || c.phi ? kSplitSlotWide : kSplitSlotBytes);
  a.split_slots = fits ? (uint32_t)c.split_slots : 0u;
  a.slot_words = (uint32_t)c.slot_bytes / 4u;
  return a;
}

// per wave: list tile + padding (16 B/entry) + owner table (64 x (16 + 4 + 4) B)
size_t walk_lds(const WalkCfg &c, int waves) {
  return (size_t)waves * ((c.list_tile + kListPad) * sizeof(float4) + 64 * 24);
}

}  // namespace

#define NB_WALK_LAUNCH(KERNEL, c, grid, lds, st, w)                           \
  do {                                                                         \
    const dim3 block_(64 * kWalkWavesPerWG);                                   \
    if ((c).compensated) {                                                     \
      if ((c).hash)                                                            \
        hipLaunchKernelGGL((KERNEL<true, true>), grid, block_, lds, st, w);    \
      else                                                                     \
        hipLaunchKernelGGL((KERNEL<true, false>), grid, block_, lds, st, w);   \
    } else {                                                                   \
      if ((c).hash)                                                            \
        hipLaunchKernelGGL((KERNEL<false, true>), grid, block_, lds, st, w);   \
      else                                                                     \
        hipLaunchKernelGGL((KERNEL<false, false>), grid, block_, lds, st, w);  \
    }                                                                          \
  } while (0)

namespace {
template <bool kComp, bool kHash, bool kPot>
void heavy_passes(const WalkCfg &c, WalkArgs a, const Ptrs &P, hipStream_t st) {
  a.frontier = P.frontier;
  a.fmask = (uint32_t)c.heavy_stack - 1u;
  hipLaunchKernelGGL((k_heavy_walk<kComp, kHash, kPot>), dim3(c.heavy_waves / kWalkWavesPerWG),
                     dim3(64 * kWalkWavesPerWG), walk_lds(c, kWalkWavesPerWG), st, a);
  a.fmask = (uint32_t)c.heavy_cap - 1u;
  hipLaunchKernelGGL((k_heavy_end<kComp, kHash, kPot>), dim3(c.heavy_end_blocks), dim3(64),
                     walk_lds(c, 1), st, a);
}
template <bool kComp>
void heavy_passes_of(const WalkCfg &c, const WalkArgs &a, const Ptrs &P, hipStream_t st) {
  if (c.phi)
    c.hash ? heavy_passes<kComp, true, true>(c, a, P, st)
           : heavy_passes<kComp, false, true>(c, a, P, st);
  else
    c.hash ? heavy_passes<kComp, true, false>(c, a, P, st)
           : heavy_passes<kComp, false, false>(c, a, P, st);
}
}  // namespace

// The main pass; the retry pass (groups that outgrew a stack smaller than the
// bound, walked again with the largest stacks, by as many wavefronts as the
// stack buffer then serves; a second overflow is reported, it cannot happen);
// the fronts of heavy groups and the sums of a split walk; the heavy groups'
// parts and their sums. (The queue counters are cleared by k_group_bounds,
// which runs before every walk.)
void launch_walk(const WalkCfg &c, const uint32_t *perm, int64_t n, float *ax, float *ay,
                 float *az, const Ptrs &P, hipStream_t st) {
  WalkArgs a = walk_args(c, perm, n, ax, ay, az, P);
  // four wavefronts for every group there may be (of 16 particles, or group_max if
  // that is smaller) are more than a tree has tasks; fewer only share
  const int blocks = (int)std::min<int64_t>(
      c.num_cu * c.waves_per_cu / kWalkWavesPerWG,
      std::max<int64_t>(cdiv(4 * n, kWalkWavesPerWG * std::min(c.group_max, 16)), 64));
  a.split_waves = (uint32_t)(blocks * kWalkWavesPerWG);
  // Small groups add little per entry, so that a second traversal costs more than
  // it saves once the queue fills the chip (potential of 40000 particles in groups
  // of up to 4, 13000 of them: 332 us unsplit, 400 with K = 2)
  if (c.phi && c.split == 0 && c.group_max <= 16)
    a.split_slots = std::min(a.split_slots, a.split_waves / 4u);
  const size_t lds = walk_lds(c, kWalkWavesPerWG);
  if (c.phi)
    NB_WALK_LAUNCH(k_walk_pot, c, dim3(blocks), lds, st, a);
  else
    NB_WALK_LAUNCH(k_walk, c, dim3(blocks), lds, st, a);
  if (a.may_retry) {
    // the split walk's sums first: they leave out the groups handed on
    hipLaunchKernelGGL(k_walk_mid, dim3(kJoinBlocks), dim3(256), 0, st, a, 0, 0u, 1);
    WalkArgs r = a;
    r.order = P.retry;
    r.qcount = &P.sc->nretry;
    r.may_retry = 0;
    r.fmask = (uint32_t)c.heavy_cap - 1u;
    r.head = &P.sc->retry_head;
    r.split_mode = -1;  // results written by the pass itself
    const dim3 rgrid(c.retry_waves / kWalkWavesPerWG);
    if (c.phi)
      NB_WALK_LAUNCH(k_walk_pot, c, rgrid, lds, st, r);
    else
      NB_WALK_LAUNCH(k_walk_retry, c, rgrid, lds, st, r);
    hipLaunchKernelGGL(k_walk_mid, dim3(kFrontBlocks), dim3(256), 0, st, a, c.hash ? 1 : 0,
                       kFrontBlocks, 0);
  } else {
    hipLaunchKernelGGL(k_walk_mid, dim3(kFrontBlocks + kJoinBlocks), dim3(256), 0, st, a, c.hash ? 1 : 0,
                       kFrontBlocks, 1);
  }
  // (a list holds no more entries than there are particles)
  if (n <= (int64_t)heavy_limit((uint32_t)n)) return;
  if (c.compensated)
    heavy_passes_of<true>(c, a, P, st);
  else
    heavy_passes_of<false>(c, a, P, st);
}

}  // namespace nb
