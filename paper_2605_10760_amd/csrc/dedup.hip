// Occupancy-aware deduplication of borrowed Gaussians (Sec. III-C, Eqs.
// (envelope), (free_carve), (dedup)).
//
// The set is a bitmap over the box of voxels the inputs touch, one bit per
// voxel (32 along x to a word), when it fits the workspace, and otherwise an
// open-addressing hash set of 64-bit voxel keys (21 bits per axis, offset
// 2^20); the device decides, so nothing is read back in between:
//   k_dd_bounds  per-workgroup bounds of the target boxes and of the segments'
//                end voxels (a walk never leaves the box of its two ends);
//   k_dd_plan    their box, and which form holds it;
//   k_dd_clear   empty the set (a fill kernel, capturable);
//   k_dd_occ     one thread per target Gaussian inserts every voxel of its
//                box [mu - k s, mu + k s] (bitmap: a masked OR per word);
//   k_dd_free    one thread per keyframe pixel walks the voxels of the
//                segment from the camera centre to the back-projected depth
//                (t in [0, 1)) and inserts them (hash set: through a
//                workgroup-local LDS set that drops the repeats of
//                neighbouring rays);
//   k_dd_count   distinct voxels of the bitmap;
//   k_dd_probe   one thread per borrowed Gaussian looks up the voxel of its
//                mean: kept only when absent.
// The bitmap of a 6 x 3 x 4 m room at 5 cm is 72 KB and stays in L2; a
// hash insert is a random 64-byte line of a table a thousand times that.
// 350k boxes and 2.46M rays of 8 keyframes: boxes 1416 -> 160 us, rays
// 984 -> 372 us (and 38 us for the bounds).
// Voxel indices are floor(x / v) in FP64 from the FP32 inputs; segment
// crossings are computed per plane as (plane - c) / (r - c) (no incremental
// sums) and walked in increasing t, ties to the lower axis, with no fused
// multiply-add, so every index is reproducible.  Inserts use 64-bit CAS with
// linear probing, bounded by DD_MAX_PROBE; an insert that finds no slot
// raises the overflow flag (bit 0).  Indices outside the key range (+-2^20
// voxels per axis, NaN included) or a box / segment of more than 2^22 voxels
// raise bit 1 and are skipped, so every thread's loop is bounded.
#include <algorithm>

#include "common.h"

namespace gsr {

constexpr unsigned long long DD_EMPTY = ~0ull;
constexpr int DD_MAX_PROBE = 1 << 14;
constexpr long long DD_OFF = 1ll << 20;
constexpr long long DD_MAX_CELLS = 1ll << 22;  // voxels of one box or one segment
constexpr int DD_BOUND_BLOCKS = 512;           // workgroups of k_dd_bounds at most

// Written by k_dd_plan, behind the counters in the workspace's header.
struct DedupGrid {
  int dense;     // the bitmap holds the set
  int lo[3];     // its first voxel
  int n[3];      // its extent
  int wx;        // words along x
  unsigned long long words;
};

struct DedupTable {
  unsigned long long* keys;  // hash set; its storage holds the bitmap instead
  unsigned int* flags;
  unsigned int* counters;  // [0] overflow flag, [1] distinct voxels
  unsigned long long mask;
  DedupGrid* grid;
  int* bounds;             // [blocks][6] partial bounds, at the start of keys
  __device__ unsigned int* bits() const { return reinterpret_cast<unsigned int*>(keys); }
};

// Reads and writes of memory that other threads write meanwhile: relaxed
// atomics of the narrowest scope, which are the plain instructions but neither
// torn nor repeated by the compiler.  Their readers bear a stale value (cells only
// gain bits or go from empty to final), not half of one and half of another.
template <class T>
__device__ __forceinline__ T dd_peek(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
template <class T>
__device__ __forceinline__ void dd_poke(T* p, T x) {
  __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Sets bits of a word of the bitmap.  A look first: a word that
// already holds them (the rays of one keyframe share most of their voxels)
// needs no atomic, and a stale one falls through to it.
__device__ __forceinline__ void dd_or(unsigned int* w, unsigned int bits) {
  if ((dd_peek(w) & bits) != bits) atomicOr(w, bits);
}
__device__ __forceinline__ unsigned int* dd_word(const DedupTable& T, const DedupGrid& G, int x,
                                                 int y, int z) {
  return T.bits() + ((unsigned long long)(z - G.lo[2]) * G.n[1] + (y - G.lo[1])) * G.wx +
         ((x - G.lo[0]) >> 5);
}

__device__ __forceinline__ unsigned long long dd_pack(long long x, long long y, long long z) {
  return (unsigned long long)((x + DD_OFF) & 0x1FFFFF) |
         ((unsigned long long)((y + DD_OFF) & 0x1FFFFF) << 21) |
         ((unsigned long long)((z + DD_OFF) & 0x1FFFFF) << 42);
}

// splitmix64 finaliser
__device__ __forceinline__ unsigned long long dd_mix(unsigned long long k) {
  k ^= k >> 30;
  k *= 0xbf58476d1ce4e5b9ull;
  k ^= k >> 27;
  k *= 0x94d049bb133111ebull;
  k ^= k >> 31;
  return k;
}

// A slot's key only ever goes from empty to its final value, so a
// read that already shows the key (or the flag) settles the insert without
// an atomic: many rays of one keyframe share the voxels near its camera, and
// their CASes would otherwise queue on the same slot.  A stale read of an
// empty slot falls through to the CAS, which decides.
__device__ void dd_insert(const DedupTable& T, unsigned long long key, unsigned int flag) {
  unsigned long long h = dd_mix(key) & T.mask;
  for (int probe = 0; probe < DD_MAX_PROBE && probe <= (long long)T.mask; ++probe) {
    unsigned long long cur = dd_peek(&T.keys[h]);
    if (cur == DD_EMPTY) {
      cur = atomicCAS(&T.keys[h], DD_EMPTY, key);
      if (cur == DD_EMPTY) {
        atomicAdd(&T.counters[1], 1u);
        atomicOr(&T.flags[h], flag);
        return;
      }
    }
    if (cur == key) {
      if ((dd_peek(&T.flags[h]) & flag) == 0u) atomicOr(&T.flags[h], flag);
      return;
    }
    h = (h + 1) & T.mask;
  }
  atomicOr(&T.counters[0], 1u);
}

// Workgroup-local filter in front of dd_insert: the rays of one workgroup
// (neighbouring pixels of one keyframe) cross mostly the same voxels, so a
// key goes to the global set only from the thread that first places it in
// this LDS set (bounded probing; a key that finds no LDS slot goes straight
// to the global set).  Every key still reaches the global set, once per
// workgroup at most.
constexpr int DD_LSLOTS = 4096;
constexpr int DD_LPROBE = 8;
__device__ void dd_insert_local(const DedupTable& T, unsigned long long* lk,
                                unsigned long long key, unsigned int flag) {
  unsigned int h = (unsigned int)(dd_mix(key) >> 40) & (DD_LSLOTS - 1);
  for (int probe = 0; probe < DD_LPROBE; ++probe) {
    unsigned long long cur = dd_peek(&lk[h]);
    if (cur == DD_EMPTY) {
      cur = atomicCAS(&lk[h], DD_EMPTY, key);
      if (cur == DD_EMPTY) {
        dd_insert(T, key, flag);
        return;
      }
    }
    if (cur == key) return;
    h = (h + 1) & (DD_LSLOTS - 1);
  }
  dd_insert(T, key, flag);
}

// Voxel box of a target Gaussian; false (and the input flag) for indices
// outside the key range or a box of more than DD_MAX_CELLS voxels.
__device__ __forceinline__ bool dd_box(const float* means, const float* log_scales, long long i,
                                       double v, double kenv, int* lo, int* hi) {
#pragma clang fp contract(off)
  double cells = 1.0;
  for (int a = 0; a < 3; ++a) {
    const double m = means[3 * i + a];
    const double s = exp((double)log_scales[3 * i + a]);
    const double l = floor((m - kenv * s) / v), h = floor((m + kenv * s) / v);
    if (!(l > -(double)DD_OFF && h < (double)DD_OFF)) return false;
    lo[a] = (int)l;
    hi[a] = (int)h;
    cells *= (double)(hi[a] - lo[a] + 1);
  }
  return cells <= (double)DD_MAX_CELLS;
}

// Segment of a keyframe pixel: origin c, direction d, start and end voxels.
// 0: nothing to carve (depth <= 0), -1: outside the key range or too long.
__device__ __forceinline__ int dd_segment(const float* depth, const float* viewmats,
                                          const float* intr, int W, int H, long long g, double v,
                                          double* c, double* d, int* cur, int* end) {
#pragma clang fp contract(off)
  int kf, j, i;
  if (g <= 0x7FFFFFFF && (long long)W * H <= 0x7FFFFFFF) {
    const unsigned int u = (unsigned int)g, hw = (unsigned int)(W * H);
    kf = (int)(u / hw);
    const unsigned int p = u - (unsigned int)kf * hw;
    j = (int)(p / (unsigned int)W);
    i = (int)(p - (unsigned int)(j * W));
  } else {
    kf = (int)(g / ((long long)W * H));
    const long long p = g - (long long)kf * W * H;
    j = (int)(p / W);
    i = (int)(p - (long long)j * W);
  }
  const double dd = depth[g];
  if (!(dd > 0.0)) return 0;
  const float* vm = viewmats + 12 * kf;
  double R[3][3], t[3];
  for (int r = 0; r < 3; ++r) {
    for (int k = 0; k < 3; ++k) R[r][k] = vm[4 * r + k];
    t[r] = vm[4 * r + 3];
  }
  const double fx = intr[4 * kf], fy = intr[4 * kf + 1], cx = intr[4 * kf + 2],
               cy = intr[4 * kf + 3];
  const double ray[3] = {((double)i + 0.5 - cx) / fx, ((double)j + 0.5 - cy) / fy, 1.0};
  double steps = 0.0;
  for (int a = 0; a < 3; ++a) {
    c[a] = -((R[0][a] * t[0] + R[1][a] * t[1]) + R[2][a] * t[2]);
    const double r = c[a] + dd * ((R[0][a] * ray[0] + R[1][a] * ray[1]) + R[2][a] * ray[2]);
    d[a] = r - c[a];
    const double fc = floor(c[a] / v), fr = floor(r / v);
    // indices must fit the key, and a segment's walk must stay bounded
    if (!(fc > -(double)DD_OFF && fc < (double)DD_OFF && fr > -(double)DD_OFF &&
          fr < (double)DD_OFF))
      return -1;
    cur[a] = (int)fc;
    end[a] = (int)fr;
    steps += fabs(fr - fc);
  }
  return steps > (double)DD_MAX_CELLS ? -1 : 1;
}

// Bounds of every voxel that the boxes and segments touch, one partial per
// workgroup (a grid of at most DD_BOUND_BLOCKS strides over the inputs).
__global__ __launch_bounds__(256) void k_dd_bounds(DedupTable T, const float* tm, const float* tls,
                                                   long long n_tgt, double kenv,
                                                   const float* depth, const float* vms,
                                                   const float* intr, int W, int H,
                                                   long long npix, double v) {
  __shared__ int red[4][6];
  int b[6];  // minimum, and minus the maximum, per axis
  for (int a = 0; a < 6; ++a) b[a] = 0x7FFFFFFF;
  const long long n = n_tgt + npix;
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n;
       i += (long long)gridDim.x * 256) {
    int lo[3], hi[3];
    bool ok;
    if (i < n_tgt) {
      ok = dd_box(tm, tls, i, v, kenv, lo, hi);
    } else {
      double c[3], d[3];
      ok = dd_segment(depth, vms, intr, W, H, i - n_tgt, v, c, d, lo, hi) > 0;
    }
    if (ok)
      for (int a = 0; a < 3; ++a) {
        b[a] = min(b[a], min(lo[a], hi[a]));
        b[3 + a] = min(b[3 + a], -max(lo[a], hi[a]));
      }
  }
  for (int a = 0; a < 6; ++a) {
    for (int o = 32; o >= 1; o >>= 1) b[a] = min(b[a], __shfl_xor(b[a], o, 64));
    if (lane_id() == 0) red[threadIdx.x >> 6][a] = b[a];
  }
  __syncthreads();
  if (threadIdx.x < 6)
    T.bounds[6 * blockIdx.x + threadIdx.x] =
        min(min(red[0][threadIdx.x], red[1][threadIdx.x]),
            min(red[2][threadIdx.x], red[3][threadIdx.x]));
}

// nb = 0: the table is too small for the partials, the hash set is used.
__global__ __launch_bounds__(64) void k_dd_plan(DedupTable T, int nb) {
  int b[6];
  for (int a = 0; a < 6; ++a) b[a] = 0x7FFFFFFF;
  for (int i = threadIdx.x; i < nb; i += 64)
    for (int a = 0; a < 6; ++a) b[a] = min(b[a], T.bounds[6 * i + a]);
  for (int a = 0; a < 6; ++a)
    for (int o = 32; o >= 1; o >>= 1) b[a] = min(b[a], __shfl_xor(b[a], o, 64));
  if (threadIdx.x != 0) return;
  DedupGrid g{};
  if (nb > 0 && b[0] != 0x7FFFFFFF)  // at most 2^21 per axis
    for (int a = 0; a < 3; ++a) {
      g.lo[a] = b[a];
      g.n[a] = -b[3 + a] - b[a] + 1;
    }
  g.wx = (g.n[0] + 31) / 32;
  g.words = (unsigned long long)g.wx * g.n[1] * g.n[2];
  g.dense = nb > 0 && g.words <= 3ull * (T.mask + 1) && g.words < 0xFFFFFFFFull;
  *T.grid = g;
  T.counters[0] = 0u;
  T.counters[1] = 0u;
}

__global__ __launch_bounds__(256) void k_dd_clear(DedupTable T) {
  const bool dense = T.grid->dense != 0;
  const unsigned long long words = T.grid->words;
  const unsigned long long stride = (unsigned long long)gridDim.x * 256;
  unsigned long long i = (unsigned long long)blockIdx.x * 256 + threadIdx.x;
  if (dense) {
    for (; i < words; i += stride) T.bits()[i] = 0u;
    return;
  }
  for (; i <= T.mask; i += stride) {
    T.keys[i] = DD_EMPTY;
    T.flags[i] = 0u;
  }
}

__global__ __launch_bounds__(256) void k_dd_occ(DedupTable T, const float* means,
                                                const float* log_scales, long long n, double v,
                                                double kenv) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  int lo[3], hi[3];
  if (!dd_box(means, log_scales, i, v, kenv, lo, hi)) {
    atomicOr(&T.counters[0], 2u);
    return;
  }
  const DedupGrid G = *T.grid;
  if (G.dense) {
    const int x0 = lo[0] - G.lo[0], x1 = hi[0] - G.lo[0];
    for (int z = lo[2]; z <= hi[2]; ++z)
      for (int y = lo[1]; y <= hi[1]; ++y) {
        unsigned int* row = dd_word(T, G, G.lo[0], y, z);
        for (int w = x0 >> 5; w <= x1 >> 5; ++w) {
          const int f = max(x0 - 32 * w, 0), l = min(x1 - 32 * w, 31);
          dd_or(row + w, (0xFFFFFFFFu >> (31 - l)) & (0xFFFFFFFFu << f));
        }
      }
    return;
  }
  for (int x = lo[0]; x <= hi[0]; ++x)
    for (int y = lo[1]; y <= hi[1]; ++y)
      for (int z = lo[2]; z <= hi[2]; ++z) dd_insert(T, dd_pack(x, y, z), 1u);
}

// Sets one bit of the bitmap through a workgroup-local cache of words
// (direct-mapped, (word + 1, bits known set) in one 64-bit slot).  Slots are
// read and written whole, but not both at once: a lost update only costs another
// look at the bitmap itself.
__device__ __forceinline__ void dd_set_local(const DedupTable& T, unsigned long long* lk,
                                             unsigned int word, unsigned int bit) {
  unsigned long long* slot = lk + (word & (DD_LSLOTS - 1));
  const unsigned long long e = dd_peek(slot);
  const bool same = (unsigned int)(e >> 32) == word + 1u;
  if (same && ((unsigned int)e & bit)) return;
  dd_or(T.bits() + word, bit);
  dd_poke(slot, ((unsigned long long)(word + 1u) << 32) | (same ? (unsigned int)e | bit : bit));
}

// Walks a segment's voxels in increasing t: step(axis, +-1) at every plane
// crossing with t in [0, 1), ties to the lower axis; the walk stops at the end
// voxel's planes.  The order is that of the correctly rounded quotients
// (plane - c) / d, but a step forms only a product with 1 / d (a few ulp off)
// for the axis it advanced: the quotients themselves decide when two
// crossings, or a crossing and t = 1, are closer than DD_NEAR (a division is
// about 14 FP64 instructions; three per step at first).
constexpr double DD_NEAR = 1e-14;
template <class F>
__device__ __forceinline__ void dd_walk(const double (&c)[3], const double (&d)[3],
                                        const int (&cur)[3], const int (&end)[3], double v,
                                        const F& step) {
#pragma clang fp contract(off)
  double inv[3], nd[3], u[3];  // next plane's index and (about) its t; 2: none
  int left[3], sg[3];          // planes left to cross, direction
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    inv[a] = 1.0 / d[a];
    sg[a] = d[a] > 0.0 ? 1 : -1;
    left[a] = d[a] == 0.0 ? 0 : sg[a] * (end[a] - cur[a]);
    nd[a] = (double)(d[a] > 0.0 ? cur[a] + 1 : cur[a]);
    // a crossing behind the start (t < 0, the exact sign) is never taken, and
    // blocks its axis; t = 0: a start on the plane, moving down, leaves its
    // voxel at once
    const double t = (nd[a] * v - c[a]) * inv[a];
    u[a] = left[a] != 0 && t >= 0.0 ? t : 2.0;
  }
  for (;;) {
    const double m01 = fmin(u[0], u[1]), M01 = fmax(u[0], u[1]);
    const double m1 = fmin(m01, u[2]), m2 = fmax(m01, fmin(M01, u[2]));
    if (m1 > 1.0 + DD_NEAR) return;
    int best = u[0] == m1 ? 0 : u[1] == m1 ? 1 : 2;
    if (m2 - m1 < DD_NEAR || m1 > 1.0 - DD_NEAR) {
      best = -1;
      double tb = 1.0;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        if (u[a] == 2.0) continue;
        const double t = (nd[a] * v - c[a]) / d[a];
        if (t < tb) {
          tb = t;
          best = a;
        }
      }
      if (best < 0) return;
    }
    int s = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a)
      if (a == best) {
        s = sg[a];
        left[a] -= 1;
        nd[a] += (double)sg[a];
        u[a] = left[a] != 0 ? (nd[a] * v - c[a]) * inv[a] : 2.0;
      }
    step(best, s);
  }
}

// One workgroup per 64 x 16 pixel tile of a keyframe, a wave per pixel row at
// a time.  Bitmap: the tile's pyramid of rays has its own box, kept as a
// bitmap in LDS (words aligned with the global one's) that is merged once
// the tile is walked: inserts are LDS reads, and the voxels near a camera,
// which every ray of the keyframe crosses, see one update per tile instead
// of queueing on one line.  A pyramid too large for LDS goes through the
// workgroup's word cache.  Hash set: through the workgroup's LDS set.
constexpr int DD_TILE = 64, DD_ROWS = 16, DD_FT = 256;
constexpr int DD_LWORDS = 2 * DD_LSLOTS;  // words of the LDS bitmap
__global__ __launch_bounds__(DD_FT) void k_dd_free(DedupTable T, const float* depth,
                                                   const float* viewmats, const float* intr,
                                                   int W, int H, int tx, int ty, double v) {
  __shared__ unsigned long long lk[DD_LSLOTS];
  __shared__ int red[DD_FT / 64][6];
  unsigned int* lw = reinterpret_cast<unsigned int*>(lk);
  const DedupGrid G = *T.grid;
  const int per = tx * ty;
  const int kf = (int)(blockIdx.x / per), t = (int)(blockIdx.x - kf * per);
  const int i = (t % tx) * DD_TILE + (int)(threadIdx.x & 63);
  const int j0 = (t / tx) * DD_ROWS + (int)(threadIdx.x >> 6);
  const int j1 = min((t / tx + 1) * DD_ROWS, H);
  const long long base = (long long)kf * W * H;
  double c[3], d[3];
  int cur[3], end[3];
  int lo[3] = {0, 0, 0}, n[3] = {0, 0, 0}, wx = 0;
  bool local = false;
  if (G.dense) {
    int b[6];  // minimum, and minus the maximum, per axis
    for (int a = 0; a < 6; ++a) b[a] = 0x7FFFFFFF;
    if (i < W)
      for (int j = j0; j < j1; j += DD_FT / 64)
        if (dd_segment(depth, viewmats, intr, W, H, base + (long long)j * W + i, v, c, d, cur,
                       end) > 0)
          for (int a = 0; a < 3; ++a) {
            b[a] = min(b[a], min(cur[a], end[a]));
            b[3 + a] = min(b[3 + a], -max(cur[a], end[a]));
          }
    for (int a = 0; a < 6; ++a) {
      for (int o = 32; o >= 1; o >>= 1) b[a] = min(b[a], __shfl_xor(b[a], o, 64));
      if (lane_id() == 0) red[threadIdx.x >> 6][a] = b[a];
    }
    __syncthreads();
    for (int a = 0; a < 6; ++a) {
      b[a] = red[0][a];
      for (int w = 1; w < DD_FT / 64; ++w) b[a] = min(b[a], red[w][a]);
    }
    if (b[0] != 0x7FFFFFFF) {
      lo[0] = G.lo[0] + ((b[0] - G.lo[0]) & ~31);
      lo[1] = b[1];
      lo[2] = b[2];
      for (int a = 0; a < 3; ++a) n[a] = -b[3 + a] - lo[a] + 1;
      wx = (n[0] + 31) / 32;
      local = (long long)wx * n[1] * n[2] <= DD_LWORDS;
    }
  }
  for (int k = threadIdx.x; k < DD_LSLOTS; k += DD_FT) lk[k] = G.dense ? 0ull : DD_EMPTY;
  __syncthreads();
  if (i < W)
    for (int j = j0; j < j1; j += DD_FT / 64) {
      const int got =
          dd_segment(depth, viewmats, intr, W, H, base + (long long)j * W + i, v, c, d, cur, end);
      if (got < 0) atomicOr(&T.counters[0], 2u);
      if (got <= 0) continue;
      if (local) {
        // bit index in the LDS bitmap
        int at = ((cur[2] - lo[2]) * n[1] + (cur[1] - lo[1])) * 32 * wx + (cur[0] - lo[0]);
        const auto set = [&]() {
          unsigned int* w = lw + (at >> 5);
          const unsigned int bit = 1u << (at & 31);
          if (!(dd_peek(w) & bit)) atomicOr(w, bit);
        };
        set();
        dd_walk(c, d, cur, end, v, [&](int axis, int sg) {
          at += sg * (axis == 0 ? 1 : axis == 1 ? 32 * wx : 32 * wx * n[1]);
          set();
        });
      } else {
        int q[3] = {cur[0], cur[1], cur[2]};
        const auto set = [&]() {
          if (G.dense) {
            const int x = q[0] - G.lo[0], y = q[1] - G.lo[1], z = q[2] - G.lo[2];
            // words < 2^32 (k_dd_plan)
            dd_set_local(T, lk,
                         ((unsigned int)z * (unsigned int)G.n[1] + (unsigned int)y) *
                                 (unsigned int)G.wx + (unsigned int)(x >> 5),
                         1u << (x & 31));
          } else {
            dd_insert_local(T, lk, dd_pack(q[0], q[1], q[2]), 2u);
          }
        };
        set();
        dd_walk(c, d, cur, end, v, [&](int axis, int sg) {
#pragma unroll
          for (int a = 0; a < 3; ++a) q[a] += a == axis ? sg : 0;
          set();
        });
      }
    }
  if (!local) return;  // uniform
  __syncthreads();
  const int words = wx * n[1] * n[2];
  for (int k = threadIdx.x; k < words; k += DD_FT) {
    const unsigned int bits = lw[k];
    if (bits == 0u) continue;
    const int r = k / wx, x = k - r * wx, z = r / n[1], y = r - z * n[1];
    dd_or(dd_word(T, G, lo[0] + 32 * x, lo[1] + y, lo[2] + z), bits);
  }
}

// Distinct voxels of the bitmap, and the overflow flag when a hash set of the
// caller's size could not have held them.
__global__ __launch_bounds__(256) void k_dd_count(DedupTable T) {
  __shared__ unsigned int red[4];
  if (!T.grid->dense) return;
  const unsigned long long words = T.grid->words;
  unsigned int s = 0u;
  for (unsigned long long i = (unsigned long long)blockIdx.x * 256 + threadIdx.x; i < words;
       i += (unsigned long long)gridDim.x * 256)
    s += (unsigned int)__popc(T.bits()[i]);
  for (int o = 32; o >= 1; o >>= 1) s += (unsigned int)__shfl_xor((int)s, o, 64);
  if (lane_id() == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    s = red[0] + red[1] + red[2] + red[3];
    if (s) {
      const unsigned long long all = (unsigned long long)atomicAdd(&T.counters[1], s) + s;
      if (all > T.mask + 1) atomicOr(&T.counters[0], 1u);
    }
  }
}

__global__ __launch_bounds__(256) void k_dd_probe(DedupTable T, const float* means, long long n,
                                                  double v, uint8_t* keep) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  int q[3];
  for (int a = 0; a < 3; ++a) {
    const double f = floor((double)means[3 * i + a] / v);
    if (!(f > -(double)DD_OFF && f < (double)DD_OFF)) {
      atomicOr(&T.counters[0], 2u);
      keep[i] = 0;
      return;
    }
    q[a] = (int)f;
  }
  const DedupGrid G = *T.grid;
  if (G.dense) {
    bool in = true;
    for (int a = 0; a < 3; ++a) in = in && q[a] >= G.lo[a] && q[a] < G.lo[a] + G.n[a];
    const bool set =
        in && ((*dd_word(T, G, q[0], q[1], q[2]) >> ((q[0] - G.lo[0]) & 31)) & 1u) != 0u;
    keep[i] = set ? 0 : 1;
    return;
  }
  const unsigned long long key = dd_pack(q[0], q[1], q[2]);
  unsigned long long h = dd_mix(key) & T.mask;
  bool found = false;
  for (long long probe = 0; probe <= (long long)T.mask; ++probe) {
    const unsigned long long k = T.keys[h];
    if (k == key) {
      found = T.flags[h] != 0u;
      break;
    }
    if (k == DD_EMPTY) break;
    h = (h + 1) & T.mask;
  }
  keep[i] = found ? 0 : 1;
}

size_t dedup_workspace_bytes(long long slots) {
  return (size_t)slots * 12 + 256;
}

hipError_t launch_dedup(long long slots, void* ws, double v, double kenv, const float* tm,
                        const float* tls, long long n_tgt, const float* depth, const float* vms,
                        const float* intr, int nk, int W, int H, const float* sm, long long n_src,
                        uint8_t* keep, hipStream_t s, unsigned int** counters) {
  DedupTable T;
  char* b = (char*)ws;
  T.counters = (unsigned int*)b;
  T.keys = (unsigned long long*)(b + 256);
  T.flags = (unsigned int*)(b + 256 + 8 * (size_t)slots);
  T.mask = (unsigned long long)slots - 1;
  T.grid = (DedupGrid*)(b + 64);
  T.bounds = (int*)(b + 256);
  *counters = T.counters;
  const auto blocks = [](long long n) { return dim3((unsigned)((n + 255) / 256)); };
  const long long npix = (long long)nk * W * H;
  int nb = (int)std::min<long long>((n_tgt + npix + 255) / 256, DD_BOUND_BLOCKS);
  // the partial bounds sit in the table's storage
  if (slots * 12 < (long long)DD_BOUND_BLOCKS * 24) nb = 0;
  if (nb > 0)
    hipLaunchKernelGGL(k_dd_bounds, dim3(nb), dim3(256), 0, s, T, tm, tls, n_tgt, kenv, depth, vms,
                       intr, W, H, npix, v);
  hipLaunchKernelGGL(k_dd_plan, dim3(1), dim3(64), 0, s, T, nb);
  const dim3 fill((unsigned)std::min<long long>((slots + 255) / 256, 2048));
  hipLaunchKernelGGL(k_dd_clear, fill, dim3(256), 0, s, T);
  if (n_tgt > 0)
    hipLaunchKernelGGL(k_dd_occ, blocks(n_tgt), dim3(256), 0, s, T, tm, tls, n_tgt, v, kenv);
  const int tx = (W + DD_TILE - 1) / DD_TILE, ty = (H + DD_ROWS - 1) / DD_ROWS;
  if (npix > 0)
    hipLaunchKernelGGL(k_dd_free, dim3((unsigned)(nk * tx * ty)), dim3(DD_FT), 0, s, T, depth, vms,
                       intr, W, H, tx, ty, v);
  hipLaunchKernelGGL(k_dd_count, dim3(256), dim3(256), 0, s, T);
  if (n_src > 0)
    hipLaunchKernelGGL(k_dd_probe, blocks(n_src), dim3(256), 0, s, T, sm, n_src, v, keep);
  return hipGetLastError();
}

}  // namespace gsr
