// Mapping-loss extras (Sec. III-A, Eq. (map_loss)) and Gaussian seeding of
// new keyframes.
//
// k_iso_grad: one thread per Gaussian, the gradient of the isotropy term
// sum_c |s_c - mean(s)| (s = exp(log-scale)) with respect to the log-scales,
// added into the caller's gradient (HBM-bound: 12 B read, 12 B read-modify-
// written per Gaussian).
// k_normal_grad: a wave marches down a strip of 64 columns (60 written, two of
// halo on either side) over NR rows.  Every pixel computes its depth-induced
// normal (central differences of back-projected points) and the gradients of its
// cosine loss with respect to its two difference vectors; each output pixel
// gathers the four difference-vector gradients that involve it, the vertical ones
// from the registers of the rows before and after, the horizontal ones from
// the neighbouring lanes, and projects them on its ray.  The difference
// vectors are formed from depth differences and the exact ray differences
// (2 / f), which keeps FP32 cancellation small.  HBM-bound, 24 B per pixel:
// 48 views of 640 x 480 in 78 us (157 by 16 x 16 tiles through LDS), 8 views in 19
// (30; 23 with 16 rows to a wave).
// k_seed_*: ordered compaction (per-block counts, summed by each later block,
// wave-ballot ranks) of the pixels with positive depth on a stride grid,
// each writing one isotropic Gaussian at its back-projected point.
// The per-block counts live in file-scope device arrays: one that the
// allocation-free variant's calls share, and a few slots of which every
// synchronising call takes its own.
#include <mutex>

#include "common.h"

namespace gsr {

__global__ __launch_bounds__(256) void k_iso_grad(long n, const float* ls, float w, float* g) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const float s0 = expf(ls[3 * i]), s1 = expf(ls[3 * i + 1]), s2 = expf(ls[3 * i + 2]);
  // sign(s_c - mean) = sign(2 s_c - s_a - s_b): equal components give an
  // exact 0, and three equal components give a zero gradient either way
  const float e0 = 2.f * s0 - (s1 + s2), e1 = 2.f * s1 - (s0 + s2), e2 = 2.f * s2 - (s0 + s1);
  const float q0 = e0 > 0.f ? 1.f : (e0 < 0.f ? -1.f : 0.f);
  const float q1 = e1 > 0.f ? 1.f : (e1 < 0.f ? -1.f : 0.f);
  const float q2 = e2 > 0.f ? 1.f : (e2 < 0.f ? -1.f : 0.f);
  const float m = (q0 + q1 + q2) * (1.f / 3.f);
  g[3 * i] += w * s0 * (q0 - m);
  g[3 * i + 1] += w * s1 * (q1 - m);
  g[3 * i + 2] += w * s2 * (q2 - m);
}

hipError_t launch_iso_grad(long n, const float* ls, float w, float* g, hipStream_t s) {
  if (n > 0)
    hipLaunchKernelGGL(k_iso_grad, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, ls, w,
                       g);
  return hipGetLastError();
}

// ------------------------------------------------------------ normal loss
constexpr int NR = 8;        // rows per wave
constexpr int NC = 60;       // columns written per wave

struct F3 {
  float x, y, z;
};
__device__ __forceinline__ F3 cross3(F3 a, F3 b) {
  return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}

// The value of the lane before / after (0 past the wave's ends).
__device__ __forceinline__ float lane_before(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                                       0, __builtin_bit_cast(int, x), 0x138, 0xF, 0xF, true));
}
__device__ __forceinline__ float lane_after(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
                                       0, __builtin_bit_cast(int, x), 0x130, 0xF, 0xF, true));
}

__global__ __launch_bounds__(256) void k_normal_grad(int W, int H, int tiles_x, int tiles_y, long n,
                                                     const float* depth, const float* prior,
                                                     const float* intr, float w, float* g_dep) {
  const long u = (long)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (u >= n) return;
  const int tpv = tiles_x * tiles_y;
  const int v = (int)(u / tpv), t = (int)(u - (long)v * tpv);
  const int r0 = (t / tiles_x) * NR, r1 = min(H, r0 + NR);
  const int lane = lane_id(), i = (t % tiles_x) * NC - 2 + lane;
  const bool in = i >= 0 && i < W;                        // a pixel of the image
  const bool out = in && lane >= 2 && lane < 2 + NC;      // written
  const size_t HW = (size_t)H * W;
  const float* dv = depth + v * HW + i;
  const float* pv = prior + v * 3 * HW + i;
  float* gv = g_dep + v * HW + i;
  const float fx = intr[4 * v], fy = intr[4 * v + 1], cx = intr[4 * v + 2], cy = intr[4 * v + 3];
  const float ifx = 1.f / fx, ify = 1.f / fy;
  const float xi = ((float)i + 0.5f - cx) * ifx, xr = ((float)(i + 1) + 0.5f - cx) * ifx;
  const auto load_d = [&](int j) { return in && j >= 0 && j < H ? dv[(size_t)j * W] : 0.f; };
  const auto load_p = [&](int j) {
    F3 p{0.f, 0.f, 0.f};
    if (in && j >= 0 && j < H) {
      const size_t q = (size_t)j * W;
      p = F3{pv[q], pv[q + HW], pv[q + 2 * HW]};
    }
    return p;
  };
  const auto load_g = [&](int j) { return out && j >= r0 && j < r1 ? gv[(size_t)j * W] : 0.f; };
  // depth of rows j - 1, j, j + 1; prior of row j, gradient of row j - 1: the
  // loads of a step are issued one step ahead
  float dd = load_d(r0 - 2), d0 = load_d(r0 - 1), du = load_d(r0), g = 0.f;
  F3 p = load_p(r0 - 1);
  F3 ga2{0.f, 0.f, 0.f}, ga1{0.f, 0.f, 0.f}, gb1{0.f, 0.f, 0.f};  // of rows j - 2, j - 1
  for (int j = r0 - 1; j <= r1; ++j) {
    const float dn = load_d(j + 2), gn = load_g(j);
    const F3 pn = load_p(j + 1);
    const float dr = lane_after(d0), dl = lane_before(d0);
    F3 ga{0.f, 0.f, 0.f}, gb{0.f, 0.f, 0.f};
    if (j >= 1 && j < H - 1 && i >= 1 && i < W - 1 && du > 0.f && dd > 0.f && dr > 0.f &&
        dl > 0.f) {
      const float yj = ((float)j + 0.5f - cy) * ify, yu = ((float)(j + 1) + 0.5f - cy) * ify;
      // a = P(i, j+1) - P(i, j-1), b = P(i+1, j) - P(i-1, j)
      const float ev = du - dd, eh = dr - dl;
      const F3 a{ev * xi, ev * yu + dd * (2.f * ify), ev};
      const F3 b{eh * xr + dl * (2.f * ifx), eh * yj, eh};
      const F3 c = cross3(a, b);
      const float n2 = c.x * c.x + c.y * c.y + c.z * c.z;
      if (n2 > 0.f) {
        const float inr = rsqrtf(n2);
        const F3 n{c.x * inr, c.y * inr, c.z * inr};
        const float dot = n.x * p.x + n.y * p.y + n.z * p.z;
        const float sc = w * inr;
        const F3 gc{sc * (dot * n.x - p.x), sc * (dot * n.y - p.y), sc * (dot * n.z - p.z)};
        ga = cross3(b, gc);
        gb = cross3(gc, a);
      }
    }
    // the point P(i, j-1) is the "+" end of the vertical difference of
    // (i, j-2), the "-" end of that of (i, j), and likewise horizontally
    const float px = ga2.x - ga.x + lane_before(gb1.x) - lane_after(gb1.x);
    const float py = ga2.y - ga.y + lane_before(gb1.y) - lane_after(gb1.y);
    const float pz = ga2.z - ga.z + lane_before(gb1.z) - lane_after(gb1.z);
    if (out && j > r0) {
      const float ry = ((float)(j - 1) + 0.5f - cy) * ify;
      gv[(size_t)(j - 1) * W] = g + (xi * px + ry * py + pz);
    }
    dd = d0; d0 = du; du = dn;
    p = pn;
    g = gn;
    ga2 = ga1; ga1 = ga; gb1 = gb;
  }
}

hipError_t launch_normal_grad(int nv, int W, int H, const float* depth, const float* prior,
                              const float* intr, float w, float* g_dep, hipStream_t s) {
  const int tx = (W + NC - 1) / NC, ty = (H + NR - 1) / NR;
  const long n = (long)nv * tx * ty;  // waves
  hipLaunchKernelGGL(k_normal_grad, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, W, H, tx, ty, n,
                     depth, prior, intr, w, g_dep);
  return hipGetLastError();
}

// ---------------------------------------------------------------- seeding
constexpr int SEED_SUM_BLOCKS = 4096;
struct SeedGrid {
  int W, H, stride, gw;  // gw grid columns
  long m;                // grid points
};

__device__ __forceinline__ bool seed_valid(const SeedGrid& sgd, const float* d, long k, int* pj,
                                           int* pi) {
  if (k >= sgd.m) return false;
  const int gj = (int)(k / sgd.gw), gi = (int)(k - (long)gj * sgd.gw);
  *pj = gj * sgd.stride;
  *pi = gi * sgd.stride;
  return d[(size_t)*pj * sgd.W + *pi] > 0.f;
}

__global__ __launch_bounds__(256) void k_seed_count(SeedGrid sgd, const float* d, uint32_t* blk) {
  int j, i;
  const bool ok = seed_valid(sgd, d, (long)blockIdx.x * 256 + threadIdx.x, &j, &i);
  const int c = __syncthreads_count(ok);
  if (threadIdx.x == 0) blk[blockIdx.x] = (uint32_t)c;
}

template <bool SCANNED>
__global__ __launch_bounds__(256) void k_seed_write(SeedGrid sgd, const float* d,
                                                    const float* col, const float* vm,
                                                    const float* intr, float opac_logit,
                                                    long max_out, uint32_t* blk, int64_t* n_out,
                                                    float* m, float* ls, float* q, float* o,
                                                    float* c) {
  __shared__ uint32_t wc[4], sh[4];
  const uint32_t before = SCANNED ? blk[blockIdx.x] : block_prefix_256(blk, sh);
  int j = 0, i = 0;
  const bool ok = seed_valid(sgd, d, (long)blockIdx.x * 256 + threadIdx.x, &j, &i);
  const unsigned long long bal = __ballot(ok);
  const int lane = lane_id(), w = threadIdx.x >> 6;
  if (lane == 0) wc[w] = (uint32_t)__popcll(bal);
  __syncthreads();
  if (threadIdx.x == 0 && blockIdx.x == gridDim.x - 1) {
    const uint32_t all = before + wc[0] + wc[1] + wc[2] + wc[3];
    if (!SCANNED) blk[gridDim.x] = all;
    if (n_out) n_out[0] = (int64_t)all;
  }
  if (!ok) return;
  long pos = before + __popcll(bal & ((1ull << lane) - 1ull));
  for (int k = 0; k < w; ++k) pos += wc[k];
  if (pos >= max_out) return;
  const float fx = intr[0], fy = intr[1], cx = intr[2], cy = intr[3];
  const float ifx = 1.f / fx, ify = 1.f / fy;
  const int W = sgd.W, H = sgd.H, s = sgd.stride;
  const float z = d[(size_t)j * W + i];
  const float xi = ((float)i + 0.5f - cx) * ifx, yj = ((float)j + 0.5f - cy) * ify;
  // mean distance to the grid neighbours with positive depth; a neighbour's
  // offset is (z' - z) ray' + z (ray' - ray), the ray step being s / f
  float sum = 0.f;
  int cnt = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int dj = e < 2 ? 0 : (e == 2 ? -s : s), di = e < 2 ? (e == 0 ? -s : s) : 0;
    const int jj = j + dj, ii = i + di;
    if (jj < 0 || jj >= H || ii < 0 || ii >= W) continue;
    const float zn = d[(size_t)jj * W + ii];
    if (!(zn > 0.f)) continue;
    const float xn = ((float)ii + 0.5f - cx) * ifx, yn = ((float)jj + 0.5f - cy) * ify;
    const float dz = zn - z;
    const float ox = dz * xn + z * ((float)di * ifx), oy = dz * yn + z * ((float)dj * ify);
    sum += sqrtf(ox * ox + oy * oy + dz * dz);
    ++cnt;
  }
  const float sc = cnt ? sum / (float)cnt : z * (float)s * ifx;
  const float p0 = z * xi - vm[3], p1 = z * yj - vm[7], p2 = z - vm[11];
#pragma unroll
  for (int a = 0; a < 3; ++a) m[3 * pos + a] = vm[a] * p0 + vm[4 + a] * p1 + vm[8 + a] * p2;
  const float lsc = logf(sc);
  ls[3 * pos] = lsc;
  ls[3 * pos + 1] = lsc;
  ls[3 * pos + 2] = lsc;
  *reinterpret_cast<float4*>(q + 4 * pos) = make_float4(1.f, 0.f, 0.f, 0.f);
  o[pos] = opac_logit;
  const size_t HW = (size_t)H * W, px = (size_t)j * W + i;
  c[3 * pos] = col[px];
  c[3 * pos + 1] = col[HW + px];
  c[3 * pos + 2] = col[2 * HW + px];
}

// ------------------------------------------------- allocation-free seeding
// Block counts of gsr_seed_noalloc: one word per 256 grid points plus the
// total, at most SEED_NOALLOC_MAX_POINTS points.  Every GPU the library runs
// on holds its own copy until the process ends; every call on a GPU shares
// it, so calls that overlap on one GPU race.  Nothing in it needs clearing:
// the count kernel writes every word the write kernel reads.
static __device__ __align__(256) uint32_t scratch[SEED_NOALLOC_MAX_POINTS / 256 + 64];

// Scratch of the calls that synchronise before they return (gsr_seed,
// gsr_prune): a few slots that a call takes for itself and gives back, so that
// an ordinary call neither allocates nor frees device memory (seeding a 1200x680
// keyframe: 67 -> 53 us together with the scan kernel and one host wait less).
static __device__ __align__(256) uint32_t call_slots[CALL_SLOTS][CALL_SLOT_BYTES / 4];

// Device address of a file-scope array on the current device, looked up once
// per device with that device current (an array's name is a host-side stand-in
// in host code and must never reach a kernel).
static hipError_t symbol_addr(const void* symbol, uint32_t** table, int dev, uint32_t** out) {
  if (!table[dev]) {
    void* p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, symbol);
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    table[dev] = (uint32_t*)p;
  }
  *out = table[dev];
  return hipSuccess;
}

static std::mutex scratch_mu;

hipError_t seed_scratch(uint32_t** out) {
  static uint32_t* addr[GSR_MAX_DEVICES] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= GSR_MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(scratch_mu);
  return symbol_addr(HIP_SYMBOL(scratch), addr, dev, out);
}

// A call's scratch of at least `bytes`: a free slot of the current device, or
// an allocation when it does not fit one or every slot is taken (calls of
// other host threads).  The destructor gives it back; the caller has
// synchronised the stream that used it by then.
static unsigned call_busy[GSR_MAX_DEVICES];

hipError_t CallScratch::get(size_t bytes) {
  if (hipGetDevice(&dev) != hipSuccess) dev = -1;
  if (bytes <= CALL_SLOT_BYTES && dev >= 0 && dev < GSR_MAX_DEVICES) {
    static uint32_t* addr[GSR_MAX_DEVICES] = {};
    std::lock_guard<std::mutex> lock(scratch_mu);
    uint32_t* base = nullptr;
    if (symbol_addr(HIP_SYMBOL(call_slots), addr, dev, &base) == hipSuccess)
      for (int k = 0; k < CALL_SLOTS; ++k)
        if (!((call_busy[dev] >> k) & 1u)) {
          call_busy[dev] |= 1u << k;
          slot = k;
          ptr = base + (size_t)k * (CALL_SLOT_BYTES / 4);
          return hipSuccess;
        }
  }
  (void)hipGetLastError();
  return hipMalloc(&ptr, bytes);
}

CallScratch::~CallScratch() {
  if (slot >= 0) {
    std::lock_guard<std::mutex> lock(scratch_mu);
    call_busy[dev] &= ~(1u << slot);
  } else if (ptr) {
    (void)hipFree(ptr);
  }
}

hipError_t launch_seed(int W, int H, int stride, const float* depth, const float* color,
                       const float* vm, const float* intr, float opac_logit, long max_out,
                       uint32_t* blk, int64_t* n_out, float* m, float* ls, float* q, float* o,
                       float* c, hipStream_t s) {
  SeedGrid g;
  g.W = W;
  g.H = H;
  g.stride = stride;
  g.gw = (W + stride - 1) / stride;
  g.m = (long)g.gw * ((H + stride - 1) / stride);
  const int nb = (int)((g.m + 255) / 256);
  hipLaunchKernelGGL(k_seed_count, dim3(nb), dim3(256), 0, s, g, depth, blk);
  // Points before a block: up to SEED_SUM_BLOCKS every block sums the counts
  // before it (at most 16 KB from L2), which costs less than a scan kernel
  // between the two (1200x680 keyframe, 3,188 blocks: 5.7 us and a launch
  // against 2.2 us); beyond, the sums would grow with the square.
  const auto k = nb <= SEED_SUM_BLOCKS ? k_seed_write<false> : k_seed_write<true>;
  if (nb > SEED_SUM_BLOCKS) {
    hipError_t e = launch_block_scan(nb, blk, s);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k, dim3(nb), dim3(256), 0, s, g, depth, color, vm, intr, opac_logit, max_out,
                     blk, n_out, m, ls, q, o, c);
  return hipGetLastError();
}

}  // namespace gsr
