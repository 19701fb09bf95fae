// SSIM term of the refinement loss (Sec. III-C, Eq. (refine_loss)) on the
// exposure-compensated render I~ = exp(a_v) I^ + b_v, and its gradient.
//
// Statistics under an 11 x 11 Gaussian window (sigma 1.5, zero outside the
// image), per colour channel: the moments of (x, y) -> S and the gradient maps
// f1 = dS/dmx - 2 mx dS/dsxx - my dS/dsxy, f2 = dS/dsxx, f3 = dS/dsxy, then
// blurs of f1..f3 -> d mean(S)/dx = (w*f1 + 2 x w*f2 + y w*f3) / N, chained
// through the exposure into d_color (accumulated).  S and its derivatives need
// sxx and syy only as their sum, so four moments are blurred: x, y, x^2 + y^2
// and xy.
//
// k_ssim: a workgroup of one to four waves takes a strip of output columns (40,
// 104, 168 or 232: its columns less two windows, in fours) and marches down
// the image four rows at a time, a column per lane.  A separable blur is a product with a
// band matrix, and it runs on the matrix unit in 4 x 4 blocks (4x4x1, FP32
// throughout, a fused multiply-add per element): four output rows of 64
// columns take the 14 input rows of their windows, one instruction per row
// with the weights as the left operand (vertical), or four columns of 16
// column groups take 14 columns each, one instruction per column with the
// weights as the right operand (horizontal).  The narrow blocks keep the band
// dense (11 of 14; 11 of 26 in a 16 x 16 block), and both products leave a
// column per lane and a row per register, so only the horizontal blurs'
// left operands pass through LDS (four 16-byte reads per map and four rows).
// The rows of x and y, and of f1..f3, that the next windows need stay in
// registers (rings of 16 rows, the march unrolled by four steps).
// One workgroup per 32 x 32 tile with blurs through LDS took 1050 us at 48 x 3
// x 480 x 640 (bound by LDS reads: about 118 per pixel, and 310 multiply-adds
// with the tile's halo); this form took 463 us when it was chosen (one wave per
// strip, 40 of its 64 columns its own: 585 us; loads at their use instead of a
// step ahead and one chain of products at a time: 692).  Since its sums are
// FP64 and its registers held to two waves a SIMD it takes 408 back to back
// (425 before); in a trace, the clocks lower, 494.
//
// k_ssim_reduce: per-wave partial sums (S, and the exposure gradients) summed
// per view in a fixed order: no float atomics on a few hot addresses.
#include <algorithm>

#include "common.h"

namespace gsr {

constexpr float SS_C1 = 0.01f * 0.01f, SS_C2 = 0.03f * 0.03f;

struct SsimArgs {
  float w[SS_K];
  int W, H, TX, nv;     // TX: strips
  int rows;             // output rows of a workgroup (a multiple of 4)
  float weight_over_n;  // weight / (3 V H W)
};

__device__ __forceinline__ float block_sum_256(float x, float* red) {
  x = wave_total(x);
  if (lane_id() == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  const float t = red[0] + red[1] + red[2] + red[3];
  __syncthreads();
  return t;
}

typedef float ss_v4 __attribute__((ext_vector_type(4)));
// LDS row pitch: the workgroup's columns and the last groups' overhang; 16 mod
// 64 words, so the four rows a read touches hit distinct banks
constexpr int ss_ld(int nw) { return 64 * nw + 16; }

// Vertical blurs of four rows of NM maps: in(k, t) is row t of the 14 of map k
// (a column per lane); d[k][i] is its output row i.  The maps' chains of
// dependent products are interleaved.
//
// The band product also multiplies the rows outside an output's window, by
// zero: an infinite or NaN input there would reach outputs it must not.  Each
// output row sums all 14 inputs, so row 0 shows whether there is one; the
// wave then sums its windows alone, by vector instructions.  Returns whether
// it did (uniform over the wave): the horizontal blur of these rows must too.
template <int NM, class F>
__device__ __forceinline__ bool ss_vert(const SsimArgs& A, const float (&wt)[SS_W], const F& in,
                                        ss_v4 (&d)[NM]) {
#pragma unroll
  for (int k = 0; k < NM; ++k) d[k] = ss_v4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < SS_W; ++t)
#pragma unroll
    for (int k = 0; k < NM; ++k)
      d[k] = __builtin_amdgcn_mfma_f32_4x4x1f32(wt[t], in(k, t), d[k], 0, 0, 0);
  float all = d[0][0];
#pragma unroll
  for (int k = 1; k < NM; ++k) all += d[k][0];
  if (__ballot(!(fabsf(all) < INFINITY)) == 0ull) return false;
#pragma unroll
  for (int k = 0; k < NM; ++k)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float a = 0.f;
#pragma unroll
      for (int t = 0; t < SS_K; ++t) a = fmaf(A.w[t], in(k, i + t), a);
      d[k][i] = a;
    }
  return true;
}

// Horizontal blurs of the four rows of NM maps, handed over through buf (row i
// of map k at [k][i]): output column o (thread o) is the window over columns o
// .. o + 10.  One barrier: a step's two calls use two buffers, so a buffer is
// written again only after a barrier behind its last read.  alone: this wave's
// rows hold infinite or NaN values; the workgroup agrees through *flag, which
// holds the last step (counted from 1) where a wave's did.
template <int NM, int NW>
__device__ __forceinline__ void ss_horiz(const SsimArgs& A, const float (&wt)[SS_W],
                                         float (*buf)[4][ss_ld(NW)], bool alone, int step,
                                         int* flag, ss_v4 (&d)[NM]) {
  const int lane = threadIdx.x;
#pragma unroll
  for (int k = 0; k < NM; ++k)
#pragma unroll
    for (int i = 0; i < 4; ++i) buf[k][i][lane] = d[k][i];
  if (NW > 1) {
    if (alone && lane_id() == 0) *flag = step;
    __syncthreads();
    alone = __builtin_amdgcn_readfirstlane(*flag) == step;
  } else {
    __builtin_amdgcn_wave_barrier();
  }
  if (alone) {
#pragma unroll
    for (int k = 0; k < NM; ++k)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float a = 0.f;
#pragma unroll
        for (int t = 0; t < SS_K; ++t) a = fmaf(A.w[t], buf[k][i][lane + t], a);
        d[k][i] = a;
      }
  } else {
#pragma unroll
    for (int k = 0; k < NM; ++k) d[k] = ss_v4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      float4 x[NM];
#pragma unroll
      for (int k = 0; k < NM; ++k)
        x[k] = *reinterpret_cast<const float4*>(&buf[k][lane & 3][(lane & ~3) + 4 * c]);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (4 * c + e < SS_W) {
#pragma unroll
          for (int k = 0; k < NM; ++k)
            d[k] = __builtin_amdgcn_mfma_f32_4x4x1f32(
                e == 0 ? x[k].x : e == 1 ? x[k].y : e == 2 ? x[k].z : x[k].w, wt[4 * c + e], d[k],
                0, 0, 0);
        }
    }
  }
  if (NW == 1) __builtin_amdgcn_wave_barrier();
}

template <int NW>
__global__ __launch_bounds__(64 * NW, 2) void k_ssim(SsimArgs A, const float* color, const float* target,
                                             const float* expo, float* d_color, float* ssim_part,
                                             float* e_part) {
  constexpr int OW = ss_out(NW), SW = ss_stats(NW);
  __shared__ __align__(16) float buf[4][4][ss_ld(NW)], buf2[3][4][ss_ld(NW)];
  __shared__ float red[3][NW];
  __shared__ int flag[2];
  const int lane = threadIdx.x;  // the thread's column
  const int vc = blockIdx.y, v = vc / 3;
  const int sy = blockIdx.x / A.TX, sx = blockIdx.x - sy * A.TX;
  const int y0 = sy * A.rows, y1 = min(y0 + A.rows, A.H);  // the workgroup's output rows
  const int xi = sx * OW - 2 * SS_R + lane;                // the lane's input column,
  const int xs = xi + SS_R, xo = xs + SS_R;                // statistics and output column
  const float ea = expo ? expf(expo[2 * v]) : 1.f, eb = expo ? expo[2 * v + 1] : 0.f;
  const size_t plane = (size_t)A.W * A.H;
  const float* ci = color + (size_t)vc * plane;
  const float* ti = target + (size_t)vc * plane;
  float* di = d_color + (size_t)vc * plane;
  // the weight of input t in output lane mod 4: both operands' tables
  float wt[SS_W];
#pragma unroll
  for (int t = 0; t < SS_W; ++t) {
    wt[t] = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (t - i >= 0 && t - i < SS_K) wt[t] = (lane & 3) == i ? A.w[t - i] : wt[t];
  }
  const bool xi_in = xi >= 0 && xi < A.W, xs_in = xs >= 0 && xs < A.W && lane < SW;
  const bool own_col = lane >= SS_R && lane < SS_R + OW && xs < A.W;  // counted in S
  const bool xo_in = lane < OW && xo < A.W;
  const int xc = min(max(xi, 0), A.W - 1), oxc = min(max(xo, 0), A.W - 1);
  float rx[4][4], ry[4][4];  // input rows y0 - 10 + 4 g + i at [g mod 4][i]
  float f[3][4][4];          // gradient maps of statistics rows y0 - 5 + 4 s + i at [.][s mod 4][i]
  // raw rows of input group g, and their values (loaded a step ahead of use)
  const auto fetch = [&](int g, float (&x)[4], float (&y)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = min(max(y0 - 2 * SS_R + 4 * g + i, 0), A.H - 1);
      x[i] = (ci + (size_t)r * A.W)[xc];
      y[i] = (ti + (size_t)r * A.W)[xc];
    }
  };
  const auto place = [&](int g, const float (&a)[4], const float (&b)[4], float (&x)[4],
                         float (&y)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = y0 - 2 * SS_R + 4 * g + i;
      const bool in = r >= 0 && r < A.H && xi_in;
      x[i] = in ? ea * a[i] + eb : 0.f;
      y[i] = in ? b[i] : 0.f;
    }
  };
  if (lane < 2) flag[lane] = 0;
  if (NW > 1) __syncthreads();
  float nx[4], ny[4];
#pragma unroll
  for (int g = 0; g < 3; ++g) {
    fetch(g, nx, ny);
    place(g, nx, ny, rx[g], ry[g]);
  }
  fetch(3, nx, ny);
  // a lane sums four rows in FP32 and the steps, as many as the march is long,
  // in FP64: a chain of hundreds of FP32 additions would lose digits that the
  // tree over lanes and workgroups does not (240 rows: 3e-6 of the sum, now 2e-7).
  double sd = 0.0, sad = 0.0, sbd = 0.0;
  const int steps = (y1 - y0 + 3) / 4 + 3;
  for (int s0 = 0; s0 < steps; s0 += 4) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int st = s0 + u;
      if (st >= steps) break;  // uniform
      place(st + 3, nx, ny, rx[(u + 3) & 3], ry[(u + 3) & 3]);
      fetch(st + 4, nx, ny);
      // the output rows' own pixels, for the end of the step
      float oc[4], oy[4], od[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const size_t q = (size_t)min(max(y0 + 4 * (st - 3) + i, 0), A.H - 1) * A.W;
        oc[i] = (ci + q)[oxc];
        oy[i] = (ti + q)[oxc];
        od[i] = (di + q)[oxc];
      }
      // moments of the statistics rows y0 - 5 + 4 st + i
      ss_v4 m[4];
      bool alone = ss_vert<4>(
          A, wt,
          [&](int k, int t) {
            const float x = rx[(u + (t >> 2)) & 3][t & 3], y = ry[(u + (t >> 2)) & 3][t & 3];
            return k == 0 ? x : k == 1 ? y : k == 2 ? x * x + y * y : x * y;
          },
          m);
      ss_horiz<4, NW>(A, wt, buf, alone, st + 1, flag, m);
      float s4 = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = y0 - SS_R + 4 * st + i;
        const float mx = m[0][i], my = m[1][i];
        const float mm = mx * mx + my * my;
        const float a1 = 2.f * mx * my + SS_C1, a2 = 2.f * (m[3][i] - mx * my) + SS_C2;
        const float b1 = mm + SS_C1, b2 = (m[2][i] - mm) + SS_C2;
        // b1, b2 >= C1, C2 > 0: reciprocals by the hardware (about 1 ulp)
        const float rb1 = __builtin_amdgcn_rcpf(b1), rb2 = __builtin_amdgcn_rcpf(b2);
        const float ib = rb1 * rb2;
        const float so = a1 * a2 * ib;
        const float d_mx = 2.f * my * a2 * ib - 2.f * mx * so * rb1;
        const float d_sxx = -so * rb2;
        const float d_sxy = 2.f * a1 * ib;
        const bool in = r >= 0 && r < A.H && xs_in;
        f[0][u][i] = in ? d_mx - 2.f * mx * d_sxx - my * d_sxy : 0.f;
        f[1][u][i] = in ? d_sxx : 0.f;
        f[2][u][i] = in ? d_sxy : 0.f;
        // the workgroup's own pixels carry S
        if (r >= y0 && r < y1) s4 += own_col ? so : 0.f;
      }
      sd += (double)s4;
      if (st < 3) {  // uniform: the first output rows need four groups
        if (NW > 1) __syncthreads();
        continue;
      }
      // blurred maps at the output rows y0 + 4 (st - 3) + i
      ss_v4 bl[3];
      alone = ss_vert<3>(A, wt, [&](int k, int t) { return f[k][(u + 1 + (t >> 2)) & 3][t & 3]; }, bl);
      ss_horiz<3, NW>(A, wt, buf2, alone, st + 1, flag + 1, bl);
      float sa4 = 0.f, sb4 = 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = y0 + 4 * (st - 3) + i;
        const float x = ea * oc[i] + eb;
        // loss = weight (1 - mean S): dL/dx~ = -weight/N (w*f1 + 2 x w*f2 + y w*f3)
        float g = -A.weight_over_n * (bl[0][i] + 2.f * x * bl[1][i] + oy[i] * bl[2][i]);
        g = r < y1 && xo_in ? g : 0.f;
        if (r < y1 && xo_in) (di + (size_t)r * A.W)[oxc] = od[i] + ea * g;
        sa4 += g * oc[i];
        sb4 += g;
      }
      sad += (double)sa4;
      sbd += (double)sb4;
    }
  }
  const size_t bb = (size_t)blockIdx.y * gridDim.x + blockIdx.x;
  float s = wave_total((float)sd);
  float sa = wave_total((float)sad), sb = wave_total((float)sbd);
  const int w = lane >> 6;
  if (lane_id() == 0) {
    red[0][w] = s;
    red[1][w] = sa;
    red[2][w] = sb;
  }
  __syncthreads();
  if (lane == 0) {
    for (int k = 1; k < NW; ++k) {
      s += red[0][k];
      sa += red[1][k];
      sb += red[2][k];
    }
    ssim_part[bb] = s;
    if (e_part) {
      e_part[2 * bb] = ea * sa;
      e_part[2 * bb + 1] = sb;
    }
  }
}

// One workgroup per view: the view's block partials of the exposure sums
// (added to d_expo) and of S (to s_view[v]).  Sums run in a fixed order
// (deterministic).
__global__ __launch_bounds__(256) void k_ssim_reduce(int nb_view, const float* s_part,
                                                     const float* e_part, float* d_expo,
                                                     float* s_view) {
  __shared__ float red[4];
  const int v = blockIdx.x;
  const size_t k0 = (size_t)v * 3 * nb_view;
  float a = 0.f, b = 0.f, t = 0.f;
  for (int i = threadIdx.x; i < 3 * nb_view; i += 256) {
    t += s_part[k0 + i];
    if (e_part) {
      a += e_part[2 * (k0 + i)];
      b += e_part[2 * (k0 + i) + 1];
    }
  }
  t = block_sum_256(t, red);
  if (e_part) {
    a = block_sum_256(a, red);
    b = block_sum_256(b, red);
  }
  if (threadIdx.x == 0) {
    s_view[v] = t;
    if (e_part) {
      d_expo[2 * v] += a;
      d_expo[2 * v + 1] += b;
    }
  }
}

__global__ __launch_bounds__(64) void k_ssim_mean(int nv, const float* s_view, float inv_n,
                                                  float* out) {
  float t = 0.f;
  for (int v = threadIdx.x; v < nv; v += 64) t += s_view[v];
  t = wave_total(t);
  if (threadIdx.x == 0) out[0] = t * inv_n;
}

static size_t align_up(size_t x) { return (x + 255) / 256 * 256; }

size_t ssim_workspace_bytes(int nv, int W, int H) {
  // partials of a call: at most its 32 x 32 tiles, or a small call's waves
  const size_t tiles = (size_t)((W + SS_T - 1) / SS_T) * ((H + SS_T - 1) / SS_T) * 3 * nv;
  const size_t nb = std::max<size_t>(tiles, 2 * SS_SIMDS);
  return align_up(nb * 4) + align_up(nb * 8) + align_up((size_t)nv * 4);
}

hipError_t launch_ssim(int nv, int W, int H, float weight, const float* color,
                       const float* target, const float* expo, void* ws, float* d_color,
                       float* d_expo, float* ssim_out, hipStream_t s) {
  SsimArgs A{};
  double g[SS_K], tot = 0.0;
  for (int d = -SS_R; d <= SS_R; ++d) tot += g[d + SS_R] = exp(-(double)(d * d) / (2.0 * 1.5 * 1.5));
  for (int d = 0; d <= 2 * SS_R; ++d) A.w[d] = (float)(g[d] / tot);
  A.W = W;
  A.H = H;
  const SsimShape sh = ssim_shape(nv, W, H);
  const int nw = sh.nw;
  A.TX = sh.strips;
  A.nv = nv;
  A.rows = sh.rows;
  const double n = 3.0 * nv * (double)W * H;
  A.weight_over_n = (float)(weight / n);
  const int nb_view = A.TX * ((H + A.rows - 1) / A.rows);
  const size_t nb = (size_t)nb_view * 3 * nv;
  char* w8 = (char*)ws;
  float* s_part = (float*)w8;
  float* e_part = (float*)(w8 + align_up(nb * 4));
  float* s_view = (float*)(w8 + align_up(nb * 4) + align_up(nb * 8));
  const dim3 grid(nb_view, 3 * nv);
  const auto k = nw == 1 ? k_ssim<1> : nw == 2 ? k_ssim<2> : nw == 3 ? k_ssim<3> : k_ssim<4>;
  hipLaunchKernelGGL(k, grid, dim3(64 * nw), 0, s, A, color, target, expo, d_color, s_part,
                     d_expo ? e_part : (float*)nullptr);
  if (d_expo || ssim_out)
    hipLaunchKernelGGL(k_ssim_reduce, dim3(nv), dim3(256), 0, s, nb_view, s_part,
                       d_expo ? e_part : (const float*)nullptr, d_expo, s_view);
  if (ssim_out)
    hipLaunchKernelGGL(k_ssim_mean, dim3(1), dim3(64), 0, s, nv, s_view, (float)(1.0 / n),
                       ssim_out);
  return hipGetLastError();
}

}  // namespace gsr
