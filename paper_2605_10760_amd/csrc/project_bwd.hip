// Chain rule from the per-pair screen-space gradients to the Gaussian
// parameters and each view's pose.
//
// One thread per Gaussian; it goes through grad-needing views of its set,
// recomputes the projection in FP64 (the forward's code), accumulates the
// parameter gradients in registers (the colour sums of SH degrees above 0 in
// its own LDS column) and writes them once (no atomics, so summing over views
// is deterministic).
#include "common.h"

namespace gsr {

#define SHK0 0.28209479177387814f
#define SHK1 0.4886025119029199f
#define SHK2A 1.0925484305920792f
#define SHK2B 0.31539156525252005f
#define SHK2C 0.5462742152960396f
#define SHK3A 0.5900435899266435f
#define SHK3B 2.890611442640554f
#define SHK3C 0.4570457994644658f
#define SHK3D 0.3731763325901154f
#define SHK3E 1.445305721320277f

// Real SH basis (as in the forward) and its partial derivatives with respect
// to the direction components, as polynomials on R^3.
template <int D>
__device__ __forceinline__ void sh_eval_grad(float x, float y, float z, float* Y, float (*dY)[3]) {
  Y[0] = SHK0; dY[0][0] = dY[0][1] = dY[0][2] = 0.f;
  if (D >= 1) {
    Y[1] = -SHK1 * y; dY[1][0] = 0.f; dY[1][1] = -SHK1; dY[1][2] = 0.f;
    Y[2] = SHK1 * z;  dY[2][0] = 0.f; dY[2][1] = 0.f;   dY[2][2] = SHK1;
    Y[3] = -SHK1 * x; dY[3][0] = -SHK1; dY[3][1] = 0.f; dY[3][2] = 0.f;
  }
  if (D >= 2) {
    const float xx = x * x, yy = y * y, zz = z * z;
    Y[4] = SHK2A * x * y;  dY[4][0] = SHK2A * y; dY[4][1] = SHK2A * x; dY[4][2] = 0.f;
    Y[5] = -SHK2A * y * z; dY[5][0] = 0.f; dY[5][1] = -SHK2A * z; dY[5][2] = -SHK2A * y;
    Y[6] = SHK2B * (2.f * zz - xx - yy);
    dY[6][0] = -2.f * SHK2B * x; dY[6][1] = -2.f * SHK2B * y; dY[6][2] = 4.f * SHK2B * z;
    Y[7] = -SHK2A * x * z; dY[7][0] = -SHK2A * z; dY[7][1] = 0.f; dY[7][2] = -SHK2A * x;
    Y[8] = SHK2C * (xx - yy); dY[8][0] = 2.f * SHK2C * x; dY[8][1] = -2.f * SHK2C * y; dY[8][2] = 0.f;
    if (D >= 3) {
      Y[9] = -SHK3A * y * (3.f * xx - yy);
      dY[9][0] = -6.f * SHK3A * x * y; dY[9][1] = -SHK3A * (3.f * xx - 3.f * yy); dY[9][2] = 0.f;
      Y[10] = SHK3B * x * y * z;
      dY[10][0] = SHK3B * y * z; dY[10][1] = SHK3B * x * z; dY[10][2] = SHK3B * x * y;
      Y[11] = -SHK3C * y * (4.f * zz - xx - yy);
      dY[11][0] = 2.f * SHK3C * x * y; dY[11][1] = -SHK3C * (4.f * zz - xx - 3.f * yy);
      dY[11][2] = -8.f * SHK3C * y * z;
      Y[12] = SHK3D * z * (2.f * zz - 3.f * xx - 3.f * yy);
      dY[12][0] = -6.f * SHK3D * x * z; dY[12][1] = -6.f * SHK3D * y * z;
      dY[12][2] = SHK3D * (6.f * zz - 3.f * xx - 3.f * yy);
      Y[13] = -SHK3C * x * (4.f * zz - xx - yy);
      dY[13][0] = -SHK3C * (4.f * zz - 3.f * xx - yy); dY[13][1] = 2.f * SHK3C * x * y;
      dY[13][2] = -8.f * SHK3C * x * z;
      Y[14] = SHK3E * z * (xx - yy);
      dY[14][0] = 2.f * SHK3E * x * z; dY[14][1] = -2.f * SHK3E * y * z; dY[14][2] = SHK3E * (xx - yy);
      Y[15] = -SHK3A * x * (xx - 3.f * yy);
      dY[15][0] = -SHK3A * (3.f * xx - 3.f * yy); dY[15][1] = 6.f * SHK3A * x * y; dY[15][2] = 0.f;
    }
  }
}

// Normalised quaternion, scales and rotation matrix of a Gaussian; returns the
// quaternion's norm.
__device__ __forceinline__ float rot_scale(const float* lsv, const float* q4v, float* qh, float* sv,
                                           float (*R)[3]) {
  for (int k = 0; k < 3; ++k) sv[k] = expf(lsv[k]);
  const float qn = sqrtf(q4v[0] * q4v[0] + q4v[1] * q4v[1] + q4v[2] * q4v[2] + q4v[3] * q4v[3]);
  for (int k = 0; k < 4; ++k) qh[k] = q4v[k] / qn;
  const float w = qh[0], x = qh[1], y = qh[2], z = qh[3];
  R[0][0] = 1.f - 2.f * (y * y + z * z); R[0][1] = 2.f * (x * y - w * z); R[0][2] = 2.f * (x * z + w * y);
  R[1][0] = 2.f * (x * y + w * z); R[1][1] = 1.f - 2.f * (x * x + z * z); R[1][2] = 2.f * (y * z - w * x);
  R[2][0] = 2.f * (x * z - w * y); R[2][1] = 2.f * (y * z + w * x); R[2][2] = 1.f - 2.f * (x * x + y * y);
  return qn;
}

// A view as the kernel uses it: rotation, translation, focal lengths, guard
// limits.
struct BwdView {
  float Rc[3][3], tc[3];
  float fx, fy;
  float lx, ly;
  double dx, dy;
};

// What a Gaussian's pairs add up to.
struct GaussSums {
  float m[3];     // dL/dmean
  float S3[6];    // dL/dSigma, symmetric: 00 01 02 11 12 22
  float sig;      // dL/dsigma
  float col[3];   // dL/dcolour (degree 0)
};

// One pair: from its screen-space gradient (u, v, A, B, C, sigma, r, g, b, z)
// to the Gaussian's sums and the view's pose gradient.  gk: the thread's LDS
// column of colour sums (degrees above 0, stride gks words).
template <int SHD>
__device__ __forceinline__ void pair_bwd(const BwdView& w, const float* m, const double Sd[3][3],
                                         const float* g10, const float* kk, GaussSums& G,
                                         float* gk, int gks, float* pose) {
  constexpr int NB = (SHD + 1) * (SHD + 1);
  const float fx = w.fx, fy = w.fy;
  const float gu = g10[0], gv = g10[1], gA = g10[2], gB = g10[3], gC = g10[4];
  const float gs = g10[5], gz = g10[9];
  float gc[3] = {g10[6], g10[7], g10[8]};
  // the forward's FP64 projection again (no read of the record): the conic (A,
  // B, C) = (c, -b, a) / det, and, rounded once, the mean and covariance in the
  // camera
  const ScreenCov s2 = screen_cov_fp64(Sd, &w.Rc[0][0], w.tc, m, fx, fy, w.dx, w.dy);
  const double idet = 1.0 / (s2.a * s2.c - s2.b * s2.b);
  const float p[3] = {(float)s2.p[0], (float)s2.p[1], (float)s2.p[2]};
  float V[3][3];
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) V[i][j] = (float)s2.V[i][j];
  const float iz = (float)s2.iz, iz2 = iz * iz;
  const float rx = p[0] * iz, ry = p[1] * iz;
  const bool inx = !(rx < -w.lx || rx > w.lx), iny = !(ry < -w.ly || ry > w.ly);
  const float rxc = inx ? rx : (rx < 0.f ? -w.lx : w.lx);
  const float ryc = iny ? ry : (ry < 0.f ? -w.ly : w.ly);
  const float j00 = fx * iz, j02 = -fx * rxc * iz, j11 = fy * iz, j12 = -fy * ryc * iz;

  // conic -> 2D covariance:  G_S2 = -Q G_Q Q, in FP64: the products of an
  // elongated splat's conic cancel
  float s00, s01, s11;
  {
    const double A = s2.c * idet, B = -s2.b * idet, C = s2.a * idet;
    const double hB = 0.5 * gB;
    const double X00 = gA * A + hB * B, X01 = gA * B + hB * C;
    const double X10 = hB * A + gC * B, X11 = hB * B + gC * C;
    s00 = (float)-(A * X00 + B * X10);
    s01 = (float)(-0.5 * ((A * X01 + B * X11) + (B * X00 + C * X10)));
    s11 = (float)-(B * X01 + C * X11);
  }
  // 2D -> camera covariance (J^T G J) and Jacobian (2 G J V)
  float GV[3][3];
  GV[0][0] = j00 * j00 * s00;
  GV[0][1] = j00 * j11 * s01;
  GV[0][2] = j00 * (j02 * s00 + j12 * s01);
  GV[1][1] = j11 * j11 * s11;
  GV[1][2] = j11 * (j02 * s01 + j12 * s11);
  GV[2][2] = j02 * j02 * s00 + 2.f * j02 * j12 * s01 + j12 * j12 * s11;
  GV[1][0] = GV[0][1]; GV[2][0] = GV[0][2]; GV[2][1] = GV[1][2];
  float JV0[3], JV1[3];
  for (int k = 0; k < 3; ++k) {
    JV0[k] = j00 * V[0][k] + j02 * V[2][k];
    JV1[k] = j11 * V[1][k] + j12 * V[2][k];
  }
  const float GJ00 = 2.f * (s00 * JV0[0] + s01 * JV1[0]);
  const float GJ02 = 2.f * (s00 * JV0[2] + s01 * JV1[2]);
  const float GJ11 = 2.f * (s01 * JV0[1] + s11 * JV1[1]);
  const float GJ12 = 2.f * (s01 * JV0[2] + s11 * JV1[2]);
  // camera-space mean
  float gp[3];
  gp[0] = gu * fx * iz;
  gp[1] = gv * fy * iz;
  gp[2] = -(gu * fx * p[0] + gv * fy * p[1]) * iz2 + gz;
  gp[2] += -(GJ00 * fx + GJ11 * fy) * iz2;
  gp[2] += GJ02 * fx * rxc * iz2 + GJ12 * fy * ryc * iz2;
  if (inx) {
    gp[0] += -GJ02 * fx * iz2;
    gp[2] += GJ02 * fx * p[0] * iz2 * iz;
  }
  if (iny) {
    gp[1] += -GJ12 * fy * iz2;
    gp[2] += GJ12 * fy * p[1] * iz2 * iz;
  }
  for (int k = 0; k < 3; ++k)
    G.m[k] += w.Rc[0][k] * gp[0] + w.Rc[1][k] * gp[1] + w.Rc[2][k] * gp[2];
  // world covariance: Rc^T G_V Rc
  float Y3[3][3];
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j)
      Y3[i][j] = GV[i][0] * w.Rc[0][j] + GV[i][1] * w.Rc[1][j] + GV[i][2] * w.Rc[2][j];
  {
    int e = 0;
    for (int i = 0; i < 3; ++i)
      for (int j = i; j < 3; ++j)
        G.S3[e++] += w.Rc[0][i] * Y3[0][j] + w.Rc[1][i] * Y3[1][j] + w.Rc[2][i] * Y3[2][j];
  }
  G.sig += gs;
  // pose: rho <- dL/dp (+ SH term below), phi <- p x dL/dp + covariance rotation
  pose[0] = gp[0]; pose[1] = gp[1]; pose[2] = gp[2];
  pose[3] = p[1] * gp[2] - p[2] * gp[1];
  pose[4] = p[2] * gp[0] - p[0] * gp[2];
  pose[5] = p[0] * gp[1] - p[1] * gp[0];
  float VG[3][3];
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j)
      VG[i][j] = V[i][0] * GV[0][j] + V[i][1] * GV[1][j] + V[i][2] * GV[2][j];
  // M = V G - G V = VG - VG^T
  pose[3] += 2.f * (VG[1][2] - VG[2][1]);
  pose[4] += 2.f * (VG[2][0] - VG[0][2]);
  pose[5] += 2.f * (VG[0][1] - VG[1][0]);
  // colour
  if (SHD == 0) {
    G.col[0] += gc[0]; G.col[1] += gc[1]; G.col[2] += gc[2];
  } else {
    const float ox = -(w.Rc[0][0] * w.tc[0] + w.Rc[1][0] * w.tc[1] + w.Rc[2][0] * w.tc[2]);
    const float oy = -(w.Rc[0][1] * w.tc[0] + w.Rc[1][1] * w.tc[1] + w.Rc[2][1] * w.tc[2]);
    const float oz = -(w.Rc[0][2] * w.tc[0] + w.Rc[1][2] * w.tc[1] + w.Rc[2][2] * w.tc[2]);
    float d[3] = {m[0] - ox, m[1] - oy, m[2] - oz};
    const float dist = sqrtf(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
    const float idist = 1.f / dist;
    d[0] *= idist; d[1] *= idist; d[2] *= idist;
    float Y[16], dY[16][3];
    sh_eval_grad<SHD>(d[0], d[1], d[2], Y, dY);
    // the colour and its Jacobian with respect to the direction,
    // Jr[c][k] = sum_i k_ic dY_i/dd_k, in one pass over the coefficients
    // (each coefficient and basis derivative is used once, so neither
    // stays live past it)
    float raw[3] = {0.5f, 0.5f, 0.5f};
    float Jr[3][3] = {{0.f, 0.f, 0.f}, {0.f, 0.f, 0.f}, {0.f, 0.f, 0.f}};
    for (int i = 0; i < NB; ++i)
      for (int c = 0; c < 3; ++c) {
        const float kc = kk[3 * i + c];
        raw[c] += Y[i] * kc;
        Jr[c][0] += kc * dY[i][0]; Jr[c][1] += kc * dY[i][1]; Jr[c][2] += kc * dY[i][2];
      }
    for (int c = 0; c < 3; ++c) gc[c] = raw[c] > 0.f ? gc[c] : 0.f;
    // d L/d d = Jr^T gc
    float gdir[3];
    for (int k = 0; k < 3; ++k) gdir[k] = gc[0] * Jr[0][k] + gc[1] * Jr[1][k] + gc[2] * Jr[2][k];
    for (int i = 0; i < NB; ++i)
      for (int c = 0; c < 3; ++c) gk[(3 * i + c) * gks] += Y[i] * gc[c];
    const float dd = d[0] * gdir[0] + d[1] * gdir[1] + d[2] * gdir[2];
    float gmd[3];
    for (int k = 0; k < 3; ++k) {
      gmd[k] = (gdir[k] - d[k] * dd) * idist;
      G.m[k] += gmd[k];
    }
    for (int i = 0; i < 3; ++i)
      pose[i] += w.Rc[i][0] * gmd[0] + w.Rc[i][1] * gmd[1] + w.Rc[i][2] * gmd[2];
  }
}

// A wave takes the set's views in turn, a lane idling where its Gaussian is
// culled, or (`own`) every lane takes the views that see its own Gaussian, from
// a starting view of its own, so that the lanes spread over the views.  The
// first form reads gradient rows and view constants together and sums a
// view's pose gradient over the wave; the second does as many steps as the
// wave's most visible Gaussian has views, and adds each pair's pose gradient
// to the views' sums in LDS.  The second is taken where it saves enough steps:
// from 4 steps for 3 on (3M Gaussians of degree 3 in 32 views: 1500 us, in
// turn 2670; 400k in 8 views 105 and 152; 1.6M of degree 0 in 8 views of each
// submap, where most waves save nothing: 223 in turn, all `own` 348).
// Pose sums are FP64 from the workgroup's LDS on (a chain of up to 256 FP32
// additions in `own`, no tree, lost 4 times the rounding of the result; the FP64
// LDS atomics are the faster ones too: 3M Gaussians of degree 3 in 32 views 1401 ->
// 1196 us), and the last workgroup to finish writes d_pose and clears them for the
// next call (no clearing kernel, and the rounding of thousands of FP32 additions
// per component does not reach the result).
// SPLIT: a loop for each way.  One loop for both keeps the registers of degrees 1 to 3
// within 125, 124 and 167 (152, 190 and 246 with two), and LDS for the views there are
// leaves degree 3 room for three workgroups a CU; two loops are faster where lanes
// mostly take their own views, and for degree 0.  Two loops | one, us: one view of 1M
// Gaussians of degree 1 51 | 45, 2 90 | 79, 3 124 | 109; three submaps of 200k of degree 2
// in 2 keyframes each 75 | 70, in 4 118 | 120, in 6 154 | 162; of degree 3 in 8 226 | 198;
// 300k of degree 3 in 12 views all around 85 | 88, 200k in 20 83 | 97; six submaps of 200k
// of degree 0 in 8 keyframes 153 | 162, of degree 1 211 | 190.
constexpr size_t BWD_VIEW_BYTES = 64 + 48 + 16 + 32 + 16;  // LDS of a view
template <int SHD, bool SPLIT>
__global__ __launch_bounds__(256) void k_project_bwd(SetTab t, SceneDev sc, CamDev cam, StateDev st,
                                                     float* grad2d, PoseAcc* pa, gsr_grads out) {
  constexpr int NB = (SHD + 1) * (SHD + 1);
  const int nblk = t.set_blk[t.ns];
  const int b = xcd_remap(blockIdx.x, nblk);
  if (b < 0) return;
  const int share = (int)blockIdx.x & 7;
  const int s = find_seg(t.set_blk, t.ns, b);
  const int lb = b - t.set_blk[s];
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int local = lb * 256 + (int)threadIdx.x;
  const int nset = t.set_goff[s + 1] - t.set_goff[s];
  const int v0 = t.set_voff[s], nv = t.set_voff[s + 1] - v0;
  const bool valid = local < nset;
  const long gi = (long)t.set_goff[s] + (valid ? local : 0);

  // the set's views: parameters, pose sums, and per wave the visible bits and the
  // position of the first visible pair (SPLIT: at fixed addresses, else as many as
  // the largest set has)
  constexpr int NV = SPLIT ? MAXV : 1;
  __shared__ float4 vw_s[NV][4];  // (R row, t component) x 3, (fx, fy, limits)
  __shared__ double psum_s[NV][6], vlim_s[NV][2];
  __shared__ unsigned long long vmask_s[NV][4];
  __shared__ uint32_t vrow_s[NV][4];
  extern __shared__ float4 views_lds[];
  const int most = SPLIT ? 0 : t.most;
  float4 (*vw)[4] = SPLIT ? vw_s : reinterpret_cast<float4(*)[4]>(views_lds);
  double (*psum)[6] = SPLIT ? psum_s : reinterpret_cast<double(*)[6]>(vw + most);
  double (*vlim)[2] = SPLIT ? vlim_s : reinterpret_cast<double(*)[2]>(psum + most);
  unsigned long long (*vmask)[4] =
      SPLIT ? vmask_s : reinterpret_cast<unsigned long long(*)[4]>(vlim + most);
  uint32_t (*vrow)[4] = SPLIT ? vrow_s : reinterpret_cast<uint32_t(*)[4]>(vmask + most);
  if ((int)threadIdx.x < nv) {
    const int v = t.view_by_set[v0 + (int)threadIdx.x];
    const float* vm = cam.viewmats + 12 * v;
    const float* f = cam.intrinsics + 4 * v;
    const ViewLim lm = view_lim(f[0], f[1], t.W, t.H);
    for (int i = 0; i < 3; ++i)
      vw[threadIdx.x][i] = make_float4(vm[4 * i], vm[4 * i + 1], vm[4 * i + 2], vm[4 * i + 3]);
    vw[threadIdx.x][3] = make_float4(f[0], f[1], lm.lx, lm.ly);
    vlim[threadIdx.x][0] = lm.dx;
    vlim[threadIdx.x][1] = lm.dy;
    const size_t bi = (size_t)(t.blk_off[v] + lb);
    uint32_t row = st.vbase[bi];
    for (int w = 0; w < 4; ++w) {
      const unsigned long long mk = st.vmask[4 * bi + w];
      vmask[threadIdx.x][w] = mk;
      vrow[threadIdx.x][w] = row;
      row += (uint32_t)__popcll(mk);
    }
    for (int k = 0; k < 6; ++k) psum[threadIdx.x][k] = 0.0;
  }

  // The mean and the forward's FP64 covariance (the conic is recomputed per view
  // from it rather than read back from the screen-space record).  The
  // rotation and scale factors are formed again after the loop, so they hold
  // no registers during it.
  float m[3] = {0.f, 0.f, 0.f};
  double Sd[3][3];
  {
    float lsv[3] = {0.f, 0.f, 0.f}, q4v[4] = {1.f, 0.f, 0.f, 0.f};
    if (valid) {
      for (int k = 0; k < 3; ++k) {
        m[k] = sc.means[3 * gi + k];
        lsv[k] = sc.log_scales[3 * gi + k];
      }
      const float4 q4 = *reinterpret_cast<const float4*>(sc.quats + 4 * gi);
      q4v[0] = q4.x; q4v[1] = q4.y; q4v[2] = q4.z; q4v[3] = q4.w;
    }
    cov3_fp64(lsv, q4v, Sd);
  }

  GaussSums G{};
  // colour gradients: in registers for degree 0; for higher degrees (up to
  // 48 per Gaussian) in the thread's own LDS column (the lanes of a
  // wave hit distinct banks), out of the registers during the view loop
  __shared__ float gkl[SHD > 0 ? 3 * NB : 1][256];
  if (SHD > 0)
    for (int j = 0; j < 3 * NB; ++j) gkl[j][threadIdx.x] = 0.f;
  const float* kk = SHD > 0 ? sc.colors + (long)3 * sc.sh_stride * gi : nullptr;
  __syncthreads();

  const auto load_view = [&](int k) {
    BwdView w;
    for (int i = 0; i < 3; ++i) {
      const float4 r = vw[k][i];
      w.Rc[i][0] = r.x; w.Rc[i][1] = r.y; w.Rc[i][2] = r.z;
      w.tc[i] = r.w;
    }
    const float4 f = vw[k][3];
    w.fx = f.x; w.fy = f.y; w.lx = f.z; w.ly = f.w;
    w.dx = vlim[k][0];
    w.dy = vlim[k][1];
    return w;
  };
  const auto read_row = [&](int k, float (&g)[GRAD2D]) {
    const unsigned long long mk = vmask[k][wv];
    const uint32_t row =
        vrow[k][wv] + __builtin_amdgcn_mbcnt_hi((uint32_t)(mk >> 32),
                                                __builtin_amdgcn_mbcnt_lo((uint32_t)mk, 0u));
    const float2* p = reinterpret_cast<const float2*>(grad2d + (size_t)GRAD2D * row);
#pragma unroll
    for (int i = 0; i < GRAD2D / 2; ++i) {
      const float2 x = p[i];
      g[2 * i] = x.x;
      g[2 * i + 1] = x.y;
    }
  };
  float* gk = SHD > 0 ? &gkl[0][threadIdx.x] : nullptr;
  // bit k: view k of the set sees the lane's Gaussian, one of the wave's
  unsigned long long see = 0ull, any = 0ull;
  for (int k = 0; k < nv; ++k) {
    const unsigned long long mk = vmask[k][wv];
    see |= ((mk >> lane_id()) & 1ull) << k;
    any |= (unsigned long long)(mk != 0ull) << k;
  }
  int steps = (int)__popcll(see);
  for (int d = 1; d < 64; d *= 2) steps = max(steps, __shfl_xor(steps, d));
  steps = __builtin_amdgcn_readfirstlane(steps);
  // `own`: the lane's views in cyclic order from view `first` (hi, then lo); in turn:
  // the views that see one of the wave's Gaussians
  const bool own = 4 * steps < 3 * (int)__popcll(any);
  if constexpr (SPLIT) {
    if (own) {
      const int first = (lane_id() * nv) >> 6;
      unsigned long long hi = see & (~0ull << first), lo = see & ~(~0ull << first);
      while (hi | lo) {
        const int k = (int)__builtin_ctzll(hi ? hi : lo);
        if (hi)
          hi &= hi - 1ull;
        else
          lo &= lo - 1ull;
        float g10[GRAD2D], pose[6];
        read_row(k, g10);
        pair_bwd<SHD>(load_view(k), m, Sd, g10, kk, G, gk, 256, pose);
#pragma unroll
        for (int i = 0; i < 6; ++i) unsafeAtomicAdd(&psum[k][i], (double)pose[i]);
      }
    } else {
      while (any) {
        const int k = __builtin_amdgcn_readfirstlane((int)__builtin_ctzll(any));
        any &= any - 1ull;
        float pose[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if ((see >> k) & 1ull) {
          float g10[GRAD2D];
          read_row(k, g10);
          pair_bwd<SHD>(load_view(k), m, Sd, g10, kk, G, gk, 256, pose);
        }
        for (int i = 0; i < 6; ++i) pose[i] = wave_total(pose[i]);
        if (lane_id() == 0)
          for (int i = 0; i < 6; ++i) unsafeAtomicAdd(&psum[k][i], (double)pose[i]);
      }
    }
  } else {
    const int first = own ? (lane_id() * nv) >> 6 : 0;
    const unsigned long long walk = own ? see : any;
    unsigned long long hi = walk & (~0ull << first), lo = walk & ~(~0ull << first);
    while (__ballot((hi | lo) != 0ull) != 0ull) {
      int k = (hi | lo) != 0ull ? (int)__builtin_ctzll(hi ? hi : lo) : 0;
      bool on = (hi | lo) != 0ull;
      if (hi)
        hi &= hi - 1ull;
      else
        lo &= lo - 1ull;
      if (!own) {
        k = __builtin_amdgcn_readfirstlane(k);
        on = (see >> k) & 1ull;
      }
      float pose[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      if (on) {
        float g10[GRAD2D];
        read_row(k, g10);
        pair_bwd<SHD>(load_view(k), m, Sd, g10, kk, G, gk, 256, pose);
      }
      if (!own)
        for (int i = 0; i < 6; ++i) pose[i] = wave_total(pose[i]);
      if (own ? on : lane_id() == 0)
#pragma unroll
        for (int i = 0; i < 6; ++i) unsafeAtomicAdd(&psum[k][i], (double)pose[i]);
    }
  }
  __syncthreads();
  // The rows read are cleared (zero between backward calls), a view's rows of
  // the workgroup lying together: whole lines, where clearing each row as it
  // was read (40 bytes a lane) wrote most lines in parts: 1.5 ms
  // instead of 2.1 for 3M Gaussians in 32 views
  for (int k = wv; k < nv; k += 4) {
    const uint32_t r0 = vrow[k][0];
    const uint32_t n = vrow[k][3] + (uint32_t)__popcll(vmask[k][3]) - r0;
    float2* p = reinterpret_cast<float2*>(grad2d + (size_t)GRAD2D * r0);
    for (uint32_t i = lane_id(); i < n * (GRAD2D / 2); i += 64u) p[i] = make_float2(0.f, 0.f);
  }
  for (int i = threadIdx.x; i < 6 * nv; i += 256) {
    const int k = i / 6;
    const double tot = psum[k][i - 6 * k];
    if (tot != 0.0)
      unsafeAtomicAdd(&pa->share[share].sum[6 * t.view_by_set[v0 + k] + (i - 6 * k)], tot);
  }
  // The last workgroup writes the call's sums and clears them: the last of each
  // XCD's share finds itself by the share's count, the last of these by the
  // count of shares (the counts and sums of a share lie together, so that
  // most atomics meet only those of their own XCD).  Only device-scope atomics
  // touch the sums, so each wave need only wait until its own are performed: no
  // cache is written back.
  {
    __shared__ unsigned int last;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
      const int per = (nblk + 7) / 8, shares = (nblk + per - 1) / per;
      const int mine = min(per, nblk - share * per);
      last = atomicAdd(&pa->share[share].done, 1u) == (unsigned int)mine - 1u &&
             atomicAdd(&pa->done, 1u) == (unsigned int)shares - 1u;
    }
    __syncthreads();
    if (last) {
      for (int i = threadIdx.x; i < 6 * t.nv; i += 256) {
        double x = 0.0;
        for (int j = 0; j < 8; ++j)
          x += __longlong_as_double((long long)atomicExch(
              reinterpret_cast<unsigned long long*>(&pa->share[j].sum[i]), 0ull));
        out.d_pose[i] = (float)x;
      }
      if (threadIdx.x < 8) atomicExch(&pa->share[threadIdx.x].done, 0u);
      if (threadIdx.x == 8) atomicExch(&pa->done, 0u);
    }
  }
  if (!valid) return;
  // covariance -> scales and rotation:  Sigma = M M^T, M = R diag(s)
  float R[3][3], M[3][3], qh[4], sv[3];
  float qn;
  {
    float lsv[3], q4v[4];
    for (int k = 0; k < 3; ++k) lsv[k] = sc.log_scales[3 * gi + k];
    const float4 q4 = *reinterpret_cast<const float4*>(sc.quats + 4 * gi);
    q4v[0] = q4.x; q4v[1] = q4.y; q4v[2] = q4.z; q4v[3] = q4.w;
    qn = rot_scale(lsv, q4v, qh, sv, R);
  }
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) M[i][j] = R[i][j] * sv[j];
  const float* S = G.S3;
  const float G3[3][3] = {{S[0], S[1], S[2]}, {S[1], S[3], S[4]}, {S[2], S[4], S[5]}};
  float GM[3][3];
  for (int i = 0; i < 3; ++i)
    for (int k = 0; k < 3; ++k)
      GM[i][k] = 2.f * (G3[i][0] * M[0][k] + G3[i][1] * M[1][k] + G3[i][2] * M[2][k]);
  float GR[3][3];
  for (int k = 0; k < 3; ++k) {
    const float gsk = GM[0][k] * R[0][k] + GM[1][k] * R[1][k] + GM[2][k] * R[2][k];
    out.d_log_scales[3 * gi + k] = gsk * sv[k];
    for (int i = 0; i < 3; ++i) GR[i][k] = GM[i][k] * sv[k];
  }
  const float w = qh[0], x = qh[1], y = qh[2], z = qh[3];
  float gq[4];
  gq[0] = 2.f * (-z * GR[0][1] + y * GR[0][2] + z * GR[1][0] - x * GR[1][2] - y * GR[2][0] + x * GR[2][1]);
  gq[1] = 2.f * (y * GR[0][1] + z * GR[0][2] + y * GR[1][0] - 2.f * x * GR[1][1] - w * GR[1][2] +
                 z * GR[2][0] + w * GR[2][1] - 2.f * x * GR[2][2]);
  gq[2] = 2.f * (-2.f * y * GR[0][0] + x * GR[0][1] + w * GR[0][2] + x * GR[1][0] + z * GR[1][2] -
                 w * GR[2][0] + z * GR[2][1] - 2.f * y * GR[2][2]);
  gq[3] = 2.f * (-2.f * z * GR[0][0] - w * GR[0][1] + x * GR[0][2] + w * GR[1][0] -
                 2.f * z * GR[1][1] + y * GR[1][2] + x * GR[2][0] + y * GR[2][1]);
  const float dq = qh[0] * gq[0] + qh[1] * gq[1] + qh[2] * gq[2] + qh[3] * gq[3];
  const float4 gq4 = make_float4((gq[0] - qh[0] * dq) / qn, (gq[1] - qh[1] * dq) / qn,
                                 (gq[2] - qh[2] * dq) / qn, (gq[3] - qh[3] * dq) / qn);
  *reinterpret_cast<float4*>(out.d_quats + 4 * gi) = gq4;
  for (int k = 0; k < 3; ++k) out.d_means[3 * gi + k] = G.m[k];
  // d sigmoid(o)/do = e/(1 + e)^2 with e = exp(-|o|) <= 1: accurate for
  // every logit (sigma (1 - sigma) in FP32 is exactly 0 once sigma rounds
  // to 1, at o above about 16.6)
  const float eo = expf(-fabsf(sc.opac[gi]));
  const float ro = 1.f / (1.f + eo);
  out.d_opacity_logits[gi] = G.sig * (eo * ro * ro);
  if (SHD == 0) {
    for (int c = 0; c < 3; ++c) out.d_colors[3 * gi + c] = G.col[c];
  } else {
    float* dk = out.d_colors + (long)3 * sc.sh_stride * gi;
    for (int i = 0; i < NB; ++i)
      for (int c = 0; c < 3; ++c) dk[3 * i + c] = gkl[3 * i + c][threadIdx.x];
    for (int i = 3 * NB; i < 3 * sc.sh_stride; ++i) dk[i] = 0.f;
  }
}

hipError_t launch_project_bwd(const SetTab& t, const SceneDev& sc, const CamDev& cam, StateDev st,
                              float* grad2d, PoseAcc* pa, const gsr_grads& g,
                              hipStream_t s) {
  const int nb = t.set_blk[t.ns];
  if (nb == 0) return hipSuccess;
  const bool split = bwd_by_two_loops(sc.sh_degree, t.most);
  const auto k = sc.sh_degree == 0   ? k_project_bwd<0, true>
                 : sc.sh_degree == 1 ? k_project_bwd<1, false>
                 : sc.sh_degree == 2 ? (split ? k_project_bwd<2, true> : k_project_bwd<2, false>)
                                     : (split ? k_project_bwd<3, true> : k_project_bwd<3, false>);
  hipLaunchKernelGGL(k, dim3(xcd_grid(nb)), dim3(256), split ? 0 : (size_t)t.most * BWD_VIEW_BYTES, s,
                     t, sc, cam, st, grad2d, pa, g);
  return hipGetLastError();
}

}  // namespace gsr
