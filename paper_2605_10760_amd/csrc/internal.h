// Internal declarations shared by the HIP translation units of libgsr.
// Host code builds small per-kernel tables of the call's structure (which
// view renders which Gaussian set, block offsets); they travel as kernel
// arguments so a launch needs no host-to-device copy and can be captured.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gsr.h"

namespace gsr {

constexpr int MAXV = GSR_MAX_VIEWS;
constexpr int MAXS = GSR_MAX_SETS;

constexpr int PROJ_BLOCK = 256;   // pairs per projection / compaction block
constexpr int SORT_THREADS = 256;
constexpr int SORT_ITEMS = 8;
constexpr int SORT_TILE = SORT_THREADS * SORT_ITEMS;  // keys per radix-sort block
constexpr int RADIX_BITS = 8;
constexpr int RADIX = 1 << RADIX_BITS;
constexpr int GRAD2D = 10;        // u, v, A, B, C, sigma, r, g, b, z
constexpr uint32_t CULLED = 0xFFFFFFFFu;
constexpr int MAX_ROWS = 512;     // tile rows per view (binning LDS arrays)
constexpr int MAX_COLS = 512;     // tile columns per view
constexpr int VIS_GRID = 8192;   // most workgroups of a kernel over visible pairs
// The grid of such a kernel whose items are at most `bound`: a multiple of 8.
inline int vis_grid(size_t bound) {
  return (int)((bound < (size_t)VIS_GRID ? bound : (size_t)VIS_GRID) + 7) / 8 * 8;
}
constexpr int MAX_CHUNK = 256;   // depth-sorted pairs per row-binning chunk
// Depth-sorted pairs per chunk where the plan leaves it open: small calls need many
// chunks to fill the device, large ones take longer runs per chunk.  Binning with
// 64 | 128 | 256, us: 8 views of 50k pairs 31 | 32 | 32, one of 600k 39 | 36 | 38, 8 of
// 130k 42 | 37 | 37, 48 of 25k 38 | 34 | 35, one of 1.5M 65 | 49 | 45, 8 of 200k 55 | 45 |
// 40, one of 3M 105 | 80 | 68.
inline int auto_chunk(long pairs) { return pairs <= 640000 ? 64 : pairs <= 1280000 ? 128 : 256; }
constexpr int RC_SUB = 4;        // row-binning chunks per counting workgroup
constexpr int SCHED_WORDS = 2 + 2 * 33;  // tile cursors + length-bucket counts (render.hip)
constexpr int GSR_MAX_DEVICES = 64;  // devices with a looked-up library-held buffer
constexpr long SEED_NOALLOC_MAX_POINTS = GSR_SEED_NOALLOC_MAX_POINTS;

// Pair p of view v is Gaussian (set_goff[view_set[v]] + p - pair_off[v]).
struct ProjTab {
  int nv;
  int P;                      // total pairs of the call
  int W, H, TX, TY;
  float itw, ith;             // 1 / tile width, height (exact: powers of two)
  int pair_off[MAXV + 1];
  int blk_off[MAXV + 1];      // PROJ_BLOCK-pair blocks per view, prefix
  int g_off[MAXV];            // first global Gaussian of the view's set
  int ns;                     // sets
  int set_goff[MAXS + 1];     // Gaussian offsets of the sets
  int set_gblk[MAXS + 1];     // PROJ_BLOCK-Gaussian blocks of the rendered sets, prefix
  int set_voff[MAXS + 1];     // views of each set in vset
  int vset[MAXV];             // view ids grouped by set (every view)
};

struct SortTab {
  int nv;
  int sblk_off[MAXV + 1];     // SORT_TILE blocks per view, prefix (upper bound)
};

// Whether the sort goes without scan kernels: each scatter block then walks its
// view's digit counts itself (1 KB a block of the view), which saves four launches
// and, in each pass, one workgroup's walk down the largest view.  A pass reads the
// sum over the views of (visible blocks)^2 KB that way; the host knows the bound of
// that sum, where all is visible.  Sort, without | with scan kernels, us:
//   all visible: one view of 1M pairs 125 | 137, 2M 224 | 211, 2.3M 296 | 231, 3M 420 |
//     281, 4M 665 | 350; 3 views of 1M 202 | 169, 4 253 | 194; 8 of 400k 156 | 146, of 800k
//     334 | 234; 48 of 85k 143 | 148;
//   half of it: one view of 2M 124 | 138, 2.3M 137 | 153; 3 of 1M 106 | 123, 4 120 | 130; 8
//     of 500k 100 | 110; a fifth: one of 3M 99 | 111, 3 of 1M 76 | 88.
// Most calls see a fifth to a half and gain 10 to 17 us; the line lies where one that
// sees all loses two or three times that.  Calls of more than 2048 blocks have more
// to sort than launches to save.
constexpr int FOLD_BLOCKS = 2048;
constexpr long FOLD_SQUARES = 750000, FOLD_PER_BLOCK = 250;
inline bool sort_folds(const SortTab& t) {
  long squares = 0, most = 0;
  for (int v = 0; v < t.nv; ++v) {
    const long b = t.sblk_off[v + 1] - t.sblk_off[v];
    squares += b * b;
    most = b > most ? b : most;
  }
  return t.sblk_off[t.nv] <= FOLD_BLOCKS && squares <= FOLD_SQUARES + FOLD_PER_BLOCK * most;
}

struct BinTab {
  int nv;
  int chunk;                  // pairs per chunk
  int TX, TY, T;              // tiles per view = T
  int cblk_off[MAXV + 1];     // chunks per view, prefix (upper bound)
};

struct SetTab {
  int ns, nv;
  int most;                   // grad-needing views of the set that has the most
  int set_goff[MAXS + 1];     // Gaussian offsets of the sets
  int set_blk[MAXS + 1];      // PROJ_BLOCK-Gaussian blocks per set, prefix
  int set_voff[MAXS + 1];     // views of each set in view_by_set
  int view_by_set[MAXV];      // view ids grouped by set (grad-needing only)
  int blk_off[MAXV + 1];      // PROJ_BLOCK-pair blocks per view, prefix (ProjTab's)
  int W, H;
};

// Pose sums of a backward call (context-owned, zero between calls): a share per
// XCD, with the count of its workgroups that have added theirs, and the count
// of shares that are complete.
struct PoseAcc {
  struct alignas(128) Share {
    double sum[6 * MAXV];
    unsigned int done;
  } share[8];
  unsigned int done;
};

struct SceneDev {
  const float* means;
  const float* log_scales;
  const float* quats;
  const float* opac;
  const float* colors;
  int sh_degree;
  int sh_stride;
};

struct CamDev {
  const float* viewmats;    // [V,12]
  const float* intrinsics;  // [V,4]
  float z_near;
  float bg0, bg1, bg2;
};

// Device header at the start of every saved-state buffer.
struct StateHeader {
  unsigned long long inst_total;  // (pair, tile) copies of the rects (reported only)
  unsigned int overflow;          // the row entries exceeded the capacity
  unsigned int vis_total;
  unsigned long long row_total;   // (pair, tile row) entries of the binning
  unsigned int vis_off[MAXV + 1]; // visible-pair offsets per view (compacted order)
  unsigned int pair_off[MAXV + 1]; // pair offsets per view (for the debug export)
};
constexpr size_t STATE_HEADER_BYTES = 1024;
static_assert(sizeof(StateHeader) <= STATE_HEADER_BYTES, "header");

// Byte offsets of the arrays inside a saved-state buffer (all 256-aligned).
struct StateLayout {
  size_t hdr, vmask, vbase, vkey, skey, rect, rec, order, row_rg, rows, torder, tfinal, last, total;
};

// Pointers into a saved-state buffer.
struct StateDev {
  StateHeader* hdr;
  // A view's pairs are cut into blocks of PROJ_BLOCK (ProjTab::blk_off); pair
  // 64 w + l of block b is visible iff bit l of vmask[4 b + w] is set, and
  // its position in the compacted visible list (view-major, pair order) is
  // vbase[b] plus the set bits before it in the block.
  unsigned long long* vmask;  // [4 blocks]
  uint32_t* vbase;    // [blocks]
  uint32_t* vkey;     // [Pv] by visible position: FP32 bits of camera z
  uint32_t* skey;     // [Pv] scratch of the forward: keys of the depth sort's odd passes
  uint2* rect;        // [Pv] by visible position: packed (x0 | y0 << 16, x1 | y1 << 16)
  float4* rec;        // [Pv][3] by visible position: (u, v, A', B'), (C', sigma, z, ex),
                      //   (r, g, b, ey)
  uint32_t* order;    // [Pv] visible positions in (view, depth, id) order
  uint2* row_rg;      // [V*TY] range of each (view, tile row) list in rows
  uint2* rows;        // [cap] row lists: (visible position, x0 | x1 << 16) in
                      //   (depth, id) order
  uint32_t* torder;   // [V*T] tiles by decreasing row-list length (persistent render)
  float* tfinal;      // [V*H*W]
  uint32_t* last;     // [V*H*W]
  unsigned long long cap;
};

// Binning workspace (context-owned).
struct BinWork {
  uint32_t* counts;     // [chunks][TY] per-chunk row counts -> exclusive bases
  uint32_t* row_tot;    // [V*TY] entries per (view, row)
  uint32_t* rect_lo;    // [P] the rects in depth order (rect.x and rect.y), in sort
  uint32_t* rect_hi;    //   buffers that the depth sort has done with
  unsigned long long* area_part;  // [<= VIS_GRID] (pair, tile) copies per counting workgroup
};

// SSIM: window, and the strips and rows of a call's workgroups.
constexpr int SS_R = 5;                // window radius
constexpr int SS_K = 2 * SS_R + 1;     // taps
constexpr int SS_W = SS_K + 3;         // inputs of four neighbouring outputs
constexpr int SS_MAXW = 4;             // waves per workgroup at most
// statistics and output columns of a workgroup of nw waves
constexpr int ss_stats(int nw) { return 4 * ((64 * nw - SS_W) / 4 + 1); }
constexpr int ss_out(int nw) { return 4 * ((ss_stats(nw) - SS_W) / 4 + 1); }
constexpr int SS_T = 32;               // tile edge the workspace is sized for
constexpr int SS_SIMDS = 1024;         // of the device
struct SsimShape {
  int nw, strips, rows;  // waves per workgroup, workgroups across, output rows of one
};
inline SsimShape ssim_shape(int nv, int W, int H) {
  SsimShape s{1, 0, SS_T};
  const auto strips_of = [&](int k) { return (W + ss_out(k) - 1) / ss_out(k); };
  // A call of few waves: a march's steps (four rows each, and three before the
  // first) follow one another, about 2 us each, so the rows are as few as fill the
  // SIMDs with one wave each, or with two where that, at 1.45 times the time a
  // step, takes less: one view of 64 x 64 9.7 us, of 320 x 240 13.0, of 640 x 480
  // 23.2.  Marches of 32 rows at least took 26, 28 and 30, and workgroups of 32 x
  // 32 pixels with all blurs through LDS 11.7, 12.6 and 31.
  const long waves32 = 3L * nv * strips_of(1) * ((H + SS_T - 1) / SS_T);
  if (waves32 <= SS_SIMDS) {
    s.strips = strips_of(1);
    double best = 0.0;
    for (int rows = 4; rows <= SS_T; rows += 4) {
      const long waves = 3L * nv * s.strips * ((H + rows - 1) / rows);
      if (waves > 2 * SS_SIMDS) continue;
      const double cost = (rows / 4 + 3) * (waves <= SS_SIMDS ? 1.0 : 1.45);
      if (best == 0.0 || cost < best) {
        best = cost;
        s.rows = rows;
      }
    }
    return s;
  }
  // waves per workgroup: the fewest waves over the strips of a row (each strip
  // recomputes two windows of columns), the larger workgroup on a tie (640
  // columns: 3 x 4 waves 463 us, 4 x 3 572, 7 x 2 534, 16 x 1 585, measured together)
  for (int k = 2; k <= SS_MAXW; ++k)
    if (k * strips_of(k) <= s.nw * strips_of(s.nw)) s.nw = k;
  s.strips = strips_of(s.nw);
  // rows per workgroup: it recomputes the statistics of 12 rows, so long marches
  // are cheaper, but about 8192 waves fill the chip (8 per SIMD); never below
  // SS_T rows (the partials then fit the workspace)
  const int waves = 3 * nv * s.strips * s.nw, most = (H + SS_T - 1) / SS_T;
  int segs = (8192 + waves - 1) / waves;
  segs = segs < 1 ? 1 : segs > most ? most : segs;
  const int rows = ((H + segs - 1) / segs + 3) / 4 * 4;
  s.rows = rows > SS_T ? rows : SS_T;
  return s;
}

// Sim(3) corrections: Gaussian set offsets, and the set of every view.
struct SimSetTab {
  int ns;
  long long off[MAXS + 1];
};
struct SimViewTab {
  int nv;
  int view_set[MAXV];
};

StateLayout state_layout(const gsr_plan_desc& p);
StateDev state_ptrs(void* base, const gsr_plan_desc& p);

// ------------------------------------------------------------------ launches
hipError_t launch_project_keys(const ProjTab& t, const SceneDev& sc, const CamDev& cam,
                               StateDev st, uint32_t* blk_cnt, hipStream_t s);
hipError_t launch_project_records(const ProjTab& t, const SceneDev& sc, const CamDev& cam,
                                  StateDev st, hipStream_t s);
hipError_t launch_compact(const ProjTab& t, StateDev st, const uint32_t* blk_cnt, hipStream_t s);
hipError_t launch_depth_sort(const SortTab& t, StateDev st, uint32_t* ka, uint32_t* va,
                             uint32_t* kb, uint32_t* vb, uint32_t* hist, uint32_t* off,
                             hipStream_t s);
hipError_t launch_binning(const BinTab& t, StateDev st, const BinWork& w, hipStream_t s);
// Compositing launch options (from the plan): list entries staged per lane
// in the forward (1 or 2) and in the backward (1, 2 or 4), tiles of a tile
// row per backward wave (1 or 2), and the persistent length-ordered tile
// queue instead of one wave per tile.
struct RenderCfg {
  int fwd_batch;
  int bwd_batch;
  int bwd_cols;
  bool persistent;
};
// Whether the tiles of a call (of `blocks` 8x8 blocks each) go to a workgroup each
// instead of a wave each, where the plan does not ask for the persistent queue.
// The workgroup form spends more instructions per entry and far less time per
// tile: it wins until its waves, one per block, fill the device a few times
// over, so the line lies at their number.  A tile of one or two blocks gains
// less from its workgroup and pays its barriers, so its line lies earlier.  One-wave
// form | workgroup form, us, of 300k Gaussians in 640x480 views (48,000 blocks are ten
// of them):
//   forward, 16x16: 1 view 67 | 37, 2 69 | 55, 6 130 | 131, 16 260 | 300;
//     32x16: 1 view 114 | 39, 6 150 | 145, 16 297 | 344; 16x8: 1 50 | 37, 2 60 | 59, 6
//     128 | 133; 8x8: 320x240 35 | 32, 640x480 41 | 41, 2 62 | 64, 6 143 | 157;
//   backward, 16x16: 1 view 121 | 80, 2 132 | 134, 6 270 | 343; 32x16: 1 view 164 | 97,
//     2 165 | 161, 1200x680 147 | 181, 6 256 | 412; 16x8: 1 130 | 112, 2 160 | 174; 8x8:
//     320x240 82 | 80, 640x480 188 | 204.
inline bool fwd_by_workgroup(long tiles, int blocks) {
  const long most = 5000L * blocks * blocks;
  return tiles * blocks <= (most < 40000 ? most : 40000);
}
inline bool bwd_by_workgroup(long tiles, int blocks) {
  const long most = 2500L * blocks;
  return tiles * blocks <= (most < 10000 ? most : 10000);
}
hipError_t launch_tile_order(int nv, int TX, int TY, StateDev st, unsigned int* sched,
                             hipStream_t s);
hipError_t launch_render_fwd(int nv, int W, int H, int TW, int TH, int TX, int TY,
                             const RenderCfg& rc, const CamDev& cam, StateDev st,
                             unsigned int* sched, float* color, float* depth, float* alpha,
                             int32_t* n_eval, hipStream_t s);
hipError_t launch_render_bwd(int nv, int W, int H, int TW, int TH, int TX, int TY,
                             const RenderCfg& rc, unsigned long long grad_mask,
                             const CamDev& cam, StateDev st, unsigned int* sched,
                             const float* g_color, const float* g_depth, const float* g_alpha,
                             float* grad2d, hipStream_t s);
// Debug only: the per-tile lists filtered from the row lists, first as
// counts per tile (tile_cnt [V*T]), then written at the tiles' offsets
// (ranges [V*T], from the counts' exclusive scan) into inst.
hipError_t launch_tile_lists(int nv, int TX, int TY, StateDev st, uint32_t* tile_cnt,
                             const uint2* ranges, uint32_t* inst, hipStream_t s);
hipError_t launch_count_blend(int nv, int W, int H, int TW, int TH, int TX, int TY, StateDev st,
                              const uint2* ranges, const uint32_t* inst, int32_t* n_blend,
                              hipStream_t s);
hipError_t launch_zero_pose(float* d_pose, int nv, unsigned int* bwd_next, hipStream_t s);
// Whether the projection backward has a loop for each of its two ways through the
// views (figures at the kernel), from the degree and the most views of a set.
inline bool bwd_by_two_loops(int sh_degree, int most) {
  return sh_degree == 0 || (sh_degree == 2 && most > 4) || (sh_degree == 3 && most > 12);
}
hipError_t launch_project_bwd(const SetTab& t, const SceneDev& sc, const CamDev& cam,
                              StateDev st, float* grad2d, PoseAcc* pa,
                              const gsr_grads& g, hipStream_t s);
hipError_t launch_pose_delta(const float* vin, const float* delta, float* vout, int nv,
                             hipStream_t s);
hipError_t launch_sim3_gaussians(const SimSetTab& tab, const float* m_in, const float* ls_in,
                                 const float* q_in, const float* sims, float* m_out,
                                 float* ls_out, float* q_out, hipStream_t s);
hipError_t launch_sim3_views(const SimViewTab& tab, const float* vin, const float* sims,
                             float* vout, hipStream_t s);
hipError_t launch_l1_grad(int nv, int HW, const float* color, const float* depth,
                          const float* tcol, const float* tdep, const float* expo, float w_col,
                          float w_dep, float* g_col, float* g_dep, float* g_expo, hipStream_t s);
size_t dedup_workspace_bytes(long long slots);
hipError_t launch_dedup(long long slots, void* ws, double v, double kenv, const float* tm,
                        const float* tls, long long n_tgt, const float* depth, const float* vms,
                        const float* intr, int nk, int W, int H, const float* sm, long long n_src,
                        uint8_t* keep, hipStream_t s, unsigned int** counters);
size_t ssim_workspace_bytes(int nv, int W, int H);
hipError_t launch_ssim(int nv, int W, int H, float weight, const float* color,
                       const float* target, const float* expo, void* ws, float* d_color,
                       float* d_expo, float* ssim_out, hipStream_t s);
hipError_t launch_prune(long n, const SceneDev& in, int color_stride, float thr,
                        const SimSetTab& sets, uint32_t* blk, long long* bounds, float* m,
                        float* ls, float* q, float* o, float* col, hipStream_t s);
// exclusive scan of nb block counts in place, total at blk[nb] (one workgroup)
hipError_t launch_block_scan(int nb, uint32_t* blk, hipStream_t s);
hipError_t launch_iso_grad(long n, const float* ls, float w, float* g, hipStream_t s);
hipError_t launch_normal_grad(int nv, int W, int H, const float* depth, const float* prior,
                              const float* intr, float w, float* g_dep, hipStream_t s);
hipError_t launch_seed(int W, int H, int stride, const float* depth, const float* color,
                       const float* vm, const float* intr, float opac_logit, long max_out,
                       uint32_t* blk, int64_t* n_out, float* m, float* ls, float* q, float* o,
                       float* c, hipStream_t s);
hipError_t launch_adam(const gsr_adam_group* gr, int ng, double b1, double b2, double eps,
                       int32_t* step, hipStream_t s);
hipError_t seed_scratch(uint32_t** out);

// Device scratch of one host call that synchronises before it returns.
constexpr int CALL_SLOTS = 4;
constexpr size_t CALL_SLOT_BYTES = 256 * 1024;
struct CallScratch {
  void* ptr = nullptr;
  int dev = -1, slot = -1;
  hipError_t get(size_t bytes);
  ~CallScratch();
};

}  // namespace gsr
