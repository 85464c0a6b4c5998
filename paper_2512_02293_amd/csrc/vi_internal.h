// Internal structures of the visual-inertial step library: the per-batch plan
// (index tables built on the host from the windows' frame graphs), the
// per-window device descriptors, the workspace carve, and the kernel launchers
// shared by the translation units.
//
// A call solves a batch of independent windows (a single-window call is a
// batch of one).  Keyframes, edges and IMU factors of all windows are numbered
// globally (window after window); per-window quantities (map size, intrinsics,
// the caller's arrays, the reduced system) are reached through the window
// descriptor of the keyframe, edge or factor.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <string>
#include <vector>

#include "../../include/vi_ba.h"

namespace vi {

constexpr int kMaxOutDegree = 18;     // per-source outgoing edges (Gram tile budget)
constexpr int kVisBlock = 256;        // pixels per workgroup of the per-pixel kernels
constexpr int kCholNB = 32;           // Cholesky tile size
constexpr int kCholSmallMaxNpad = 512;  // systems up to this size are solved by one workgroup
constexpr int kPairTicketFlag = 1 << 30;  // Cholesky ticket of tile (j + 1, j) that also factors tile (j + 1, j + 1)
constexpr int kMaxIters = 64;         // cost trace capacity of vi_ba_solve
constexpr int kMaxKeyframes = 640;    // per window: the matrix of the reduced system is stored whole
constexpr int kTraceLen = 2 * (kMaxIters + 1);

// Velocity / bias unknowns ("V", 9 per keyframe) are eliminated before the
// reduced system is formed.  Only inertial factors touch them, so their block
// of the normal equations is block tridiagonal along the keyframes.  The
// keyframes are cut into segments by separator keyframes; the V of the
// keyframes inside a segment are eliminated (k_cond.h), the V of the
// separators stay in the reduced system beside their poses.
//  * A segment couples all of its poses and its two chains run one keyframe
//    after the other, so a window is cut about every kCondSpan keyframes (40 x
//    56 maps, 4 iterations, the whole window as one segment -> cut: 28
//    keyframes 785 -> 619 us with 6 edges per source and 890 -> 815 with 15; 16:
//    541 -> 515).  Shorter spans keep more unknowns: about every 6 instead of
//    every 12, 128 keyframes take 2156 instead of 2055 us; every 24, 48 take 937
//    instead of 865.
//  * A separator that fits the padding of the last tile of the reduced system
//    costs nothing there and halves a chain, so more are taken while segments
//    keep kCondMinLen keyframes (12 keyframes: 513 -> 465 us; at 6, segments of
//    3 and 2 keyframes, 443 -> 449).
//  * The elimination takes 6 to 12 us an iteration in windows of up to 7
//    keyframes, with one bias for the window 14 to 18, and saves the
//    factorisation 8 to 10 for each tile column that the reduced system is
//    shorter by.  Where it saves too few, every keyframe keeps its V (a
//    separator): us of a call of 8 iterations, all kept / eliminated, 40 x 56
//    maps: 2 keyframes (no column saved) 495 / 558, 3 (one) 578 / 566, 4 (one)
//    583 / 591, 6 (one) 665 / 701, 5 (two) 663 / 594, 7 (two) 741 / 682; with one
//    bias 3 (one) 581 / 621, 4 (none) 590 / 715, 6 (one) 675 / 741, 7 (two) 749 /
//    734, 8 (two) 753 / 752.
constexpr int kCondSpan = 12;
constexpr int kCondMinLen = 3;
constexpr int kCondNV = 9;
constexpr bool cond_pays(int N, bool bias_global, int tiles_saved) {
  return tiles_saved > 1 || (tiles_saved == 1 && !bias_global && N <= 3);
}
// Device status word of one window: first error (vi_status), its detail (e.g.
// pivot index), the number of committed steps, whether the tolerance stopped it,
// and what the elimination of velocities and biases found (elim).  That runs
// beside the vision assembly, ahead of the checks whose place its own have in
// the order of errors (a non-finite entry with the assembly's, a pivot with the
// factorisation's), so it is kept apart: kElimNonfinite or kElimPivot, plus
// kElimPivot - 1 minus the coordinate (keyframe * 15 + unknown), the largest
// kept; 0: nothing.  32 bytes, so that it is found by a shift: with 20 every
// launch paid for it (inertial initialisation 1037 -> 1050 us).
constexpr int kElimPivot = 1 << 20, kElimNonfinite = 1 << 21;
struct alignas(32) DevStatus {
  int code;
  int detail;
  int iters;
  int conv;      // tolerance stop reached: the window takes no further step
  int elim;
};

// Per-window device descriptor.
struct WinDev {
  double fx, fy, cx, cy, g[3];
  double Rbc[9], tbc[3];             // camera-IMU extrinsic (body-from-camera), row-major rotation
  int ext;                           // 1: T_bc is not the identity (vision terms go through it)
  int H, W, HW, N;
  int kf_base, e_base, f_base, F;    // global index of the first keyframe / edge / factor
  int nkr;                           // pixel ranges per source in the fused assembly + Gram
  int n, npad, nblk;                 // reduced system
  int pair_base;                     // offset of this window's pair table
  int flag_off, nflags;              // Cholesky tile flags [(nblk + 1) * nblk]
  int band;                          // tiles (i, j) with i - j > band are zero in S and in L
  int seg_base, nseg;                // segments of eliminated velocity / bias unknowns
  int tab_off;                        // dataflow path: offset of its block-column table in chol_tab
  long long pix_base;                // global offset of the first keyframe's first pixel
  long long A_off, Linv_off, x_off;  // reduced system, diagonal-tile inverses, solution
  double* pose;
  double* vel;
  double* bias;
  double* invdepth;                  // FP64 inverse depths, or null when they are FP32:
  float* invdepth32;                 // FP32 inverse depths (mixed precision), or null
  const float* target;
  const float* weight;
  const vi_preint* imu;
  double* rep_dxi;
  double* rep_dd;
  // pose-graph adjustment in Sim(3) (null / 0 for the visual-inertial step)
  double* scale;                     // [N] keyframe scales s (X_w = s R X_c + p), updated in place
  const double* rel_meas;            // [n_rel][8] measured E_ij = T_j^-1 T_i: t (3), q (4), s
  const double* rel_info;            // [n_rel][49] information, (rotation, translation, log-scale) order
  int rel_base, n_rel;               // global index of the window's first relative-pose factor
};

// One segment of eliminated velocity / bias unknowns: the V of keyframes a..b
// (window indices).  Its columns are the unknowns of the reduced system that
// they couple with: the poses of keyframes k0..k1 (the segment and its
// neighbours), the V of the separators a - 1 and b + 1 where there are any
// (columns vl.., vr..), with one global bias also its 6 unknowns (columns gb..,
// inside vr.. where the last keyframe is the right neighbour), and last (nc)
// the right-hand side.
struct SegDev {
  int32_t w, a, b, k0, k1, nc, ld;   // ld: columns rounded up to the 16 x 16 tiles of its Gram
  int32_t vl, vr, gb;                // first column of each, -1: none
  int32_t nf;                        // inertial factors that touch it
  int32_t pad;
  int64_t y_off, l_off, g_off;       // Y (9 per keyframe x ld), factors (162 per keyframe), Gram (ld x ld)
};
// 16 x 16 tiles along a side of the Gram of a source with k outgoing edges:
// 6 k rows, or with w_d one more
constexpr int vis_tiles_T(int k, bool wd_row) { return (6 * k + (wd_row ? 16 : 15)) / 16; }
constexpr int kSegGramTiles = 16;    // Gram tiles per workgroup (one per wave)

// Host-built description of one batch.
struct Plan {
  int n_win = 0;
  int N = 0, E = 0, F = 0;       // totals over the batch
  int kmax = 0;
  int nkr_max = 0;               // max pixel ranges per source
  int hw_max = 0;
  int nblk_max = 0;
  int range = 320;               // pixels per workgroup of the fused kernel
  long long pix_total = 0;       // sum over keyframes of H*W
  std::vector<WinDev> win;       // pointers filled per call
  // host tables
  std::vector<int32_t> ii, jj;                 // global keyframe indices per global edge
  std::vector<int32_t> win_of_kf, win_of_f;
  std::vector<int32_t> src_off, src_edges;     // CSR of edges by source keyframe
  std::vector<int32_t> gram_off, z_off, zb_off;
  std::vector<int32_t> pair_off, pair_z, pair_zb;
  std::vector<int32_t> chol_tiles;             // ticket -> (window, (i << 16) | j)
  // order of each window's reduced system: keyframe a (window index) has its
  // unknowns from row kf_off[kf_base + a] on (6 pose unknowns, all 15 for a
  // separator, 7 in the pose graph); row_map[x_off + r] = (a << 8) | unknown of
  // row r, -1 in the padding
  std::vector<int32_t> kf_off, row_map;
  std::vector<SegDev> segs;
  std::vector<int32_t> kf_seg;                 // [2 N] segments whose columns hold the keyframe's pose (-1: none)
  std::vector<int32_t> f_seg;                  // [F] segment that eliminates with the factor, -1: between two separators
  std::vector<int32_t> gram_map;               // (segment, first Gram tile) per workgroup of the segments' Grams
  int cond_len = 0;                            // keyframes of the longest segment
  // per window of the dataflow path: chain order of the block columns, the ends
  // and beginnings of the k-loops in it, bits of the nonzero tiles (build_plan)
  std::vector<int32_t> chol_tab;
  int pdim = 15;                               // unknowns per keyframe: 15 (visual-inertial) or 7 (Sim(3) graph)
  int R = 0;                                   // relative-pose factors (pose-graph adjustment)
  std::vector<int32_t> rel_ii, rel_jj;         // global keyframe indices per factor
  std::vector<int32_t> rel_z, rel_zb;          // offsets of each factor's four 7x7 blocks in Z and its 14 in ZB/ZV
  int n_tickets = 0;
  int n_bs = 0;                                // back-substitution columns after the tiles in chol_tiles
  size_t flags_size = 0;
  size_t gram_size = 0, z_size = 0, zb_size = 0;
  size_t A_size = 0, Linv_size = 0, x_size = 0;
  size_t cond_size = 0;                        // doubles of Y, factors and Grams of all segments
  size_t seg_cap = 0;                          // arrival counters of the segments
};

// Device pointers into the plan upload.
struct DevPlan {
  const int32_t *ii, *jj, *win_of_kf, *win_of_f, *src_off, *src_edges;
  const int32_t *gram_off, *z_off, *zb_off;
  const int32_t *pair_off, *pair_z, *pair_zb;
  const int32_t* chol_tiles;
  const int32_t *rel_ii, *rel_jj, *rel_z, *rel_zb;
  const int32_t *kf_off, *row_map, *chol_tab;
  const int32_t *kf_seg, *f_seg, *gram_map;
  const SegDev* segs;
  const WinDev* win;
};

// Workspace carve (device pointers into the caller's workspace).
struct Work {
  double* Rw;        // [N][9]
  double* rel;       // [E][12]  R_ji (9), t_ji (3)
  double* Cd;        // [pix_total]  C + eta
  double* wd;        // [pix_total]
  double* hpart;     // [E][nkr_max][32]
  double* vcost;     // [N][ncost][2]  vision cost / valid count partials
  double* gpart;     // Gram partials
  double* Z;         // per source (k+1)^2 * 36
  double* ZB;        // per source 6 (k+1)
  double* ZV;        // per source 6 (k+1)
  double* Lam;       // [F][225]
  double* Hf;        // [F][900]
  double* gf;        // [F][30]
  double* icost;     // [F]
  double* A;         // per window [(npad + NB) * npad]  reduced matrix (+ augmented rhs row)
  int32_t* flags;    // Cholesky tile flags of all windows
  int32_t* sync;     // [0] ticket counter, [1] abort flag
  double* Linv;      // per window [nblk][NB*NB]
  double* x;         // per window [npad]
  double* trace;     // [n_win][kTraceLen]  cost, n_valid per slot
  double* rcost;     // [R]  relative-pose factor costs (pose-graph adjustment)
  double* cond;      // eliminated unknowns: Y, factors and Gram of every segment
  int32_t* seg_cnt;  // [segments] inertial factors linearised so far (zero between launches)
};

struct OptsDev {
  int n_fixed, use_imu, bias_fixed, precision;
  double lambda, eta, z_min, d_min;
  double tol;        // relative cost decrease below which a window stops (0: never)
  int bias_global;   // one bias per window, in the last keyframe's slot (with use_imu)
};

// learned warm-start network (k_wnet.hip)
constexpr int kWCin = 15, kWCinPad = 16, kWC = 32, kWLayers = 4;
constexpr int kWParams = kWC * kWCin * 9 + kWC + 3 * (kWC * kWC * 9 + kWC) + kWC * 9 + 1 + 6 * kWC + 6;
constexpr int kWHQMax = 16, kWWQMax = 24;       // canvas of 4x4-pixel cells (maps up to 64 x 96)
constexpr float kWSd = 0.02f;                   // inverse-depth correction scale of the loss

// partial-sum slots per source in the cost / Hessian partial arrays
inline int cost_slots(const Plan& P) {
  return std::max(P.nkr_max, (P.hw_max + kVisBlock - 1) / kVisBlock);
}

// kernel launchers (enqueue on `s`)
void launch_preint(hipStream_t s, int F, const int32_t* off, const double* gyro,
                   const double* accel, const double* dt, const double* bias_hat,
                   vi_imu_noise noise, vi_preint* out, DevStatus* st);
void launch_imu_info(hipStream_t s, const Plan& P, const DevPlan& D, double* Lam, DevStatus* st);
void launch_predict_kf(hipStream_t s, int n, const double* pose_i, const double* vel_i, const double* bias_i,
                       const vi_preint* imu, const double* g, double tau, double* pose_j, double* vel_j,
                       double* bias_j, int32_t* used);
// Stages of one step, for per-stage event timing.
enum Stage { kStVis = 0, kStLocal, kStAssemble, kStChol, kStBacksub, kNumStages };
// `mark`, when non-null, is called between stages (used to record timing events).
typedef void (*StageMark)(void* user, int stage_done);
void launch_step(hipStream_t s, const Plan& P, const DevPlan& D, const Work& w, const OptsDev& o, int iter,
                 DevStatus* st, StageMark mark = nullptr, void* mark_user = nullptr);
// the first two stages only (autotuning of the assembly tiling)
void launch_tune_stages(hipStream_t s, const Plan& P, const DevPlan& D, const Work& w, const OptsDev& o,
                        StageMark mark, void* mark_user);
// also clears the arrival counters of the segments (cnt, ncnt)
void launch_reset_status(hipStream_t s, DevStatus* st, int n, int32_t* cnt = nullptr, int ncnt = 0);
// dd / db (optional): warm-start corrections (cells [n][HQ][WQ], [n][6]) applied
// to the state first, so that the cost is that of the corrected state
void launch_final_cost(hipStream_t s, const Plan& P, const DevPlan& D, const Work& w, const OptsDev& o,
                       int slot, double* trace = nullptr, const float* dd = nullptr, const float* db = nullptr,
                       int HQ = 0, int WQ = 0, double d_min = 0.0);   // trace: w.trace unless given
void launch_chol(hipStream_t s, const Plan& P, const DevPlan& D, const Work& w, DevStatus* st);
// the fused vision assembly alone (no inertial workgroups) and the vision cost
// of the current state (vcost in ranges of kVisBlock pixels)
void launch_vis_assembly(hipStream_t s, const Plan& P, const DevPlan& D, const Work& w, const OptsDev& o,
                         DevStatus* st);
void launch_vis_cost(hipStream_t s, const Plan& P, const DevPlan& D, const Work& w, const OptsDev& o);
// pose-graph adjustment in Sim(3) (k_pgba.hip)
size_t pg_local_lds(int kmax);
void pg_set_attributes();
int vis_wd_row(const Plan& P, const OptsDev& o);
void launch_pg_local(hipStream_t s, const Plan& P, const DevPlan& D, const Work& w, const OptsDev& o, DevStatus* st);
void launch_pg_relpose(hipStream_t s, const Plan& P, const DevPlan& D, const Work& w, DevStatus* st, bool jac);
void launch_pg_assemble(hipStream_t s, const Plan& P, const DevPlan& D, const Work& w, int n_fixed, double lambda,
                        DevStatus* st);
void launch_pg_backsub(hipStream_t s, const Plan& P, const DevPlan& D, const Work& w, const OptsDev& o,
                       DevStatus* st);
void launch_pg_cost(hipStream_t s, const Plan& P, const DevPlan& D, const Work& w, int ncost, int range_px,
                    int slot, double tol, DevStatus* st);
void step_set_attributes(int kmax, int cond_len);
// warm start
void wnet_set_attributes();
// wprep (optional device scratch of wnet_prep_bytes()): the layers' weights are
// converted to their LDS image once per call instead of once per image
void launch_wnet_forward(hipStream_t s, int n, int HQ, int WQ, const int* dims, const float* theta, const float* feat,
                         void* act, float* dd, float* db, void* wprep = nullptr);
size_t wnet_prep_bytes();
void launch_wnet_backward(hipStream_t s, int n, int HQ, int WQ, const int* dims, const float* theta, const void* act,
                          const float* dd, const float* db, const float* lab_dd, const float* lab_db, float nv,
                          float* g_dd, float* g_db, float* loss, float* partial, float* grads);
// inertial-only initialisation (k_iinit.hip): one descriptor per problem, in the workspace
struct IInitDesc {
  int N;
  int pad;
  const double* pose_vis;
  const vi_preint* imu;
  double* vel;
  double* bias;
  double* rot_wg;
  double* log_scale;
  double* cost;
  double* wf;            // whitening scratch [N-1][87]
};
constexpr int kIInitMaxKeyframes = 32;
size_t iinit_lds_bytes(int N);
size_t iinit_whiten_doubles(int N);
void launch_inertial_init(hipStream_t s, int n, const IInitDesc* descs, int max_n_kf, double G, double lambda,
                          int iters, DevStatus* status);

// loop-closure update of a Gaussian map (k_gauss.hip)
size_t reanchor_table_bytes(int n_kf);
// allocation-free variant: the keyframe table in a file-scope device array of
// k_gauss.hip.  reanchor_scratch_init (with `device` current) looks up that
// array's address on the device once; reanchor_scratch returns it (nullptr
// before a successful init).
int reanchor_noalloc_max_keyframes();
hipError_t reanchor_scratch_init(int device);
void* reanchor_scratch(int device);
int64_t reanchor_max_gaussians();
void launch_reanchor(hipStream_t s, int n_kf, const double* pose_pre, const double* pose_post, const double* ds,
                     void* table, int64_t K, const int32_t* anchor, const float* mean_in, const float* cov_in,
                     float* mean_out, float* cov_out, int* n_rej);

void launch_wnet_adamw(hipStream_t s, int P, float* theta, const float* g, float* m, float* v, int t, float lr,
                       float b1, float b2, float eps, float wd);
void launch_warm_features(hipStream_t s, const Plan& P, const DevPlan& D, const OptsDev& o, int HQ, int WQ,
                          float* feat, int* dims, double* saved_d = nullptr,
                          double* saved_b = nullptr);
void launch_warm_apply(hipStream_t s, const Plan& P, const DevPlan& D, int HQ, int WQ, const float* dd,
                       const float* db, double d_min, int apply_bias);
void launch_warm_state(hipStream_t s, const Plan& P, const DevPlan& D, double* saved_d, double* saved_b,
                       const double* trace, int restore);

}  // namespace vi
