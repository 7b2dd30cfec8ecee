// Internal declarations shared by the libdop host code and its HIP kernels.
#ifndef DOP_INTERNAL_H_
#define DOP_INTERNAL_H_

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/dop.h"

namespace dop {

// Size of the shared twiddle table: W[j] = exp(-2 pi i j / kTwN).
constexpr int kTwLog = 17;
constexpr int kTwN = 1 << kTwLog;

// Grids 2^kTriMinLM .. 2^kTriMaxLM that the three-pass path of a half-filled
// plane covers.  Behind the shared table the context keeps, per such grid,
// the path's cross twiddles exp(-2 pi i p j / M) at [p - 1][j], p = 1..8,
// j < M / 16: M / 2 entries from index tri_tw_offset(log2 M).
constexpr int kTriMinLM = 12;
constexpr int kTriMaxLM = 14;
constexpr int tri_tw_offset(int lm) { return kTwN + (1 << (lm - 1)) - (1 << (kTriMinLM - 1)); }
// Then omega_L^i, i < L, of the axis lengths that are no power of two and
// take the small-grid path, from axis_tw_offset(L).
constexpr int kAxisLengths[] = {240, 720, 1440, 2144, 3600, 5360};
constexpr int axis_tw_offset(int l) {
  int at = tri_tw_offset(kTriMaxLM + 1);
  for (int a : kAxisLengths) {
    if (a == l) return at;
    at += a;
  }
  return at;
}
// Last, the three-pass path's cross twiddles of 3600^2.
constexpr int kTri3600Tw = axis_tw_offset(0);
constexpr int kTwTotal = kTri3600Tw + 3600 / 2;

// Wavelengths per group: pass A forms, and pass A' accumulates, up to this
// many fields (one workspace field each) per launch.
constexpr int kMaxGroup = 4;

// Row pitch of the M x M workspace, in elements: M + kRowPad.  The pad keeps
// rows that are a power of two apart from landing on the same HBM channels
// (column passes read hundreds of rows at one column offset).
constexpr int kRowPad = 16;

// Pass-A input modes.
enum InMode : int {
  IN_PHASE = 0,  // E = amp * exp(i 2 pi (n-1)/lambda h)        (Eq. 1-2)
  IN_FIELD = 1,  // caller's complex field
  IN_GRAD = 2    // g_U = 2 w_k G * U_k (adjoint seed)
};

// Last-pass output modes.
enum OutMode : int {
  OUT_PSF = 0,    // psf (+)= w_k |U|^2                          (Eq. 4)
  OUT_FIELD = 1,  // complex U
  OUT_GRADH = 2   // grad_h (+)= c_k Im(g_E conj(E_k))
};

// The passes an operation takes: the five digit passes of asm_kernels.hip, or
// three passes over whole rows and columns (small_grid.hip, three_pass.hip).
enum Route : int { ROUTE_FIVE = 0, ROUTE_SMALL = 1, ROUTE_TRI = 2 };

// Everything one wavelength's passes need.  Passed by value.
struct KParams {
  float2 *ws;            // My x Mx c64 workspace (row pitch Mx + kRowPad)
  const float2 *tw;      // twiddle table, kTwN entries
  const float2 *tw3;     // cross twiddles of this grid (three-pass path)
  int pitch3;            // items from one group of column pairs to the next (three-pass path)
  int n;                 // DOE columns Nx (row length of every N-wide array)
  int plan;              // plan id of the grid (plan_id)
  int route;             // Route of the operation
  int nrows_in;          // rows of the padded input that may be nonzero
  int nrows_out;         // rows of the output plane that are needed
  int p0x, p0y;          // (Mx - Nx) / 2, (My - Ny) / 2
  int in_mode, out_mode;
  int full;              // 1: output the whole M x M plane (centred)
  int first;             // 1: overwrite the accumulator, 0: add to it
  const float *h;        // heights (IN_PHASE, OUT_GRADH): row y, column x of
                         // the Ny x Nx map is h[(y >> up_log2) * nh + (x >> up_log2)]
  int up_log2;           // log2 of the nearest-neighbour upsampling factor
  int nh;                // row length of h: Nx >> up_log2
  const float *amp;      // N x N amplitude or NULL
  const float2 *u_in;    // N x N field (IN_FIELD)
  const float2 *saved_in;// N x N field U_k (IN_GRAD)
  const float *gpsf;     // N x N dL/dPSF (IN_GRAD)
  float *psf;            // OUT_PSF destination
  float2 *u_out;         // OUT_FIELD destination
  float2 *saved_out;     // optional N x N copy of U_k (OUT_PSF, crop)
  float *grad_h;         // OUT_GRADH destination
  double phase_turns;    // (n_k - 1) / lambda_k  (turns of phase per unit h)
  double zl;             // z / lambda_k (turns at normal incidence); -z / lambda_k
                         // for the adjoint, whose transfer function is conj(H)
  double lam;            // lambda_k
  double inv_mdx;        // 1 / (Mx dx)
  double inv_mdy;        // 1 / (My dx)
  double flim_x;         // band limit on |fx| (infinity: none)
  double flim_y;         // band limit on |fy| (infinity: none)
  float wk_m4;           // w_k / (My Mx)^2: PSF weight times the squared
                         // 1/(My Mx) of the inverse DFT, which the passes
                         // leave to the output
  float two_wk;          // 2 w_k
  float ck_m2;           // 2 pi (n_k - 1) / lambda_k / (My Mx)
  float inv_m2;          // 1 / (My Mx) (inverse-DFT normalisation of output fields)
  int group;             // wavelengths in this launch of pass A (IN_PHASE) or A'
                         // (OUT_PSF, no saved fields): 1, or 2..kMaxGroup with
                         // their fields field_elems apart and the per-wavelength
                         // constants below
  size_t field_elems;    // elements from one field of a group to the next
  double phase_turns_g[kMaxGroup];
  float wk_m4_g[kMaxGroup];
  // the rest of a wavelength's constants, for the small-grid path's groups
  // (set for a group of one as well)
  double lam_g[kMaxGroup], zl_g[kMaxGroup], flim_x_g[kMaxGroup], flim_y_g[kMaxGroup];
  float two_wk_g[kMaxGroup], ck_m2_g[kMaxGroup];
};

constexpr int kNumPasses = 5;

// Route of an operation (by its input mode) on a valid problem (dop_api.cpp).
Route route_of(const dop_problem *prob, InMode in);

// Enqueue passes first..last (0 = A, 1 = B, 2 = C, 3 = B', 4 = A') of `p`;
// ev (if not NULL) gets last - first + 2 marks around them.
hipError_t launch_passes(const KParams &p, int first, int last, hipStream_t stream,
                         hipEvent_t *ev);

// Small-grid path (small_grid.hip): square power-of-two grids of
// 2^kSmallMinLM .. 2^kSmallMaxLM points per side, and the table grids whose
// rows and columns fit a block, run an operation as three passes: rows,
// columns with H, rows.  small_path says whether an operation takes them, from
// its plan id, its input mode, the rows of its first and last pass together
// and its wavelengths (1 for fields); small_max_group(plan) says how many
// wavelengths a launch takes at most;
// launch_small enqueues the three passes of p.group wavelengths (PSF and
// gradient; 1 for fields).  ev (if not NULL) gets p.group + 3 marks: before
// the first pass, after it, after each field's column pass (launched one by
// one then) and after the last pass.
constexpr int kSmallMinLM = 4;
constexpr int kSmallMaxLM = 11;
bool small_path(int plan, InMode in, int rows, int n_lambda);
int small_max_group(int plan);
hipError_t launch_small(const KParams &p, hipStream_t stream, hipEvent_t *ev);

// Three-pass path of a half-filled plane (three_pass.hip): tri_path says
// whether a problem takes it, from its plan id, DOE (n columns, rows rows) and
// window; tri_pitch
// gives KParams::pitch3 for a number of rows; launch_tri enqueues one
// wavelength in any input and output mode, with ev[0..3] (if not NULL)
// recorded before, between and after its passes, and refuses any other
// problem or group.  It needs the workspace of one field.
int tri_grid(int plan);  // points per side if the plan may take the path, else 0
bool tri_path(int plan, int n, int rows, bool full);
int tri_pitch(int plan, int nrows);
hipError_t launch_tri(const KParams &p, hipStream_t s, hipEvent_t *ev);

// Largest wavelength group of the plan's five passes (1 if pass A' ends in a
// radix-67 stage).
int plan_max_group(int plan);

// Plan id of the My x Mx grid (mx columns, my rows): log2(M) for a square
// power of two M in [16, 131072], a larger id for each grid of the plan
// table, -1 if the grid has no plan.
int plan_id(int mx, int my);

// The grids of the plan table (square grids that are not powers of two,
// and rectangular grids): writes up to `max` (rows, columns) pairs and
// returns how many there are.
int table_grids(int *rows, int *cols, int max);

// Bandwidth probes (dop_probe_bandwidth): pass C's access pattern without its
// arithmetic on the power-of-two grid of plan id `plan` (14..17), and plain
// 16-byte stream kernels over n16 16-byte vectors.  Arguments already
// validated.
hipError_t launch_probe_passc(int plan, float2 *ws, float scale, hipStream_t stream);
hipError_t launch_probe_stream(int kind, void *buf, size_t n16, float scale, hipStream_t stream);

// Super-resolved front end: fine = Wy coarse Wx^T and its adjoint for a
// coarse design of ncy rows and ncx columns (kind 0: nearest, 1: Lanczos-3;
// see dop_upsample).  Arguments already validated.
hipError_t launch_upsample(int kind, int ncy, int ncx, int s, const float *coarse, float *fine,
                           hipStream_t stream);
hipError_t launch_upsample_adjoint(int kind, int ncy, int ncx, int s, const float *grad_fine,
                                   float *grad_coarse, hipStream_t stream);

}  // namespace dop

#endif  // DOP_INTERNAL_H_
