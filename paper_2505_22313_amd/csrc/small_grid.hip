// Small-grid path: whole rows and columns in LDS, three passes.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "asm_device.h"
#include "asm_stages.h"
#include "dop_internal.h"

namespace dop {

// ---------------------------------------------------------------------------
// Small-grid path (square power-of-two M up to 2048, and the grids of the table
// whose rows and columns fit a block), three passes:
//   S1: M-point DFT over x of each of the N input rows (formed on the fly:
//       DOE field from h, Eq. 1-2, caller's field or adjoint seed), written
//       in natural frequency order;
//   S2: for a run of columns, M-point DFT over y (rows >= N are zeros and not
//       read), times H (Eq. 3), inverse DFT over y; only the rows the output
//       needs are written back;
//   S3: inverse M-point DFT over kx of those rows, then the output stage
//       (|U|^2 accumulated into the PSF with the wavelength weight, Eq. 4,
//       and the optional saved field; field; or height gradient).
// A whole row or column fits in a block, so the 2-D FFT takes two sweeps
// instead of the large path's digit passes, and the column pass touches
// only the N rows that hold data.  At these sizes the field (34 MB at 2048^2,
// 104 MB at 3600^2) stays in the 256 MB Infinity Cache between passes, and the
// five large-path launches were latency-bound.  At 4096 the column pass,
// limited to two columns (16-byte runs) by the LDS, was twice as slow as the
// large path; three-column tiles fit at 3600 rows.
// ---------------------------------------------------------------------------
// Tiles of the grids of table_plan that take the path (c = 0: the others).
// PSF of one and of four wavelengths, gradient step of one (us per call), five
// passes -> three: 240^2 25, 137, 55 -> 17, 22, 38; 720^2 30, 140, 65 -> 24,
// 41, 47; 1440^2 56, 172, 112 -> 40, 88, 81; 2144^2 149, 618, 306 -> 112,
// 457, 229; 512 x 2048 33, 135, 68 -> 29, 58, 57; 5360 x 240 60, 198, 120 ->
// 52, 105, 105.  3600^2 takes them for some operations (small_path).  3072^2
// was no faster (118, 443, 240 against 120, 491, 247: one 123 KB column tile
// per CU) and keeps the five passes, as do the grids whose columns do not fit.
struct SmallTab {
  int rb, tr;  // rows per S1 / S3 tile and threads (per wavelength of a group)
  int c, tc;   // columns per S2 tile and threads
  bool group;  // whether S1 / S3 tiles of four wavelengths fit
};
__host__ __device__ constexpr SmallTab small_tab(int i) {
  return i == 0    ? SmallTab{4, 64, 4, 64, true}       // 240^2
         : i == 1  ? SmallTab{2, 128, 4, 192, true}     // 720^2
         : i == 2  ? SmallTab{1, 192, 4, 768, true}     // 1440^2
         : i == kTab3600 - kTabBase ? SmallTab{1, 256, 3, 768, false}
         : i == 7  ? SmallTab{1, 320, 4, 512, false}    // 2144^2
         : i == 8  ? SmallTab{4, 64, 4, 192, true}      // 720 x 240
         : i == 9  ? SmallTab{1, 128, 4, 256, true}     // 512 x 2048
         : i == 10 ? SmallTab{1, 320, 8, 128, false}    // 240 x 2144
         : i == 11 ? SmallTab{4, 64, 2, 704, true}      // 5360 x 240
                   : SmallTab{0, 0, 0, 0, false};
}

template <int PID>
struct SmallPlan {
  static constexpr bool POW2 = PID < kTabBase;
  static constexpr TablePlan TP = table_plan(POW2 ? -1 : PID - kTabBase);
  static constexpr SmallTab TAB = small_tab(POW2 ? -1 : PID - kTabBase);
  static constexpr int MX = POW2 ? 1 << PID : TP.ax * TP.bx;  // columns
  static constexpr int MY = POW2 ? 1 << PID : TP.ay * TP.by;  // rows
  static constexpr size_t PITCH = (size_t)MX + kRowPad;
  // square powers of two: points per thread: 8 below 2048 (more waves to hide the latency chain of
  // these small tiles), 16 at 2048 (measured equal or better there)
  static constexpr int PPT = MX >= 2048 ? 16 : 8;
  // rows per S1/S3 tile (at least 512 points; two at 1024, measured 2 %
  // faster than one) and threads; at these sizes the passes are
  // latency-bound, so tiles are kept small and numerous
  static constexpr int RB = !POW2 ? TAB.rb : MX == 1024 ? 2 : MX >= 512 ? 1 : 512 / MX;
  static constexpr int TR = !POW2 ? TAB.tr : cmax(64, RB * MX / PPT);
  static constexpr bool GROUP = POW2 || TAB.group;
  // columns per S2 tile: M / 256 (so that there are 256 tiles), at least 1
  // and at most 4
  static constexpr int C = !POW2 ? TAB.c : cmin(4, cmax(1, MX / 256));
  // LDS row stride: conflict-free column walks where the padding fits
  static constexpr int SJ = C == 3 || MY > 4096 ? C : C + 1;
  static constexpr int TC = !POW2 ? TAB.tc : cmax(64, MX * C / PPT);
  // S1 and the first half of S2 take the radices smallest first, so that
  // every thread has items in the first stage, where the inputs' loads and
  // the phase arithmetic sit (2 % faster at 1024^2 and 2048^2); S3 was faster
  // in the natural order.  The odd radices of the other grids come last (a
  // radix-67 stage cannot take its inputs from registers).
  static constexpr bool REV = POW2;
  static_assert(MX % C == 0, "whole column tiles");
};

// The twiddle table omega_L^i, i < L, read into registers (loads issued, not
// yet waited for) and then written to LDS.
template <int L, int T>
struct SmallTw {
  static constexpr int N = (L + T - 1) / T;
  float2 r[N];
  DEV void load(const float2 *g) {
#pragma unroll
    for (int q = 0; q < N; ++q) {
      const int i = (int)threadIdx.x + q * T;
      if (L % T == 0 || i < L)
        r[q] = is_pow2c(L) ? g[i << (kTwLog - ilog2c(L))] : g[axis_tw_offset(L) + i];
    }
  }
  DEV void put(float2 *tw) const {
#pragma unroll
    for (int q = 0; q < N; ++q) {
      const int i = (int)threadIdx.x + q * T;
      if (L % T == 0 || i < L) tw[i] = r[q];
    }
  }
};

// The first Stockham stage's inputs of a tile gathered into registers, in
// the layout a register-fed first stage consumes (only the items it will
// use: b < nb_act).  Issued together with the twiddle loads, so the two
// memory latencies overlap instead of following each other; ld must not
// branch around its loads (clamp the address and select instead), so that
// all of an item's loads are in flight before the first is waited for.
// The register block a first stage of that shape consumes.
template <class G, bool REV>
using FirstRegs = float2[FirstStage<G, REV>::PER][FirstStage<G, REV>::R];
template <class G, bool REV, class LoadF>
DEV void gather_first(FirstRegs<G, REV> &pre, const LoadF &ld, const int tid, const int nb_act) {
  using FS = FirstStage<G, REV>;
#pragma unroll
  for (int i = 0; i < FS::PER; ++i) {
    const int it = tid + i * G::T;
    if (FS::EXACT || it < FS::ITEMS) {
      int j, b;
      decode_item<G, FS::R>(it, j, b);
      if (b < nb_act) {
#pragma unroll
        for (int t = 0; t < FS::R; ++t) pre[i][t] = ld(j + t * FS::LR, b);
      }
    }
  }
}

// A wavelength's constants in a group of GR (one: the plain fields).
template <int GR, class V>
DEV V pick(const V &one, const V (&g)[kMaxGroup], int q) {
  return GR == 1 ? one : group_value(g, q);
}

// S1: one tile = RB rows of M points for each of the group's wavelengths (the
// batch index of the DFT is wavelength * RB + row); the row DFT runs along x.
// GR > 1: up to kMaxGroup wavelengths in one launch.  These launches are
// latency-bound (5 us of which the arithmetic is a small part), so a launch
// of four wavelengths costs little more than one.
template <int PID, int INM, int GR>
__global__ __launch_bounds__(SmallPlan<PID>::TR * GR) void k_small_rows_fwd(KParams p) {
  using S = SmallPlan<PID>;
  constexpr int M = S::MX, RB = S::RB, T = S::TR * GR;
  // element (x, b) of the tile: x fastest across threads; wavelengths in
  // planes of their own
  using G = Geo<M, RB * GR, GR == 1 ? RB : 1, GR == 1 ? 1 : M, T, true>;
  __shared__ float2 lds[M * RB * GR];
  __shared__ float2 tw[M];
  const int nrows = p.nrows_in, n = p.n;
  const int ntiles = (nrows + RB - 1) / RB;
  const size_t nn = (size_t)nrows * n;
  // the DOE field (Eq. 1-2), the caller's field or the adjoint seed, zero
  // past column n.  Branch-free: columns past n read column 0 and are
  // replaced by zero, rows past the last read it and are not written; without
  // an amplitude the amplitude load reads h[0] and is replaced by one.
  const float *amp_src = p.amp ? p.amp : p.h;
  auto ld = [&](int y0, int x, int b) {
    const int q = GR == 1 ? 0 : b / RB, r = GR == 1 ? b : b % RB;
    const bool in = x < n;
    const int xc = in ? x : 0, y = cmin(y0 + r, nrows - 1);
    const size_t at = (size_t)y * n + xc;
    float2 v;
    if constexpr (INM == IN_PHASE) {
      const float hv = p.h[(size_t)(y >> p.up_log2) * p.nh + (xc >> p.up_log2)];
      const float av = amp_src[p.amp ? at : 0];
      v = cscale(doe_phase(hv, pick<GR>(p.phase_turns, p.phase_turns_g, q)), p.amp ? av : 1.f);
    } else if constexpr (INM == IN_FIELD) {
      v = p.u_in[at];
    } else {
      v = cscale(p.saved_in[q * nn + at], pick<GR>(p.two_wk, p.two_wk_g, q) * p.gpsf[at]);
    }
    return in ? v : make_float2(0.f, 0.f);
  };
  const int nb = RB * (GR == 1 ? 1 : p.group);
  auto gather = [&](int tile, FirstRegs<G, S::REV> &pre, int tid) {
    gather_first<G, S::REV>(pre, [&](int x, int b) { return ld(tile * RB, x, b); }, tid, nb);
  };
  SmallTw<M, T> twr;
  twr.load(p.tw);
  FirstRegs<G, S::REV> pre;
  if ((int)blockIdx.x < ntiles) gather(blockIdx.x, pre, threadIdx.x);
  twr.put(tw);  // read from the second stage on, after the first's barriers
  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int tid = loop_tid();
    const int y0 = tile * RB;
    if (tile != (int)blockIdx.x) {
      __syncthreads();
      gather(tile, pre, tid);
    }
    auto st = [&](int kx, int b, float2 v) {
      const int q = GR == 1 ? 0 : b / RB, y = y0 + (GR == 1 ? b : b % RB);
      if (RB == 1 || y < nrows) p.ws[q * p.field_elems + (size_t)y * S::PITCH + kx] = v;
    };
    dft_tile<G, false, S::REV, SRC_REG, SNK_FN, M>(lds, tw, NoLoad{}, st, pre, tid, nb);
  }
}

// S3: the inverse row DFT of the rows left by S2, then the output stage: w is
// M^2 U (the inverse DFT's 1/M^2 is in the constants).  A group's terms are
// added in the order and rounding of one wavelength at a time.
template <int PID, int OUTM, int GR>
__global__ __launch_bounds__(SmallPlan<PID>::TR * GR) void k_small_rows_inv(KParams p) {
  using S = SmallPlan<PID>;
  constexpr int M = S::MX, MY = S::MY, RB = S::RB, T = S::TR * GR;
  using G = Geo<M, RB * GR, GR == 1 ? RB : 1, GR == 1 ? 1 : M, T, true>;
  __shared__ float2 lds[M * RB * GR];
  __shared__ float2 tw[M];
  const int nrows = p.nrows_out, n = p.n;
  const int ntiles = (nrows + RB - 1) / RB;
  const int group = GR == 1 ? 1 : p.group, nb = RB * group;
  const size_t nn = (size_t)nrows * n;
  auto gather = [&](int tile, FirstRegs<G, false> &pre, int tid) {
    auto ld = [&](int kx, int b) {
      const int q = GR == 1 ? 0 : b / RB, r = GR == 1 ? b : b % RB;
      return p.ws[q * p.field_elems + (size_t)cmin(tile * RB + r, nrows - 1) * S::PITCH + kx];
    };
    gather_first<G, false>(pre, ld, tid, nb);
  };
  SmallTw<M, T> twr;
  twr.load(p.tw);
  FirstRegs<G, false> pre;
  if ((int)blockIdx.x < ntiles) gather(blockIdx.x, pre, threadIdx.x);
  twr.put(tw);
  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int tid = loop_tid();
    const int y0 = tile * RB;
    if (tile != (int)blockIdx.x) {
      __syncthreads();
      gather(tile, pre, tid);
    }
    // output element of column x of row y; false if it is not wanted
    auto place = [&](int x, int y, size_t &at) {
      if (y >= nrows) return false;
      if (p.full) {
        const int ys = y + p.p0y, xs = x + p.p0x;
        at = (size_t)(ys >= MY ? ys - MY : ys) * M + (xs >= M ? xs - M : xs);
        return true;
      }
      at = (size_t)y * n + x;
      return x < n;
    };
    // wavelength q's term on top of `acc`
    auto term = [&](float acc, float2 w, int x, int y, size_t at, int q) {
      if constexpr (OUTM == OUT_PSF) {
        if (p.saved_out) p.saved_out[q * nn + at] = cscale(w, p.inv_m2);
        return psf_add(acc, pick<GR>(p.wk_m4, p.wk_m4_g, q), w);
      } else {
        float2 e = doe_phase(p.h[(size_t)(y >> p.up_log2) * p.nh + (x >> p.up_log2)],
                             pick<GR>(p.phase_turns, p.phase_turns_g, q));
        if (p.amp) e = cscale(e, p.amp[at]);
        return grad_add(acc, pick<GR>(p.ck_m2, p.ck_m2_g, q), w, e);
      }
    };
    float *sum = OUTM == OUT_PSF ? p.psf : p.grad_h;
    if constexpr (GR == 1) {
      auto st = [&](int x, int r, float2 w) {
        size_t at;
        if (!place(x, y0 + r, at)) return;
        if constexpr (OUTM == OUT_FIELD) p.u_out[at] = cscale(w, p.inv_m2);
        else sum[at] = term(p.first ? 0.f : sum[at], w, x, y0 + r, at, 0);
      };
      dft_tile<G, true, false, SRC_REG, SNK_FN, M>(lds, tw, NoLoad{}, st, pre, tid, nb);
    } else {
      dft_tile<G, true, false, SRC_REG, SNK_LDS, M>(lds, tw, NoLoad{}, NoStore{}, pre, tid, nb);
      for (int e = tid; e < M * RB; e += T) {
        const int x = e % M, r = e / M;
        size_t at;
        if (!place(x, y0 + r, at)) continue;
        float acc = p.first ? 0.f : sum[at];
        for (int q = 0; q < group; ++q)
          acc = term(acc, lds[(q * RB + r) * M + x], x, y0 + r, at, q);
        sum[at] = acc;
      }
    }
  }
}

// S2: one tile = C consecutive columns of M points; DFT over y, times H,
// inverse DFT over y, rows < nrows_out written back.  A tile's rows are
// C * 8 bytes wide, so 128 / (C * 8) neighbouring tiles share each cache
// line: tiles go to blocks in the XCD-aware order, which puts neighbours on
// one XCD and its L2 (at 1024^2 this took the pass from 18.7 to 14.1 us).
// q0 + blockIdx.y: wavelength of the group.  GR = 1: a single wavelength, whose
// constants are the plain fields (choosing them by q ahead of the first loads
// took 0.4 of 7 us at 512^2).
template <int PID, int GR>
__global__ __launch_bounds__(SmallPlan<PID>::TC) void k_small_cols(KParams p, int q0) {
  using S = SmallPlan<PID>;
  constexpr int MX = S::MX, M = S::MY, C = S::C, SJ = S::SJ, T = S::TC;
  using G = Geo<M, C, SJ, 1, T, false>;
  using FS = FirstStage<G, S::REV>;
  __shared__ float2 lds[M * SJ];
  __shared__ float2 tw[M];
  __shared__ double a2col[C];
  constexpr int NT = MX / C;
  const int q = GR == 1 ? 0 : q0 + blockIdx.y;
  float2 *const ws = GR == 1 ? p.ws : p.ws + q * p.field_elems;
  const double lam = pick<GR>(p.lam, p.lam_g, q), zl = pick<GR>(p.zl, p.zl_g, q);
  const double flim_x = pick<GR>(p.flim_x, p.flim_x_g, q);
  const double flim_y = pick<GR>(p.flim_y, p.flim_y_g, q);
  auto gather = [&](int tile, float2 (&pre)[FS::PER][FS::R], int tid) {
    const int x0 = xcd_tile(tile, NT) * C;
    // rows at or past nrows_in are zero: read row 0 and replace (branch-free)
    auto ld = [&](int y, int c) {
      const bool in = y < p.nrows_in;
      const float2 v = ws[(size_t)(in ? y : 0) * S::PITCH + x0 + c];
      return in ? v : make_float2(0.f, 0.f);
    };
    gather_first<G, S::REV>(pre, ld, tid, C);
  };
  SmallTw<M, T> twr;
  twr.load(p.tw);
  float2 pre[FS::PER][FS::R];
  if ((int)blockIdx.x < NT) gather(blockIdx.x, pre, threadIdx.x);
  twr.put(tw);  // read from the second stage on, after the first's barriers
  for (int tile = blockIdx.x; tile < NT; tile += gridDim.x) {
    const int tid = loop_tid();
    const int x0 = xcd_tile(tile, NT) * C;
    if (tile != (int)blockIdx.x) {
      __syncthreads();
      gather(tile, pre, tid);
    }
    // frequency-x data of the tile's columns; read after the forward DFT,
    // whose stage barriers order this write before them
    for (int c = tid; c < C; c += T) a2col[c] = a2_eff(axis_freq(x0 + c, MX, p.inv_mdx, flim_x, lam));
    dft_tile<G, false, S::REV, SRC_REG, SNK_LDS, M>(lds, tw, NoLoad{}, NoStore{}, pre, tid);
    auto ld_h = [&](int ky, int c) {
      const double a2y = a2_eff(axis_freq(ky, M, p.inv_mdy, flim_y, lam));
      return cmul(lds[ky * SJ + c], transfer(a2y, a2col[c], zl));
    };
    auto st = [&](int y, int c, float2 v) {
      if (y < p.nrows_out) ws[(size_t)y * S::PITCH + x0 + c] = v;
    };
    float2 dummy[1][1];
    dft_tile<G, true, true, SRC_FN, SNK_FN, M>(lds, tw, ld_h, st, dummy, tid);
  }
}

static inline void mark(hipEvent_t *ev, int i, hipStream_t s) {
  if (ev) (void)hipEventRecord(ev[i], s);
}

template <int PID, int INM>
static void launch_rows_fwd(const KParams &p, dim3 grid, hipStream_t s) {
  using S = SmallPlan<PID>;
  if constexpr (S::GROUP && INM != IN_FIELD) {
    if (p.group > 1) {
      hipLaunchKernelGGL((k_small_rows_fwd<PID, INM, kMaxGroup>), grid, dim3(S::TR * kMaxGroup), 0, s, p);
      return;
    }
  }
  hipLaunchKernelGGL((k_small_rows_fwd<PID, INM, 1>), grid, dim3(S::TR), 0, s, p);
}

template <int PID, int OUTM>
static void launch_rows_inv(const KParams &p, dim3 grid, hipStream_t s) {
  using S = SmallPlan<PID>;
  if constexpr (S::GROUP && OUTM != OUT_FIELD) {
    if (p.group > 1) {
      hipLaunchKernelGGL((k_small_rows_inv<PID, OUTM, kMaxGroup>), grid, dim3(S::TR * kMaxGroup), 0, s, p);
      return;
    }
  }
  hipLaunchKernelGGL((k_small_rows_inv<PID, OUTM, 1>), grid, dim3(S::TR), 0, s, p);
}

// The column pass of `count` wavelengths of the group, from the q0-th on.
template <int PID>
static void launch_cols(const KParams &p, unsigned gc, int q0, int count, hipStream_t s) {
  using S = SmallPlan<PID>;
  if constexpr (S::GROUP) {
    if (p.group > 1) {
      hipLaunchKernelGGL((k_small_cols<PID, kMaxGroup>), dim3(gc, count), dim3(S::TC), 0, s, p, q0);
      return;
    }
  }
  hipLaunchKernelGGL((k_small_cols<PID, 1>), dim3(gc), dim3(S::TC), 0, s, p, 0);
}

template <int PID>
static hipError_t launch_small_plan(const KParams &p, hipStream_t s, hipEvent_t *ev) {
  using S = SmallPlan<PID>;
  if (p.group < 1 || p.group > (S::GROUP && p.in_mode != IN_FIELD ? kMaxGroup : 1))
    return hipErrorInvalidValue;
  auto grid = [](long long tiles) {
    return (unsigned)(tiles < 1 ? 1 : tiles < kMaxBlocks ? tiles : kMaxBlocks);
  };
  const dim3 gin(grid((p.nrows_in + S::RB - 1) / S::RB)), gout(grid((p.nrows_out + S::RB - 1) / S::RB));
  mark(ev, 0, s);
  if (p.in_mode == IN_FIELD) launch_rows_fwd<PID, IN_FIELD>(p, gin, s);
  else if (p.in_mode == IN_PHASE) launch_rows_fwd<PID, IN_PHASE>(p, gin, s);
  else launch_rows_fwd<PID, IN_GRAD>(p, gin, s);
  mark(ev, 1, s);
  const unsigned gc = grid(S::MX / S::C);
  if (!ev) {
    launch_cols<PID>(p, gc, 0, p.group, s);
  } else {  // a group's fields one launch each, so that each is timed
    for (int q = 0; q < p.group; ++q) {
      launch_cols<PID>(p, gc, q, 1, s);
      mark(ev, q + 2, s);
    }
  }
  if (p.out_mode == OUT_FIELD) launch_rows_inv<PID, OUT_FIELD>(p, gout, s);
  else if (p.out_mode == OUT_PSF) launch_rows_inv<PID, OUT_PSF>(p, gout, s);
  else launch_rows_inv<PID, OUT_GRADH>(p, gout, s);
  mark(ev, p.group + 2, s);
  return hipGetLastError();
}

// 3600^2: these passes cost more per row than the five, and run one wavelength
// at a time where the five group them.  us per wavelength, five passes -> three,
// by the rows of the first and last pass together: one wavelength 3960 rows 217
// -> 185, 5400 233 -> 221, 6480 240 -> 248, 6840 245 -> 258; four wavelengths
// 3960 rows 211 -> 209, 5400 225 -> 245, 6480 232 -> 266, 6840 237 -> 282; a
// field 3960 rows 209 -> 186, 5400 222 -> 221, 6480 233 -> 247, 6840 240 -> 262.
// The gradient gains at every size (6480 rows 334 -> 298).
bool small_path(int plan, InMode in, int rows, int n_lambda) {
  if (plan < kTabBase) return plan >= kSmallMinLM && plan <= kSmallMaxLM;
  if (plan == kTab3600 && in != IN_GRAD) return rows <= (n_lambda == 1 ? 5400 : 4000);
  return small_tab(plan - kTabBase).c > 0;
}

int small_max_group(int plan) {
  return plan < kTabBase || small_tab(plan - kTabBase).group ? kMaxGroup : 1;
}

hipError_t launch_small(const KParams &p, hipStream_t s, hipEvent_t *ev) {
  switch (p.plan) {
    case 4: return launch_small_plan<4>(p, s, ev);
    case 5: return launch_small_plan<5>(p, s, ev);
    case 6: return launch_small_plan<6>(p, s, ev);
    case 7: return launch_small_plan<7>(p, s, ev);
    case 8: return launch_small_plan<8>(p, s, ev);
    case 9: return launch_small_plan<9>(p, s, ev);
    case 10: return launch_small_plan<10>(p, s, ev);
    case 11: return launch_small_plan<11>(p, s, ev);
    case kTabBase + 0: return launch_small_plan<kTabBase + 0>(p, s, ev);
    case kTabBase + 1: return launch_small_plan<kTabBase + 1>(p, s, ev);
    case kTabBase + 2: return launch_small_plan<kTabBase + 2>(p, s, ev);
    case kTab3600: return launch_small_plan<kTab3600>(p, s, ev);
    case kTabBase + 7: return launch_small_plan<kTabBase + 7>(p, s, ev);
    case kTabBase + 8: return launch_small_plan<kTabBase + 8>(p, s, ev);
    case kTabBase + 9: return launch_small_plan<kTabBase + 9>(p, s, ev);
    case kTabBase + 10: return launch_small_plan<kTabBase + 10>(p, s, ev);
    case kTabBase + 11: return launch_small_plan<kTabBase + 11>(p, s, ev);
    default: return hipErrorInvalidValue;
  }
}
static_assert(kSmallMinLM == 4 && kSmallMaxLM == 11, "one launch case per small grid");

}  // namespace dop
