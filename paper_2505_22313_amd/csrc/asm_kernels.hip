// HIP kernels for CDNA4 (gfx950): FFT-based angular-spectrum propagation of a
// DOE, Eq. (1)-(4) of Wei et al., "Large-Area Fabrication-Aware Computational
// Diffractive Optics" (Sec. 3.1).
//
// One wavelength = five passes over an My x Mx complex64 field held in HBM
// (square, or rectangular as the paper's 128,640 x 85,760 grid).  Each axis
// index is split into two digits,
//     x = BX * xa + xb,   y = BY * ya + yb      (Mx = AX * BX, My = AY * BY),
// and the 2-D FFT is the row-column decomposition of the paper's Sec. 4.1
// carried one step further: the 1-D transforms along x and y are themselves
// four-step (digit) transforms.  Forward transforms work in place and leave
// the spectrum in digit-transposed order (position BX*kxa + kxb holds
// frequency kxa + AX*kxb), the single-GPU analogue of the paper keeping the
// spectrum in swapped sharding; the transfer function is evaluated at that
// order and the inverse transforms undo it.
//
//   A  : DFT over xa (stride BX) of the N input rows.  Forms the DOE field
//        from h on the fly (Eq. 1-2); columns >= N are implicit zeros.
//   B  : DFT over xb (contiguous) and over ya (stride BY rows), one tile.
//        Rows >= N are implicit zeros.
//   C  : DFT over yb, multiply by H (Eq. 3, evaluated per element with an
//        FP64 argument, never stored), inverse DFT over yb.  Fused.
//   B' : inverse of B; only the rows that are needed are written.
//   A' : inverse of A, then |U|^2 with the wavelength weight accumulated into
//        the PSF (Eq. 4), or the field, or the height gradient.
//
// The DOE sits at the corner of the padded grid internally; propagation is a
// circular convolution, so the centred placement of the paper's grids is the
// same result shifted by p0 = (M - N)/2, applied when writing a full plane.
//
// Within a pass each tile lives in LDS and its DFTs run as Stockham radix
// 16/8/4 (and 3, 5, 9, 15) stages in registers, or a radix-67 stage through
// LDS.  Inner twiddles and four-step twiddles come from one FP64-generated
// complex64 table of exp(-2 pi i j / 2^17) on power-of-two grids, and are
// generated per block in FP64 on the others.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "asm_device.h"
#include "asm_stages.h"
#include "dop_internal.h"

namespace dop {

// ---------------------------------------------------------------------------
// Pass plans.  Tiles of passes B and C hold at most 8192 points (64 KiB +
// padding), so two blocks fit in one CU's 160 KiB LDS; tiles of passes A and
// A' hold up to 16384 (one block per CU) so that every row run they move is a
// whole 128-byte line.
//
// Plan id PID < kTabBase: the square grid M = 2^PID.  PID = kTabBase + i:
// the i-th grid of table_plan, My x Mx with Mx = AX * BX and My = AY * BY
// from a hand-chosen digit split: BX a power of two >= 16, every tile within
// the limits above, and every digit length a product of the radices
// 16/8/4/2, 3, 5 and 67.
// ---------------------------------------------------------------------------
// M = 2^17 splits both axes 1024 x 128: its B tiles hold 16384 points (one
// 1024-thread block per CU), the only way to keep every digit <= 1024; its
// pass-C tiles are 1024 rows by 8 columns (see RC below).
__host__ __device__ constexpr int plan_bx(int lm) { return lm == 17 ? 7 : cmin(lm / 2, 6); }
__host__ __device__ constexpr int plan_ay(int lm) {
  return lm == 17 ? 7 : cmin(cmin(lm / 2, 7), 13 - plan_bx(lm));
}
__host__ __device__ constexpr int threads_for(int pts) {
  return round64(cmin(512, cmax(64, pts / 16)));
}

// Two 512-thread blocks per CU = 4 waves per SIMD: caps registers at 128.
#define DOP_KERNEL(T) __global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(4)))

template <int PID>
struct Plan {
  static constexpr bool POW2 = PID < kTabBase;  // square power-of-two grid
  static constexpr TablePlan TP = table_plan(POW2 ? -1 : PID - kTabBase);
  static constexpr int MX = POW2 ? 1 << PID : TP.ax * TP.bx;  // columns
  static constexpr int MY = POW2 ? 1 << PID : TP.ay * TP.by;  // rows
  static constexpr size_t PITCH = (size_t)MX + kRowPad;  // workspace row pitch
  static constexpr int BX = POW2 ? 1 << plan_bx(PID) : TP.bx;
  static constexpr int AX = MX / BX;
  static constexpr int AY = POW2 ? 1 << plan_ay(PID) : TP.ay;
  static constexpr int BY = MY / AY;
  static constexpr int RA = TP.ra ? TP.ra : cmin(16, BX);  // run in passes A / A': a 128-byte line
  // contiguous run in pass C: 16 columns (128-byte lines); 8 on the 2^17
  // grid, whose 1024-row tiles would otherwise hold one block per CU (two
  // 80 KB blocks share a CU instead: pass C 75.7 -> 71.9 ms per wavelength)
  static constexpr int RC = TP.rc ? TP.rc : PID == 17 ? 8 : cmin(16, MX);
  // A / A' tiles (up to 1024 x 16 points, 128 KiB of LDS) run one block of
  // up to 1024 threads per CU
  // (other M: about 8 points per thread, since their mixed-radix stage
  // shapes do not divide evenly among threads and need more registers each)
  static constexpr int TA = TP.ta ? TP.ta : round64(cmin(1024, cmax(64, AX * RA / (POW2 ? 16 : 8))));
  // pass-B / B' threads: about 16 points each, 8 on the 4096 grid
  // (passes B and B' at 4096^2: 61 -> 58 and 52 -> 48 us per wavelength)
  static constexpr int TB = TP.tb ? TP.tb : !POW2 ? round64(cmin(1024, cmax(64, BX * AY / 8)))
                            : BX * AY > 8192 ? 1024
                            : PID == 12 ? 2 * threads_for(BX * AY)
                                        : threads_for(BX * AY);
  // pass-C threads: about 16 points each, except 8 on the 4096 and
  // 32768 grids, whose 64- and 256-row transforms spilled registers at
  // 16 (pass C at 4096^2: 71 -> 53 us per wavelength; at 32768^2: 3.84 ->
  // 3.69 ms)
  static constexpr int TC = TP.tc ? TP.tc : !POW2 ? round64(cmin(1024, cmax(64, BY * RC / 8)))
                            : BY * RC > 8192 ? 1024
                            : (PID == 12 || PID == 15) ? 2 * threads_for(BY * RC)
                                                       : threads_for(BY * RC);
  // Twiddles in LDS: omega_M^q = HI[q / S] * LO[q % S] with HI[i] = omega_M^(i S)
  // (= omega_THI^i) and LO[i] = omega_M^i.  Power-of-two M: THI = min(M, 1024),
  // which also serves every inner DFT length.  Table grids: THI = AX (S = BX),
  // the inner table of passes A and A'; passes B, B' and C keep their own.
  static constexpr int THI = POW2 ? (MX < 1024 ? MX : 1024) : AX;
  static constexpr int S = MX / THI;
  static_assert(AX * BX == MX && AY * BY == MY, "digit split");
  static_assert(MX % 2 == 0 && MY % 2 == 0, "even axes (signed frequency split at M / 2)");
  static_assert(is_pow2c(BX) && BX % RA == 0 && MX % RC == 0, "runs");
  static_assert(AX * RA <= 16384 && BX * AY <= 16384 && BY * RC <= 16384, "tile sizes");
  static_assert(AX <= 1024 && BX <= 1024 && AY <= 1024 && BY <= 1024, "digit lengths");
};

// Four-step twiddles of one axis (x: passes A and A'; y: passes B and B').
// The y axis shares the x tables on a square grid; on a rectangular one it
// has its own, HI over AY and LO over BY (q = yb * kya < My).
template <int PID, bool Y>
struct TwAxis {
  using P = Plan<PID>;
  static constexpr bool OWN = Y && P::MX != P::MY;
  static constexpr int M = Y ? P::MY : P::MX;
  static constexpr int THI = OWN ? P::AY : P::THI;
  static constexpr int S = M / THI;
};

template <int PID, bool Y = false>
struct TwLds {
  float2 hi[TwAxis<PID, Y>::THI];
  float2 lo[TwAxis<PID, Y>::S];
};

// exp(-2 pi i num / den), 0 <= num < den, formed in FP64 and rounded once.
DEV float2 omega_fp64(int num, int den) {
  double sn, cs;
  sincospi(-2.0 * (double)num / (double)den, &sn, &cs);
  return make_float2((float)cs, (float)sn);
}

// This plan's twiddles in LDS: from the FP64-generated global table
// (power-of-two M), or generated in FP64 (table grids).
template <int PID, int T, bool Y = false>
DEV void tw_fill(TwLds<PID, Y> &t, const float2 *__restrict__ g) {
  using P = Plan<PID>;
  using A = TwAxis<PID, Y>;
  if constexpr (P::POW2) {
    for (int i = threadIdx.x; i < A::THI; i += T) t.hi[i] = g[(i * A::S) << (kTwLog - PID)];
    for (int i = threadIdx.x; i < A::S; i += T) t.lo[i] = g[i << (kTwLog - PID)];
  } else {
    for (int i = threadIdx.x; i < A::THI; i += T) t.hi[i] = omega_fp64(i * A::S, A::M);
    for (int i = threadIdx.x; i < A::S; i += T) t.lo[i] = omega_fp64(i, A::M);
  }
}

// Table of omega_L^i, i < L (the inner twiddles of an L-point DFT).
template <int L, int T>
DEV void omega_fill(float2 *t) {
  for (int i = threadIdx.x; i < L; i += T) t[i] = omega_fp64(i, L);
}

// omega_M^q (forward sign) of the axis, q >= 0.
template <int PID, bool Y = false>
DEV float2 tw_q(const TwLds<PID, Y> &t, int q) {
  using A = TwAxis<PID, Y>;
  const unsigned u = (unsigned)q % (unsigned)A::M;
  if constexpr (A::S == 1) {
    return t.hi[u];
  } else {
    return cmul(t.hi[u / A::S], t.lo[u % A::S]);
  }
}

// Passes A and A' read heights and read-modify-write the PSF in float runs
// shorter than a cache line, shared by CH sibling tiles of one row.  A block walks the siblings of a chunk back to back (the
// chunks themselves in the XCD-aware order), so each line is consumed by one
// block while it is still in L2 even with the next tile's loads in flight.
template <int CH>
struct ChunkSeq {
  int ntiles, nchunks;
  DEV explicit ChunkSeq(int n) : ntiles(n), nchunks((n + CH - 1) / CH) {}
  // k-th tile of this block (k counts the block's own tiles), or -1
  DEV int tile(int k) const {
    const int q = (int)blockIdx.x + (k / CH) * (int)gridDim.x;
    if (q >= nchunks) return -1;
    const int t = CH * xcd_tile(q, nchunks) + k % CH;
    return t < ntiles ? t : -2;  // -2: past the end of a short last chunk
  }
};

// ---------------------------------------------------------------------------
// Pass A: DFT over xa for the N input rows, input formed on the fly.
// Tile = one row y and a run of RA consecutive xb.
// ---------------------------------------------------------------------------
template <int PID, int INM>
DOP_KERNEL(Plan<PID>::TA) void k_pass_a_fwd(KParams p) {
  using P = Plan<PID>;
  constexpr int AX = P::AX, BX = P::BX, RA = P::RA, T = P::TA;
  using G = Geo<AX, RA, RA, 1, T, false>;
  using FS = FirstStage<G>;
  __shared__ float2 lds[AX * RA];
  __shared__ TwLds<PID> tw;
  tw_fill<PID, T>(tw, p.tw);
  constexpr int RUNS = BX / RA;
  const int ntiles = p.nrows_in * RUNS;
  const int n = p.n;
  // Raw inputs of one tile's first DFT stage, loaded one tile ahead:
  // (h, amp) for IN_PHASE, the field for IN_FIELD, the saved field for
  // IN_GRAD; columns x >= n are zero.
  float2 pre[FS::PER][FS::R];
  constexpr bool GRAD = INM == IN_GRAD;
  // dL/dPSF beside the saved field (read where it is used it stalled each
  // tile: 65536^2 7.07 -> 6.02 ms, 28800^2 1.89 -> 1.49 ms, 16384^2 557 -> 400 us)
  float gpre[GRAD ? FS::PER : 1][GRAD ? FS::R : 1];
  // A tile is one input row: its arrays are addressed as a tile-uniform row
  // base plus a 32-bit byte offset per element.
  auto fetch = [&](int tile, int tid) {
    const int y = tile / RUNS;
    const size_t rowin = (size_t)y * n;
    const float *hrow = p.h + (size_t)(y >> p.up_log2) * p.nh;
    const float *arow = p.amp ? p.amp + rowin : nullptr;
    const float2 *frow = INM == IN_FIELD ? p.u_in + rowin : INM == IN_GRAD ? p.saved_in + rowin
                                                                          : nullptr;
    const float *grow = GRAD ? p.gpsf + rowin : nullptr;
    const int xb0 = (tile % RUNS) * RA;
#pragma unroll
    for (int i = 0; i < FS::PER; ++i) {
      const int it = tid + i * T;
      if (FS::EXACT || it < FS::ITEMS) {
        int j, b;
        decode_item<G, FS::R>(it, j, b);
#pragma unroll
        for (int t = 0; t < FS::R; ++t) {
          const int x = BX * (j + t * FS::LR) + xb0 + b;
          float2 v = make_float2(0.f, 0.f);
          if (x < n) {
            const unsigned ux = (unsigned)x;
            if constexpr (INM == IN_PHASE)
              v = make_float2(*at_byte(hrow, (ux >> p.up_log2) * 4u),
                              arow ? *at_byte(arow, ux * 4u) : 1.f);
            else v = *at_byte(frow, ux * 8u);
          }
          if constexpr (GRAD) gpre[i][t] = x < n ? *at_byte(grow, (unsigned)x * 4u) : 0.f;
          pre[i][t] = v;
        }
      }
    }
  };
  constexpr int CH = RUNS < 4 ? RUNS : 4;
  const ChunkSeq<CH> seq(ntiles);
  const int ngroup = INM == IN_PHASE ? p.group : 1;
  if (seq.tile(0) >= 0) fetch(seq.tile(0), threadIdx.x);
  for (int k = 0;; ++k) {
    const int tile = seq.tile(k);
    if (tile == -1) break;
    if (tile < 0) continue;
    const int y = tile / RUNS;
    const int xb0 = (tile % RUNS) * RA;
    // a group of wavelengths shares the tile's heights.  On grids of 2^28
    // points and more the prefetched values stay in registers for every
    // member of the group (each forms its field from them and writes its own
    // workspace field) and the next tile's loads are issued during the last
    // member's transform, so h crosses the fabric once per group.  Smaller
    // grids re-read the tile (an L2 hit) for each member: keeping the values
    // live there made the compiler spill.  (Grids with the factor 67 in x
    // run one wavelength at a time.)
    constexpr bool KEEP_H = (size_t)P::MX * P::MY >= (1ull << 28) && n67(AX) == 0;
    for (int q = 0; q < ngroup; ++q) {
      const int tid = loop_tid();
      __syncthreads();
      const double turns = ngroup > 1 ? group_value(p.phase_turns_g, q) : p.phase_turns;
      // the DOE field (Eq. 1-2) or the caller's field, from the prefetched values
      float2 v[FS::PER][FS::R];
#pragma unroll
      for (int i = 0; i < FS::PER; ++i) {
        const int it = tid + i * T;
        if (FS::EXACT || it < FS::ITEMS) {
          int j, b;
          decode_item<G, FS::R>(it, j, b);
#pragma unroll
          for (int t = 0; t < FS::R; ++t) {
            const float2 r = pre[i][t];
            if constexpr (INM == IN_PHASE) {
              v[i][t] = cscale(doe_phase(r.x, turns), r.y);  // r.y = 0 past column n
            } else if constexpr (INM == IN_FIELD) {
              v[i][t] = r;
            } else {
              v[i][t] = cscale(r, p.two_wk * gpre[i][t]);  // r = 0 past column n
            }
          }
        }
      }
      if (q + 1 < ngroup) {
        if constexpr (!KEEP_H) fetch(tile, tid);
      } else {
        const int nt = seq.tile(k + 1) >= 0 ? seq.tile(k + 1) : seq.tile(k + 2);
        if (nt >= 0) fetch(nt, tid);
      }
      float2 *out = p.ws + (size_t)q * p.field_elems + (size_t)y * P::PITCH;
      auto st = [&](int kxa, int b, float2 w) {
        const int xb = xb0 + b;
        out[BX * kxa + xb] = cmul(w, tw_q<PID>(tw, xb * kxa));
      };
      dft_tile<G, false, false, SRC_REG, SNK_FN, P::THI>(lds, tw.hi, NoLoad{}, st, v, tid);
    }
  }
}

// ---------------------------------------------------------------------------
// Pass B: DFT over xb then over ya on a BX x AY tile (tile = (kxa, yb)).
// Rows are moved between HBM and LDS as 16-byte (two-element) vectors.
// ---------------------------------------------------------------------------
DEV f4v ld_pair(const float2 *p) { return *reinterpret_cast<const f4v *>(p); }
DEV void st_pair(float2 *p, float2 a, float2 b) {
  *reinterpret_cast<f4v *>(p) = f4v{a.x, a.y, b.x, b.y};
}

template <int PID>
DOP_KERNEL(Plan<PID>::TB) void k_pass_b_fwd(KParams p) {
  using P = Plan<PID>;
  constexpr int AX = P::AX, BX = P::BX, AY = P::AY, BY = P::BY, T = P::TB;
  constexpr int SR = BX + 1;  // odd row stride: conflict-free for both DFT directions
  constexpr int HB = BX / 2;  // 16-byte pairs per row segment
  constexpr int PF = (AY * HB + T - 1) / T;  // pairs each thread moves per tile
  __shared__ float2 lds[AY * SR];
  __shared__ TwLds<PID, true> tw;  // y four-step twiddles omega_My
  __shared__ float2 rowtw[AY];
  // inner twiddles: the shared power-of-two table, else tables of their own
  __shared__ float2 wbx[P::POW2 ? 1 : BX], way[P::POW2 ? 1 : AY];
  tw_fill<PID, T, true>(tw, p.tw);
  if constexpr (!P::POW2) {
    omega_fill<BX, T>(wbx);
    omega_fill<AY, T>(way);
  }
  constexpr int THX = P::POW2 ? P::THI : BX, THY = P::POW2 ? P::THI : AY;
  const float2 *twx = P::POW2 ? tw.hi : wbx;
  const float2 *twy = P::POW2 ? tw.hi : way;
  constexpr int NT = AX * BY;
  float2 dummy[1][1];
  // rows ya with BY*ya + yb >= nrows_in hold zeros: not read, x-DFT skipped
  auto nzrows = [&](int yb) {
    return p.nrows_in > yb ? cmin(AY, (p.nrows_in - yb + BY - 1) / BY) : 0;
  };
  // Loads of one tile's nonzero rows into registers; issued one tile ahead so
  // that they are in flight while the current tile is transformed.
  f4v pre[PF];
  auto fetch = [&](int pt, int tid) {
    const int tile = xcd_tile(pt, NT);
    const int kxa = tile % AX, yb = tile / AX, nz = nzrows(yb);
    const float2 *src = p.ws + (size_t)yb * P::PITCH + (size_t)BX * kxa;
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      const int e = tid + i * T, ya = e / HB, c = e % HB;
      pre[i] = f4v{0.f, 0.f, 0.f, 0.f};
      if ((PF * T == AY * HB || e < AY * HB) && ya < nz)
        pre[i] = ld_pair(src + (size_t)(BY * ya) * P::PITCH + 2 * c);
    }
  };
  if (blockIdx.x < NT) fetch(blockIdx.x, threadIdx.x);
  for (int pt = blockIdx.x; pt < NT; pt += gridDim.x) {
    const int tid = loop_tid();
    const int tile = xcd_tile(pt, NT);
    const int kxa = tile % AX;
    const int yb = tile / AX;
    const size_t col0 = (size_t)BX * kxa;
    const int nz = nzrows(yb);
    __syncthreads();
    for (int r = tid; r < AY; r += T) rowtw[r] = tw_q<PID, true>(tw, yb * r);  // omega_My^(yb kya)
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      const int e = tid + i * T, ya = e / HB, c = e % HB;
      if (PF * T == AY * HB || e < AY * HB) {
        lds[ya * SR + 2 * c] = make_float2(pre[i].x, pre[i].y);
        lds[ya * SR + 2 * c + 1] = make_float2(pre[i].z, pre[i].w);
      }
    }
    if (pt + (int)gridDim.x < NT) fetch(pt + gridDim.x, tid);
    __syncthreads();
    using GX = Geo<BX, AY, 1, SR, T, false>;
    dft_tile<GX, false, false, SRC_LDS, SNK_LDS, THX>(lds, twx, NoLoad{}, NoStore{}, dummy, tid, nz);
    using GY = Geo<AY, BX, SR, 1, T, false>;
    dft_tile<GY, false, false, SRC_LDS, SNK_LDS, THY>(lds, twy, NoLoad{}, NoStore{}, dummy, tid);
    for (int e = tid; e < AY * HB; e += T) {
      const int kya = e / HB, c = e % HB;
      const float2 w = rowtw[kya];
      st_pair(p.ws + (size_t)(BY * kya + yb) * P::PITCH + col0 + 2 * c,
              cmul(lds[kya * SR + 2 * c], w), cmul(lds[kya * SR + 2 * c + 1], w));
    }
  }
}

// ---------------------------------------------------------------------------
// Pass C: DFT over yb, times H, inverse DFT over yb (tile = (kya, run of RC
// columns)).
// ---------------------------------------------------------------------------
template <int PID>
DOP_KERNEL(Plan<PID>::TC) void k_pass_c(KParams p) {
  using P = Plan<PID>;
  constexpr int AX = P::AX, BX = P::BX, AY = P::AY, BY = P::BY, RC = P::RC, T = P::TC;
  // LDS row stride: one pad element for 16-column tiles; an 8-column tile
  // goes unpadded so that two blocks fit in a CU's LDS
  constexpr int SJ = RC >= 16 ? RC + 1 : RC;
  using G = Geo<BY, RC, SJ, 1, T, false>;
  using FS = FirstStage<G>;
  // A radix-67 stage cannot hand its outputs over in registers: with one, the
  // forward DFT ends in LDS (natural order) and the inverse DFT reads it
  // through a load functor that applies H.
  constexpr bool VIA_LDS = n67(BY) > 0;
  static_assert((size_t)BY * P::PITCH * sizeof(float2) <= 0xFFFFFFFFull,
                "tile byte offsets are 32-bit");
  __shared__ float2 lds[BY * SJ];
  // only BY-point DFTs run here: their twiddles omega_BY^i, i < BY
  __shared__ float2 twc[BY];
  // a2_eff of the tile's BY frequency rows (and, via LDS, of its RC columns)
  __shared__ double a2row[BY];
  __shared__ double a2col[VIA_LDS ? RC : 1];
  if constexpr (P::POW2) {
    for (int i = threadIdx.x; i < BY; i += T) twc[i] = p.tw[i << (kTwLog - ilog2c(BY))];
  } else {
    omega_fill<BY, T>(twc);
  }
  constexpr int RUNS = P::MX / RC;
  constexpr int NT = AY * RUNS;
  auto tile_base = [&](int pt) {
    const int tile = xcd_tile(pt, NT);
    return p.ws + (size_t)(BY * (tile / RUNS)) * P::PITCH + (tile % RUNS) * RC;
  };
  // frequency-x data of padded column px (spectrum position BX kxa + kxb
  // holds kx = kxa + AX kxb)
  auto col_a2 = [&](int px) {
    const int kx = (px / BX) + AX * (px % BX);
    return a2_eff(axis_freq(kx, P::MX, p.inv_mdx, p.flim_x, p));
  };
  // one tile's first-stage inputs, loaded one tile ahead
  float2 pre[FS::PER][FS::R];
  auto fetch = [&](int pt, int tid) {
    const float2 *base = tile_base(pt);
#pragma unroll
    for (int i = 0; i < FS::PER; ++i) {
      const int it = tid + i * T;
      if (FS::EXACT || it < FS::ITEMS) {
        int j, b;
        decode_item<G, FS::R>(it, j, b);
#pragma unroll
        for (int t = 0; t < FS::R; ++t)
          pre[i][t] = *at_byte(base, ((unsigned)(j + t * FS::LR) * (unsigned)P::PITCH + b) * 8u);
      }
    }
  };
  if ((int)blockIdx.x < NT) fetch(blockIdx.x, threadIdx.x);
  for (int pt = blockIdx.x; pt < NT; pt += gridDim.x) {
    const int tid = loop_tid();
    const int tile = xcd_tile(pt, NT);
    const int px0 = (tile % RUNS) * RC;
    const int kya = tile / RUNS;
    float2 *base = p.ws + (size_t)(BY * kya) * P::PITCH + px0;
    __syncthreads();
    // frequency rows of this tile: position kyb holds ky = kya + AY kyb; read
    // after the forward DFT, whose stage barriers order this write before them
    for (int r = tid; r < BY; r += T)
      a2row[r] = a2_eff(axis_freq(kya + AY * r, P::MY, p.inv_mdy, p.flim_y, p));
    if constexpr (VIA_LDS)
      for (int c = tid; c < RC; c += T) a2col[c] = col_a2(px0 + c);
    float2 v[FS::PER][FS::R];
#pragma unroll
    for (int i = 0; i < FS::PER; ++i)
#pragma unroll
      for (int t = 0; t < FS::R; ++t) v[i][t] = pre[i][t];
    auto hook = [&]() {
      if (pt + (int)gridDim.x < NT) fetch(pt + gridDim.x, tid);
    };
    auto st = [&](int yb, int b, float2 w) {
      *at_byte(base, ((unsigned)yb * (unsigned)P::PITCH + b) * 8u) = w;
    };
    if constexpr (VIA_LDS) {
      float2 dummy[1][1];
      dft_tile_hooked<G, false, false, SRC_REG, SNK_LDS, BY>(lds, twc, NoLoad{}, NoStore{}, hook,
                                                            v, dummy, tid);
      auto ld_h = [&](int kyb, int b) {
        return cmul(lds[kyb * SJ + b], transfer(a2row[kyb], a2col[b], p));
      };
      dft_tile<G, true, true, SRC_FN, SNK_FN, BY>(lds, twc, ld_h, st, dummy, tid);
    } else {
      using LR_ = LastRegs<G, false>;
      float2 regs[LR_::PER][LR_::R];
      dft_tile_hooked<G, false, false, SRC_REG, SNK_REG, BY>(lds, twc, NoLoad{}, NoStore{}, hook,
                                                            v, regs, tid);
      {
        constexpr int R = LR_::R;
        constexpr int LRn = BY / R;
        using SS = StageShape<G, R>;
#pragma unroll
        for (int i = 0; i < LR_::PER; ++i) {
          const int it = tid + i * T;
          if (SS::EXACT || it < SS::ITEMS) {
            int j, b;
            decode_item<G, R>(it, j, b);
            const double a2x = col_a2(px0 + b);
#pragma unroll
            for (int t = 0; t < R; ++t)
              regs[i][t] = cmul(regs[i][t], transfer(a2row[j + t * LRn], a2x, p));
          }
        }
      }
      dft_tile<G, true, true, SRC_REG, SNK_FN, BY>(lds, twc, NoLoad{}, st, regs, tid);
    }
  }
}

// ---------------------------------------------------------------------------
// Pass B': inverse DFT over kya then over kxb (tile = (kxa, yb)); writes the
// rows y < nrows_out.
// ---------------------------------------------------------------------------
template <int PID>
DOP_KERNEL(Plan<PID>::TB) void k_pass_b_inv(KParams p) {
  using P = Plan<PID>;
  constexpr int AX = P::AX, BX = P::BX, AY = P::AY, BY = P::BY, T = P::TB;
  constexpr int SR = BX + 1;
  constexpr int HB = BX / 2;
  constexpr int PF = (AY * HB + T - 1) / T;
  __shared__ float2 lds[AY * SR];
  __shared__ TwLds<PID, true> tw;
  __shared__ float2 rowtw[AY];
  __shared__ float2 wbx[P::POW2 ? 1 : BX], way[P::POW2 ? 1 : AY];
  tw_fill<PID, T, true>(tw, p.tw);
  if constexpr (!P::POW2) {
    omega_fill<BX, T>(wbx);
    omega_fill<AY, T>(way);
  }
  constexpr int THX = P::POW2 ? P::THI : BX, THY = P::POW2 ? P::THI : AY;
  const float2 *twx = P::POW2 ? tw.hi : wbx;
  const float2 *twy = P::POW2 ? tw.hi : way;
  constexpr int NT = AX * BY;
  float2 dummy[1][1];
  f4v pre[PF];
  auto fetch = [&](int pt, int tid) {
    const int tile = xcd_tile(pt, NT);
    const int kxa = tile % AX, yb = tile / AX;
    const float2 *src = p.ws + (size_t)yb * P::PITCH + (size_t)BX * kxa;
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      const int e = tid + i * T, kya = e / HB, c = e % HB;
      if (PF * T == AY * HB || e < AY * HB) pre[i] = ld_pair(src + (size_t)(BY * kya) * P::PITCH + 2 * c);
    }
  };
  if (blockIdx.x < NT) fetch(blockIdx.x, threadIdx.x);
  for (int pt = blockIdx.x; pt < NT; pt += gridDim.x) {
    const int tid = loop_tid();
    const int tile = xcd_tile(pt, NT);
    const int kxa = tile % AX;
    const int yb = tile / AX;
    const size_t col0 = (size_t)BX * kxa;
    // only the rows ya with BY*ya + yb < nrows_out are needed
    const int nz = p.nrows_out > yb ? cmin(AY, (p.nrows_out - yb + BY - 1) / BY) : 0;
    __syncthreads();
    for (int r = tid; r < AY; r += T) rowtw[r] = tw_q<PID, true>(tw, yb * r);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      const int e = tid + i * T, kya = e / HB, c = e % HB;
      if (PF * T == AY * HB || e < AY * HB) {
        const float2 w = rowtw[kya];
        lds[kya * SR + 2 * c] = cmulc(make_float2(pre[i].x, pre[i].y), w);
        lds[kya * SR + 2 * c + 1] = cmulc(make_float2(pre[i].z, pre[i].w), w);
      }
    }
    if (pt + (int)gridDim.x < NT) fetch(pt + gridDim.x, tid);
    __syncthreads();
    using GY = Geo<AY, BX, SR, 1, T, false>;
    dft_tile<GY, true, false, SRC_LDS, SNK_LDS, THY>(lds, twy, NoLoad{}, NoStore{}, dummy, tid);
    using GX = Geo<BX, AY, 1, SR, T, false>;
    dft_tile<GX, true, false, SRC_LDS, SNK_LDS, THX>(lds, twx, NoLoad{}, NoStore{}, dummy, tid, nz);
    for (int e = tid; e < nz * HB; e += T) {
      const int ya = e / HB, c = e % HB;
      st_pair(p.ws + (size_t)(BY * ya + yb) * P::PITCH + col0 + 2 * c, lds[ya * SR + 2 * c],
              lds[ya * SR + 2 * c + 1]);
    }
  }
}

// ---------------------------------------------------------------------------
// Pass A': inverse DFT over kxa for the rows y < nrows_out, then the output
// stage: PSF accumulation (Eq. 4), field, or height gradient.
// ---------------------------------------------------------------------------
template <int PID, int OUTM>
DOP_KERNEL(Plan<PID>::TA) void k_pass_a_inv(KParams p) {
  using P = Plan<PID>;
  constexpr int AX = P::AX, BX = P::BX, RA = P::RA, MX = P::MX, MY = P::MY, T = P::TA;
  using G = Geo<AX, RA, RA, 1, T, false>;
  using FS = FirstStage<G>;
  // A radix-67 last stage writes through a store functor that does the
  // output stage; otherwise the last stage's registers are finished here.
  constexpr bool VIA_FN = n67(AX) > 0;
  using LS = LastRegs<G, false>;
  constexpr int LRL = AX / LS::R;
  using SSL = StageShape<G, LS::R>;
  constexpr int APER = VIA_FN ? 1 : LS::PER, AR = VIA_FN ? 1 : LS::R;
  // Whether the gradient's output stage reads its heights (and aperture) in
  // batches ahead of the stores: 16384^2 grid 522 -> 408 us, 28800^2 2.31 ->
  // 2.02 ms, 40000^2 3.36 -> 3.06 ms.  The 512- and 1024-thread tiles of the
  // larger powers of two have no registers left for a batch (92 bytes of
  // spills: 65536^2 7.4 -> 10.7 ms).
  constexpr bool GRAD_BATCH = OUTM == OUT_GRADH && !VIA_FN && !(P::POW2 && T >= 512);
  __shared__ float2 lds[AX * RA];
  __shared__ TwLds<PID> tw;
  tw_fill<PID, T>(tw, p.tw);
  constexpr int RUNS = BX / RA;
  const int ntiles = p.nrows_out * RUNS;
  const int n = p.n;
  const bool accumulate = (OUTM == OUT_PSF || OUTM == OUT_GRADH) && !p.first;
  // a group of wavelengths (PSF output, no saved fields) adds all its
  // intensities to one read-modify-write of the PSF; field q of the group
  // sits q * field_elems after the first
  const int ngroup = (OUTM == OUT_PSF && !VIA_FN) ? p.group : 1;
  // spectrum values of one tile's first inverse stage, loaded one tile ahead
  float2 pre[FS::PER][FS::R];
  auto fetch = [&](int tile, int tid, int q) {
    const float2 *row = p.ws + (size_t)q * p.field_elems + (size_t)(tile / RUNS) * P::PITCH +
                        (tile % RUNS) * RA;
#pragma unroll
    for (int i = 0; i < FS::PER; ++i) {
      const int it = tid + i * T;
      if (FS::EXACT || it < FS::ITEMS) {
        int j, b;
        decode_item<G, FS::R>(it, j, b);
#pragma unroll
        for (int t = 0; t < FS::R; ++t) pre[i][t] = row[BX * (j + t * FS::LR) + b];
      }
    }
  };
  // A tile is one row y, so every output array is addressed as a
  // tile-uniform row base plus a 32-bit column offset.  Element offset of
  // the output row of row y (full plane: centred, wrapped):
  auto out_row = [&](int y) -> size_t {
    if (p.full) {
      const int ys = y + p.p0y;  // < 2 My
      return (size_t)(ys >= MY ? ys - MY : ys) * MX;
    }
    return (size_t)y * n;
  };
  // output column of element (xa, b) of the current tile; false if outside
  auto out_col = [&](int xb0, int xa, int b, unsigned &c) {
    const int x = BX * xa + xb0 + b;
    if (p.full) {
      const int xs = x + p.p0x;  // < 2 Mx
      c = (unsigned)(xs >= MX ? xs - MX : xs);
      return true;
    }
    c = (unsigned)x;
    return x < n;
  };
  // Row bases of the outputs (and, for the gradient, of h and amp).
  struct Rows {
    float *acc;         // PSF or gradient row
    float2 *field;      // saved or output field row (NULL if none)
    const float *h;     // height row (gradient)
    const float *amp;   // aperture row (gradient, NULL if none)
  };
  auto rows_of = [&](int y) {
    const size_t r = out_row(y);
    Rows o{nullptr, nullptr, nullptr, nullptr};
    if constexpr (OUTM == OUT_PSF) {
      o.acc = p.psf + r;
      if (p.saved_out) o.field = p.saved_out + r;
    } else if constexpr (OUTM == OUT_FIELD) {
      o.field = p.u_out + r;
    } else {
      o.acc = p.grad_h + r;
      o.h = p.h + (size_t)(y >> p.up_log2) * p.nh;
      if (p.amp) o.amp = p.amp + r;
    }
    return o;
  };
  // output stage of one element at column c: w is My Mx U (the inverse DFT's
  // 1/(My Mx) is applied here), accv the accumulator value it adds to, wk
  // the PSF weight
  auto finish = [&](const Rows &o, unsigned c, float2 w, float accv, float wk) {
    if constexpr (OUTM == OUT_PSF) {
      *at_byte(o.acc, c * 4u) = psf_add(accv, wk, w);
      if (o.field) *at_byte(o.field, c * 8u) = cscale(w, p.inv_m2);
    } else if constexpr (OUTM == OUT_FIELD) {
      *at_byte(o.field, c * 8u) = cscale(w, p.inv_m2);
    } else {
      // crop only: the column is x < n
      float2 e = doe_phase(o.h[c >> p.up_log2], p.phase_turns);
      if (o.amp) e = cscale(e, *at_byte(o.amp, c * 4u));
      // c_k Im(g_E conj(E)), g_E = w / (My Mx)
      *at_byte(o.acc, c * 4u) = grad_add(accv, p.ck_m2, w, e);
    }
  };
  constexpr int CH = RUNS < 4 ? RUNS : 4;
  const ChunkSeq<CH> seq(ntiles);
  if (seq.tile(0) >= 0) fetch(seq.tile(0), threadIdx.x, 0);
  for (int k = 0;; ++k) {
    const int tile = seq.tile(k);
    if (tile == -1) break;
    if (tile < 0) continue;
    const int y = tile / RUNS;
    const int xb0 = (tile % RUNS) * RA;
    const Rows orow = rows_of(y);
    float acc[APER][AR];
    for (int q = 0; q < ngroup; ++q) {
      const int tid = loop_tid();
      __syncthreads();
      const float wk = ngroup > 1 ? group_value(p.wk_m4_g, q) : p.wk_m4;
      float2 v[FS::PER][FS::R];
#pragma unroll
      for (int i = 0; i < FS::PER; ++i) {
        const int it = tid + i * T;
        if (FS::EXACT || it < FS::ITEMS) {
          int j, b;
          decode_item<G, FS::R>(it, j, b);
#pragma unroll
          for (int t = 0; t < FS::R; ++t)
            v[i][t] = cmulc(pre[i][t], tw_q<PID>(tw, (xb0 + b) * (j + t * FS::LR)));
        }
      }
      // After the first stage: read the accumulator values this tile will
      // add to (once per group), then start the next loads (the group's next
      // field of this tile, else the next tile).  Loads complete in issue
      // order, so the accumulator reads go first: waiting for them at the end
      // of this tile must not also wait for the prefetch.
      auto hook = [&]() {
        if constexpr (!VIA_FN) {
          if (q == 0) {
#pragma unroll
            for (int i = 0; i < LS::PER; ++i) {
              const int it = tid + i * T;
              int j = 0, b = 0;
              if (SSL::EXACT || it < SSL::ITEMS) decode_item<G, LS::R>(it, j, b);
#pragma unroll
              for (int t = 0; t < LS::R; ++t) {
                acc[i][t] = 0.f;
                unsigned c;
                if (accumulate && (SSL::EXACT || it < SSL::ITEMS) &&
                    out_col(xb0, j + t * LRL, b, c))
                  acc[i][t] = *at_byte(orow.acc, c * 4u);
              }
            }
          }
        }
        if (q + 1 < ngroup) {
          fetch(tile, tid, q + 1);
        } else {
          const int nt = seq.tile(k + 1) >= 0 ? seq.tile(k + 1) : seq.tile(k + 2);
          if (nt >= 0) fetch(nt, tid, 0);
        }
      };
      if constexpr (VIA_FN) {
        float2 dummy[1][1];
        auto st = [&](int xa, int b, float2 w) {
          unsigned c;
          if (!out_col(xb0, xa, b, c)) return;
          const float accv = accumulate ? *at_byte(orow.acc, c * 4u) : 0.f;
          finish(orow, c, w, accv, wk);
        };
        dft_tile_hooked<G, true, false, SRC_REG, SNK_FN, P::THI>(lds, tw.hi, NoLoad{}, st, hook, v,
                                                                dummy, tid);
      } else {
        float2 u[LS::PER][LS::R];
        dft_tile_hooked<G, true, false, SRC_REG, SNK_REG, P::THI>(lds, tw.hi, NoLoad{}, NoStore{},
                                                                 hook, v, u, tid);
        const bool last = q + 1 == ngroup;
        if constexpr (GRAD_BATCH) {
          // the output stage's own reads come ahead of the stores, which the
          // compiler must assume to alias them, in batches that the registers
          // beside the prefetch hold
          constexpr int NB = 8;
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int i = 0; i < LS::PER; ++i) {
            const int it = loop_tid() + i * T;
            int j = 0, b = 0;
            if (SSL::EXACT || it < SSL::ITEMS) decode_item<G, LS::R>(it, j, b);
#pragma unroll
            for (int t0 = 0; t0 < LS::R; t0 += NB) {
              float hv[NB], av[NB];
#pragma unroll
              for (int t = t0; t < t0 + NB && t < LS::R; ++t) {
                unsigned c;
                if (!out_col(xb0, j + t * LRL, b, c)) c = 0;
                hv[t - t0] = orow.h[c >> p.up_log2];
                av[t - t0] = orow.amp ? *at_byte(orow.amp, c * 4u) : 1.f;
              }
#pragma unroll
              for (int t = t0; t < t0 + NB && t < LS::R; ++t) {
                const float2 e = cscale(doe_phase(hv[t - t0], p.phase_turns), av[t - t0]);
                acc[i][t] = grad_add(acc[i][t], p.ck_m2, u[i][t], e);
              }
              __builtin_amdgcn_sched_barrier(0);
            }
          }
#pragma unroll
          for (int i = 0; i < LS::PER; ++i) {
            const int it = loop_tid() + i * T;
            if (SSL::EXACT || it < SSL::ITEMS) {
              int j, b;
              decode_item<G, LS::R>(it, j, b);
#pragma unroll
              for (int t = 0; t < LS::R; ++t) {
                unsigned c;
                if (out_col(xb0, j + t * LRL, b, c)) *at_byte(orow.acc, c * 4u) = acc[i][t];
              }
            }
          }
        } else {
#pragma unroll
        for (int i = 0; i < LS::PER; ++i) {
          const int it = tid + i * T;
          if (SSL::EXACT || it < SSL::ITEMS) {
            int j, b;
            decode_item<G, LS::R>(it, j, b);
#pragma unroll
            for (int t = 0; t < LS::R; ++t) {
              unsigned c;
              if (!out_col(xb0, j + t * LRL, b, c)) continue;
              if (last) finish(orow, c, u[i][t], acc[i][t], wk);
              else acc[i][t] = psf_add(acc[i][t], wk, u[i][t]);
            }
          }
        }
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Ceiling probe with pass C's memory access pattern and none of its
// arithmetic: the same tiles (BY rows x RC columns of the padded-pitch
// field), the same persistent grid and XCD-aware tile order, the same
// one-tile-ahead prefetch into the first stage's register layout (which is
// also the last inverse stage's store layout), the same LDS footprint (so as
// many blocks share a CU), and each element written back in place times
// `scale`.  What pass C achieves against this is the share of the pattern's
// bandwidth its arithmetic leaves.
// ---------------------------------------------------------------------------
template <int PID>
DOP_KERNEL(Plan<PID>::TC) void k_probe_passc(float2 *ws, float scale) {
  using P = Plan<PID>;
  constexpr int AY = P::AY, BY = P::BY, RC = P::RC, T = P::TC;
  constexpr int SJ = RC >= 16 ? RC + 1 : RC;
  using G = Geo<BY, RC, SJ, 1, T, false>;
  using FS = FirstStage<G>;
  static_assert((size_t)BY * P::PITCH * sizeof(float2) <= 0xFFFFFFFFull,
                "tile byte offsets are 32-bit");
  constexpr int RUNS = P::MX / RC;
  constexpr int NT = AY * RUNS;
  auto tile_base = [&](int pt) {
    const int tile = xcd_tile(pt, NT);
    return ws + (size_t)(BY * (tile / RUNS)) * P::PITCH + (tile % RUNS) * RC;
  };
  auto off = [&](int j, int b) { return ((unsigned)j * (unsigned)P::PITCH + b) * 8u; };
  float2 pre[FS::PER][FS::R];
  auto fetch = [&](int pt, int tid) {
    const float2 *base = tile_base(pt);
#pragma unroll
    for (int i = 0; i < FS::PER; ++i) {
      const int it = tid + i * T;
      if (FS::EXACT || it < FS::ITEMS) {
        int j, b;
        decode_item<G, FS::R>(it, j, b);
#pragma unroll
        for (int t = 0; t < FS::R; ++t) pre[i][t] = *at_byte(base, off(j + t * FS::LR, b));
      }
    }
  };
  if ((int)blockIdx.x < NT) fetch(blockIdx.x, threadIdx.x);
  for (int pt = blockIdx.x; pt < NT; pt += gridDim.x) {
    const int tid = loop_tid();
    float2 v[FS::PER][FS::R];
#pragma unroll
    for (int i = 0; i < FS::PER; ++i)
#pragma unroll
      for (int t = 0; t < FS::R; ++t) v[i][t] = pre[i][t];
    if (pt + (int)gridDim.x < NT) fetch(pt + gridDim.x, tid);
    float2 *base = tile_base(pt);
#pragma unroll
    for (int i = 0; i < FS::PER; ++i) {
      const int it = tid + i * T;
      if (FS::EXACT || it < FS::ITEMS) {
        int j, b;
        decode_item<G, FS::R>(it, j, b);
#pragma unroll
        for (int t = 0; t < FS::R; ++t) *at_byte(base, off(j + t * FS::LR, b)) = cscale(v[i][t], scale);
      }
    }
  }
}

// LDS bytes of pass C of plan PID (the probe reserves as much, dynamically).
template <int PID>
constexpr size_t pass_c_lds_bytes() {
  using P = Plan<PID>;
  constexpr int SJ = P::RC >= 16 ? P::RC + 1 : P::RC;
  constexpr bool VIA_LDS = n67(P::BY) > 0;
  return sizeof(float2) * (P::BY * SJ + P::BY) + sizeof(double) * (P::BY + (VIA_LDS ? P::RC : 1));
}

template <int PID>
static hipError_t launch_probe(float2 *ws, float scale, hipStream_t s) {
  using P = Plan<PID>;
  const long long tiles = (long long)P::AY * (P::MX / P::RC);
  const unsigned grid = (unsigned)(tiles < kMaxBlocks ? tiles : kMaxBlocks);
  hipLaunchKernelGGL(k_probe_passc<PID>, dim3(grid), dim3(P::TC), pass_c_lds_bytes<PID>(), s, ws,
                     scale);
  return hipGetLastError();
}

hipError_t launch_probe_passc(int plan, float2 *ws, float scale, hipStream_t s) {
  switch (plan) {
    case 14: return launch_probe<14>(ws, scale, s);
    case 15: return launch_probe<15>(ws, scale, s);
    case 16: return launch_probe<16>(ws, scale, s);
    case 17: return launch_probe<17>(ws, scale, s);
    default: return hipErrorInvalidValue;
  }
}

// ---------------------------------------------------------------------------
// Host-side launch of the five passes.
// ---------------------------------------------------------------------------
static inline void mark(hipEvent_t *ev, int i, hipStream_t s) {
  if (ev) (void)hipEventRecord(ev[i], s);
}

template <int PID>
static hipError_t launch_range(const KParams &p, int first, int last, hipStream_t s,
                               hipEvent_t *ev) {
  using P = Plan<PID>;
  // the gradient on 3600^2 takes the small grids' passes at every size
  constexpr bool GRAD = PID != kTab3600;
  if (!GRAD && p.in_mode == IN_GRAD) return hipErrorInvalidValue;
  auto grid = [](long long tiles) {
    return (unsigned)(tiles < kMaxBlocks ? tiles : kMaxBlocks);
  };
  const unsigned ga = grid((long long)p.nrows_in * (P::BX / P::RA));
  const unsigned gb = grid((long long)P::AX * P::BY);
  const unsigned gc = grid((long long)P::AY * (P::MX / P::RC));
  const unsigned gai = grid((long long)p.nrows_out * (P::BX / P::RA));
  for (int pass = first; pass <= last; ++pass) {
    mark(ev, pass - first, s);
    switch (pass) {
      case 0:
        if (p.in_mode == IN_PHASE)
          hipLaunchKernelGGL((k_pass_a_fwd<PID, IN_PHASE>), dim3(ga), dim3(P::TA), 0, s, p);
        else if (p.in_mode == IN_FIELD)
          hipLaunchKernelGGL((k_pass_a_fwd<PID, IN_FIELD>), dim3(ga), dim3(P::TA), 0, s, p);
        else if constexpr (GRAD)
          hipLaunchKernelGGL((k_pass_a_fwd<PID, IN_GRAD>), dim3(ga), dim3(P::TA), 0, s, p);
        break;
      case 1: hipLaunchKernelGGL(k_pass_b_fwd<PID>, dim3(gb), dim3(P::TB), 0, s, p); break;
      case 2: hipLaunchKernelGGL(k_pass_c<PID>, dim3(gc), dim3(P::TC), 0, s, p); break;
      case 3: hipLaunchKernelGGL(k_pass_b_inv<PID>, dim3(gb), dim3(P::TB), 0, s, p); break;
      default:
        if (p.out_mode == OUT_PSF)
          hipLaunchKernelGGL((k_pass_a_inv<PID, OUT_PSF>), dim3(gai), dim3(P::TA), 0, s, p);
        else if (p.out_mode == OUT_FIELD)
          hipLaunchKernelGGL((k_pass_a_inv<PID, OUT_FIELD>), dim3(gai), dim3(P::TA), 0, s, p);
        else if constexpr (GRAD)
          hipLaunchKernelGGL((k_pass_a_inv<PID, OUT_GRADH>), dim3(gai), dim3(P::TA), 0, s, p);
        break;
    }
  }
  mark(ev, last - first + 1, s);
  return hipGetLastError();
}

hipError_t launch_passes(const KParams &p, int first, int last, hipStream_t s, hipEvent_t *ev) {
  if (first < 0 || last >= kNumPasses || first > last) return hipErrorInvalidValue;
  switch (p.plan) {
    case 12: return launch_range<12>(p, first, last, s, ev);
    case 13: return launch_range<13>(p, first, last, s, ev);
    case 14: return launch_range<14>(p, first, last, s, ev);
    case 15: return launch_range<15>(p, first, last, s, ev);
    case 16: return launch_range<16>(p, first, last, s, ev);
    case 17: return launch_range<17>(p, first, last, s, ev);
    case kTabBase + 3: return launch_range<kTabBase + 3>(p, first, last, s, ev);
    case kTab3600: return launch_range<kTab3600>(p, first, last, s, ev);
    case kTabBase + 5: return launch_range<kTabBase + 5>(p, first, last, s, ev);
    case kTabBase + 6: return launch_range<kTabBase + 6>(p, first, last, s, ev);
    case kTabBase + 12: return launch_range<kTabBase + 12>(p, first, last, s, ev);
    case kTabBase + 13: return launch_range<kTabBase + 13>(p, first, last, s, ev);
    default: return hipErrorInvalidValue;
  }
}

static_assert(kNumTab == 14, "a launch case here or in launch_small per grid of table_plan");

int plan_id(int mx, int my) {
  if (mx == my && mx >= 16 && mx <= (1 << 17) && is_pow2c(mx)) return ilog2c(mx);
  for (int i = 0; i < kNumTab; ++i) {
    const TablePlan t = table_plan(i);
    if (t.ax * t.bx == mx && t.ay * t.by == my) return kTabBase + i;
  }
  return -1;
}

int table_grids(int *rows, int *cols, int max) {
  for (int i = 0; i < kNumTab && i < max; ++i) {
    const TablePlan t = table_plan(i);
    rows[i] = t.ay * t.by;
    cols[i] = t.ax * t.bx;
  }
  return kNumTab;
}

// A group of wavelengths needs pass A' to hold the accumulator in registers,
// which a radix-67 last stage (writing through a store functor) does not.
int plan_max_group(int plan) {
  return plan >= kTabBase && table_plan(plan - kTabBase).ax % kP == 0 ? 1 : kMaxGroup;
}

}  // namespace dop
