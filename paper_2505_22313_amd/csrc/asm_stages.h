// The tile DFT engine: Stockham stages of an L-point DFT over a tile in LDS,
// and the table of grids that are not square powers of two.
#ifndef DOP_ASM_STAGES_H_
#define DOP_ASM_STAGES_H_

#include "asm_device.h"

namespace dop {

// ---------------------------------------------------------------------------
// Stockham stage plan for an L-point DFT, L = 2^a 3^b 5^c 67^d <= 1024: the
// power-of-two factor in radix 16/8/4 stages (as for a power-of-two L), then
// the odd factor: a radix-15 stage per (3, 5) pair, radix 9 per pair of the
// remaining threes, radix 5 per remaining five, a last radix 3, and last of
// all a radix-67 stage (the prime factor of the paper's 128,640 x 85,760
// grid; see stage_prime).  (Radix 25 would save more stages, but 25 points
// per item plus the prefetched inputs overflow the 128 registers a thread
// has at this occupancy.)
// ---------------------------------------------------------------------------
__host__ __device__ constexpr int ilog2c(int v) { return v <= 1 ? 0 : 1 + ilog2c(v / 2); }
__host__ __device__ constexpr bool is_pow2c(int v) { return v > 0 && (v & (v - 1)) == 0; }
__host__ __device__ constexpr int pow2_part(int v) { return v % 2 ? 1 : 2 * pow2_part(v / 2); }
__host__ __device__ constexpr int cmin_(int a, int b) { return a < b ? a : b; }
__host__ __device__ constexpr int count_factor(int v, int f) {
  return v % f ? 0 : 1 + count_factor(v / f, f);
}

__host__ __device__ constexpr int num_stages_p2(int L) {
  return L <= 1 ? 0 : L <= 16 ? 1 : (L <= 256 ? 2 : 3);
}

__host__ __device__ constexpr int fwd_radix_p2(int L, int s) {
  return L <= 16 ? L
       : L == 32 ? (s == 0 ? 8 : 4)
       : L == 64 ? 8
       : L == 128 ? (s == 0 ? 16 : 8)
       : L == 256 ? 16
       : L == 512 ? (s == 0 ? 16 : (s == 1 ? 8 : 4))
       : L == 1024 ? (s == 0 ? 16 : 8)
       : L == 2048 ? (s < 2 ? 16 : 8)
       : 16;  // 4096 (whole rows and columns of the small-grid path)
}

__host__ __device__ constexpr int n15(int L) {
  return cmin_(count_factor(L, 3), count_factor(L, 5));
}
__host__ __device__ constexpr int n9(int L) { return (count_factor(L, 3) - n15(L)) / 2; }
__host__ __device__ constexpr int n5(int L) { return count_factor(L, 5) - n15(L); }
__host__ __device__ constexpr int n3(int L) { return (count_factor(L, 3) - n15(L)) % 2; }
constexpr int kP = 67;  // the prime radix
__host__ __device__ constexpr int n67(int L) { return count_factor(L, kP); }

__host__ __device__ constexpr int num_stages(int L) {
  return L <= 1 ? 1 : num_stages_p2(pow2_part(L)) + n15(L) + n9(L) + n5(L) + n3(L) + n67(L);
}

// radix of odd-factor stage s (s counted from the first odd stage)
__host__ __device__ constexpr int odd_radix(int L, int s) {
  return s < n15(L)                         ? 15
         : s < n15(L) + n9(L)               ? 9
         : s < n15(L) + n9(L) + n5(L)       ? 5
         : s < n15(L) + n9(L) + n5(L) + n3(L) ? 3
                                            : kP;
}

__host__ __device__ constexpr int fwd_radix(int L, int s) {
  return L <= 1 ? 1
       : s < num_stages_p2(pow2_part(L)) ? fwd_radix_p2(pow2_part(L), s)
                                         : odd_radix(L, s - num_stages_p2(pow2_part(L)));
}

// REV reverses the radix order (used by the inverse half of the fused middle
// pass so that it starts with the radix the forward half ended with).
__host__ __device__ constexpr int stage_radix(int L, int s, bool rev) {
  return rev ? fwd_radix(L, num_stages(L) - 1 - s) : fwd_radix(L, s);
}

__host__ __device__ constexpr int stage_ns(int L, int s, bool rev) {
  return s == 0 ? 1 : stage_ns(L, s - 1, rev) * stage_radix(L, s - 1, rev);
}

// Tile geometry: element (j, b) of the tile (j = transform index in [0, L),
// b = batch index in [0, NB)) lives at LDS offset j*SJ + b*SB.  JFAST chooses
// whether consecutive threads walk j or b.
template <int L_, int NB_, int SJ_, int SB_, int T_, bool JFAST_>
struct Geo {
  static constexpr int L = L_, NB = NB_, SJ = SJ_, SB = SB_, T = T_;
  static constexpr bool JFAST = JFAST_;
};

enum { SRC_LDS = 0, SRC_FN = 1, SRC_REG = 2 };
enum { SNK_LDS = 0, SNK_FN = 1, SNK_REG = 2 };

template <class G, int R>
struct StageShape {
  static constexpr int LR = G::L / R;
  static constexpr int ITEMS = LR * G::NB;
  static constexpr int PER = (ITEMS + G::T - 1) / G::T;
  static constexpr bool EXACT = (ITEMS % G::T) == 0;
};

template <class G, int R>
DEV void decode_item(int it, int &j, int &b) {
  constexpr int LR = G::L / R;
  if constexpr (G::JFAST) {
    j = is_pow2c(LR) ? it & (LR - 1) : (int)((unsigned)it % LR);
    b = it / LR;
  } else {
    b = is_pow2c(G::NB) ? it & (G::NB - 1) : (int)((unsigned)it % G::NB);
    j = it / G::NB;
  }
}

// Register block handed between the forward and inverse halves of pass C.
template <class G, bool REV>
struct LastRegs {
  static constexpr int R = stage_radix(G::L, num_stages(G::L) - 1, REV);
  static constexpr int PER = StageShape<G, R>::PER;
};

// ---------------------------------------------------------------------------
// Radix-67 Stockham stage.  67 points per item do not fit in registers, so
// the stage works through the tile in LDS, in place:
//  1. fold: for every item and t = 1..33 (one thread per pair), read v_t and
//     v_{67-t} (after the stage twiddles) and write v_t + v_{67-t} to slot t
//     and v_t - v_{67-t} to slot 67 - t (slot 0 keeps v_0);
//  2. three or four threads per item (whichever spreads the tile's
//     wavefronts evenly over the four SIMDs) each form a share of the 33
//     output pairs from the folded values, X_k, X_{67-k} = v_0 + sum_t s_t cos(2 pi t k / 67)
//     -/+ i sum_t d_t sin(2 pi t k / 67) (forward sign; the symmetric form of
//     the direct DFT, 2 real multiply-adds per input pair and output), with
//     the constants folded in at compile time; a share is uniform across a
//     wavefront so that the code paths of the shares do not diverge;
//  3. the outputs go to the stage's Stockham positions, in LDS or through the
//     store functor.
// Inputs come from LDS or the load functor, never from registers, and
// outputs never go to registers.
// ---------------------------------------------------------------------------
constexpr int kPH = (kP - 1) / 2;  // folded input pairs
// With NSH shares per item, share rb covers output pairs k = share_k0 ..
// share_k0 + share_np - 1: 11 + 11 + 11 or 9 + 8 + 8 + 8.
__host__ __device__ constexpr int share_np(int nsh, int rb) {
  return nsh == 3 ? 11 : (rb == 0 ? 9 : 8);
}
__host__ __device__ constexpr int share_k0(int nsh, int rb) {
  return nsh == 3 ? 1 + 11 * rb : (rb == 0 ? 1 : 10 + 8 * (rb - 1));
}
constexpr int kPBMax = 11;
static_assert(share_k0(3, 2) + share_np(3, 2) == kPH + 1, "three shares cover 1..33");
static_assert(share_k0(4, 3) + share_np(4, 3) == kPH + 1, "four shares cover 1..33");

template <class G, int NSH, int RB, bool INV>
DEV void prime_outputs(const float2 *lds, const int e0, float2 (&o)[2 * kPBMax + 1]) {
  constexpr int STEP = (G::L / kP) * G::SJ;
  constexpr int K0 = share_k0(NSH, RB), NP = share_np(NSH, RB);
  const float2 x0 = lds[e0];
  float2 a[NP], q[NP];
  float2 sum = x0;
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    a[i] = x0;
    q[i] = make_float2(0.f, 0.f);
  }
#pragma unroll
  for (int t = 1; t <= kPH; ++t) {
    const float2 sv = lds[e0 + t * STEP], dv = lds[e0 + (kP - t) * STEP];
    if constexpr (RB == 0) sum = cadd(sum, sv);
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int e = (t * (K0 + i)) % kP;
      const float c = UnitRoots<kP>::c[e], sn_ = UnitRoots<kP>::s[e];
      a[i].x += sv.x * c;
      a[i].y += sv.y * c;
      q[i].x += dv.x * sn_;
      q[i].y += dv.y * sn_;
    }
  }
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    const float2 iq = INV ? mul_pi(q[i]) : mul_mi(q[i]);
    o[2 * i] = cadd(a[i], iq);      // X_{K0 + i}
    o[2 * i + 1] = csub(a[i], iq);  // X_{67 - K0 - i}
  }
  o[2 * kPBMax] = sum;              // X_0 (share 0)
}

template <class G, bool INV, bool FIRST, bool LAST, int NS, int TWMUL, int SRC, int SNK,
          class LoadF, class StoreF, class Hook>
DEV void stage_prime(float2 *lds, const float2 *twl, const LoadF &ld, const StoreF &st,
                     const Hook &hook, const int tid, const int nb_act) {
  static_assert(SRC != SRC_REG && SNK != SNK_REG,
                "a radix-67 stage reads and writes LDS or functors, not registers");
  constexpr int LR = G::L / kP, ITEMS = LR * G::NB;
  auto at = [](int j, int b) { return j * G::SJ + b * G::SB; };
  // 1. fold, one thread per (item, pair), in place; item fastest so that
  // neighbouring threads touch neighbouring LDS words
  for (int u = tid; u < ITEMS * (kPH + 1); u += G::T) {
    const int it = u % ITEMS, t = u / ITEMS;
    int j, b;
    decode_item<G, kP>(it, j, b);
    if (b >= nb_act) continue;
    if (t == 0) {
      if constexpr (SRC == SRC_FN) lds[at(j, b)] = ld(j, b);
      continue;
    }
    const int k = FIRST ? 0 : (is_pow2c(NS) ? j & (NS - 1) : (int)((unsigned)j % NS));
    auto in = [&](int tt) {
      float2 x;
      if constexpr (SRC == SRC_FN) x = ld(j + tt * LR, b);
      else x = lds[at(j + tt * LR, b)];
      if constexpr (!FIRST) {
        const float2 w = twl[(tt * k) * TWMUL];
        x = INV ? cmulc(x, w) : cmul(x, w);
      }
      return x;
    };
    const float2 v1 = in(t), v2 = in(kP - t);
    lds[at(j + t * LR, b)] = cadd(v1, v2);
    lds[at(j + (kP - t) * LR, b)] = csub(v1, v2);
  }
  if constexpr (FIRST) hook();
  __syncthreads();
  // 2. outputs: wavefront w takes share w / IW of items (w % IW) * 64 + lane
  constexpr int IW = (ITEMS + 63) / 64;
  constexpr int NSH = (3 * IW) % 4 == 0 || 4 * IW * 64 > G::T ? 3 : 4;
  static_assert(NSH * IW * 64 <= G::T, "one output share per thread");
  const int wv = tid >> 6, rb = wv / IW, it = (wv % IW) * 64 + (tid & 63);
  int j = 0, b = 0;
  bool act = rb < NSH && it < ITEMS;
  if (act) {
    decode_item<G, kP>(it, j, b);
    act = b < nb_act;
  }
  float2 o[2 * kPBMax + 1];
  if (act) {
    const int e0 = at(j, b);
    if (rb == 0) prime_outputs<G, NSH, 0, INV>(lds, e0, o);
    else if (rb == 1) prime_outputs<G, NSH, 1, INV>(lds, e0, o);
    else if (NSH == 3 || rb == 2) prime_outputs<G, NSH, 2, INV>(lds, e0, o);
    else prime_outputs<G, NSH, NSH == 3 ? 2 : 3, INV>(lds, e0, o);
  }
  // 3. output t of item (j, b) goes to (j - k) * 67 + k + t * NS, k = j mod NS
  constexpr bool TO_LDS = !LAST || SNK == SNK_LDS;
  if constexpr (TO_LDS) __syncthreads();  // every fold slot has been read
  if (act) {
    const int k = is_pow2c(NS) ? j & (NS - 1) : (int)((unsigned)j % NS);
    const int base = (j - k) * kP + k;
    auto put = [&](int t, float2 val) {
      if constexpr (TO_LDS) lds[at(base + t * NS, b)] = val;
      else st(base + t * NS, b, val);
    };
    const int k0 = share_k0(NSH, rb), np = share_np(NSH, rb);
#pragma unroll
    for (int i = 0; i < kPBMax; ++i) {
      if (i < np) {
        put(k0 + i, o[2 * i]);
        put(kP - k0 - i, o[2 * i + 1]);
      }
    }
    if (rb == 0) put(0, o[2 * kPBMax]);
  }
  if constexpr (TO_LDS) __syncthreads();
}

// One Stockham stage S of the L-point DFT along j for every b, followed by the
// remaining stages.  The first stage reads from SRC (LDS, a load functor
// ld(j, b), or the register block rin), every later stage from LDS.  The last
// stage writes natural-order results to SNK (LDS, a store functor
// st(j, b, v), or the register block rout).  hook() runs once, right after
// the first stage has consumed its inputs (so prefetches issued there do not
// overlap the first stage's registers).  All threads of the block must call.
template <class G, bool INV, bool REV, int S, int SRC, int SNK, int THI, class LoadF, class StoreF,
          class Hook, int PI, int RI, int PO, int RO>
DEV void stages(float2 *lds, const float2 *twl, const LoadF &ld, const StoreF &st,
                const Hook &hook, float2 (&rin)[PI][RI], float2 (&rout)[PO][RO], const int tid,
                const int nb_act) {
  constexpr int NSTG = num_stages(G::L);
  constexpr int R = stage_radix(G::L, S, REV);
  constexpr int NS = stage_ns(G::L, S, REV);
  constexpr bool FIRST = (S == 0), LAST = (S == NSTG - 1);
  using SS = StageShape<G, R>;
  constexpr int LR = SS::LR, PER = SS::PER, ITEMS = SS::ITEMS;
  static_assert(NS * R <= THI, "twiddle table too small");
  constexpr int TWMUL = THI / (NS * R);  // omega_{NS R}^e = twl[e * TWMUL]
  if constexpr (R == kP) {
    stage_prime<G, INV, FIRST, LAST, NS, TWMUL, SRC, SNK>(lds, twl, ld, st, hook, tid, nb_act);
    if constexpr (!LAST)
      stages<G, INV, REV, S + 1, SRC_LDS, SNK, THI>(lds, twl, ld, st, hook, rin, rout, tid, nb_act);
  } else {
  float2 v[PER][R];
  // an item is live if it exists and its batch column is below nb_act (the
  // columns at or beyond nb_act are known to be zero, or are not needed)
  auto live = [&](int it, int &j, int &b) {
    if (!(SS::EXACT || it < ITEMS)) return false;
    decode_item<G, R>(it, j, b);
    return b < nb_act;
  };
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int it = tid + i * G::T;
    int j, b;
    if (live(it, j, b)) {
      if constexpr (FIRST && SRC == SRC_REG) {
        static_assert(PI == PER && RI == R, "register input shape");
#pragma unroll
        for (int t = 0; t < R; ++t) v[i][t] = rin[i][t];
      } else if constexpr (FIRST && SRC == SRC_FN) {
#pragma unroll
        for (int t = 0; t < R; ++t) v[i][t] = ld(j + t * LR, b);
      } else {
#pragma unroll
        for (int t = 0; t < R; ++t) v[i][t] = lds[(j + t * LR) * G::SJ + b * G::SB];
      }
    }
  }

#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int it = tid + i * G::T;
    int j, b;
    if (live(it, j, b)) {
      if constexpr (!FIRST) {
        const int k = is_pow2c(NS) ? j & (NS - 1) : (int)((unsigned)j % NS);
#pragma unroll
        for (int t = 1; t < R; ++t) {
          const float2 w = twl[(t * k) * TWMUL];
          v[i][t] = INV ? cmulc(v[i][t], w) : cmul(v[i][t], w);
        }
      }
      Dft<R, INV>::run(v[i]);
    }
  }

  if constexpr (LAST) {
    if constexpr (FIRST) hook();
    if constexpr (SNK == SNK_LDS) __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int it = tid + i * G::T;
      int j, b;
      if (live(it, j, b)) {
#pragma unroll
        for (int t = 0; t < R; ++t) {
          if constexpr (SNK == SNK_REG) {
            static_assert(PO == PER && RO == R, "register output shape");
            rout[i][t] = v[i][t];
          } else if constexpr (SNK == SNK_FN) {
            st(j + t * LR, b, v[i][t]);
          } else {
            lds[(j + t * LR) * G::SJ + b * G::SB] = v[i][t];
          }
        }
      }
    }
    if constexpr (SNK == SNK_LDS) __syncthreads();
  } else {
    __syncthreads();  // every read of this stage is done before LDS is reused
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int it = tid + i * G::T;
      int j, b;
      if (live(it, j, b)) {
        const int k = is_pow2c(NS) ? j & (NS - 1) : (int)((unsigned)j % NS);
        const int base = (j - k) * R + k;
#pragma unroll
        for (int t = 0; t < R; ++t) lds[(base + t * NS) * G::SJ + b * G::SB] = v[i][t];
      }
    }
    if constexpr (FIRST) hook();
    __syncthreads();
    stages<G, INV, REV, S + 1, SRC_LDS, SNK, THI>(lds, twl, ld, st, hook, rin, rout, tid, nb_act);
  }
  }
}

struct NoHook {
  DEV void operator()() const {}
};

// L-point DFT of every batch column of a tile; twl is the LDS table
// omega_THI^i, i < THI (THI a multiple of L).  One register block serves as
// input (SRC_REG) and output (SNK_REG).
template <class G, bool INV, bool REV, int SRC, int SNK, int THI, class LoadF, class StoreF,
          int PERR, int RR>
DEV void dft_tile(float2 *lds, const float2 *twl, const LoadF &ld, const StoreF &st,
                  float2 (&regs)[PERR][RR], const int tid, const int nb_act = G::NB) {
  stages<G, INV, REV, 0, SRC, SNK, THI>(lds, twl, ld, st, NoHook{}, regs, regs, tid, nb_act);
}

// As dft_tile, with separate input and output register blocks and a hook run
// after the first stage.
template <class G, bool INV, bool REV, int SRC, int SNK, int THI, class LoadF, class StoreF,
          class Hook, int PI, int RI, int PO, int RO>
DEV void dft_tile_hooked(float2 *lds, const float2 *twl, const LoadF &ld, const StoreF &st,
                         const Hook &hook, float2 (&rin)[PI][RI], float2 (&rout)[PO][RO],
                         const int tid, const int nb_act = G::NB) {
  stages<G, INV, REV, 0, SRC, SNK, THI>(lds, twl, ld, st, hook, rin, rout, tid, nb_act);
}

// Thread index re-read in every tile iteration through an empty asm
// statement, so per-thread LDS addresses are recomputed inside the tile loop
// instead of being hoisted out of it and spilled.
DEV int loop_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// Shape of the first Stockham stage of a tile (what a prefetch must gather);
// REV: of the reversed radix order.
template <class G, bool REV = false>
struct FirstStage {
  static constexpr int R = stage_radix(G::L, 0, REV);
  using SS = StageShape<G, R>;
  static constexpr int PER = SS::PER, LR = SS::LR, ITEMS = SS::ITEMS;
  static constexpr bool EXACT = SS::EXACT;
};

struct NoLoad {
  DEV float2 operator()(int, int) const { return make_float2(0.f, 0.f); }
};
struct NoStore {
  DEV void operator()(int, int, float2) const {}
};

__host__ __device__ constexpr int cmin(int a, int b) { return a < b ? a : b; }
__host__ __device__ constexpr int cmax(int a, int b) { return a > b ? a : b; }
__host__ __device__ constexpr int round64(int v) { return (v + 63) / 64 * 64; }

struct TablePlan {
  int ax, bx, ay, by;  // Mx = ax * bx columns, My = ay * by rows
  // pass-C run and threads (0: 16 columns, about 8 points per thread); the
  // 1005-row tiles of the paper's grid take 8 columns and 512 threads, so two
  // blocks share a CU and one block's ALU work overlaps the other's traffic
  int rc = 0, tc = 0;
  // pass-A / A' run and threads (0: 16 columns, about 8 points per thread);
  // the 28,800 grid's 450 x 16 tiles take 512 threads, so two blocks share a CU
  int ra = 0, ta = 0;
  // pass-B / B' threads (0: about 8 points per thread); the 40,000 grid's
  // B, B' and C tiles take 512 threads, so two blocks share a CU
  int tb = 0;
};
constexpr int kTabBase = 100;
constexpr int kNumTab = 14;
constexpr int kTab3600 = kTabBase + 4;  // 3600^2, the grid all three paths share
// 28800^2: C tiles have 240 and 256 items a stage, so 256 threads (two more
// blocks per CU than with 512): 3.08 -> 2.80 ms per wavelength, 4.8 TB/s.
// 16080 x 10720: 16 x 16 B tiles fill a quarter of a wavefront's lanes, and a
// 1005-row C tile (153 KB) leaves one block per CU.  With 120 x 134 rows the B
// tiles hold 1920 points, and 32 columns give the 67-point stage of C 64
// items, a whole wavefront per share, in a 34 KB tile: per wavelength B 789 ->
// 428, B' 726 -> 425, C 1530 -> 1016 us (A and A' 441 and 511 -> 527 and 590
// beside the faster C).
__host__ __device__ constexpr TablePlan table_plan(int i) {
  return i == 0    ? TablePlan{15, 16, 15, 16}        // 240^2
         : i == 1  ? TablePlan{45, 16, 45, 16}        // 720^2
         : i == 2  ? TablePlan{45, 32, 45, 32}        // 1440^2
         : i == 3  ? TablePlan{48, 64, 48, 64}        // 3072^2
         : i == 4  ? TablePlan{225, 16, 15, 240}      // 3600^2
         : i == 5  ? TablePlan{450, 64, 120, 240, 16, 256, 0, 512}      // 28800^2, 2^7 3^2 5^2
         : i == 6  ? TablePlan{625, 64, 100, 400, 0, 512, 0, 0, 512}    // 40000^2, 2^6 5^4
         : i == 7  ? TablePlan{134, 16, 16, 134}      // 2144^2, 2^5 67
         : i == 8  ? TablePlan{15, 16, 45, 16}        // 720 rows x 240 columns
         : i == 9  ? TablePlan{128, 16, 16, 32}       // 512 x 2048
         : i == 10 ? TablePlan{134, 16, 15, 16}       // 240 x 2144
         : i == 11 ? TablePlan{15, 16, 16, 335}       // 5360 x 240
         : i == 12 ? TablePlan{670, 16, 120, 134, 32, 256}  // 16080 x 10720
         : i == 13 ? TablePlan{670, 128, 128, 1005, 8, 512}  // 128640 x 85760: 2^7 3 5 67 x 2^8 5 67
                   : TablePlan{0, 0, 0, 0};
}

}  // namespace dop

#endif  // DOP_ASM_STAGES_H_
