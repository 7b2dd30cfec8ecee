// Three-pass propagation of a zero-padded field on the square power-of-two
// grids of 4096 .. 16384 points per side and on 3600^2, where whole rows and
// columns fit in one block:
//   R : DFT along x of each DOE row (the input formed on the fly), written
//       column by column;
//   K : per column, DFT along y, times H (Eq. 3), inverse DFT along y;
//   R': inverse DFT along x of the DOE's rows, then the output stage.
// The five digit passes of asm_kernels.hip move 51 bytes per padded point and
// wavelength, these 19: only the N rows that hold data ever leave the chip,
// and each row and column crosses HBM once per pass.  It applies when the DOE
// covers at most half of each axis and only the DOE window is wanted, which
// is what the factor-of-two padding of a linear convolution gives.
//
// Transform.  M = CR * L2, an index splits as x = j + L2 t (t < CR) and a
// frequency as k = k1 + CR k2.  The cross stage is a CR-point DFT over t
// (t >= CR/2 are the padding and are not computed on), then the twiddle
// omega_M^(j k1), and per k1 an L2-point DFT over j.  A wavefront owns whole
// L2-point transforms, so past the one exchange that follows the cross stage
// all LDS traffic is inside a wavefront and needs no block barrier.
//
// Frequencies go in pairs (p, -p): the transforms k1 = p and k1 = CR - p run
// side by side in the same threads, the first with the forward sign and the
// second, on input twiddled by conj(omega_M^(j p)), with the opposite one, so
// that the same registers hold the frequencies p + CR k2 and -(p + CR k2).
// One twiddle serves both, one value of H serves both in pass K (H is even),
// and a pair of frequency columns is one 16-byte item of the layout below.
// The pair p = 0 is made of k1 = 0 and k1 = CR / 2.
//
// Layout between the passes: pair q = p L2 + k2 of columns (kx = p + CR k2
// and its partner) holds one 16-byte item per DOE row y; groups of QG pairs
// lie pitch3 items apart, each as (row, pair) items.  Pass K streams one
// pair; passes R and R' write and read the runs of their block's rows.
// pitch3 is an odd number of 128-byte lines, which spreads neighbouring
// groups over the channels.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "asm_device.h"
#include "asm_stages.h"
#include "dop_internal.h"

namespace dop {
namespace {

// LM: log2 M of a power of two, or the plan id of 3600^2 (3600 = 16 * 15 * 15).
template <int LM>
struct Tri {
  static constexpr bool POW2 = LM < kTabBase;
  static constexpr TablePlan TP = table_plan(POW2 ? -1 : LM - kTabBase);
  static constexpr int M = POW2 ? 1 << LM : TP.ax * TP.bx;
  static constexpr int CR = 16;           // cross radix
  static constexpr int NP = CR / 2;       // frequency pairs p
  static constexpr int L2 = M / CR;       // wave-local transform: LP * RX * LP
  static constexpr int LP = POW2 ? 16 : 15;           // points of it per lane
  static constexpr int RX = L2 / (LP * LP);           // its middle radix: 1 (none), 2, 4
  static constexpr int IW = L2 / LP;                  // lanes per pair of transforms
  static constexpr int NW = 64 / IW;                  // pairs of transforms per wavefront
  static constexpr int ROWS = NW;                     // rows per block of passes R and R'
  static constexpr int TROW = 64 * NP;                // threads of passes R and R'
  static constexpr int HALF = TROW / ROWS;            // from a thread's first item to its second
  static constexpr int TCOL = 64 * 2 * NP / NW;       // threads of pass K: a column pair
  // Lanes and items past the end (3600: four lanes of a wavefront, 31 threads
  // of a row's or column's items) repeat the last one, and store what it stores.
  static constexpr bool EXACT = IW * NW == 64;
  // LDS position of element pos: one pad element per 16 keeps the first
  // exchange (stride 16) free of bank conflicts; stride 15 needs none
  static constexpr int pad(int pos) { return POW2 ? pos + pos / 16 : pos; }
  static constexpr int SUB = pad(L2);     // of one pair of transforms
  static constexpr int REG = SUB * NW;    // of one wavefront's
  static_assert(M == CR * L2 && L2 == LP * RX * LP && L2 == LP * IW, "transform");
  // Pairs interleaved in memory: passes R and R' touch runs of 16 QG ROWS
  // bytes, pass K 128 / QG bytes of each line.  Runs under 64 bytes cost the
  // row passes more than the split lines cost pass K (us per wavelength of
  // R + K + R'): 16384 grid 717 + 1054 + 527 at QG = 1, 599 + 1215 + 447 at
  // 2, 339 + 1457 + 346 at 4; 8192 grid 119 + 267 + 122, 101 + 285 + 99,
  // 91 + 322 + 88; 4096 grid 21 + 59 + 21 at 1, 22 + 61 + 23 at 2.
  static constexpr int QG = LM == 14 ? 4 : LM == 13 ? 2 : 1;
  // item of pair q, row 0 (row y lies QG y on)
  DEV static size_t pair_item(int q, int pitch) { return (size_t)(q / QG) * pitch + q % QG; }
};

// Twiddles of the wave-local transform, in LDS: omega_L2^(t i) at [t - 1][i],
// t < LP, i < IW, and omega_(16 RX)^(t k) at [t - 1][k], k < 16.
template <int LM>
struct LocalTw {
  using P = Tri<LM>;
  float2 a[(P::LP - 1) * P::IW];
  float2 b[P::RX > 1 ? (P::RX - 1) * 16 : 1];
  DEV void fill(const float2 *__restrict__ tw, int threads) {
    for (int i = threadIdx.x; i < (P::LP - 1) * P::IW; i += threads) {
      const int e = (i / P::IW + 1) * (i % P::IW);
      a[i] = P::POW2 ? tw[e << (kTwLog - LM + 4)] : tw[axis_tw_offset(P::M) + e * P::CR];
    }
    if constexpr (P::RX > 1)
      for (int i = threadIdx.x; i < (P::RX - 1) * 16; i += threads)
        b[i] = tw[((i / 16 + 1) * (i % 16)) << (kTwLog - 4 - (P::RX == 2 ? 1 : 2))];
  }
};

// The mirror transform of pair p: k1 = 16 - p (8 for p = 0).
__host__ __device__ constexpr int mir(int p) { return p ? 16 - p : 8; }

// Orders one wavefront's LDS accesses: LDS serves a wavefront in program
// order, so only the compiler has to be held back.
DEV void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Keeps the instruction scheduler from interleaving the work on both sides,
// which would hold more values at once than the 128 registers a thread has.
DEV void sched_fence() { __builtin_amdgcn_sched_barrier(0); }

// Exchange of 2 x 16 points inside a wavefront's LDS region, real parts then
// imaginary parts (one 8-byte access moves a component of both transforms).
// Register t goes to put[PS idx(t)], and is taken from get[GS t].
template <int LP, int PS, int GS, class Idx>
DEV void wave_exchange(float2 (&a)[16], float2 (&b)[16], float2 *put, const float2 *get,
                       const Idx &idx) {
  float2 re[LP];
  wave_sync();
#pragma unroll
  for (int t = 0; t < LP; ++t) put[PS * idx(t)] = make_float2(a[t].x, b[t].x);
  wave_sync();
#pragma unroll
  for (int t = 0; t < LP; ++t) re[t] = get[GS * t];
  wave_sync();
#pragma unroll
  for (int t = 0; t < LP; ++t) put[PS * idx(t)] = make_float2(a[t].y, b[t].y);
  wave_sync();
#pragma unroll
  for (int t = 0; t < LP; ++t) {
    const float2 im = get[GS * t];
    a[t] = make_float2(re[t].x, im.x);
    b[t] = make_float2(re[t].y, im.y);
  }
}

// L2-point DFTs of a (sign INV) and b (the opposite sign) over the IW lanes
// `it` that share them.  In and out, register t of lane it holds element
// it + IW t, t < LP.  reg is the LDS element of position 0; position pos lies
// pad(pos) S elements on.  Every access is one of three bases plus a
// constant, so no address is kept per element.
template <int LM, int S, bool INV>
DEV void local_dft(float2 (&a)[16], float2 (&b)[16], float2 *reg, const int it,
                   const LocalTw<LM> &tw) {
  using P = Tri<LM>;
  constexpr int IW = P::IW, RX = P::RX, LP = P::LP;
  constexpr int NAT = P::pad(IW) * S;  // from element it + IW t to the next t
  Dft<LP, INV>::run(a);
  sched_fence();
  Dft<LP, !INV>::run(b);
  float2 *nat = reg + P::pad(it) * S;
  wave_exchange<LP, S, NAT>(a, b, reg + P::pad(LP) * it * S, nat, [](int t) { return t; });
  if constexpr (RX > 1) {
    constexpr int NI = 16 / RX;  // radix-RX items per lane: it + IW i
    const int k = it & 15;
#pragma unroll
    for (int t = 1; t < RX; ++t) {
      const float2 w = tw.b[(t - 1) * 16 + k];
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        float2 &x = a[i + NI * t], &y = b[i + NI * t];
        x = INV ? cmulc(x, w) : cmul(x, w);
        y = INV ? cmul(y, w) : cmulc(y, w);
      }
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      float2 u[RX], v[RX];
#pragma unroll
      for (int t = 0; t < RX; ++t) {
        u[t] = a[i + NI * t];
        v[t] = b[i + NI * t];
      }
      Dft<RX, INV>::run(u);
      Dft<RX, !INV>::run(v);
#pragma unroll
      for (int t = 0; t < RX; ++t) {
        a[i + NI * t] = u[t];
        b[i + NI * t] = v[t];
      }
    }
    // output t of item i goes to (item - k) RX + k + 16 t
    wave_exchange<LP, 17 * S, NAT>(a, b, reg + (17 * RX * (it >> 4) + k) * S, nat, [](int s) {
      const int i = s % NI, t = s / NI;
      return IW / 16 * RX * i + t;
    });
  }
#pragma unroll
  for (int t = 1; t < LP; ++t) {
    const float2 w = tw.a[(t - 1) * IW + it];
    a[t] = INV ? cmulc(a[t], w) : cmul(a[t], w);
    b[t] = INV ? cmul(b[t], w) : cmulc(b[t], w);
    if (t % 4 == 3) sched_fence();
  }
  Dft<LP, INV>::run(a);
  sched_fence();
  Dft<LP, !INV>::run(b);
}

// 16-point DFT whose inputs 8..15 are zero (forward): the zeros' butterflies
// are left out, the rest is Dft<16>'s arithmetic.
DEV void dft16_half_in(float2 (&a)[16]) {
  float2 t[16];
#pragma unroll
  for (int n2 = 0; n2 < 4; ++n2) {
    const float2 x = a[n2], y = a[4 + n2], iy = mul_mi(y);
    const float2 o[4] = {cadd(x, y), cadd(x, iy), csub(x, y), csub(x, iy)};
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1) t[k1 * 4 + n2] = mulw16<false>(o[k1], n2 * k1);
  }
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1) {
    float2 c[4] = {t[k1 * 4], t[k1 * 4 + 1], t[k1 * 4 + 2], t[k1 * 4 + 3]};
    Dft<4, false>::run(c);
#pragma unroll
    for (int k2 = 0; k2 < 4; ++k2) a[k1 + 4 * k2] = c[k2];
  }
}

// Inverse 16-point DFT of which only outputs 0..7 are wanted.
DEV void idft16_half_out(float2 (&a)[16]) {
  float2 t[16];
#pragma unroll
  for (int n2 = 0; n2 < 4; ++n2) {
    float2 b[4] = {a[n2], a[4 + n2], a[8 + n2], a[12 + n2]};
    Dft<4, true>::run(b);
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1) t[k1 * 4 + n2] = mulw16<true>(b[k1], n2 * k1);
  }
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1) {
    const float2 *c = t + 4 * k1;
    a[k1] = cadd(cadd(c[0], c[2]), cadd(c[1], c[3]));
    a[k1 + 4] = cadd(csub(c[0], c[2]), mul_pi(csub(c[1], c[3])));
  }
}

// Cross twiddles omega_M^(p j), p = 1..8, of items j, from the global table
// [p - 1][L2] (consecutive lanes read consecutive elements).
template <int LM>
DEV void load_cross(float2 (&w)[8], const float2 *__restrict__ tw3, int j) {
#pragma unroll
  for (int p = 0; p < 8; ++p) w[p] = tw3[p * Tri<LM>::L2 + j];
}

// Forward: k1 = p by omega^(p j), its mirror by the conjugate.  The inverse
// applies the conjugates of those.
template <bool INV>
DEV void cross_twiddle(float2 (&v)[16], const float2 (&w)[8]) {
#pragma unroll
  for (int p = 1; p < 8; ++p) {
    v[p] = INV ? cmulc(v[p], w[p - 1]) : cmul(v[p], w[p - 1]);
    v[16 - p] = INV ? cmul(v[16 - p], w[p - 1]) : cmulc(v[16 - p], w[p - 1]);
  }
  v[8] = INV ? cmul(v[8], w[7]) : cmulc(v[8], w[7]);
}

// Block exchange after the forward cross stage: the two items' 2 x 16 values
// go out as (k1 = p, mirror) pairs, and each lane takes its wave-local
// transform's.  Pair p of the first / second item is put0 / put1[PP p], the
// lane's element t is get[GS t].
template <int LP, int PP, int GS>
DEV void cross_exchange_fwd(float2 (&v0)[16], float2 (&v1)[16], float2 *put0, float2 *put1,
                            const float2 *get) {
  float2 re[LP];
#pragma unroll
  for (int p = 0; p < 8; ++p) {
    put0[PP * p] = make_float2(v0[p].x, v0[mir(p)].x);
    put1[PP * p] = make_float2(v1[p].x, v1[mir(p)].x);
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < LP; ++t) re[t] = get[GS * t];
  __syncthreads();
#pragma unroll
  for (int p = 0; p < 8; ++p) {
    put0[PP * p] = make_float2(v0[p].y, v0[mir(p)].y);
    put1[PP * p] = make_float2(v1[p].y, v1[mir(p)].y);
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < LP; ++t) {
    const float2 im = get[GS * t];
    v0[t] = make_float2(re[t].x, im.x);
    v1[t] = make_float2(re[t].y, im.y);
  }
}

// The way back: lanes hold their wave-local transform's values (v0: k1 = p,
// v1: mirror) and take the 2 x 16 values of their two items.  The first
// writes go to the wavefront's own region, which only it has read since.
template <int LP, int PP, int GS>
DEV void cross_exchange_inv(float2 (&v0)[16], float2 (&v1)[16], float2 *put, const float2 *get0,
                            const float2 *get1) {
  float2 r0[8], r1[8];
  wave_sync();
#pragma unroll
  for (int t = 0; t < LP; ++t) put[GS * t] = make_float2(v0[t].x, v1[t].x);
  __syncthreads();
#pragma unroll
  for (int p = 0; p < 8; ++p) {
    r0[p] = get0[PP * p];
    r1[p] = get1[PP * p];
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < LP; ++t) put[GS * t] = make_float2(v0[t].y, v1[t].y);
  __syncthreads();
#pragma unroll
  for (int p = 0; p < 8; ++p) {
    const float2 i0 = get0[PP * p], i1 = get1[PP * p];
    v0[p] = make_float2(r0[p].x, i0.x);
    v0[mir(p)] = make_float2(r0[p].y, i0.y);
    v1[p] = make_float2(r1[p].x, i1.x);
    v1[mir(p)] = make_float2(r1[p].y, i1.y);
  }
}

// A value the compiler may not trace back: addresses and masks formed from it
// are formed where they are used and not kept (spilled) from an earlier use.
DEV int fresh(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

#define TRI_KERNEL(T) __global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(4)))

// LDS geometry of passes R and R': a wavefront is one pair p with the block's
// ROWS rows interleaved, so that lanes of one frequency are neighbours.
template <int LM>
struct RowGeo {
  using P = Tri<LM>;
  // item threads: row r, items j and j2; whether the second is this thread's own
  int r, j, j2;
  bool own2;
  // transform lanes: pair p, row rw, lane `it` of the transform
  int p, rw, it;
  DEV explicit RowGeo(int tid) {
    r = tid % P::ROWS;
    j = tid / P::ROWS;
    own2 = P::EXACT || j + P::HALF < P::L2;
    j2 = own2 ? j + P::HALF : P::L2 - 1;
    p = tid >> 6;
    rw = (tid & 63) % P::ROWS;
    it = (tid & 63) / P::ROWS;
    if (!P::EXACT) it = it < P::IW ? it : P::IW - 1;
  }
  // LDS element of an item in pair 0 (pair p lies REG p on), of this lane's
  // transform, and of its element 0 (NAT from one element to the next)
  static constexpr int NAT = P::pad(P::IW) * P::ROWS;
  DEV int item(int i) const { return P::pad(i) * P::ROWS + r; }
  DEV int region() const { return p * P::REG + rw; }
  DEV int natural() const { return region() + P::pad(it) * P::ROWS; }
};

// ---------------------------------------------------------------------------
// Pass R.  One block: ROWS rows.
// ---------------------------------------------------------------------------
template <int LM, int INM>
TRI_KERNEL(Tri<LM>::TROW) void k_tri_rows_fwd(KParams p) {
  using P = Tri<LM>;
  using G = RowGeo<LM>;
  constexpr int L2 = P::L2, IW = P::IW, T = P::TROW;
  __shared__ float2 lds[P::NP * P::REG];
  __shared__ LocalTw<LM> tw;
  const G g(threadIdx.x);
  const int y0 = xcd_tile(blockIdx.x, gridDim.x) * P::ROWS;
  const int n = p.n;
  float2 v0[16], v1[16];
  {
    // branch-free: a point outside the DOE reads a point inside and is
    // replaced by zero, so that all loads are in flight together
    const int y = y0 + g.r;
    const bool row = y < p.nrows_in;
    const size_t rowin = (size_t)(row ? y : 0) * n;
    const float *hrow = p.h + (size_t)((row ? y : 0) >> p.up_log2) * p.nh;
    auto load = [&](int x) {
      const bool in = row && x < n;
      const int xc = in ? x : 0;
      float2 v;
      if constexpr (INM == IN_PHASE) {
        v = make_float2(hrow[xc >> p.up_log2], p.amp ? p.amp[rowin + xc] : 1.f);
        v.y = in ? v.y : 0.f;
      } else {
        v = (INM == IN_FIELD ? p.u_in : p.saved_in)[rowin + xc];
        if constexpr (INM == IN_GRAD) v = cscale(v, p.two_wk * p.gpsf[rowin + xc]);
        v = in ? v : make_float2(0.f, 0.f);
      }
      return v;
    };
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      v0[t] = load(g.j + L2 * t);
      v1[t] = load(g.j2 + L2 * t);
    }
  }
  tw.fill(p.tw, T);
  if constexpr (INM == IN_PHASE) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      v0[t] = cscale(doe_phase(v0[t].x, p.phase_turns), v0[t].y);
      v1[t] = cscale(doe_phase(v1[t].x, p.phase_turns), v1[t].y);
    }
  }
  {
    float2 w[8];
    load_cross<LM>(w, p.tw3, g.j);
    dft16_half_in(v0);
    cross_twiddle<false>(v0, w);
    load_cross<LM>(w, p.tw3, g.j2);
    dft16_half_in(v1);
    cross_twiddle<false>(v1, w);
  }
  cross_exchange_fwd<P::LP, P::REG, G::NAT>(v0, v1, lds + g.item(g.j), lds + g.item(g.j2),
                                            lds + g.natural());
  local_dft<LM, P::ROWS, false>(v0, v1, lds + g.region(), g.it, tw);
  const int y = y0 + g.rw;
  if (y < p.nrows_in) {
    f4v *out = reinterpret_cast<f4v *>(p.ws) + y * P::QG;
#pragma unroll
    for (int t = 0; t < P::LP; ++t)
      out[P::pair_item(g.p * L2 + g.it + IW * t, p.pitch3)] = f4v{v0[t].x, v0[t].y, v1[t].x, v1[t].y};
  }
}

// ---------------------------------------------------------------------------
// Pass K.  One block: the column pair q, in place.
// ---------------------------------------------------------------------------
template <int LM>
TRI_KERNEL(Tri<LM>::TCOL) void k_tri_cols(KParams p) {
  using P = Tri<LM>;
  constexpr int M = P::M, L2 = P::L2, IW = P::IW, CR = P::CR, T = P::TCOL;
  __shared__ float2 lds[2 * P::NP * P::SUB];
  __shared__ LocalTw<LM> tw;
  const int q = xcd_tile(blockIdx.x, gridDim.x);
  f4v *col = reinterpret_cast<f4v *>(p.ws) + P::pair_item(q, p.pitch3);
  float2 v0[16], v1[16];  // item j of the cross stage in the two columns
  {
    const int j = P::EXACT ? threadIdx.x : min((int)threadIdx.x, L2 - 1);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int y = j + L2 * t;
      const bool in = y < p.nrows_in;
      const f4v x = col[in ? y * P::QG : 0];
      v0[t] = in ? make_float2(x.x, x.y) : make_float2(0.f, 0.f);
      v1[t] = in ? make_float2(x.z, x.w) : make_float2(0.f, 0.f);
    }
    tw.fill(p.tw, T);
    float2 w[8];
    load_cross<LM>(w, p.tw3, j);
    dft16_half_in(v0);
    sched_fence();
    cross_twiddle<false>(v0, w);
    sched_fence();
    dft16_half_in(v1);
    sched_fence();
    cross_twiddle<false>(v1, w);
  }
  // unit = (pair p, column c), P::NW of them per wavefront
  struct Place {
    int it, unit;
    float2 *item, *reg, *nat;  // column 0's pair 0, the unit's region, element 0
    DEV Place(float2 *lds, int tid) {
      const int lane = P::EXACT ? tid & 63 : min(tid & 63, IW * P::NW - 1);
      it = lane % IW;
      unit = (tid >> 6) * P::NW + lane / IW;
      item = lds + P::pad(P::EXACT ? tid : min(tid, L2 - 1));
      reg = lds + unit * P::SUB;
      nat = reg + P::pad(it);
    }
  };
  constexpr int NAT = P::pad(IW), PP = 2 * P::SUB, LP = P::LP;
  {
    const Place at(lds, fresh(threadIdx.x));
    cross_exchange_fwd<LP, PP, NAT>(v0, v1, at.item, at.item + P::SUB, at.nat);
    local_dft<LM, 1, false>(v0, v1, at.reg, at.it, tw);
  }
  {
    // this lane's kx, and its ky = pk + CR (it + IW t) with their partners
    const Place at(lds, fresh(threadIdx.x));
    const int it = at.it, pq = q / L2, kq = q % L2, pk = at.unit >> 1;
    int kx = pq + CR * kq;
    if (at.unit & 1) kx = M - (pq ? kx : kx + CR / 2);
    const double a2x = a2_eff(axis_freq(kx, M, p.inv_mdx, p.flim_x, p));
    auto h = [&](int ky) {
      return transfer(a2_eff(axis_freq(ky, M, p.inv_mdy, p.flim_y, p)), a2x, p);
    };
    if (pk) {
      const int ky0 = pk + CR * it;
#pragma unroll
      for (int t = 0; t < LP; ++t) {
        const float2 hv = h(fresh(ky0) + CR * IW * t);  // H(-ky) = H(ky)
        v0[t] = cmul(v0[t], hv);
        v1[t] = cmul(v1[t], hv);
        sched_fence();
      }
    } else {
#pragma unroll
      for (int t = 0; t < LP; ++t) {
        const int ky = fresh(CR * it) + CR * IW * t;
        v0[t] = cmul(v0[t], h(ky));
        sched_fence();
        v1[t] = cmul(v1[t], h(M - CR / 2 - ky));
        sched_fence();
      }
    }
  }
  {
    const Place at(lds, fresh(threadIdx.x));
    local_dft<LM, 1, true>(v0, v1, at.reg, at.it, tw);
    cross_exchange_inv<LP, PP, NAT>(v0, v1, at.nat, at.item, at.item + P::SUB);
  }
  const int j = P::EXACT ? fresh(threadIdx.x) : min(fresh(threadIdx.x), L2 - 1);
  {
    float2 w[8];
    load_cross<LM>(w, p.tw3, j);
    cross_twiddle<true>(v0, w);
    sched_fence();
    idft16_half_out(v0);
    sched_fence();
    cross_twiddle<true>(v1, w);
    sched_fence();
    idft16_half_out(v1);
  }
  if (p.nrows_out == M / 2) {
#pragma unroll
    for (int t = 0; t < 8; ++t)
      col[(j + L2 * t) * P::QG] = f4v{v0[t].x, v0[t].y, v1[t].x, v1[t].y};
  } else {
#pragma unroll
    for (int t = 0; t < 8; ++t)
      if (j + L2 * t < p.nrows_out)
        col[(j + L2 * t) * P::QG] = f4v{v0[t].x, v0[t].y, v1[t].x, v1[t].y};
  }
}

// ---------------------------------------------------------------------------
// Pass R'.  One block: ROWS rows, then the output stage of asm_kernels.hip's
// pass A': PSF accumulation (Eq. 4), field, or height gradient.
// ---------------------------------------------------------------------------
template <int LM, int OUTM>
TRI_KERNEL(Tri<LM>::TROW) void k_tri_rows_inv(KParams p) {
  using P = Tri<LM>;
  using G = RowGeo<LM>;
  constexpr int L2 = P::L2, IW = P::IW, T = P::TROW;
  __shared__ float2 lds[P::NP * P::REG];
  __shared__ LocalTw<LM> tw;
  const G g(threadIdx.x);
  const int y0 = xcd_tile(blockIdx.x, gridDim.x) * P::ROWS;
  const int n = p.n;
  float2 v0[16], v1[16];
  {
    const int y = y0 + g.rw;
    const f4v *in = reinterpret_cast<const f4v *>(p.ws) + (y < p.nrows_out ? y : 0) * P::QG;
#pragma unroll
    for (int t = 0; t < P::LP; ++t) {
      const f4v x = in[P::pair_item(g.p * L2 + g.it + IW * t, p.pitch3)];
      v0[t] = make_float2(x.x, x.y);
      v1[t] = make_float2(x.z, x.w);
    }
  }
  tw.fill(p.tw, T);
  __syncthreads();
  local_dft<LM, P::ROWS, true>(v0, v1, lds + g.region(), g.it, tw);
  cross_exchange_inv<P::LP, P::REG, G::NAT>(v0, v1, lds + g.natural(), lds + g.item(g.j),
                                            lds + g.item(g.j2));
  const int y = y0 + g.r;
  const bool live = y < p.nrows_out;
  const size_t row = (size_t)(live ? y : 0) * n;
  {
    float2 w[8];
    load_cross<LM>(w, p.tw3, g.j);
    cross_twiddle<true>(v0, w);
    sched_fence();
    idft16_half_out(v0);
    sched_fence();
    load_cross<LM>(w, p.tw3, g.j2);
    cross_twiddle<true>(v1, w);
    sched_fence();
    idft16_half_out(v1);
  }
  if (!live) return;
  // Value 2 t + i of this thread is column t of its item i.  Straight-line
  // loads, then straight-line stores: one branch on a DOE that fills the half
  // plane, where no column has to be masked.  (A repeated item is left out:
  // its sums would be added to twice.)
  const int j = fresh(g.j), j2 = fresh(g.j2);
  const bool own2 = g.own2;
  auto col = [&](int t) { return (t % 2 ? j2 : j) + L2 * (t / 2); };
  auto emit = [&](auto whole) {
    constexpr bool WHOLE = decltype(whole)::value;
    auto wanted = [&](int t) { return (WHOLE || col(t) < n) && (P::EXACT || t % 2 == 0 || own2); };
    auto value = [&](int t) { return t % 2 ? v1[t / 2] : v0[t / 2]; };
    float acc[16] = {};
    if (OUTM != OUT_FIELD && !p.first) {
      const float *sum = (OUTM == OUT_PSF ? p.psf : p.grad_h) + row;
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        const int x = col(t);
        acc[t] = sum[WHOLE || x < n ? x : 0];
      }
    }
    if constexpr (OUTM == OUT_GRADH) {
      const float *hrow = p.h + (size_t)(y >> p.up_log2) * p.nh;
      const float *arow = p.amp ? p.amp + row : nullptr;
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        const int x = col(t), xc = WHOLE || x < n ? x : 0;
        float2 e = doe_phase(hrow[xc >> p.up_log2], p.phase_turns);
        if (arow) e = cscale(e, arow[xc]);
        const float2 w = value(t);
        acc[t] = grad_add(acc[t], p.ck_m2, w, e);
      }
    } else if constexpr (OUTM == OUT_PSF) {
#pragma unroll
      for (int t = 0; t < 16; ++t) acc[t] = psf_add(acc[t], p.wk_m4, value(t));
    }
    if constexpr (OUTM != OUT_FIELD) {
      float *out = (OUTM == OUT_PSF ? p.psf : p.grad_h) + row;
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        const int x = col(t);
        if (wanted(t)) out[x] = acc[t];
      }
    }
    float2 *field = OUTM == OUT_FIELD ? p.u_out : OUTM == OUT_PSF ? p.saved_out : nullptr;
    if (OUTM != OUT_GRADH && field) {
      field += row;
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        const int x = col(t);
        if (wanted(t)) field[x] = cscale(value(t), p.inv_m2);
      }
    }
  };
  if (n == P::M / 2) emit(std::true_type{});
  else emit(std::false_type{});
}

void mark(hipEvent_t *ev, int i, hipStream_t s) {
  if (ev) (void)hipEventRecord(ev[i], s);
}

template <int LM>
hipError_t launch_lm(const KParams &p, hipStream_t s, hipEvent_t *ev) {
  using P = Tri<LM>;
  const dim3 gin((p.nrows_in + P::ROWS - 1) / P::ROWS), gout((p.nrows_out + P::ROWS - 1) / P::ROWS);
  const dim3 t(P::TROW);
  mark(ev, 0, s);
  if (p.in_mode == IN_PHASE)
    hipLaunchKernelGGL((k_tri_rows_fwd<LM, IN_PHASE>), gin, t, 0, s, p);
  else if (p.in_mode == IN_FIELD)
    hipLaunchKernelGGL((k_tri_rows_fwd<LM, IN_FIELD>), gin, t, 0, s, p);
  else
    hipLaunchKernelGGL((k_tri_rows_fwd<LM, IN_GRAD>), gin, t, 0, s, p);
  mark(ev, 1, s);
  hipLaunchKernelGGL(k_tri_cols<LM>, dim3(P::M / 2), dim3(P::TCOL), 0, s, p);
  mark(ev, 2, s);
  if (p.out_mode == OUT_PSF)
    hipLaunchKernelGGL((k_tri_rows_inv<LM, OUT_PSF>), gout, t, 0, s, p);
  else if (p.out_mode == OUT_FIELD)
    hipLaunchKernelGGL((k_tri_rows_inv<LM, OUT_FIELD>), gout, t, 0, s, p);
  else
    hipLaunchKernelGGL((k_tri_rows_inv<LM, OUT_GRADH>), gout, t, 0, s, p);
  mark(ev, 3, s);
  return hipGetLastError();
}

}  // namespace

// The grids of the path by plan id; 0: none.
int tri_grid(int plan) {
  return plan >= kTriMinLM && plan <= kTriMaxLM ? 1 << plan : plan == kTab3600 ? 3600 : 0;
}
static_assert(Tri<kTab3600>::M == 3600, "the table's 3600^2 grid");

bool tri_path(int plan, int n, int rows, bool full) {
  const int half = tri_grid(plan) / 2;
  return half && !full && n <= half && rows <= half;
}

// Items of QG pairs' rows, rounded up to an odd number of 128-byte lines.
int tri_pitch(int plan, int nrows) {
  const int qg = plan == 14 ? Tri<14>::QG : plan == 13 ? Tri<13>::QG : 1;
  return ((nrows * qg + 7) / 8 | 1) * 8;
}

hipError_t launch_tri(const KParams &p, hipStream_t s, hipEvent_t *ev) {
  // the kernels run one wavelength, in the window and half planes of tri_path
  if (p.group != 1 || p.nrows_out != p.nrows_in || !tri_path(p.plan, p.n, p.nrows_in, p.full))
    return hipErrorInvalidValue;
  switch (p.plan) {
    case 12: return launch_lm<12>(p, s, ev);
    case 13: return launch_lm<13>(p, s, ev);
    case 14: return launch_lm<14>(p, s, ev);
    case kTab3600: return launch_lm<kTab3600>(p, s, ev);
    default: return hipErrorInvalidValue;
  }
}
static_assert(kTriMinLM == 12 && kTriMaxLM == 14, "one launch case per grid");

}  // namespace dop
