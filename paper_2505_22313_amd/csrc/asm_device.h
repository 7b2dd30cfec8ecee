// Device helpers shared by the propagation kernels: complex arithmetic, the
// in-register DFTs, the tile order over the XCDs, and the element-wise
// physics (DOE phase, transfer function, PSF term).
#ifndef DOP_ASM_DEVICE_H_
#define DOP_ASM_DEVICE_H_

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "dop_internal.h"

namespace dop {

#define DEV __device__ __forceinline__

// ---------------------------------------------------------------------------
// complex helpers
// ---------------------------------------------------------------------------
DEV float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
DEV float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
DEV float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// a * conj(b)
DEV float2 cmulc(float2 a, float2 b) {
  return make_float2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}
DEV float2 mul_mi(float2 a) { return make_float2(a.y, -a.x); }   // -i a
DEV float2 mul_pi(float2 a) { return make_float2(-a.y, a.x); }   // +i a
DEV float2 cscale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }

// v * w16^q with w16 = exp(-2 pi i / 16) (forward) or its conjugate (INV).
// q is a compile-time constant after unrolling, so the switch folds away.
template <bool INV>
DEV float2 mulw16(float2 v, int q) {
  q &= 15;
  if (q == 0) return v;
  if (q == 4) return INV ? mul_pi(v) : mul_mi(v);
  if (q == 8) return make_float2(-v.x, -v.y);
  if (q == 12) return INV ? mul_mi(v) : mul_pi(v);
  // cos(2 pi q/16), sin(2 pi q/16)
  constexpr float C1 = 0.923879532511286756128f;  // cos(pi/8)
  constexpr float S1 = 0.382683432365089771728f;  // sin(pi/8)
  constexpr float RT = 0.707106781186547524401f;  // cos(pi/4)
  float c = 0.f, s = 0.f;
  switch (q) {
    case 1: c = C1; s = S1; break;
    case 2: c = RT; s = RT; break;
    case 3: c = S1; s = C1; break;
    case 5: c = -S1; s = C1; break;
    case 6: c = -RT; s = RT; break;
    case 7: c = -C1; s = S1; break;
    case 9: c = -C1; s = -S1; break;
    case 10: c = -RT; s = -RT; break;
    case 11: c = -S1; s = -C1; break;
    case 13: c = S1; s = -C1; break;
    case 14: c = RT; s = -RT; break;
    case 15: c = C1; s = -S1; break;
    default: break;
  }
  const float sn = INV ? s : -s;  // w = c + i*sn
  return make_float2(v.x * c - v.y * sn, v.x * sn + v.y * c);
}

// ---------------------------------------------------------------------------
// In-register DFTs of length 2, 4, 8, 16 (natural order in and out).
// Forward: X[k] = sum_n a[n] exp(-2 pi i n k / R); INV flips the sign.
// ---------------------------------------------------------------------------
template <int R, bool INV>
struct Dft;

template <bool INV>
struct Dft<1, INV> {
  DEV static void run(float2 *) {}
};

template <bool INV>
struct Dft<2, INV> {
  DEV static void run(float2 *a) {
    const float2 t = a[0];
    a[0] = cadd(t, a[1]);
    a[1] = csub(t, a[1]);
  }
};

template <bool INV>
struct Dft<4, INV> {
  DEV static void run(float2 *a) {
    const float2 t0 = cadd(a[0], a[2]), t1 = csub(a[0], a[2]);
    const float2 t2 = cadd(a[1], a[3]), t3 = csub(a[1], a[3]);
    const float2 it3 = INV ? mul_pi(t3) : mul_mi(t3);
    a[0] = cadd(t0, t2);
    a[2] = csub(t0, t2);
    a[1] = cadd(t1, it3);
    a[3] = csub(t1, it3);
  }
};

template <bool INV>
struct Dft<3, INV> {
  // X1,2 = a0 - (a1 + a2)/2 -/+ i (sqrt(3)/2) (a1 - a2)   (forward sign)
  DEV static void run(float2 *a) {
    constexpr float H = 0.866025403784438646764f;  // sin(2 pi / 3)
    const float2 t1 = cadd(a[1], a[2]);
    const float2 t2 = make_float2(a[0].x - 0.5f * t1.x, a[0].y - 0.5f * t1.y);
    const float2 d = cscale(csub(a[1], a[2]), H);
    const float2 t3 = INV ? mul_pi(d) : mul_mi(d);
    a[0] = cadd(a[0], t1);
    a[1] = cadd(t2, t3);
    a[2] = csub(t2, t3);
  }
};

template <bool INV>
struct Dft<5, INV> {
  // with t1 = a1 + a4, t2 = a2 + a3, t3 = a1 - a4, t4 = a2 - a3 (forward sign):
  // X1,4 = a0 + c1 t1 + c2 t2 -/+ i (s1 t3 + s2 t4)
  // X2,3 = a0 + c2 t1 + c1 t2 -/+ i (s2 t3 - s1 t4)
  DEV static void run(float2 *a) {
    constexpr float C1 = 0.309016994374947424102f;   // cos(2 pi / 5)
    constexpr float C2 = -0.809016994374947424102f;  // cos(4 pi / 5)
    constexpr float S1 = 0.951056516295153572116f;   // sin(2 pi / 5)
    constexpr float S2 = 0.587785252292473129169f;   // sin(4 pi / 5)
    const float2 t1 = cadd(a[1], a[4]), t2 = cadd(a[2], a[3]);
    const float2 t3 = csub(a[1], a[4]), t4 = csub(a[2], a[3]);
    const float2 r1 = make_float2(a[0].x + C1 * t1.x + C2 * t2.x, a[0].y + C1 * t1.y + C2 * t2.y);
    const float2 r2 = make_float2(a[0].x + C2 * t1.x + C1 * t2.x, a[0].y + C2 * t1.y + C1 * t2.y);
    const float2 q1 = make_float2(S1 * t3.x + S2 * t4.x, S1 * t3.y + S2 * t4.y);
    const float2 q2 = make_float2(S2 * t3.x - S1 * t4.x, S2 * t3.y - S1 * t4.y);
    const float2 i1 = INV ? mul_pi(q1) : mul_mi(q1);
    const float2 i2 = INV ? mul_pi(q2) : mul_mi(q2);
    a[0] = cadd(a[0], cadd(t1, t2));
    a[1] = cadd(r1, i1);
    a[4] = csub(r1, i1);
    a[2] = cadd(r2, i2);
    a[3] = csub(r2, i2);
  }
};

// cos(2 pi q / R) and sin(2 pi q / R), q < R, for the composite radices
// (values of the unit circle rounded to float).
template <int R>
struct UnitRoots;
template <>
struct UnitRoots<9> {
  static constexpr float c[9] = {
      1.000000000e+00f, 7.660444431e-01f, 1.736481777e-01f, -5.000000000e-01f,
      -9.396926208e-01f, -9.396926208e-01f, -5.000000000e-01f, 1.736481777e-01f,
      7.660444431e-01f};
  static constexpr float s[9] = {
      0.000000000e+00f, 6.427876097e-01f, 9.848077530e-01f, 8.660254038e-01f,
      3.420201433e-01f, -3.420201433e-01f, -8.660254038e-01f, -9.848077530e-01f,
      -6.427876097e-01f};
};
template <>
struct UnitRoots<15> {
  static constexpr float c[15] = {
      1.000000000e+00f, 9.135454576e-01f, 6.691306064e-01f, 3.090169944e-01f,
      -1.045284633e-01f, -5.000000000e-01f, -8.090169944e-01f, -9.781476007e-01f,
      -9.781476007e-01f, -8.090169944e-01f, -5.000000000e-01f, -1.045284633e-01f,
      3.090169944e-01f, 6.691306064e-01f, 9.135454576e-01f};
  static constexpr float s[15] = {
      0.000000000e+00f, 4.067366431e-01f, 7.431448255e-01f, 9.510565163e-01f,
      9.945218954e-01f, 8.660254038e-01f, 5.877852523e-01f, 2.079116908e-01f,
      -2.079116908e-01f, -5.877852523e-01f, -8.660254038e-01f, -9.945218954e-01f,
      -9.510565163e-01f, -7.431448255e-01f, -4.067366431e-01f};
};

template <>
struct UnitRoots<67> {
  static constexpr float c[67] = {
      1.000000000e+00f, 9.956059820e-01f, 9.824625429e-01f, 9.606851876e-01f,
      9.304652963e-01f, 8.920684426e-01f, 8.458320593e-01f, 7.921624734e-01f,
      7.315313353e-01f, 6.644714734e-01f, 5.915722124e-01f, 5.134741935e-01f,
      4.308637449e-01f, 3.444668503e-01f, 2.550427686e-01f, 1.633773618e-01f,
      7.027618895e-02f, -2.344257360e-02f, -1.169553220e-01f, -2.094402628e-01f,
      -3.000846350e-01f, -3.880918527e-01f, -4.726885052e-01f, -5.531311541e-01f,
      -6.287128666e-01f, -6.987694278e-01f, -7.626851781e-01f, -8.198984237e-01f,
      -8.699063724e-01f, -9.122695527e-01f, -9.466156753e-01f, -9.726429053e-01f,
      -9.901225145e-01f, -9.989008915e-01f, -9.989008915e-01f, -9.901225145e-01f,
      -9.726429053e-01f, -9.466156753e-01f, -9.122695527e-01f, -8.699063724e-01f,
      -8.198984237e-01f, -7.626851781e-01f, -6.987694278e-01f, -6.287128666e-01f,
      -5.531311541e-01f, -4.726885052e-01f, -3.880918527e-01f, -3.000846350e-01f,
      -2.094402628e-01f, -1.169553220e-01f, -2.344257360e-02f, 7.027618895e-02f,
      1.633773618e-01f, 2.550427686e-01f, 3.444668503e-01f, 4.308637449e-01f,
      5.134741935e-01f, 5.915722124e-01f, 6.644714734e-01f, 7.315313353e-01f,
      7.921624734e-01f, 8.458320593e-01f, 8.920684426e-01f, 9.304652963e-01f,
      9.606851876e-01f, 9.824625429e-01f, 9.956059820e-01f};
  static constexpr float s[67] = {
      0.000000000e+00f, 9.364148953e-02f, 1.864600543e-01f, 2.776400014e-01f,
      3.663800382e-01f, 4.519003140e-01f, 5.334492736e-01f, 6.103102618e-01f,
      6.818078216e-01f, 7.473136296e-01f, 8.062520186e-01f, 8.581050359e-01f,
      9.024169952e-01f, 9.387984816e-01f, 9.669297732e-01f, 9.865636511e-01f,
      9.975275722e-01f, 9.997251851e-01f, 9.931371772e-01f, 9.778214440e-01f,
      9.539125808e-01f, 9.216206996e-01f, 8.812295825e-01f, 8.330941882e-01f,
      7.776375321e-01f, 7.153469695e-01f, 6.467699120e-01f, 5.725090173e-01f,
      4.932168927e-01f, 4.095903603e-01f, 3.223643332e-01f, 2.323053566e-01f,
      1.402048723e-01f, 4.687226247e-02f, -4.687226247e-02f, -1.402048723e-01f,
      -2.323053566e-01f, -3.223643332e-01f, -4.095903603e-01f, -4.932168927e-01f,
      -5.725090173e-01f, -6.467699120e-01f, -7.153469695e-01f, -7.776375321e-01f,
      -8.330941882e-01f, -8.812295825e-01f, -9.216206996e-01f, -9.539125808e-01f,
      -9.778214440e-01f, -9.931371772e-01f, -9.997251851e-01f, -9.975275722e-01f,
      -9.865636511e-01f, -9.669297732e-01f, -9.387984816e-01f, -9.024169952e-01f,
      -8.581050359e-01f, -8.062520186e-01f, -7.473136296e-01f, -6.818078216e-01f,
      -6.103102618e-01f, -5.334492736e-01f, -4.519003140e-01f, -3.663800382e-01f,
      -2.776400014e-01f, -1.864600543e-01f, -9.364148953e-02f};
};

// R = R1 * R2 from two in-register DFTs (four-step split n = n1 R2 + n2,
// k = k1 + R1 k2, twiddles omega_R^(n2 k1) from UnitRoots<R>).
template <int R1, int R2, bool INV>
struct DftComposite {
  static constexpr int R = R1 * R2;
  DEV static void run(float2 *a) {
    float2 t[R];
#pragma unroll
    for (int n2 = 0; n2 < R2; ++n2) {
      float2 b[R1];
#pragma unroll
      for (int n1 = 0; n1 < R1; ++n1) b[n1] = a[n1 * R2 + n2];
      Dft<R1, INV>::run(b);
#pragma unroll
      for (int k1 = 0; k1 < R1; ++k1) {
        const int q = (n2 * k1) % R;
        if (q == 0) {
          t[k1 * R2 + n2] = b[k1];
        } else {
          const float c = UnitRoots<R>::c[q];
          const float sn = INV ? UnitRoots<R>::s[q] : -UnitRoots<R>::s[q];
          t[k1 * R2 + n2] = make_float2(b[k1].x * c - b[k1].y * sn, b[k1].x * sn + b[k1].y * c);
        }
      }
    }
#pragma unroll
    for (int k1 = 0; k1 < R1; ++k1) {
      float2 c[R2];
#pragma unroll
      for (int n2 = 0; n2 < R2; ++n2) c[n2] = t[k1 * R2 + n2];
      Dft<R2, INV>::run(c);
#pragma unroll
      for (int k2 = 0; k2 < R2; ++k2) a[k1 + R1 * k2] = c[k2];
    }
  }
};

template <bool INV>
struct Dft<9, INV> : DftComposite<3, 3, INV> {};
template <bool INV>
struct Dft<15, INV> : DftComposite<3, 5, INV> {};

// R = 4 * R2 (R = 8, 16): four-step split n = n1*R2 + n2, k = k1 + 4*k2.
template <int R, bool INV>
struct Dft {
  static_assert(R == 8 || R == 16, "radix");
  static constexpr int R2 = R / 4;
  DEV static void run(float2 *a) {
    float2 t[R];
#pragma unroll
    for (int n2 = 0; n2 < R2; ++n2) {
      float2 b[4];
#pragma unroll
      for (int n1 = 0; n1 < 4; ++n1) b[n1] = a[n1 * R2 + n2];
      Dft<4, INV>::run(b);
#pragma unroll
      for (int k1 = 0; k1 < 4; ++k1)
        t[k1 * R2 + n2] = mulw16<INV>(b[k1], n2 * k1 * (16 / R));
    }
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1) {
      float2 c[R2];
#pragma unroll
      for (int n2 = 0; n2 < R2; ++n2) c[n2] = t[k1 * R2 + n2];
      Dft<R2, INV>::run(c);
#pragma unroll
      for (int k2 = 0; k2 < R2; ++k2) a[k1 + 4 * k2] = c[k2];
    }
  }
};

typedef float f4v __attribute__((ext_vector_type(4)));

// Tiles per launch are walked by a grid of resident blocks.  Blocks are
// handed to the eight XCDs round-robin, so tile ids are permuted within each
// run of 64 to give every XCD eight consecutive tiles at a time (neighbouring
// tiles share cache lines and DRAM pages).
constexpr int kMaxBlocks = 4096;
DEV int xcd_tile(int p, int ntiles) {
  if (p >= (ntiles & ~63)) return p;
  return (p & ~63) | ((p & 7) << 3) | ((p >> 3) & 7);
}

// ---------------------------------------------------------------------------
// Element-wise physics.
// ---------------------------------------------------------------------------

// exp(i 2 pi f) for f in [-1/2, 1/2] turn: the hardware sine and cosine take
// their argument in turns (max abs error 1.3e-7 over [-1/2, 1/2], measured
// against FP64 on gfx950).
DEV float2 cis_turns(float f) {
  return make_float2(__builtin_amdgcn_cosf(f), __builtin_amdgcn_sinf(f));
}

// exp(i 2 pi q), q = turns_per_h * h formed in FP64 and reduced to
// [-1/2, 1/2] turn before the cast to FP32 (Eq. 1-2).
DEV float2 doe_phase(float hv, double turns_per_h) {
  const double q = turns_per_h * (double)hv;
  return cis_turns((float)(q - rint(q)));
}

// sqrt(q) for q in (0, 1] in FP64: FP32 reciprocal-square-root seed (relative
// error below 2^-22) and one Goldschmidt iteration, which squares the error:
// below 3e-14 relative.  Times z/lambda <= 2^17 turns that is under 4e-9 turn
// of phase, far below the 1.3e-7 turn error of the FP32 sin/cos that follows.
DEV double sqrt_unit(double q) {
  const double r = (double)__builtin_amdgcn_rsqf((float)q);
  const double g = q * r, h = 0.5 * r;
  const double e = fma(-g, h, 0.5);
  return fma(g, e, g);
}

// Per-axis frequency data of DFT bin k of an M-point axis: f = k_signed / (M dx), the
// square (lambda f)^2 with each product rounded once in FP64 (no
// contraction), as the evanescent test needs, and whether |f| is inside the
// band limit (always, unless DOP_BANDLIMIT).
struct AxisFreq {
  double a2;
  bool inband;
};
DEV AxisFreq axis_freq(int k, int m, double inv_md, double flim, double lam) {
#pragma clang fp contract(off)
  const int ks = k < (m >> 1) ? k : k - m;
  const double f = (double)ks * inv_md;
  const double a = lam * f;
  return AxisFreq{a * a, fabs(f) < flim};
}
DEV AxisFreq axis_freq(int k, int m, double inv_md, double flim, const KParams &p) {
  return axis_freq(k, m, inv_md, flim, p.lam);
}

// (lambda f)^2 of one axis with the band limit folded in: a frequency outside
// the band gets 2, so that s >= 1 below whatever the other axis holds (an
// in-band s is unchanged).
DEV double a2_eff(AxisFreq f) { return f.inband ? f.a2 : 2.0; }

// H(ky, kx) from the two axes' a2_eff: zero unless s = a2y + a2x < 1; else
// exp(i 2 pi zl sqrt(1 - s)) with the argument formed and reduced mod one
// turn in FP64.  zl = z / lambda, negated for the adjoint (conj(H) is H at
// -z).  The inverse DFT's 1/M^2 is left to the last pass's output constants.
// Branch-free: cut bins evaluate a harmless dummy root (1 - s is floored at
// 2^-60, below any propagating 1 - s >= 2^-53) and are replaced by zero.
DEV float2 transfer(double a2y, double a2x, double zl) {
#pragma clang fp contract(off)
  const double s = a2y + a2x;
  const double t = zl * sqrt_unit(fmax(1.0 - s, 0x1p-60));
  const float2 w = cis_turns((float)(t - rint(t)));
  return s < 1.0 ? w : make_float2(0.f, 0.f);
}
DEV float2 transfer(double a2y, double a2x, const KParams &p) { return transfer(a2y, a2x, p.zl); }

// Entry q of a per-group constant, selected with constant indices: indexing
// a kernel-argument array with a run-time value would copy the whole
// parameter block to scratch memory.
template <class T>
DEV T group_value(const T (&a)[kMaxGroup], int q) {
  static_assert(kMaxGroup == 4, "one select per entry");
  return q == 0 ? a[0] : q == 1 ? a[1] : q == 2 ? a[2] : a[3];
}

// One wavelength's term of the PSF (Eq. 4) added to an accumulator: acc +
// w_k |U|^2 with U = w / (My Mx) folded into wk.  Shared by the per-wavelength
// and the grouped output stages, with the fused operations spelled out, so
// that all round alike however the compiler arranges the code around it.
DEV float psf_add(float acc, float wk, float2 w) {
  return fmaf(wk, fmaf(w.x, w.x, w.y * w.y), acc);
}

// One wavelength's term of the height gradient: acc + ck Im(g_E conj(E)).
DEV float grad_add(float acc, float ck, float2 w, float2 e) {
  return fmaf(ck, fmaf(w.y, e.x, -(w.x * e.y)), acc);
}

// Element at a 32-bit byte offset from a block-uniform base: the offset is
// formed in 32-bit arithmetic so the access can take a scalar base plus one
// 32-bit vector offset instead of a 64-bit address per lane.
template <class T>
DEV T *at_byte(T *base, unsigned off) {
  return reinterpret_cast<T *>(reinterpret_cast<char *>(base) + off);
}
template <class T>
DEV const T *at_byte(const T *base, unsigned off) {
  return reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + off);
}

}  // namespace dop

#endif  // DOP_ASM_DEVICE_H_
