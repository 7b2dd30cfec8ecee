// Super-resolved front end: the coarse design is filled onto the simulation
// grid by a separable interpolation kernel (paper Sec. 3.2, Table 2), and the
// design gradient is carried back by the adjoint map.
//
//   fine = Wy coarse Wx^T,   grad_coarse = Wy^T grad_fine Wx,   W: (nc s) x nc
//
// for a coarse design of ncy rows and ncx columns (each axis has its own W).
//
// Nearest: W[j][i] = [i == j / s].  Lanczos-3: fine sample j sits at coarse
// coordinate u_j = (j + 0.5)/s - 0.5 and takes the six coarse samples
// i0 .. i0+5, i0 = floor(u_j) - 2, weighted by L(u_j - i) with
// L(x) = sinc(x) sinc(x/3) (zero for |x| >= 3 and for i outside [0, nc)),
// each row divided by its sum.  Weights are formed in FP64 and rounded to
// float32; the sums run in float32.
//
// The fine map is s^2 times the coarse one, so both directions are bound by
// streaming it once: a thread walks down fine columns with a window of six
// coarse rows in registers (interpolated rows forward, partial sums in the
// adjoint), and the taps of a row are the same for the whole block.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "dop_internal.h"

namespace dop {
namespace {

#define DEV __device__ __forceinline__

constexpr int kUpMaxS = 16;

// Lanczos-3 kernel L(x) = sinc(x) sinc(x/3), |x| < 3.
DEV double lanczos3(double x) {
  const double ax = fabs(x);
  if (ax >= 3.0) return 0.0;
  if (ax == 0.0) return 1.0;
  return 3.0 * sinpi(x) * sinpi(x / 3.0) / (M_PI * M_PI * x * x);
}

// Fine sample j = q s + r sits at coarse coordinate u = q + f_r with
// f_r = (r + 0.5)/s - 0.5 in (-1/2, 1/2), so its first tap i0 = floor(u) - 2
// = q + shift_r and its offsets u - i depend on the residue r only.  A block
// tabulates, per residue, the raw kernel values L(u - i0 - t) (FP64) and the
// normalised weights of an interior sample; a sample whose taps leave
// [0, nc) renormalises over the taps inside.
struct TapTable {
  double raw[kUpMaxS][6];
  float wint[kUpMaxS][6];
  int shift[kUpMaxS];
};

// All threads of the block must call; one kernel value per thread, so that
// the FP64 sines of a residue do not queue up in one lane.
DEV void tap_table_fill(TapTable &tt, int s) {
  for (int e = threadIdx.x; e < 6 * s; e += blockDim.x) {
    const int r = e / 6, t = e % 6;
    const double f = ((double)r + 0.5) / (double)s - 0.5;
    const int fl = f < 0.0 ? -1 : 0;
    tt.raw[r][t] = lanczos3(f - (double)(fl - 2 + t));
    if (t == 0) tt.shift[r] = fl - 2;
  }
  __syncthreads();
  for (int r = threadIdx.x; r < s; r += blockDim.x) {
    double sum = 0.0;
#pragma unroll
    for (int t = 0; t < 6; ++t) sum += tt.raw[r][t];
#pragma unroll
    for (int t = 0; t < 6; ++t) tt.wint[r][t] = (float)(tt.raw[r][t] / sum);
  }
  __syncthreads();
}

// Taps of fine sample j: returns i0 and writes the six normalised weights of
// coarse samples i0 .. i0+5 (zero outside [0, nc)).
DEV int lanczos_taps(int j, int s, int nc, const TapTable &tt, float *w) {
  const int q = j / s, r = j - q * s;
  const int i0 = q + tt.shift[r];
  if (i0 >= 0 && i0 + 5 < nc) {
#pragma unroll
    for (int t = 0; t < 6; ++t) w[t] = tt.wint[r][t];
  } else {
    double v[6];
    double sum = 0.0;
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      v[t] = (i0 + t >= 0 && i0 + t < nc) ? tt.raw[r][t] : 0.0;
      sum += v[t];
    }
#pragma unroll
    for (int t = 0; t < 6; ++t) w[t] = (float)(v[t] / sum);
  }
  return i0;
}

// ---------------------------------------------------------------------------
// Nearest neighbour.
// ---------------------------------------------------------------------------
typedef float f4v __attribute__((ext_vector_type(4)));

// One thread: V adjacent fine columns of the s rows of a coarse row (V = 4
// with 16-byte stores where every row starts on a 16-byte boundary).
template <int V>
__global__ __launch_bounds__(256) void k_up_nearest(int ncy, int ncx, int s,
                                                    const float *__restrict__ in,
                                                    float *__restrict__ out) {
  const int nfx = ncx * s, nv = nfx / V;
  for (int i = blockIdx.y; i < ncy; i += gridDim.y) {
    const float *src = in + (size_t)i * ncx;
    float *dst = out + (size_t)i * s * nfx;
    for (int x = blockIdx.x * blockDim.x + threadIdx.x; x < nv; x += gridDim.x * blockDim.x) {
      if constexpr (V == 4) {
        const f4v v = f4v{src[4 * x / s], src[(4 * x + 1) / s], src[(4 * x + 2) / s],
                          src[(4 * x + 3) / s]};
        for (int dy = 0; dy < s; ++dy)
          *reinterpret_cast<f4v *>(dst + (size_t)dy * nfx + 4 * x) = v;
      } else {
        const float v = src[x / s];
        for (int dy = 0; dy < s; ++dy) dst[(size_t)dy * nfx + x] = v;
      }
    }
  }
}

// Sum of each s x s block of a (ncy s) x (ncx s) map, rows in order, columns
// in order within a row.  S > 0: s = S, a multiple of 4, read as 16-byte
// vectors (rows start on 16-byte boundaries), so that a wavefront's loads
// cover whole lines; S = 0: any s.  14400^2, s = 8: 457 us at S = 0, 152 us
// at S = 8 (5.5 TB/s), the same bits.
template <int S>
__global__ __launch_bounds__(256) void k_up_nearest_adj(int ncy, int ncx, int s,
                                                        const float *__restrict__ g,
                                                        float *__restrict__ out) {
  const int nfx = ncx * s;
  for (int i = blockIdx.y; i < ncy; i += gridDim.y) {
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < ncx; k += gridDim.x * blockDim.x) {
      float a = 0.f;
      if constexpr (S > 0) {
        f4v v[4][S / 4];
#pragma unroll
        for (int d0 = 0; d0 < S; d0 += 4) {
#pragma unroll
          for (int dy = 0; dy < 4; ++dy)
#pragma unroll
            for (int c = 0; c < S / 4; ++c)
              v[dy][c] = *reinterpret_cast<const f4v *>(g + (size_t)(i * S + d0 + dy) * nfx +
                                                        (size_t)k * S + 4 * c);
#pragma unroll
          for (int dy = 0; dy < 4; ++dy)
#pragma unroll
            for (int c = 0; c < S / 4; ++c) a = (((a + v[dy][c].x) + v[dy][c].y) + v[dy][c].z) + v[dy][c].w;
        }
      } else {
        for (int dy = 0; dy < s; ++dy) {
          const float *row = g + (size_t)(i * s + dy) * nfx + (size_t)k * s;
          for (int dx = 0; dx < s; ++dx) a += row[dx];
        }
      }
      out[(size_t)i * ncx + k] = a;
    }
  }
}

// The fine samples whose first tap is b are the s samples from seg_lo(b) on
// (some of them outside the grid): floor(u_j) = b + 2 there.
DEV int seg_lo(int b, int s) { return s * (b + 2) + s / 2; }

// ---------------------------------------------------------------------------
// Lanczos-3, forward.  A block interpolates its coarse rows along x once, into
// LDS, its four wavefronts taking rows in turn; then each wavefront walks down
// nseg segments of s fine rows that share their six coarse rows, the window of
// six in registers, so that a fine sample costs six multiply-adds.  A thread
// owns COLS fine columns: four (adjacent and stored as one 16-byte vector where
// every fine row starts on a 16-byte boundary, V4; else 64 apart, so that a
// wavefront stores whole lines), or one.  The launcher picks the columns and
// the segment count so that small and narrow maps still fill the chip.
// 2048^2, s = 8 (1.09 GB): 647 -> 220 us, of the 215 that plain stores take; a
// tile in LDS spent its time on two LDS reads per product and on FP64 taps per
// 4096 samples.  The taps of all the block's rows are formed at its start:
// formed per segment, they kept s = 1 at 510 us on 8192^2 (now 289).
// ---------------------------------------------------------------------------
constexpr int kUpRows = 256;  // fine rows per block, at most: one row's taps per thread
// segments per wavefront, at most, where a thread owns `cols` columns
__host__ __device__ constexpr int up_max_seg(int cols, int s) {
  return cols == 4 ? 4 : 64 / s < 16 ? 64 / s : 16;
}

// NEAR > 0 (V4 only): the first taps of a thread's four columns lie within
// NEAR samples of each other (1 for s >= 3, 2 for s = 2, 3 for s = 1), so 6 +
// NEAR samples serve them all.
template <bool V4, int NEAR, int COLS = 4>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_up_lanczos(int ncy, int ncx, int s, int nseg,
                                                    const float *__restrict__ in,
                                                    float *__restrict__ out) {
  const int nfy = ncy * s, nfx = ncx * s;
  constexpr int SPAN = 64 * COLS;  // fine columns per block
  __shared__ TapTable tt;
  // taps of the block's fine rows
  __shared__ __align__(16) float rws[kUpRows][8];
  // coarse rows interpolated along x, from the block's first on; [lane][column]
  // (before them, the taps of the block's fine columns)
  __shared__ __align__(16) float hs[4 * up_max_seg(COLS, 1) + 5][SPAN];
  float (*const cws)[SPAN] = hs;
  int *const cxs = reinterpret_cast<int *>(hs[6]);
  tap_table_fill(tt, s);
  // segments -3 .. ncy - 2 cover the fine rows
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int bb = -3 + (int)blockIdx.y * 4 * nseg, b0 = bb + wave * nseg;
  const int b1 = min(b0 + nseg, ncy - 1);
  {
    float w[6];
    if (threadIdx.x < SPAN) {
      cxs[threadIdx.x] =
          lanczos_taps(min((int)(blockIdx.x * SPAN + threadIdx.x), nfx - 1), s, ncx, tt, w);
#pragma unroll
      for (int t = 0; t < 6; ++t) cws[t][threadIdx.x] = w[t];
    }
    const int e = threadIdx.x, j = seg_lo(bb, s) + e;
    if (e < 4 * nseg * s && j >= 0 && j < nfy) {
      lanczos_taps(j, s, ncy, tt, w);
#pragma unroll
      for (int t = 0; t < 6; ++t) rws[e][t] = w[t];
    }
  }
  __syncthreads();
  auto col = [&](int c) { return V4 ? 4 * lane + c : lane + 64 * c; };
  const int x0 = blockIdx.x * SPAN;
  int cx[COLS];
  float cw[COLS][6];
#pragma unroll
  for (int c = 0; c < COLS; ++c) {
    cx[c] = cxs[col(c)];
#pragma unroll
    for (int t = 0; t < 6; ++t) cw[c][t] = cws[t][col(c)];
  }
  __syncthreads();  // the column taps have been read
  // coarse row `row` interpolated at this thread's columns (taps outside the
  // grid have weight zero and their samples count as zero)
  auto interp = [&](int row, float (&o)[COLS]) {
    const float *src = in + (size_t)min(max(row, 0), ncy - 1) * ncx;
    const bool live = row >= 0 && row < ncy;
    auto sample = [&](int x) {
      const float v = src[min(max(x, 0), ncx - 1)];
      return x >= 0 && x < ncx ? v : 0.f;
    };
    float near[6 + NEAR];
    if constexpr (NEAR > 0) {
#pragma unroll
      for (int t = 0; t < 6 + NEAR; ++t) near[t] = sample(cx[0] + t);
    }
    auto tap = [&](int c, int t) {
      if constexpr (NEAR == 0) {
        return sample(cx[c] + t);
      } else if constexpr (NEAR == 3) {  // s = 1: neighbouring first taps
        return near[t + c];
      } else {
        float v = near[t];
#pragma unroll
        for (int d = 1; d <= NEAR; ++d) v = cx[c] == cx[0] + d ? near[t + d] : v;
        return v;
      }
    };
#pragma unroll
    for (int c = 0; c < COLS; ++c) {
      float a = 0.f;
#pragma unroll
      for (int t = 0; t < 6; ++t) a += cw[c][t] * tap(c, t);
      o[c] = live ? a : 0.f;
    }
  };
#pragma unroll 2
  for (int e = wave; e < 4 * nseg + 5; e += 4) {
    float o[COLS];
    interp(bb + e, o);
    if constexpr (COLS == 4) {
      *reinterpret_cast<f4v *>(&hs[e][4 * lane]) = f4v{o[0], o[1], o[2], o[3]};
    } else {
      hs[e][lane] = o[0];
    }
  }
  __syncthreads();
  float win[6][COLS];
  auto row_in = [&](int row, float (&o)[COLS]) {
    if constexpr (COLS == 4) {
      const f4v v = *reinterpret_cast<const f4v *>(&hs[row - bb][4 * lane]);
      o[0] = v.x, o[1] = v.y, o[2] = v.z, o[3] = v.w;
    } else {
      o[0] = hs[row - bb][lane];
    }
  };
#pragma unroll
  for (int t = 0; t < 5; ++t) row_in(b0 + t, win[t + 1]);
  for (int b = b0; b < b1; ++b) {
#pragma unroll
    for (int t = 0; t < 5; ++t)
#pragma unroll
      for (int c = 0; c < COLS; ++c) win[t][c] = win[t + 1][c];
    row_in(b + 5, win[5]);
    const int lo = seg_lo(b, s);
    const int j0 = max(lo, 0), j1 = min(lo + s, nfy);
#pragma unroll 4
    for (int j = j0; j < j1; ++j) {
      const float *rw = rws[(b - bb) * s + j - lo];
      float *dst = out + (size_t)j * nfx + x0;
      float a[COLS];
#pragma unroll
      for (int c = 0; c < COLS; ++c) {
        a[c] = 0.f;
#pragma unroll
        for (int t = 0; t < 6; ++t) a[c] += rw[t] * win[t][c];
      }
      if constexpr (V4) {
        if (x0 + 4 * lane < nfx)
          *reinterpret_cast<f4v *>(dst + 4 * lane) = f4v{a[0], a[1], a[2], a[3]};
      } else {
#pragma unroll
        for (int c = 0; c < COLS; ++c)
          if (x0 + col(c) < nfx) dst[col(c)] = a[c];
      }
    }
  }
}
static_assert(4 * up_max_seg(4, 1) * kUpMaxS <= kUpRows, "taps of a block's rows");

// ---------------------------------------------------------------------------
// Lanczos-3, adjoint.  The same walk with six coarse rows of partial sums: a
// fine sample adds to all six, and when a segment ends its first row is
// complete along y.  That row goes to LDS, where each thread sums the fine
// columns of its coarse samples.  A block has SPAN fine columns and the
// coarse columns whose taps lie among them; a thread has COLS of them, four, or
// one where the map is that narrow (8000 x 8, s = 1: 24.8 -> 13.7 us, from the
// taps of fewer columns and five blocks on a CU instead of three).  V4: a
// thread's fine columns are
// one 16-byte vector (rows start on 16-byte boundaries, and the block's first
// column is rounded down to one).  2048^2, s = 8: 2255 -> 303 us (3.6 TB/s);
// the former tile of 16 x 16 coarse samples read the fine map 1.9 times and
// tested each of its samples for each coarse one.
// ---------------------------------------------------------------------------
constexpr int kAdjThreads = 256;
constexpr int kAdjMaxRows = 560;  // fine rows of a block, (rows + 5) s: three blocks share a CU

// coarse columns per block: the fine columns from seg_lo(k0 - 5) to the end
// of segment k0 + n - 1
__host__ __device__ constexpr int adj_groups(int s, int cols) { return (kAdjThreads * cols - 3) / s; }
__host__ __device__ constexpr int adj_cols(int s, int cols) { return adj_groups(s, cols) - 5; }

template <bool V4, int COLS = 4>
__global__ __launch_bounds__(kAdjThreads) void k_up_lanczos_adj(int ncy, int ncx, int s, int nrow,
                                                                const float *__restrict__ g,
                                                                float *__restrict__ out) {
  constexpr int SPAN = kAdjThreads * COLS;
  const int nfy = ncy * s, nfx = ncx * s;
  __shared__ TapTable tt;
  // taps of the block's fine rows, and of its fine columns; column x of the
  // block is residue x % s of group x / s, stored [residue][group] (with an
  // odd pitch) so that threads of neighbouring coarse
  // columns read neighbouring words
  __shared__ __align__(16) float rw[kAdjMaxRows][8];
  __shared__ float cw[6][SPAN + 16], vs[2][SPAN + 16];
  const int i0 = blockIdx.y * nrow, i1 = min(i0 + nrow, ncy);
  const int kc = adj_cols(s, COLS), k0 = blockIdx.x * kc, k1 = min(k0 + kc, ncx);
  const int j00 = seg_lo(i0 - 5, s), x00 = seg_lo(k0 - 5, s);
  const int ng = adj_groups(s, COLS), pitch = ng | 1;
  const int tid = threadIdx.x;
  tap_table_fill(tt, s);
  for (int e = tid; e < (i1 - i0 + 5) * s; e += kAdjThreads) {
    const int j = j00 + e;
    if (j >= 0 && j < nfy) lanczos_taps(j, s, ncy, tt, rw[e]);
  }
  for (int e = tid; e < ng * s; e += kAdjThreads) {
    const int x = x00 + e, at = (e % s) * pitch + e / s;
    float w[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (x >= 0 && x < nfx) lanczos_taps(x, s, ncx, tt, w);
#pragma unroll
    for (int t = 0; t < 6; ++t) cw[t][at] = w[t];
  }
  // this thread's fine columns: where they are read, whether they count, and
  // their words of vs (a spare one for columns outside the block's groups)
  const int xa = V4 ? x00 & ~3 : x00;  // rounds towards minus infinity
  int xc[COLS], at[COLS];
  bool in[COLS];
#pragma unroll
  for (int c = 0; c < COLS; ++c) {
    const int x = xa + (V4 ? COLS * tid + c : tid + c * kAdjThreads), e = x - x00;
    in[c] = x >= 0 && x < nfx;
    xc[c] = in[c] ? x : 0;
    at[c] = e >= 0 && e < ng * s ? (e % s) * pitch + e / s : SPAN + 15;
  }
  __syncthreads();
  float acc[6][COLS] = {};
  for (int b = i0 - 5; b < i1; ++b) {
    const int lo = seg_lo(b, s);
    const int j0 = max(lo, 0), j1 = min(lo + s, nfy);
#pragma unroll 4
    for (int j = j0; j < j1; ++j) {
      const float *row = g + (size_t)j * nfx;
      const float *w = rw[j - j00];
      float v[COLS];
#pragma unroll
      for (int c = 0; c < COLS; ++c)
        if constexpr (!V4) v[c] = row[xc[c]];
      if constexpr (V4) {
        const f4v q = *reinterpret_cast<const f4v *>(row + xc[0]);
        v[0] = q.x, v[1] = q.y, v[2] = q.z, v[3] = q.w;
      }
#pragma unroll
      for (int c = 0; c < COLS; ++c) v[c] = in[c] ? v[c] : 0.f;
#pragma unroll
      for (int t = 0; t < 6; ++t)
#pragma unroll
        for (int c = 0; c < COLS; ++c) acc[t][c] += w[t] * v[c];
    }
    if (b >= i0) {
      float *line = vs[b & 1];  // the other line may still be read
#pragma unroll
      for (int c = 0; c < COLS; ++c) line[at[c]] = acc[0][c];
      __syncthreads();
      // coarse column k takes tap t of the columns of segment k - t, which is
      // group k - t - (k0 - 5)
      for (int k = k0 + tid; k < k1; k += kAdjThreads) {
        float a = 0.f;
#pragma unroll
        for (int t = 5; t >= 0; --t) {
          const int grp = k - k0 + 5 - t;
#pragma unroll 4
          for (int r = 0; r < s; ++r) a += cw[t][r * pitch + grp] * line[r * pitch + grp];
        }
        out[(size_t)b * ncx + k] = a;
      }
    }
#pragma unroll
    for (int t = 0; t < 6; ++t)
#pragma unroll
      for (int c = 0; c < COLS; ++c) acc[t][c] = t < 5 ? acc[t + 1][c] : 0.f;
  }
}

unsigned cdiv(int a, int b) { return (unsigned)((a + b - 1) / b); }

bool aligned16(const void *p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }

}  // namespace

hipError_t launch_upsample(int kind, int ncy, int ncx, int s, const float *coarse, float *fine,
                           hipStream_t stream) {
  const int nfx = ncx * s;
  if (kind == 0) {
    const bool v4 = nfx % 4 == 0 && aligned16(fine);
    const unsigned bx = cdiv(v4 ? nfx / 4 : nfx, 256);
    const dim3 grid(bx < 64 ? bx : 64, ncy < 4096 ? ncy : 4096);
    if (v4)
      hipLaunchKernelGGL(k_up_nearest<4>, grid, dim3(256), 0, stream, ncy, ncx, s, coarse, fine);
    else
      hipLaunchKernelGGL(k_up_nearest<1>, grid, dim3(256), 0, stream, ncy, ncx, s, coarse, fine);
  } else {
    // ncy + 2 segments of rows, 4 nseg per block (whose LDS starts with five
    // more rows): fewer while the chip has not two or three blocks for each CU
    // (at 1024 blocks and more a second, partly filled round of them began:
    // 600 x 599, s = 2, 722 blocks 9.3 us, 1444 blocks 11.4)
    const bool v4 = nfx % 4 == 0 && aligned16(fine);
    auto blocks = [&](int cols, int n) { return (long long)cdiv(nfx, 64 * cols) * cdiv(ncy + 2, 4 * n); };
    // One column per thread where four leave lanes or CUs without work, and
    // where rows are not whole 16-byte vectors up to s = 4 (us of 4 -> 1
    // columns: 500 x 333, s = 3, 11.5 -> 7.9; 8000 x 48, s = 2, 17.9 -> 9.8;
    // 4000 x 3999, s = 2, 326 -> 215; but 2047^2, s = 5, 222 -> 243)
    const bool small = blocks(4, 1) < 640 || nfx <= 192;
    const int cols = small || (!v4 && (s <= 4 || blocks(4, 1) < 8192)) ? 1 : 4;
    int nseg = up_max_seg(cols, s);
    while (nseg > 1 && blocks(cols, nseg) < 640) nseg /= 2;
    const dim3 grid(cdiv(nfx, 64 * cols), cdiv(ncy + 2, 4 * nseg));
    const auto kernel = cols == 1 ? k_up_lanczos<false, 0, 1>
                        : !v4    ? k_up_lanczos<false, 0>
                        : s >= 3 ? k_up_lanczos<true, 1>
                        : s == 2 ? k_up_lanczos<true, 2>
                                 : k_up_lanczos<true, 3>;
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, ncy, ncx, s, nseg, coarse, fine);
  }
  return hipGetLastError();
}

hipError_t launch_upsample_adjoint(int kind, int ncy, int ncx, int s, const float *grad_fine,
                                   float *grad_coarse, hipStream_t stream) {
  if (kind == 0) {
    const dim3 grid(cdiv(ncx, 256) < 64 ? cdiv(ncx, 256) : 64, ncy < 4096 ? ncy : 4096), t(256);
    const int v = aligned16(grad_fine) ? s : 0;
    if (v == 4)
      hipLaunchKernelGGL(k_up_nearest_adj<4>, grid, t, 0, stream, ncy, ncx, s, grad_fine, grad_coarse);
    else if (v == 8)
      hipLaunchKernelGGL(k_up_nearest_adj<8>, grid, t, 0, stream, ncy, ncx, s, grad_fine, grad_coarse);
    else if (v == 16)
      hipLaunchKernelGGL(k_up_nearest_adj<16>, grid, t, 0, stream, ncy, ncx, s, grad_fine, grad_coarse);
    else
      hipLaunchKernelGGL(k_up_nearest_adj<0>, grid, t, 0, stream, ncy, ncx, s, grad_fine, grad_coarse);
  } else {
    // nrow coarse rows per block: up to 64 (five segments of lead-in each),
    // as many as their taps' LDS holds, fewer while the grid has less than
    // two blocks for each CU
    const bool narrow = ncx <= adj_cols(s, 1);
    const unsigned bx = cdiv(ncx, adj_cols(s, narrow ? 1 : 4));
    int nrow = kAdjMaxRows / s - 5;
    if (nrow > 64) nrow = 64;
    while (nrow > 4 && bx * cdiv(ncy, nrow) < 512) nrow = (nrow + 1) / 2;
    const dim3 grid(bx, cdiv(ncy, nrow)), t(kAdjThreads);
    if (narrow)
      hipLaunchKernelGGL((k_up_lanczos_adj<false, 1>), grid, t, 0, stream, ncy, ncx, s, nrow, grad_fine, grad_coarse);
    else if (ncx * s % 4 == 0 && aligned16(grad_fine))
      hipLaunchKernelGGL(k_up_lanczos_adj<true>, grid, t, 0, stream, ncy, ncx, s, nrow, grad_fine, grad_coarse);
    else
      hipLaunchKernelGGL(k_up_lanczos_adj<false>, grid, t, 0, stream, ncy, ncx, s, nrow, grad_fine, grad_coarse);
  }
  return hipGetLastError();
}

}  // namespace dop
