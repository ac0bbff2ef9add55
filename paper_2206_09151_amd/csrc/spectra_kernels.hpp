// Filtered spectra of the contrast images by two kernels of 1D transforms that fill the GPU whatever
// the number of views (the whole-image kernel of fft_kernels.hpp takes one workgroup per view).
//
//   k_rows_fwd  g = ln(I/I_in) (eq. 4 left side) and the transforms along x, two real rows per
//               complex transform; the row pairs' packed spectra Z[view][pair][M] go to memory.
//   k_cols_fwd  takes the pairs apart (X_a = (Z(k) + conj Z(-k)) / 2, X_b = (Z(k) - conj Z(-k)) / 2i)
//               for a group of columns 0 <= kx <= M/2, transforms them along y -- half of the
//               spectrum, G(-ky, -kx) = conj G(ky, kx) is the rest -- and multiplies by the plan's
//               filter table: Q1 = (1+i) F_h G / M^2, Q2 = -(1+i) F_a G / M^2.
//
// Both transforms run in FP64 (the rate of FP32 without packed instructions) between FP32 storage:
// two roundings instead of one per butterfly (128^3 from 180 views by slices: relative error 1.5e-7
// instead of 2.9e-7).
//
// Bound at M = 128, 180 views: k_rows_fwd (14 us) by its logarithms and transforms (vector issue a third of
// the time, 5.6 workgroups of two waves per CU) and its loads; k_cols_fwd (13 us by slices, 29 for the
// whole filtered plane) by its 60 MB (106 MB) of traffic; small launches by the latency of their loads, which
// every thread of a workgroup shares (transforming threads alone: 10 instead of 6 us for 60 views at
// M = 48).  The whole-image kernel of fft_kernels.hpp, us for the whole plane / these two: 60 views at 48^2
// 14.3 / 14.8, 180 at 128^2 40 / 41 (27 for the half that slices take), 60 at 160^2 91 / 30, 96 at 256^2
// 217 / 76, 360 at 256^2 728 / 319.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "fft.hpp"
#include "tomo_internal.hpp"

namespace tomo {

template <int M_, int R1_, int R2_>
struct FwdShapeOf {
  static constexpr int M = M_, R1 = R1_, R2 = R2_;
  static constexpr int E = (R1 + R2 - 1) / R2;         // second-stage transforms per thread
  static constexpr int XN = E * R2 > R1 ? E * R2 : R1;
  static constexpr int PAIRS = (M + 1) / 2;            // row pairs
  static constexpr int PB = 8;                         // row pairs per workgroup
  static constexpr int RT = PB * R2 <= 64 ? 128 : 256;  // threads of k_rows_fwd (PB R2 of them transform)
  static constexpr int WPV = (PAIRS + PB - 1) / PB;
  static constexpr int HALF = M / 2 + 1;               // columns
  static constexpr int G = (HALF + 15) / 16;           // column groups per view (at most 9)
  static constexpr int C = (HALF + G - 1) / G;         // columns per group
  static constexpr int CT = C * R2 <= 256 ? 256 : 512; // threads of k_cols_fwd (C R2 of them transform)
  static constexpr int P = M | 1;                      // LDS pitch of a line (double2)
  static_assert(R1 * R2 == M && R1 >= R2, "shape");
};
template <int M>
struct FwdShape;
template <> struct FwdShape<16> : FwdShapeOf<16, 4, 4> {};
template <> struct FwdShape<18> : FwdShapeOf<18, 6, 3> {};
template <> struct FwdShape<20> : FwdShapeOf<20, 5, 4> {};
template <> struct FwdShape<24> : FwdShapeOf<24, 6, 4> {};
template <> struct FwdShape<25> : FwdShapeOf<25, 5, 5> {};
template <> struct FwdShape<27> : FwdShapeOf<27, 9, 3> {};
template <> struct FwdShape<30> : FwdShapeOf<30, 6, 5> {};
template <> struct FwdShape<32> : FwdShapeOf<32, 8, 4> {};
template <> struct FwdShape<36> : FwdShapeOf<36, 6, 6> {};
template <> struct FwdShape<40> : FwdShapeOf<40, 8, 5> {};
template <> struct FwdShape<45> : FwdShapeOf<45, 9, 5> {};
template <> struct FwdShape<48> : FwdShapeOf<48, 8, 6> {};
template <> struct FwdShape<50> : FwdShapeOf<50, 10, 5> {};
template <> struct FwdShape<54> : FwdShapeOf<54, 9, 6> {};
template <> struct FwdShape<60> : FwdShapeOf<60, 10, 6> {};
template <> struct FwdShape<64> : FwdShapeOf<64, 8, 8> {};
template <> struct FwdShape<72> : FwdShapeOf<72, 9, 8> {};
template <> struct FwdShape<75> : FwdShapeOf<75, 15, 5> {};
template <> struct FwdShape<80> : FwdShapeOf<80, 10, 8> {};
template <> struct FwdShape<81> : FwdShapeOf<81, 9, 9> {};
template <> struct FwdShape<90> : FwdShapeOf<90, 10, 9> {};
template <> struct FwdShape<96> : FwdShapeOf<96, 12, 8> {};
template <> struct FwdShape<100> : FwdShapeOf<100, 10, 10> {};
template <> struct FwdShape<108> : FwdShapeOf<108, 12, 9> {};
template <> struct FwdShape<120> : FwdShapeOf<120, 12, 10> {};
template <> struct FwdShape<125> : FwdShapeOf<125, 25, 5> {};
template <> struct FwdShape<128> : FwdShapeOf<128, 16, 8> {};
template <> struct FwdShape<135> : FwdShapeOf<135, 15, 9> {};
template <> struct FwdShape<144> : FwdShapeOf<144, 12, 12> {};
template <> struct FwdShape<150> : FwdShapeOf<150, 15, 10> {};
template <> struct FwdShape<160> : FwdShapeOf<160, 16, 10> {};
template <> struct FwdShape<162> : FwdShapeOf<162, 18, 9> {};
template <> struct FwdShape<180> : FwdShapeOf<180, 15, 12> {};
template <> struct FwdShape<192> : FwdShapeOf<192, 16, 12> {};
template <> struct FwdShape<200> : FwdShapeOf<200, 20, 10> {};
template <> struct FwdShape<216> : FwdShapeOf<216, 18, 12> {};
template <> struct FwdShape<225> : FwdShapeOf<225, 15, 15> {};
template <> struct FwdShape<240> : FwdShapeOf<240, 16, 15> {};
template <> struct FwdShape<243> : FwdShapeOf<243, 27, 9> {};
template <> struct FwdShape<250> : FwdShapeOf<250, 25, 10> {};
template <> struct FwdShape<256> : FwdShapeOf<256, 16, 16> {};

// Workgroup -> (view, part): a view's workgroups on one XCD (dealt round robin), in both kernels,
// so that Z is read from the L2 that wrote it.
template <int PARTS>
__device__ __forceinline__ bool view_part(int nb, int& view, int& part) {
  const int k = int(blockIdx.x >> 3);
  view = int(blockIdx.x & 7) + 8 * (k / PARTS);
  part = k % PARTS;
  return view < nb;
}
template <int PARTS>
__host__ inline dim3 view_parts(int nb) { return dim3(unsigned(8 * PARTS * ((nb + 7) / 8))); }

// Forward transform of the lines of one workgroup: thread (line, r) holds inputs r + R2 m in x; the
// cells of its line: mine.  Leaves the outputs s + R1 k2, s = E r + e, in x[e R2 + k2] of thread
// (line, r).  Every thread of the workgroup calls it (barriers); active ones transform.
template <class S>
__device__ __forceinline__ void fwd_line(double2 (&x)[S::XN], double2* mine, int r, const double2* tw, bool active) {
  if (active) {
    Dft<S::R1, false>::run(x);
#pragma unroll
    for (int k = 1; k < S::R1; ++k) x[k] = cmul(x[k], tw[(r * k) % S::M]);
  }
  __syncthreads();
  if (active) {
#pragma unroll
    for (int k = 0; k < S::R1; ++k) mine[k * S::R2 + r] = x[k];
  }
  __syncthreads();
  if (active) {
#pragma unroll
    for (int e = 0; e < S::E; ++e) {
      const int k = r * S::E + e;
      if (S::E * S::R2 > S::R1 && k >= S::R1) continue;
#pragma unroll
      for (int rr = 0; rr < S::R2; ++rr) x[e * S::R2 + rr] = mine[k * S::R2 + rr];
      Dft<S::R2, false>::run(&x[e * S::R2]);
    }
  }
}
// The outputs of fwd_line into the line's cells in order of frequency.
template <class S>
__device__ __forceinline__ void put_line(const double2 (&x)[S::XN], double2* mine, int r) {
#pragma unroll
  for (int e = 0; e < S::E; ++e) {
    const int k = r * S::E + e;
    if (S::E * S::R2 > S::R1 && k >= S::R1) continue;
#pragma unroll
    for (int k2 = 0; k2 < S::R2; ++k2) mine[k + S::R1 * k2] = x[e * S::R2 + k2];
  }
}

// Natural logarithm of a positive finite double to about 1e-13 relative: x = 2^e m, m in
// [1/sqrt 2, sqrt 2), ln m = 2 atanh(s) = 2 s (1 + s^2/3 + s^4/5 + ...), s = (m-1)/(m+1), |s| < 0.172.
// A third of the library function's instructions (whose last bits the FP32 storage does not hold).
// 0 (an I/I_in below FP64's range, from an extreme I_in) gives -infinity, infinity NaN.
__device__ __forceinline__ double log_positive(double x) {
  double m = __builtin_amdgcn_frexp_mant(x);             // [1/2, 1)
  int e = __builtin_amdgcn_frexp_exp(x);
  const bool low = m < 0.70710678118654752;
  m = low ? 2.0 * m : m;
  e -= low ? 1 : 0;
  const double d = m + 1.0;
  double r = __builtin_amdgcn_rcp(d);
  r = fma(fma(-d, r, 1.0), r, r);
  r = fma(fma(-d, r, 1.0), r, r);
  const double s = (m - 1.0) * r, z = s * s;
  double p = 1.0 / 17.0;
  p = fma(p, z, 1.0 / 15.0);
  p = fma(p, z, 1.0 / 13.0);
  p = fma(p, z, 1.0 / 11.0);
  p = fma(p, z, 1.0 / 9.0);
  p = fma(p, z, 1.0 / 7.0);
  p = fma(p, z, 1.0 / 5.0);
  p = fma(p, z, 1.0 / 3.0);
  const double ln = fma(double(e), 0.69314718055994530942, 2.0 * fma(s * z, p, s));
  return x > 0.0 ? ln : -INFINITY;
}

template <int M>
__global__ __launch_bounds__(FwdShape<M>::RT) void k_rows_fwd(const float* __restrict__ images,
                                                              const double2* __restrict__ twiddles,
                                                              float2* __restrict__ z, int* __restrict__ status,
                                                              double inv_iin, int nb) {
  using S = FwdShape<M>;
  __shared__ double2 cells[S::PB * S::P];
  __shared__ double2 tw[M];                            // exp(-i 2 pi k / M)
  int view, part;
  if (!view_part<S::WPV>(nb, view, part)) return;      // whole workgroup
  const int t = threadIdx.x;
  for (int i = t; i < M; i += S::RT) tw[i] = twiddles[i];
  // contrast of the workgroup's rows, by every thread in memory order: row 2 p + 1 is the imaginary
  // part of line p (odd M: the last line has none)
  const int row0 = 2 * S::PB * part, rows = min(2 * S::PB, M - row0);
  const float* img = images + (size_t(view) * M + row0) * M;
  double* flat = reinterpret_cast<double*>(cells);
  int bad = 0;
#pragma unroll 4
  for (int i = t; i < 2 * S::PB * M; i += S::RT) {
    const int row = i / M, col = i % M;
    const float iv = row < rows ? img[i] : 1.0f;
    const bool ok = (iv > 0.0f) && (iv < INFINITY);
    bad |= !ok;
    flat[((row >> 1) * S::P + col) * 2 + (row & 1)] = row < rows && ok ? log_positive(double(iv) * inv_iin) : 0.0;
  }
  // a host word: a store (every writer stores the same) rather than an atomic over the bus
  if (bad) __hip_atomic_store(status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __syncthreads();
  const bool transforms = t < S::PB * S::R2;
  const int line = transforms ? t / S::R2 : 0, r = t % S::R2;
  double2* mine = cells + line * S::P;
  double2 x[S::XN];
  if (transforms) {
#pragma unroll
    for (int m = 0; m < S::R1; ++m) x[m] = mine[r + S::R2 * m];
  }
  fwd_line<S>(x, mine, r, tw, transforms);
  // back through LDS in order of frequency: whole rows leave
  __syncthreads();
  if (transforms) put_line<S>(x, mine, r);
  __syncthreads();
  float2* out = z + (size_t(view) * S::PAIRS + part * S::PB) * M;
  const int lines = min(S::PB, S::PAIRS - part * S::PB);
  for (int i = t; i < lines * M; i += S::RT) {
    const double2 v = cells[(i / M) * S::P + i % M];
    out[i] = make_float2(float(v.x), float(v.y));
  }
}

// (Q1, Q2) at -k from those at k: Q1(-k) = i conj Q1(k), Q2(-k) = -i conj Q2(k) (F_h G is Hermitian,
// F_a G anti-Hermitian).
__device__ __forceinline__ float4 q_mirror(float4 a) { return make_float4(a.y, a.x, -a.w, -a.z); }
// (Q1, Q2) of one coefficient: the filter table's entry times G.
__device__ __forceinline__ float4 q_filtered(float4 f, double2 g) {
  return make_float4(float(f.x * g.x - f.y * g.y), float(f.x * g.y + f.y * g.x), float(f.z * g.x - f.w * g.y),
                     float(f.z * g.y + f.w * g.x));
}

// What k_cols_fwd writes (q [view] of 16 M^2 bytes and more, see the launchers):
//   kFull    q[ky][kx]: the filtered spectrum, both halves.
//   kComplex q[ky][kx] as float2: G times a complex filter (the Fourier-space form's), both halves.
//   kSlices  q[2 r + c][kx <= M/2], r <= M/2: the even (c = 0) and odd (c = 1) part of the rows +-r,
//            (Q(r) + Q(-r)) / 2 and (Q(r) - Q(-r)) / 2i; pair r = 0 holds rows 0 and (even M) M/2.
//   kRows    q[ky][kx], ky <= M/2.
// l1 (kComplex; or NULL): [view][G] sums of the output's magnitudes (fixed order).
enum ColsOut { kFull, kComplex, kSlices, kRows };
template <ColsOut OUT>
using QValue = std::conditional_t<OUT == kComplex, float2, float4>;
__device__ __forceinline__ float2 q_filtered(float2 f, double2 g) {
  return make_float2(float(f.x * g.x - f.y * g.y), float(f.x * g.y + f.y * g.x));
}
__device__ __forceinline__ float q_magnitude(float2 a) { return fabsf(a.x) + fabsf(a.y); }

template <int M, ColsOut OUT>
__global__ __launch_bounds__(FwdShape<M>::CT) void k_cols_fwd(const float2* __restrict__ z,
                                                              const double2* __restrict__ twiddles,
                                                              const QValue<OUT>* __restrict__ filt,
                                                              QValue<OUT>* __restrict__ q,
                                                              float* __restrict__ l1, int nb) {
  using S = FwdShape<M>;
  __shared__ double2 cells[S::C * S::P];
  __shared__ double2 tw[M];
  int view, part;
  if (!view_part<S::G>(nb, view, part)) return;        // whole workgroup
  const int t = threadIdx.x;
  for (int i = t; i < M; i += S::CT) tw[i] = twiddles[i];
  const float2* zv = z + size_t(view) * S::PAIRS * M;
  const int k0 = part * S::C;
#pragma unroll 4
  for (int i = t; i < S::PAIRS * S::C; i += S::CT) {
    const int p = i / S::C, cl = i % S::C, k = min(k0 + cl, S::HALF - 1);
    const float2 a = zv[p * M + k], b = zv[p * M + (k == 0 ? 0 : M - k)];
    double2* col = cells + cl * S::P + 2 * p;
    col[0] = make_double2(0.5 * (double(a.x) + double(b.x)), 0.5 * (double(a.y) - double(b.y)));
    if (2 * p + 1 < M) col[1] = make_double2(0.5 * (double(a.y) + double(b.y)), 0.5 * (double(b.x) - double(a.x)));
  }
  __syncthreads();
  {
    const bool transforms = t < S::C * S::R2;
    const int cl = t % S::C, r = t / S::C;
    double2* mine = cells + cl * S::P;
    double2 x[S::XN];
    if (transforms) {
#pragma unroll
      for (int m = 0; m < S::R1; ++m) x[m] = mine[r + S::R2 * m];
    }
    fwd_line<S>(x, mine, r, tw, transforms);
    __syncthreads();
    if (transforms) put_line<S>(x, mine, r);
  }
  __syncthreads();
  // filtered outputs, neighbouring columns side by side
  const QValue<OUT>* fv = filt + size_t(view) * M * M;
  const int cols = min(S::C, S::HALF - k0);
  if constexpr (OUT == kFull || OUT == kComplex) {
    QValue<OUT>* qv = q + size_t(view) * M * M;
    float sum = 0.0f;
#pragma unroll 4
    for (int i = t; i < M * S::C; i += S::CT) {
      const int ky = i / S::C, cl = i % S::C, k = k0 + cl;
      if (cl >= cols) continue;
      const double2 g = cells[cl * S::P + ky];
      const QValue<OUT> a = q_filtered(fv[ky * M + k], g);
      qv[ky * M + k] = a;
      if constexpr (OUT == kComplex) sum += q_magnitude(a);
      if (k > 0 && 2 * k < M) {
        const int o = (ky == 0 ? 0 : M - ky) * M + M - k;
        const QValue<OUT> b = q_filtered(fv[o], make_double2(g.x, -g.y));
        qv[o] = b;
        if constexpr (OUT == kComplex) sum += q_magnitude(b);
      }
    }
    if (OUT == kComplex && l1) {
      __shared__ float red[(S::CT + 63) / 64];
      for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
      if ((t & 63) == 0) red[t >> 6] = sum;
      __syncthreads();
      if (t == 0) {
        float tot = 0.0f;
        for (int w = 0; w < (S::CT + 63) / 64; ++w) tot += red[w];
        l1[view * S::G + part] = tot;
      }
    }
  } else {
    float4* qv = q + size_t(view) * (OUT == kRows ? S::HALF * M : 2 * S::PAIRS * S::HALF);
#pragma unroll 2
    for (int i = t; i < S::PAIRS * S::C; i += S::CT) {
      const int r = i / S::C, cl = i % S::C, k = k0 + cl;
      if (cl >= cols) continue;
      const int rm = r > 0 ? M - r : M % 2 == 0 ? M / 2 : 0;   // pair 0: rows 0 and M/2
      float4 a = q_filtered(fv[r * M + k], cells[cl * S::P + r]);
      float4 b = q_filtered(fv[rm * M + k], cells[cl * S::P + rm]);
      if constexpr (OUT == kRows) {
        const bool both = k > 0 && 2 * k < M;
        qv[r * M + k] = a;
        if (r > 0) {
          if (both) qv[r * M + M - k] = q_mirror(b);
        } else {
          if (both) qv[M - k] = q_mirror(a);
          if (M % 2 == 0) {
            qv[M / 2 * M + k] = b;
            if (both) qv[M / 2 * M + M - k] = q_mirror(b);
          }
        }
      } else {
        if (r > 0) {
          const float4 e = make_float4(0.5f * (a.x + b.x), 0.5f * (a.y + b.y), 0.5f * (a.z + b.z), 0.5f * (a.w + b.w));
          b = make_float4(0.5f * (a.y - b.y), -0.5f * (a.x - b.x), 0.5f * (a.w - b.w), -0.5f * (a.z - b.z));
          a = e;
        }
        qv[(2 * r) * S::HALF + k] = a;
        qv[(2 * r + 1) * S::HALF + k] = b;
      }
    }
  }
}

// Spectra of nb views.  z: the row pairs' spectra, room for `room` views of (M + 1) / 2 M float2 (the
// views are taken in turns of that many).  l1 (or NULL): [nb][G] out.
struct SpectraLaunch {
  const float* images;
  const double2* tw;       // [M] exp(-i 2 pi k / M)
  const void* filt;
  void* q;
  float2* z;
  size_t room;
  int* status;
  double inv_iin;
  float* l1;
  int nb;
  hipStream_t s;
};

template <int M, ColsOut OUT>
hipError_t half_spectra(const SpectraLaunch& a) {
  using S = FwdShape<M>;
  if (a.room < 1) return hipErrorInvalidValue;
  const size_t per = OUT == kSlices ? size_t(2 * S::PAIRS) * S::HALF : OUT == kRows ? size_t(S::HALF) * M : size_t(M) * M;
  const int step = int(std::min<size_t>(a.room, size_t(a.nb)));
  for (int v = 0; v < a.nb; v += step) {
    const int nb = std::min(step, a.nb - v);
    hipLaunchKernelGGL(k_rows_fwd<M>, view_parts<S::WPV>(nb), dim3(S::RT), 0, a.s, a.images + size_t(v) * M * M,
                       a.tw, a.z, a.status, a.inv_iin, nb);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_cols_fwd<M, OUT>), view_parts<S::G>(nb), dim3(S::CT), 0, a.s, a.z, a.tw,
                       static_cast<const QValue<OUT>*>(a.filt) + size_t(v) * M * M,
                       static_cast<QValue<OUT>*>(a.q) + size_t(v) * per, a.l1 ? a.l1 + size_t(v) * S::G : nullptr, nb);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace tomo
