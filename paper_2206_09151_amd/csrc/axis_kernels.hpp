// Whole single-axis reconstructions without plane stacks, for detector sizes up to 192.
//
// With every view rotated about the volume's y axis and detector rows on voxel rows, the
// gridding interpolates inside (plane, column) slices only, with the same weights in every
// row.  It therefore commutes with the inverse transform along y: the slices can be gridded
// row frequency by row frequency, and one inverse transform per voxel column of the finished
// volume takes the place of one per column of every plane (half of the plane transforms), and
// a row frequency's slice (at most 192 x 192 values) is small enough to stay in one CU's LDS
// between its transforms along x and its gridding, so no plane is ever written to memory.
//
//   k_axis_slices  workgroup (row unit, block of views): per view, the transforms along x of one
//                  row frequency of the propagated spectrum for every depth plane, into LDS, then
//                  the bilinear gather of the N x N voxels of the slice, summed over the block's
//                  views in ascending order in registers; partial slices out.
//   k_axis_columns sums the partial slices of the blocks in ascending order and runs the inverse
//                  transform along y of every voxel column, two columns per complex transform,
//                  in FP64: errors of the views' transforms average out over the scan, those of
//                  this one would not.
//
// The planes are real, so row frequencies 0 .. M/2 carry everything: M real slices, two for each
// frequency r (the real and the imaginary part of its row transforms) and one each for 0 and, with
// even M, M/2, which share slice pair 0.  With Y_j = Herm[F e^{-i phi_j} G] and the spectra kernel's
// Q1 = (1+i) F_h G / M^2, Q2 = -(1+i) F_a G / M^2 there are two ways to have two real slices or
// planes per complex transform:
//   complex cells (small M): a workgroup takes a slice pair; a lane transforms one plane,
//       Y_j / M^2 = (1-i)/2 (cos(phi_j) Q1 + i sin(phi_j) Q2), and the slice's cells are complex
//       (the constant is applied to the sums);
//   real cells: a workgroup takes one slice; its spectrum row is the even or odd part of Q over
//       the rows +-r, a lane transforms the planes j and K-1-j together,
//       Y_j + i Y_{K-1-j} = cos(phi_j) Q1 + sin(phi_j) Q2, and the cells are real.
// Complex cells compute a voxel's weights once for two slices, real cells need half the LDS: at
// M = 128 two workgroups share a CU and fill each other's barriers (337 us for 180 views, against
// 376 with complex cells and one workgroup); up to M = 64 the complex slice is small enough for
// four, and real cells would leave half of every wave's lanes without a plane pair.
//
// What bounds k_axis_slices at 128^3, 180 views (329 us): vector issue, 69-73 % of the time, and
// LDS, 64-68 % (30 % of it bank conflicts of the rotated taps), between three barriers per view
// at four waves per SIMD.  28.1 TFLOP/s of transform and interpolation, of the 78.6 that FP32
// reaches without packed instructions.  It replaces plane stacks of 8.4 MB per view: 452 us of 2D
// plane transforms and 386 us of gridding per reconstruction.  What moved it: rows of the spectrum
// fetched into LDS one view ahead (650 -> 393 us; as scalar loads their latency was exposed on
// every view), the four voxels of a quarter-turn orbit sharing one set of weights (393 -> 376),
// two workgroups per CU (376 -> 337).  From M = 135 on one workgroup fills a CU, and from 160 on
// some of a thread's 40 to 60 transform and propagation values spill: 160^3 from 60 views takes
// 391 us (plane stacks: 817 + 264), 192^3 869 us (882 + 474).  Where stacks are the faster way:
// stacks_faster in tomo_kernels.hip.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "fft.hpp"
#include "spectra_kernels.hpp"
#include "tomo_internal.hpp"

namespace tomo {

typedef __attribute__((address_space(3))) void lds_ptr_t;

constexpr int axis_pitch(int M) {
  // cells per staged plane: odd, so that the lanes of a wave (one plane each in the transform)
  // fall on different LDS banks, with at least two zero cells between planes; the rotated taps
  // of an 8 x 8 patch meet 1.95 bank cycles per read at these residues in a count over a
  // half-turn, 2.4 at 15 and 17 and 4.4 at 1 and 31
  int p = (M + 2) | 1;
  if (M == 192) return 195;                             // 197 cells would not fit in LDS
  while (p % 32 < 5 || p % 32 > 27 || (p % 32 > 13 && p % 32 < 19)) p += 2;
  return p;
}

// M = R1 R2: every lane holds one depth plane (REAL: a pair of planes), every wave the inputs
// s + R2 r of one s for 64 of them.
template <int M_, int R1_, int R2_, bool REAL_>
struct AxisShapeOf {
  static constexpr int M = M_, R1 = R1_, R2 = R2_;
  static constexpr bool REAL = REAL_;
  static constexpr int PAIRS = (M + 1) / 2;           // slice pairs
  static constexpr int UNITS = REAL ? 2 * PAIRS : PAIRS;   // workgroups per block of views
  static constexpr int LANES = REAL ? (M + 1) / 2 : M;
  static constexpr int KW = (LANES + 63) / 64;        // waves across the planes (K <= M)
  static constexpr int NW = R2 * KW, T = 64 * NW;
  static constexpr int E = (R1 + R2 - 1) / R2;        // second-stage transforms per wave
  static constexpr int XN = E * R2 > R1 ? E * R2 : R1;
  static constexpr int P = axis_pitch(M);
  static constexpr int CB = REAL ? 4 : 8;             // bytes per cell
  // two zero planes on either side; REAL: one more for the unused half of an odd K's middle pair
  static constexpr int CELLS = (M + 4 + (REAL ? 1 : 0)) * P + 4;
  static constexpr int HALF = M / 2 + 1;
  static constexpr int QN = REAL ? HALF : 2 * M;      // values of the spectrum row(s) transformed next
  static constexpr int LDS = CELLS * CB + QN * 16;
  static constexpr int XW = ((M + 1) / 2 + 7) / 8;
  static constexpr int VPT = (XW * XW + NW - 1) / NW;  // voxel orbits per thread (8 x 8 patches per wave)
  // registers for as many workgroups per CU as their LDS allows, where the values leave room
  static constexpr int WG = 160 * 1024 / LDS < 16 / NW ? 160 * 1024 / LDS : 16 / NW;
  static constexpr int WAVES = (4 * R1 + VPT * (REAL ? 4 : 8) <= 100 && WG > 0) ? (WG * NW + 3) / 4 : 1;
  static_assert(R1 * R2 == M && T <= 1024 && LDS <= 160 * 1024, "shape");
  // k_axis_columns: 16 column pairs per workgroup, transformed by R2 threads each and summed by 32
  static constexpr int CP = M | 1, CL = 16, CT = 32 * CL;
};
template <int M>
struct AxisShape;
template <> struct AxisShape<16> : AxisShapeOf<16, 4, 4, false> {};
template <> struct AxisShape<18> : AxisShapeOf<18, 6, 3, false> {};
template <> struct AxisShape<20> : AxisShapeOf<20, 5, 4, false> {};
template <> struct AxisShape<24> : AxisShapeOf<24, 6, 4, false> {};
template <> struct AxisShape<25> : AxisShapeOf<25, 5, 5, false> {};
template <> struct AxisShape<27> : AxisShapeOf<27, 9, 3, false> {};
template <> struct AxisShape<30> : AxisShapeOf<30, 6, 5, false> {};
template <> struct AxisShape<32> : AxisShapeOf<32, 8, 4, false> {};
template <> struct AxisShape<36> : AxisShapeOf<36, 9, 4, false> {};
template <> struct AxisShape<40> : AxisShapeOf<40, 10, 4, false> {};
template <> struct AxisShape<45> : AxisShapeOf<45, 9, 5, false> {};
template <> struct AxisShape<48> : AxisShapeOf<48, 12, 4, false> {};
template <> struct AxisShape<50> : AxisShapeOf<50, 10, 5, false> {};
template <> struct AxisShape<54> : AxisShapeOf<54, 9, 6, false> {};
template <> struct AxisShape<60> : AxisShapeOf<60, 15, 4, false> {};
template <> struct AxisShape<64> : AxisShapeOf<64, 16, 4, false> {};
template <> struct AxisShape<72> : AxisShapeOf<72, 12, 6, true> {};
template <> struct AxisShape<75> : AxisShapeOf<75, 15, 5, true> {};
template <> struct AxisShape<80> : AxisShapeOf<80, 16, 5, true> {};
template <> struct AxisShape<81> : AxisShapeOf<81, 9, 9, true> {};
template <> struct AxisShape<90> : AxisShapeOf<90, 15, 6, true> {};
template <> struct AxisShape<96> : AxisShapeOf<96, 16, 6, true> {};
template <> struct AxisShape<100> : AxisShapeOf<100, 10, 10, true> {};
template <> struct AxisShape<108> : AxisShapeOf<108, 12, 9, true> {};
template <> struct AxisShape<120> : AxisShapeOf<120, 15, 8, true> {};
template <> struct AxisShape<125> : AxisShapeOf<125, 25, 5, true> {};
template <> struct AxisShape<128> : AxisShapeOf<128, 16, 8, true> {};
template <> struct AxisShape<135> : AxisShapeOf<135, 27, 5, true> {};
template <> struct AxisShape<144> : AxisShapeOf<144, 18, 8, true> {};
template <> struct AxisShape<150> : AxisShapeOf<150, 25, 6, true> {};
template <> struct AxisShape<160> : AxisShapeOf<160, 20, 8, true> {};
template <> struct AxisShape<162> : AxisShapeOf<162, 27, 6, true> {};
template <> struct AxisShape<180> : AxisShapeOf<180, 30, 6, true> {};
template <> struct AxisShape<192> : AxisShapeOf<192, 24, 8, true> {};

// Partial slices: [block][2 PAIRS][pitch] float, pitch = N^2 rounded up to even.
__host__ __device__ inline unsigned axis_slice_pitch(int N) { return (unsigned(N) * unsigned(N) + 1u) & ~1u; }

// SQUARE: K = M, every slice is square
template <int M, bool SQUARE>
__global__ __launch_bounds__(AxisShape<M>::T, AxisShape<M>::WAVES) void k_axis_slices(
    const float4* __restrict__ q, const float2* __restrict__ prop, const float2* __restrict__ tw,
    const ViewGeom* __restrict__ geom, float* __restrict__ part, int N, int K, int npairs, int n, int blocks,
    double hm, double hk) {
  using S = AxisShape<M>;
  constexpr int R1 = S::R1, R2 = S::R2, NW = S::NW, E = S::E, P = S::P, VPT = S::VPT;
  constexpr bool EVEN = M % 2 == 0, REAL = S::REAL;
  using Cell = std::conditional_t<REAL, float, float2>;
  __shared__ Cell cells[S::CELLS];
  // the spectrum row transformed next: REAL the slice's part of rows +-r, kx <= M/2; else row r
  // (pair 0: rows 0 and M/2)
  __shared__ __attribute__((aligned(16))) float4 qrow[S::QN];
  const int t = threadIdx.x, lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int unit = int(blockIdx.x % S::UNITS), block = int(blockIdx.x / S::UNITS);
  // REAL: the two slices of a pair lie eight workgroups apart, on one XCD, and read the same rows
  int row, part2 = 0;                                    // row frequency; 1: imaginary part
  if constexpr (REAL) {
    constexpr int FULL = S::UNITS / 16 * 16;
    const int k = unit < FULL ? (unit / 16) * 8 + unit % 8 : FULL / 2 + (unit - FULL) / 2;
    part2 = unit < FULL ? (unit / 8) & 1 : (unit - FULL) & 1;
    row = k;
  } else {
    row = unit;
  }
  const int slice = 2 * row + part2;                     // where the partial slice goes
  if (REAL && !EVEN && slice == 1) return;               // odd M: pair 0 has one slice (whole workgroup leaves)
  if (REAL && EVEN && row == 0) {
    row = part2 ? M / 2 : 0;                             // pair 0: the real rows 0 and M/2
    part2 = 0;
  }
  const int n0 = int((long long)n * block / blocks), n1 = int((long long)n * (block + 1) / blocks);
  const int s = w % R2, j = (w / R2) * 64 + lane;       // input residue; plane (REAL: pair of planes)
  const bool plane = j < (REAL ? npairs : K);

  // propagation factors of this thread's inputs, the same for every view: (cos, sin)(phi_x + phi_y)
  // of plane j (the tables hold the planes of z' <= 0; the others are their mirror images)
  float2 ph[R1];
  float2 ph_half = make_float2(1.0f, 0.0f);              // step from frequency 0 to M/2 (complex pair 0)
  {
    constexpr int TP = M | 1;
    static_assert((M + 1) / 2 * TP * 8 <= S::CELLS * S::CB, "the propagator table fits in the cells");
    float2* table = reinterpret_cast<float2*>(cells);
    for (int i = t; i < npairs * M; i += S::T) table[(i / M) * TP + i % M] = prop[i];
    __syncthreads();
    const int pj = plane ? min(j, K - 1 - j) : 0;
    const float sg = j < npairs ? 1.0f : -1.0f;
    const float2 cy = table[pj * TP + row];
#pragma unroll
    for (int r = 0; r < R1; ++r) {
      const float2 cx = table[pj * TP + s + R2 * r];
      ph[r] = make_float2(cx.x * cy.x - cx.y * cy.y, sg * (cx.y * cy.x + cx.x * cy.y));
    }
    if constexpr (EVEN && !REAL) {
      const float2 ch = table[pj * TP + M / 2];
      ph_half = make_float2(ch.x, sg * ch.y);
    }
    __syncthreads();
    for (int i = t; i < S::CELLS; i += S::T) cells[i] = Cell{};
  }

  // voxel orbits: a quarter turn of the slice about the rotation axis takes the coordinate pair
  // (column, plane) of a voxel to (hm - (plane - hk), hk + (column - hm)), so the four voxels
  // (x, z), (-x, -z), (-z, x), (z, -x) of an orbit share their interpolation weights.  One of
  // each lies in the quadrant x, z < ceil(N / 2); wave w's i-th patch of 8 x 8 orbits is patch
  // w + NW i of the quadrant, row by row
  const int half = (N + 1) / 2;
  const int xw = (half + 7) / 8;
  const int x0 = 8 * (w % xw) + (lane & 7), z0 = 8 * (w / xw) + (lane >> 3);
  const int dx = NW % xw, dz = NW / xw;
  unsigned wraps = 0;                                     // bit i: patch i + 1 starts a new patch row
  for (int i = 0, xp = w % xw; i + 1 < VPT; ++i) {
    xp += dx;
    if (xp >= xw) {
      xp -= xw;
      wraps |= 1u << i;
    }
  }
  const double c = 0.5 * (N - 1);
  const double rx = x0 - c, rz = z0 - c;
  // coordinates are held as 1.5 2^20 + coordinate: the high word ends in the integer part, the
  // low word is the fraction in units of 2^-32
  constexpr double kBias = 1572864.0;
  constexpr unsigned kBiasHi = 0x41380000u;
  // Index bounds into the zero border, in this form (as bit patterns of floats near 11.5 the high
  // words keep their order, and a median is exact), of columns and planes, and of the quarter-turned
  // voxels' planes (column - (M - K) / 2) and columns (plane + (M - K) / 2)
  const unsigned mk = SQUARE ? 0u : unsigned(M - K) / 2u;
  float lo = __uint_as_float(kBiasHi - 2u);
  const float hi_c = __uint_as_float(kBiasHi + unsigned(M)), hi_p = __uint_as_float(kBiasHi + unsigned(K));
  float lo_qp = __uint_as_float(kBiasHi - 2u + mk), lo_qc = __uint_as_float(kBiasHi - 2u - mk);
  const float hi_qp = __uint_as_float(kBiasHi + K + mk), hi_qc = __uint_as_float(kBiasHi + M - mk);
  // byte address of a tap: CB (P (plane + 2) + column + 2)
  constexpr unsigned CB = S::CB, LOG_CB = REAL ? 2 : 3;
  unsigned mul_p = P * CB;
  unsigned ofs = (2u * P + 2u) * CB - (kBiasHi & 0xffffffu) * (P * CB) - kBiasHi * CB;
  // (operands of one instruction each: all but one of an instruction's constants in VGPRs)
  asm volatile("" : "+v"(lo), "+v"(lo_qp), "+v"(lo_qc), "+v"(mul_p), "+s"(ofs));
  // the opposite voxel's taps: plane K - 2 - plane, column M - 2 - column
  const unsigned opp = ((K + 2u) * P + M + 2u) * CB;
  // the quarter-turned voxel's: plane column - mk, column M - 2 - mk - plane
  const unsigned ofs_q = (2u * P + M) * CB - ((kBiasHi & 0xffffffu) + mk) * (P * CB) + (kBiasHi - mk) * CB;
  Cell acc[VPT][4];
#pragma unroll
  for (int i = 0; i < VPT; ++i)
#pragma unroll
    for (int o = 0; o < 4; ++o) acc[i][o] = Cell{};
  // the thread's transform row; REAL: real parts in the row of plane j, imaginary parts in that of
  // plane K-1-j (the middle pair of an odd K has one plane: the other half goes to the spare row)
  Cell* mine = cells + (j + 2) * P + 2;
  Cell* mine2 = cells + ((K - 1 - j == j ? K + 2 : K - 1 - j) + 2) * P + 2;
  // rows fetched straight into LDS (lane l's 16 bytes land 16 l bytes after the wave's base) while
  // the view before is in its second stage
  constexpr int LEN = REAL ? S::HALF : M, ROWS = REAL ? 2 * S::PAIRS : M / 2 + 1;
  auto fetch_row = [&](int v, int r, int to) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float4*>(q + size_t(v) * ROWS * LEN), short(0), ROWS * LEN * 16, 0x00020000);
    if (t < LEN)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_ptr_t*)(qrow + to + 64 * w), 16, t * 16, r * LEN * 16, 0, 0);
  };
  auto fetch = [&](int v) {
    fetch_row(v, REAL ? slice : row, 0);
    if (!REAL && EVEN && row == 0) fetch_row(v, M / 2, M);
  };
  // barriers: one waits for the fetches too, the other leaves them in flight
  auto barrier = [&]() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  auto full_sync = [&]() {
    __builtin_amdgcn_s_waitcnt(0x0070);                   // vmcnt(0) lgkmcnt(0)
    barrier();
  };
  auto light_sync = [&]() {
    __builtin_amdgcn_s_waitcnt(0xc07f);                   // lgkmcnt(0)
    barrier();
  };
  // (Q1, Q2) at the thread's input kx = s + R2 r.  REAL: those above M/2 from the mirror image; the
  // side is known at compile time but for the middle r of an odd R1.  (Two addresses with constant
  // offsets up: kx, and M - kx counted from the last r.)
  const float4* base = qrow + s;
  const float4* above = qrow + (M - s - R2 * (R1 - 1));
  auto input = [&](int r) {
    if (!REAL || 2 * r + 1 < R1) return base[R2 * r];     // kx < R2 (r + 1) <= M/2
    if (2 * r + 1 > R1) return q_mirror(above[R2 * (R1 - 1 - r)]);   // kx >= R2 r >= M/2
    if (2 * (s + R2 * r) <= M) return base[R2 * r];       // uniform
    return q_mirror(above[R2 * (R1 - 1 - r)]);
  };
  if (n0 < n1) fetch(n0);
  full_sync();

  for (int v = n0; v < n1; ++v) {
    // ---- row transforms, stage 1: inputs s + R2 r of plane j
    float2 x[S::XN];
    const ViewGeom& g = geom[v];
    const double u0 = g.u[0], u2 = g.u[2], d0 = g.d[0], d2 = g.d[2];
#pragma unroll
    for (int r = 0; r < R1; ++r) {
      const float4 a = input(r);
      if constexpr (REAL) {
        x[r] = make_float2(ph[r].x * a.x + ph[r].y * a.z, ph[r].x * a.y + ph[r].y * a.w);
        asm volatile("" : "+v"(x[r].x), "+v"(x[r].y));    // formed here: sunk past the barrier, the row values would spill
      }
      else x[r] = make_float2(ph[r].x * a.x - ph[r].y * a.w, ph[r].x * a.y + ph[r].y * a.z);
    }
    if (!REAL && EVEN && row == 0) {                      // uniform: frequency M/2 joins as imaginary part
      float2 st = ph_half;
      asm volatile("" : "+v"(st.x), "+v"(st.y));          // formed here: kept over the views it would spill
#pragma unroll
      for (int r = 0; r < R1; ++r) {
        const float4 a = base[M + R2 * r];
        const float cc = ph[r].x * st.x - ph[r].y * st.y;
        const float ss = ph[r].y * st.x + ph[r].x * st.y;
        x[r].x -= cc * a.y + ss * a.z;
        x[r].y += cc * a.x - ss * a.w;
      }
    }
    Dft<R1, true>::run(x);
#pragma unroll
    for (int k = 1; k < R1; ++k) x[k] = cmul(x[k], tw[(s * k) % M]);
    light_sync();                                         // the previous view's taps and this row are read
    if (v + 1 < n1) fetch(v + 1);
    if (plane) {
#pragma unroll
      for (int k = 0; k < R1; ++k) {
        if constexpr (REAL) mine[s * R1 + k] = x[k].x;
        else mine[s * R1 + k] = x[k];
      }
      if constexpr (REAL) {                               // by row: adjacent cells leave in pairs
#pragma unroll
        for (int k = 0; k < R1; ++k) mine2[s * R1 + k] = x[k].y;
      }
    }
    light_sync();
    // ---- stage 2, in place: output k + R1 k2 takes the cells its inputs k + R1 rr came from
    if (plane) {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int k = s * E + e;
        if (E * R2 > R1 && k >= R1) continue;
#pragma unroll
        for (int rr = 0; rr < R2; ++rr) {
          if constexpr (REAL) x[e * R2 + rr].x = mine[k + R1 * rr];
          else x[e * R2 + rr] = mine[k + R1 * rr];
        }
        if constexpr (REAL) {
#pragma unroll
          for (int rr = 0; rr < R2; ++rr) x[e * R2 + rr].y = mine2[k + R1 * rr];
        }
        Dft<R2, true>::run(&x[e * R2]);
#pragma unroll
        for (int k2 = 0; k2 < R2; ++k2) {
          if constexpr (REAL) mine[k + R1 * k2] = x[e * R2 + k2].x;
          else mine[k + R1 * k2] = x[e * R2 + k2];
        }
        if constexpr (REAL) {
#pragma unroll
          for (int k2 = 0; k2 < R2; ++k2) mine2[k + R1 * k2] = x[e * R2 + k2].y;
        }
      }
    }
    full_sync();
    // ---- bilinear gather of the slice
    unsigned wr = __builtin_amdgcn_readfirstlane(wraps);
    asm volatile("" : "+s"(wr));                          // tested bit by bit: sixteen kept conditions would spill
    double fc = u0 * rx + u2 * rz + (hm + kBias), fp = d0 * rx + d2 * rz + (hk + kBias);
    const double ac = 8.0 * (dx * u0 + dz * u2), ap = 8.0 * (dx * d0 + dz * d2);
    const double bc = ac + 8.0 * (u2 - xw * u0), bp = ap + 8.0 * (d2 - xw * d0);
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      const unsigned long long ic = __double_as_longlong(fc), ip = __double_as_longlong(fp);
      // indices clamped into the zero border (the weights of a clamped index do not matter)
      const float fhc = __uint_as_float(unsigned(ic >> 32)), fhp = __uint_as_float(unsigned(ip >> 32));
      const unsigned hc = __float_as_uint(__builtin_amdgcn_fmed3f(fhc, lo, hi_c));
      const unsigned hp = __float_as_uint(__builtin_amdgcn_fmed3f(fhp, lo, hi_p));
      unsigned qp = hc, qc = hp;
      if constexpr (!SQUARE) {
        qp = __float_as_uint(__builtin_amdgcn_fmed3f(fhc, lo_qp, hi_qp));
        qc = __float_as_uint(__builtin_amdgcn_fmed3f(fhp, lo_qc, hi_qc));
      }
      const float tx = float(unsigned(ic)) * 0x1p-32f, tz = float(unsigned(ip)) * 0x1p-32f;
      const float w11 = tx * tz, w10 = tz - w11, w01 = tx - w11, w00 = (1.0f - tx) - w10;
      const unsigned a0 = (__umul24(hp, mul_p) + ofs) + (hc << LOG_CB);
      const unsigned a2 = (__umul24(qp, mul_p) + ofs_q) - (qc << LOG_CB);
      // one rounding of the running sums per view; taps in the order of their addresses
      auto gather = [&](unsigned a, float v00, float v01, float v10, float v11, Cell& sum) {
        const Cell* tap = reinterpret_cast<const Cell*>(reinterpret_cast<const char*>(cells) + a);
        const Cell t00 = tap[0], t01 = tap[1], t10 = tap[P], t11 = tap[P + 1];
        if constexpr (REAL) {
          sum += fmaf(v11, t11, fmaf(v10, t10, fmaf(v01, t01, v00 * t00)));
        } else {
          sum.x += fmaf(v11, t11.x, fmaf(v10, t10.x, fmaf(v01, t01.x, v00 * t00.x)));
          sum.y += fmaf(v11, t11.y, fmaf(v10, t10.y, fmaf(v01, t01.y, v00 * t00.y)));
        }
      };
      gather(a0, w00, w01, w10, w11, acc[i][0]);
      gather(opp - a0, w11, w10, w01, w00, acc[i][1]);
      gather(a2, w10, w00, w11, w01, acc[i][2]);
      gather(opp - a2, w01, w11, w00, w10, acc[i][3]);
      const bool wrap = (wr >> i) & 1u;
      fc += wrap ? bc : ac;
      fp += wrap ? bp : ap;
      if (VPT > 4) __builtin_amdgcn_sched_barrier(0);     // one orbit's taps at a time: more would spill
    }
  }
  const unsigned pitch = axis_slice_pitch(N);
  float* out = part + (size_t(block) * (2 * S::PAIRS) + slice) * pitch;
  auto store = [&](int i, const Cell& v) {
    if constexpr (REAL) {
      out[i] = v;
    } else {
      out[i] = 0.5f * (v.x + v.y);
      out[pitch + i] = 0.5f * (v.y - v.x);
    }
  };
  int xx = x0, zz = z0;
#pragma unroll
  for (int i = 0; i < VPT; ++i) {
    // odd N: the orbits of the middle row z = half - 1 are those of the middle column
    const bool centre = N % 2 != 0 && xx == half - 1 && zz == half - 1;
    if (xx < half && zz < half && (N % 2 == 0 || zz < half - 1 || centre)) {
      store(zz * N + xx, acc[i][0]);
      if (!centre) {
        store((N - 1 - zz) * N + (N - 1 - xx), acc[i][1]);
        store(xx * N + (N - 1 - zz), acc[i][2]);
        store((N - 1 - xx) * N + zz, acc[i][3]);
      }
    }
    const bool wrap = (wraps >> i) & 1u;
    xx += 8 * (wrap ? dx - xw : dx);
    zz += 8 * (wrap ? dz + 1 : dz);
  }
}

template <int M>
__global__ __launch_bounds__(AxisShape<M>::CT) void k_axis_columns(const float* __restrict__ part,
                                                                   const double2* __restrict__ twiddles,
                                                                   float* __restrict__ vol, int N, int blocks) {
  using S = AxisShape<M>;
  constexpr int R1 = S::R1, R2 = S::R2, E = S::E, CP = S::CP, CL = S::CL;
  __shared__ double2 cells[CL * CP];
  __shared__ double2 tw[M];                               // exp(+i 2 pi k / M)
  const int t = threadIdx.x, s = t / CL;
  const int nn = N * N;
  const int col = (blockIdx.x * CL + t % CL) * 2;       // flattened (z, x) column pair col, col + 1
  const bool live = col < nn;
  const unsigned pitch = axis_slice_pitch(N);
  for (int i = t; i < M; i += S::CT) tw[i] = make_double2(twiddles[i].x, -twiddles[i].y);
  double2* mine = cells + (t % CL) * CP;
  // sum of the blocks' partial slices, and the full spectrum a + i b of the column pair from the
  // half spectra a, b of its columns
  for (int r = s; r < S::PAIRS; r += S::CT / CL) {
    double2 o = make_double2(0.0, 0.0), p = make_double2(0.0, 0.0);   // the columns' two slices of pair r
    if (live) {
      const float2* src = reinterpret_cast<const float2*>(part + size_t(2 * r) * pitch + col);
      const size_t step = size_t(S::PAIRS) * pitch;
#pragma unroll 4
      for (int b = 0; b < blocks; ++b) {
        const float2 f = src[b * step], g = src[b * step + pitch / 2];
        o.x += f.x, o.y += f.y, p.x += g.x, p.y += g.y;
      }
    }
    // odd N: the last pair has one column; odd M: pair 0 has one slice
    if (col + 1 >= nn) o.y = p.y = 0.0;
    if (M % 2 != 0 && r == 0) p = make_double2(0.0, 0.0);
    const double2 a = make_double2(o.x, p.x), b = make_double2(o.y, p.y);
    if (r == 0) {
      mine[0] = make_double2(a.x, b.x);
      if (M % 2 == 0) mine[M / 2] = make_double2(a.y, b.y);
    } else {
      mine[r] = make_double2(a.x - b.y, a.y + b.x);
      mine[M - r] = make_double2(a.x + b.y, b.x - a.y);
    }
  }
  __syncthreads();
  const bool transforms = s < R2;
  double2 x[S::XN];
  if (transforms) {
#pragma unroll
    for (int r = 0; r < R1; ++r) x[r] = mine[s + R2 * r];
  }
  __syncthreads();
  if (transforms) {
    Dft<R1, true>::run(x);
#pragma unroll
    for (int k = 1; k < R1; ++k) x[k] = cmul(x[k], tw[(s * k) % M]);
#pragma unroll
    for (int k = 0; k < R1; ++k) mine[s * R1 + k] = x[k];
  }
  __syncthreads();
  if (!live || !transforms) return;
  const int off = (M - N) / 2;
  const int za = col / N, xa = col % N, zb = (col + 1) / N, xb = (col + 1) % N;
  float* va = vol + size_t(za) * nn + xa;
  float* vb = vol + size_t(zb) * nn + xb;
  const bool pair = N % 2 == 0, second = col + 1 < nn;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int k = s * E + e;
    if (E * R2 > R1 && k >= R1) continue;
    double2 y[R2];
#pragma unroll
    for (int rr = 0; rr < R2; ++rr) y[rr] = mine[k + R1 * rr];
    Dft<R2, true>::run(y);
#pragma unroll
    for (int k2 = 0; k2 < R2; ++k2) {
      const int iy = k + R1 * k2 - off;
      if (unsigned(iy) >= unsigned(N)) continue;
      if (pair) {
        *reinterpret_cast<float2*>(va + iy * N) = make_float2(float(y[k2].x), float(y[k2].y));
      } else {
        va[iy * N] = float(y[k2].x);
        if (second) vb[iy * N] = float(y[k2].y);
      }
    }
  }
}

// ------------------------------------------------------------------ launchers
struct AxisLaunch {
  const float4* q;
  const float2* prop;
  const float2* tw;
  const double2* tw64;     // k_axis_columns: [M] exp(-i 2 pi k / M)
  const ViewGeom* geom;
  float* part;
  float* vol;
  int N, K, npairs, n, blocks;
  hipStream_t s;
};
struct AxisSize {
  int M, units, n_slices, lds, waves;
  hipError_t (*spectra)(const SpectraLaunch&);
  hipError_t (*slices)(const AxisLaunch&);
  hipError_t (*columns)(const AxisLaunch&);
};

template <int M>
hipError_t axis_slices(const AxisLaunch& a) {
  using S = AxisShape<M>;
  if (a.N > M || a.K > M || (M - a.N) % 2 || (M - a.K) % 2) return hipErrorInvalidValue;
  const auto kernel = a.K == M ? &k_axis_slices<M, true> : &k_axis_slices<M, false>;
  hipLaunchKernelGGL(kernel, dim3(unsigned(S::UNITS * a.blocks)), dim3(S::T), 0, a.s, a.q, a.prop, a.tw, a.geom,
                     a.part, a.N, a.K, a.npairs, a.n, a.blocks, 0.5 * (M - 1), 0.5 * (a.K - 1));
  return hipGetLastError();
}

template <int M>
hipError_t axis_columns(const AxisLaunch& a) {
  const unsigned pairs = (unsigned(a.N) * unsigned(a.N) + 1u) / 2u;
  hipLaunchKernelGGL(k_axis_columns<M>, dim3((pairs + AxisShape<M>::CL - 1u) / AxisShape<M>::CL), dim3(AxisShape<M>::CT), 0, a.s, a.part,
                     a.tw64, a.vol, a.N, a.blocks);
  return hipGetLastError();
}

template <int M>
__host__ AxisSize axis_size() {
  using S = AxisShape<M>;
  return AxisSize{M, S::UNITS, 2 * S::PAIRS, S::LDS, S::NW, &half_spectra<M, S::REAL ? kSlices : kRows>,
                  &axis_slices<M>, &axis_columns<M>};
}

extern const AxisSize kAxisSizesA[], kAxisSizesB[], kAxisSizesC[], kAxisSizesD[], kAxisSizesE[];
extern const int kAxisSizesACount, kAxisSizesBCount, kAxisSizesCCount, kAxisSizesDCount, kAxisSizesECount;

}  // namespace tomo
