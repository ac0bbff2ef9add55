// gfx950 kernels of the reconstruction hot path.
//
//   k_rows_fwd, k_cols_fwd, k_planes (spectra_kernels.hpp, fft_kernels.hpp, instantiated per size in
//               fft_sizes_*.hip):
//               contrast, 2D DFT and the eq. 11 filter; depth propagation (eq. 3) and
//               the inverse 2D FFTs that write the plane stacks.  This file keeps
//               the size table that dispatches them.
//   k_grid_*    trilinear gather of the stacks at every voxel's view-frame position
//               (text after eq. 11), summed over the batch's views in ascending
//               order in registers, then one read-modify-write of V (no atomics).
//   k_filter_table, k_sampling_*: plan-time tables in FP64, stored FP32.
#include <hip/hip_bf16.h>
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "fft_kernels.hpp"
#include "axis_kernels.hpp"
#include "fft_sizes.hpp"
#include "geom.hpp"
#include "tomo_internal.hpp"

namespace tomo {

// ------------------------------------------------------------------ inspection
__global__ void k_spectra_out(const float4* __restrict__ q, float2* __restrict__ out, size_t count,
                              float m2) {
  const size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const float4 v = q[i];
  // F G = M^2 (Q1 - Q2) / (1 + i),  1/(1+i) = (1 - i)/2
  const float a = v.x - v.z, b = v.y - v.w;
  out[i] = make_float2(0.5f * m2 * (a + b), 0.5f * m2 * (b - a));
}

// ------------------------------------------------------------------ K4: gridding
constexpr int GT = 16;  // voxel tile edge (x) x (z or y) per 256-thread workgroup

// Box geometry shared by the LDS-staged gridding kernels: 16-byte chunks of VEC stored
// values, BOXW columns per staged (row, plane), LDS pitch BOXP, AX_BOXH planes per row.
template <class InT>
struct AxisBox;
template <>
struct AxisBox<float> {   // 4 values per 16-byte chunk
  static constexpr int VEC = 4, BOXW = 28, BOXP = 28;
};
template <>
struct AxisBox<__hip_bfloat16> {   // 8 values per chunk
  static constexpr int VEC = 8, BOXW = 32, BOXP = 36;
};
template <>
struct AxisBox<__half> {
  static constexpr int VEC = 8, BOXW = 32, BOXP = 36;
};
constexpr int AX_BOXH = 24;     // planes staged per row

union Chunk16 {
  uint4 u;
  float f[4];
  unsigned short h[8];
};

template <class InT>
__device__ __forceinline__ float chunk_value(const Chunk16& c, int k);
template <>
__device__ __forceinline__ float chunk_value<float>(const Chunk16& c, int k) { return c.f[k]; }
template <>
__device__ __forceinline__ float chunk_value<__hip_bfloat16>(const Chunk16& c, int k) {
  return __uint_as_float(unsigned(c.h[k]) << 16);
}
template <>
__device__ __forceinline__ float chunk_value<__half>(const Chunk16& c, int k) {
  return __half2float(__ushort_as_half(c.h[k]));
}

// Keeps v in a register as an opaque value: the compiler may not hoist what is computed
// from it out of the loop it sits in (for values needed only on rarely taken paths).
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Single-axis views (v = y exactly, M - N even): the detector row of voxel row iy is
// iy + (M-N)/2 exactly, so the trilinear weights reduce to bilinear ones in (plane, col),
// shared by the YB voxel rows of a thread.  Per view, the workgroup's 16 x 16 (x, z) tile
// maps into a rotated square of the (plane, col) grid; its bounding box with every tap (at
// most 24 planes x 28 columns; the column start rounded down to a 16-byte boundary) is staged
// in LDS for the YB rows, zero outside the stack, so the bilinear taps are plain LDS reads.
// Only the view's own box is fetched (17 x 20 at 0 degrees, the full 24 x 28 near 45): over a
// half-turn scan that is 17% fewer bytes into LDS than the fixed 24 x 28 box.
//
// The footprints of FP32, BF16 or FP16 planes are fetched straight into LDS in their
// storage type.  The staged box is chunk-linear in 16-byte slots: 7 chunks per (row, plane)
// for FP32; for 16-bit values 4 chunks and a fifth slot that is never fetched, so that a
// (row, plane) spans 20 dwords rather than 16 and planes lp and lp + 2 of the rotated tap
// pattern fall on different LDS banks (at 16 dwords a wave's reads met 3.3 bank cycles per
// half-wave against 1.8 at 20, in a count over the scan's angles).  Wave w's
// i-th load of a view covers slots 256 i + 64 w + lane, and buffer loads with the LDS
// destination write them in place (lane l's 16 bytes land 16 l bytes after the wave's LDS
// base; lanes past the last chunk are switched off and write nothing).  Chunks outside the
// stack get an offset beyond the buffer's range, which the hardware fills with zeros, so no
// masks or register staging are needed.  Two box buffers alternate: view n + 1 is in flight
// while view n is interpolated, and each view takes one barrier.  The 4- and 8-row FP32 kernels
// keep one box instead (fetch, wait, interpolate, two barriers per view): at 4 rows half the
// LDS lets eight workgroups share a CU instead of seven, so a 128^3 volume's 2048 tiles run in
// one round rather than 1.14 (32.3 against 34.5 us per 15-view launch); at 8 rows seven instead
// of three (34.1 against 42.3 us).  The 16-bit 4-row kernel fits eight workgroups with two
// boxes; at 8 rows one box (eight workgroups instead of five) made the 16-bit kernel slower
// (50.8 against 47.2 us per 32-view launch).  A 16-bit tap pair (lc, lc + 1) is the 32-bit
// window at bit 16 (lc & 1) of the two dwords from element 2 (lc >> 1); FP16 values are
// unscaled through the interpolation weights (the per-view scale is a power of two).
//
// CH: bytes per fetched slot.  Stack rows that are not whole 16-byte chunks are fetched dword by
// dword (CH = 4) into boxes of the same pitches: 28 us per 16-view BF16 launch at N = 96, M = 100,
// where the general-frame cubic tiles, which served those rows before, took 182 us.
template <class InT>
struct DmaBox;
template <>
struct DmaBox<float> {
  static constexpr int VEC = 4, BOXW = 28;
};
template <>
struct DmaBox<__hip_bfloat16> {
  static constexpr int VEC = 8, BOXW = 32;
};
template <>
struct DmaBox<__half> {
  static constexpr int VEC = 8, BOXW = 32;
};
typedef __attribute__((address_space(3))) void lds_void_t;
constexpr unsigned kOutOfRange = 0x80000000u;      // beyond every buffer range: reads as zero

// Detector coordinates of the general kernels in fixed point: adding kFixBias to an FP64
// coordinate rounds it to 2^-23 and leaves it in the low word, modulo 512 = 2^32 steps.  Relative to a
// box origin the word holds the tap index in its upper nine bits and the interpolation fraction in
// the lower 23, so that the index costs a shift and the weight two operations, and a step to
// the next voxel is an integer addition.
constexpr double kFixBias = 805306368.0;           // 1.5 2^29
__device__ __forceinline__ unsigned fix_of(double biased) { return unsigned(__double_as_longlong(biased)); }
__device__ __forceinline__ unsigned fix_index(unsigned v) { return v >> 23; }
// (the mask is kept in a scalar register: as a literal it would cost the and-or a second operation)
__device__ __forceinline__ unsigned fix_mask() {
  unsigned m = 0x7fffffu;
  asm("" : "+s"(m));
  return m;
}
__device__ __forceinline__ float fix_frac(unsigned v, unsigned mask) {
  return __uint_as_float((v & mask) | 0x3f800000u) - 1.0f;
}
// low + t (high - low) of two packed 16-bit values; FP16 operands are widened inside the multiply-adds
template <class InT>
__device__ __forceinline__ float lerp_pair(unsigned pr, float t) {
  if constexpr (std::is_same<InT, __half>::value) {
    float d;
    asm("v_fma_mix_f32 %0, %1, 1.0, -%1 op_sel:[1,0,0] op_sel_hi:[1,0,1]" : "=v"(d) : "v"(pr));
    return fmaf(t, d, __half2float(__ushort_as_half((unsigned short)(pr & 0xffffu))));
  } else {
    const float a = __uint_as_float(pr << 16);
    return fmaf(t, __uint_as_float(pr & 0xffff0000u) - a, a);
  }
}
// Slots of a box: row, plane and column offset packed as bytes of seven bits, so that one
// subtraction compares all three with a view's extent (a byte's guard bit survives where the offset is
// inside).  A slot that is never fetched has row 127.
constexpr unsigned kSlotGuard = 0x808080u;
__device__ __forceinline__ unsigned slot_pack(int row, int plane, int col) {
  return unsigned(row) | unsigned(plane) << 8 | unsigned(col) << 16;
}
__device__ __forceinline__ unsigned slot_extent(int rows, int planes, int cols) {
  return slot_pack(rows - 1, planes - 1, cols - 1) | kSlotGuard;
}
__device__ __forceinline__ bool slot_inside(unsigned extent, unsigned slot) {
  return ((extent - slot) & kSlotGuard) == kSlotGuard;
}
// A box starts this far below the least corner coordinate, so that no rounding puts a voxel below
// it.  The corners are summed in FP32: coordinates are below 2048 (N <= 1024, M <= 256, K <= 2048), three
// products and three additions err by less than 2^-11; the extents keep a whole row, plane and
// column beyond the last tap for the other side.
constexpr float kBoxMargin = 0x1p-10f;

template <int YB, class InT, int CH>
__global__ __launch_bounds__(256) void k_grid_axis_dma(const InT* __restrict__ stack,
                                                       const ViewGeom* __restrict__ geom,
                                                       const float* __restrict__ scale,
                                                       float* __restrict__ vol, int N, int M, int K, int nb,
                                                       int accumulate, double hm, double hk) {
  constexpr int ES = int(sizeof(InT));                  // bytes per stored value
  constexpr int VEC = CH / ES;                          // values per chunk (slot) of CH bytes
  constexpr int BOXW = CH == 16 ? DmaBox<InT>::BOXW : 28;
  constexpr int PITCH = ES == 2 ? 20 : 28;              // dwords per staged (row, plane)
  constexpr int QP = PITCH * 4 / CH;                    // slots per staged (row, plane)
  constexpr int DW = CH / 4;                            // dwords per slot
  constexpr int NE = YB * AX_BOXH * QP;                 // slots per staged view
  constexpr int PER = (NE + 255) / 256;                 // loads per thread per view
  // 16-bit values: one dword of padding, the pair read may touch the dword after a row's last
  constexpr int PAD = ES == 2 ? 4 : 0;
  constexpr bool ONE_BOX = YB >= 4 && ES == 4;
  __shared__ __attribute__((aligned(16))) unsigned box0[NE * DW + PAD];
  __shared__ __attribute__((aligned(16))) unsigned box1[ONE_BOX ? 4 : NE * DW + PAD];
  const int ntx = (N + GT - 1) / GT;
  const int tiles = ntx * ntx;
  const int wg = blockIdx.x, xcd = wg & 7, k = wg >> 3;
  const int yblk = xcd + 8 * (k / tiles), tile = k % tiles;
  const int y0 = yblk * YB;
  if (y0 >= N) return;                                  // uniform
  const int tx0 = (tile % ntx) * GT, tz0 = (tile / ntx) * GT;
  const int ix = tx0 + (threadIdx.x % GT);
  const int iz = tz0 + (threadIdx.x / GT);
  const bool live = ix < N && iz < N;
  const double c = 0.5 * (N - 1);
  const double rx = ix - c, rz = iz - c;
  const int rowoff = (M - N) / 2;
  const size_t view_sz = size_t(K) * M * M;
  const int wbase = (threadIdx.x & ~63) * DW;           // this wave's first dword in a box, per load
  const int lane = threadIdx.x & 63;

  // Box origins: lane l of every wave computes the origin of view obase + l (FP64, from
  // the tile corners); per view the workgroup-uniform origin is read out of lane n - obase
  // into scalar registers, so the per-view cost is two lane reads.
  // The box of a view: columns c0 .. c0 + cw - 1 (cw a multiple of VEC) and planes
  // p0 .. p0 + bh - 1, from the tile's corner extremes; the taps of a voxel lie at most one
  // past the floor of its coordinates, and one more column and plane absorb a last-bit
  // difference between the corner and the voxel arithmetic (within the 24 x 28 maximum).
  int obase = -64, lane_c0 = 0, lane_p0 = 0, lane_cw = 0, lane_bh = 0;
  auto origin = [&](int n, int& c0, int& p0, int& cw, int& bh) {
    if (n >= obase + 64) {
      obase = n;
      const int v = n + lane;
      int cc = 0, pp = 0, ww = 0, hh = 0;
      if (v < nb) {
        const int t0 = opaque(tx0), z0 = opaque(tz0);
        const double ax = t0 - c, bx = t0 + GT - 1 - c, az = z0 - c, bz = z0 + GT - 1 - c;
        const ViewGeom& g = geom[v];
        const double cmin = fmin(g.u[0] * ax, g.u[0] * bx) + fmin(g.u[2] * az, g.u[2] * bz) + hm;
        const double cmax = fmax(g.u[0] * ax, g.u[0] * bx) + fmax(g.u[2] * az, g.u[2] * bz) + hm;
        const double pmin = fmin(g.d[0] * ax, g.d[0] * bx) + fmin(g.d[2] * az, g.d[2] * bz) + hk;
        const double pmax = fmax(g.d[0] * ax, g.d[0] * bx) + fmax(g.d[2] * az, g.d[2] * bz) + hk;
        cc = int(floor(cmin)) & ~(VEC - 1);
        pp = int(floor(pmin));
        ww = min(BOXW, (int(floor(cmax)) - cc + 3 + VEC - 1) & ~(VEC - 1));
        hh = min(AX_BOXH, int(floor(pmax)) - pp + 3);
      }
      lane_c0 = cc;
      lane_p0 = pp;
      lane_cw = ww;
      lane_bh = hh;
    }
    c0 = __builtin_amdgcn_readlane(lane_c0, n - obase);
    p0 = __builtin_amdgcn_readlane(lane_p0, n - obase);
    cw = __builtin_amdgcn_readlane(lane_cw, n - obase);
    bh = __builtin_amdgcn_readlane(lane_bh, n - obase);
  };
  // per chunk slot: byte offset from the box origin (rows all present), and for boxes that
  // cross the stack's edge its (plane, column) position and detector-row term
  // (the host launches this kernel only for M a multiple of VEC and views below 2^31 bytes)
  const bool rows_in = y0 + YB <= N && y0 + rowoff >= 0 && y0 + YB - 1 + rowoff < M;
  unsigned cfo[PER];
  int cq[PER], cpl[PER], crow[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int e = threadIdx.x + 256 * i;
    const int q = e % QP, pl = (e / QP) % AX_BOXH, j = e / (QP * AX_BOXH);
    const int row = y0 + j + rowoff;
    cq[i] = VEC * q;                                    // spare slots have cq >= BOXW >= cw
    cpl[i] = pl;
    crow[i] = (e < NE && y0 + j < N && unsigned(row) < unsigned(M)) ? row * K : -1;
    cfo[i] = rows_in ? unsigned((row * K + pl) * M + VEC * q) * unsigned(ES) : kOutOfRange;
  }
  // slot i exists for every thread below the last load; in the last one only below NE
  auto has = [&](int i) { return NE % 256 == 0 || i < PER - 1 || int(threadIdx.x) + 256 * i < NE; };
  auto fetch_slot = [&](const __amdgpu_buffer_rsrc_t& rs, unsigned* to, unsigned ofs, int base) {
    if constexpr (CH == 16) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)to, 16, int(ofs), base, 0, 0);
    else __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)to, 4, int(ofs), base, 0, 0);
  };
  auto load = [&](int n, int c0, int p0, int cw, int bh, unsigned* dst) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<InT*>(stack + size_t(n) * view_sz), short(0), int(view_sz * ES), 0x00020000);
    // slots outside the view's box fetch nothing (their LDS words are never read)
    if (rows_in && p0 >= 0 && p0 + bh <= K && c0 >= 0 && c0 + cw <= M) {
      const int so = (p0 * M + c0) * ES;
#pragma unroll
      for (int i = 0; i < PER; ++i)
        if (has(i) && cpl[i] < bh && cq[i] < cw)
          fetch_slot(rs, dst + 256 * DW * i + wbase, cfo[i], so);
    } else {
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        if (has(i) && cpl[i] < bh && cq[i] < cw) {
          const int pp = p0 + cpl[i], cc = c0 + cq[i];
          const bool ok = crow[i] >= 0 && unsigned(pp) < unsigned(K) && unsigned(cc) < unsigned(M);
          const unsigned off = ok ? unsigned((crow[i] + pp) * M + cc) * unsigned(ES) : kOutOfRange;
          fetch_slot(rs, dst + 256 * DW * i + wbase, off, 0);
        }
      }
    }
  };

  float acc[YB];
#pragma unroll
  for (int j = 0; j < YB; ++j) acc[j] = 0.0f;
  int oc0 = 0, op0 = 0, oc1 = 0, op1 = 0;              // origins of the views in each buffer
  int ow0 = 0, oh0 = 0, ow1 = 0, oh1 = 0;              // and their box extents
  // view n from buffer b: wait for this wave's loads of it (and for its own reads of the
  // other buffer), barrier (every wave's share has landed; every wave is done with the
  // other buffer), issue view n + 1 into the other buffer, interpolate
  // wait for this wave's loads and LDS reads, then for every wave (a plain barrier: the
  // workgroup fence of __syncthreads is not needed after the wait)
  auto sync = [&]() {
    __builtin_amdgcn_s_waitcnt(7 << 4);                 // vmcnt(0) lgkmcnt(0)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // interpolation of view n from its staged box bx (origin column cb, plane pb)
  auto interp = [&](const unsigned* bx, int cb, int pb, int n) {
    if (live) {
      const ViewGeom& g = geom[n];
      const double fc = fmax(g.u[0] * rx + g.u[2] * rz + (hm - cb), 0.0);
      const double fp = fmax(g.d[0] * rx + g.d[2] * rz + (hk - pb), 0.0);
      // fc, fp >= 0: truncation is the floor, fract the remainder (exact in FP64)
      const int lc = int(fc), lp = int(fp);
      float tx = float(__builtin_amdgcn_fract(fc));
      const float tz = float(__builtin_amdgcn_fract(fp));
      float ux = 1.0f - tx;
      if constexpr (std::is_same<InT, __half>::value) {
        const float inv = 1.0f / scale[n];              // exact: the scale is a power of two
        ux *= inv;
        tx *= inv;
      }
      const float w00 = (1.0f - tz) * ux, w01 = (1.0f - tz) * tx;
      const float w10 = tz * ux, w11 = tz * tx;
      const int pofs = int(__umul24(unsigned(lp), unsigned(PITCH)));   // lp < AX_BOXH
#pragma unroll
      for (int j = 0; j < YB; ++j) {
        float a0, a1, b0, b1;                           // taps (lp, lc), (lp, lc+1), (lp+1, lc), (lp+1, lc+1)
        if constexpr (ES == 4) {
          const float* r0 = reinterpret_cast<const float*>(bx) + j * AX_BOXH * PITCH + pofs + lc;
          const float* r1 = r0 + PITCH;
          a0 = r0[0], a1 = r0[1], b0 = r1[0], b1 = r1[1];
        } else {
          const unsigned* r0 = bx + j * AX_BOXH * PITCH + pofs + (lc >> 1);
          const unsigned* r1 = r0 + PITCH;
          const unsigned sh = unsigned(lc & 1) * 16u;
          const unsigned pa = __builtin_amdgcn_alignbit(r0[1], r0[0], sh);
          const unsigned pb2 = __builtin_amdgcn_alignbit(r1[1], r1[0], sh);
          if constexpr (std::is_same<InT, __half>::value) {
            a0 = __half2float(__ushort_as_half((unsigned short)(pa & 0xffffu)));
            a1 = __half2float(__ushort_as_half((unsigned short)(pa >> 16)));
            b0 = __half2float(__ushort_as_half((unsigned short)(pb2 & 0xffffu)));
            b1 = __half2float(__ushort_as_half((unsigned short)(pb2 >> 16)));
          } else {
            a0 = __uint_as_float(pa << 16), a1 = __uint_as_float(pa & 0xffff0000u);
            b0 = __uint_as_float(pb2 << 16), b1 = __uint_as_float(pb2 & 0xffff0000u);
          }
        }
        acc[j] = fmaf(w11, b1, fmaf(w10, b0, fmaf(w01, a1, fmaf(w00, a0, acc[j]))));
      }
    }
  };
  auto step = [&](unsigned* bx, int& cb, int& pb, unsigned* other, int& co, int& po, int& wo, int& ho, int n) {
    if (n >= nb) return;                                // uniform
    sync();
    if (n + 1 < nb) {
      origin(n + 1, co, po, wo, ho);
      load(n + 1, co, po, wo, ho, other);
    }
    interp(bx, cb, pb, n);
  };
  if constexpr (ONE_BOX) {
    // one box: every wave is done with the previous view, fetch, every wave's share has
    // landed, interpolate
    for (int n = 0; n < nb; ++n) {
      if (n > 0) sync();
      origin(n, oc0, op0, ow0, oh0);
      load(n, oc0, op0, ow0, oh0, box0);
      sync();
      interp(box0, oc0, op0, n);
    }
  } else {
    if (nb > 0) {
      origin(0, oc0, op0, ow0, oh0);
      load(0, oc0, op0, ow0, oh0, box0);
    }
    for (int n0 = 0; n0 < nb; n0 += 2) {
      step(box0, oc0, op0, box1, oc1, op1, ow1, oh1, n0);
      step(box1, oc1, op1, box0, oc0, op0, ow0, oh0, n0 + 1);
    }
  }
  if (!live) return;
#pragma unroll
  for (int j = 0; j < YB; ++j) {
    const int iy = y0 + j;
    if (iy < N) {
      float* dst = vol + (size_t(iz) * N + iy) * N + ix;
      *dst = accumulate ? *dst + acc[j] : acc[j];
    }
  }
}

// Single-axis views without depth planes (one plane per view, linear in the detector column): the
// footprint of a 16 x 16 (x, z) tile is a run of at most 26 columns of each of its YB rows.  Every
// thread fetches one value per view (row t % YB, column t / YB of the view's window of 256 / YB
// columns, zero outside the stack), VB views ahead of their use; in LDS the YB rows of a column lie
// side by side, so a voxel column's taps are 2 YB consecutive values, read 16 bytes at a time, and
// the column coordinate and its weights are computed once for the YB rows.  Two LDS buffers of VB
// views alternate, one barrier per VB views.  Lanes are laid out in 4 x 2 blocks of voxels, whose
// taps fall into at most five adjacent columns.
// Bound by LDS reads (8 bytes per update) and vector issue (about 5 instructions per update): 60 us
// for 180 views at 128^3 (6.3e12 updates/s); staged as a general (plane, column) box, whose second
// plane is empty, with one row per read, it took 222 us.
template <int YB, class InT>
__global__ __launch_bounds__(256) void k_grid_axis_flat(const InT* __restrict__ stack,
                                                        const ViewGeom* __restrict__ geom,
                                                        const float* __restrict__ scale,
                                                        float* __restrict__ vol, int N, int M, int nb,
                                                        int accumulate, double hm) {
  constexpr int VB = 4, W = 256 / YB;                   // views per round, columns per window
  constexpr int ES = int(sizeof(InT));
  static_assert(YB == 8, "a window of 32 columns holds the 26 of a footprint");
  __shared__ __attribute__((aligned(16))) float win[2][VB][W * YB];
  const int ntx = (N + GT - 1) / GT;
  const int tiles = ntx * ntx;
  const int wg = blockIdx.x, xcd = wg & 7, k = wg >> 3;
  const int yblk = xcd + 8 * (k / tiles), tile = k % tiles;
  const int y0 = yblk * YB;
  if (y0 >= N) return;                                  // uniform
  const int tx0 = (tile % ntx) * GT, tz0 = (tile / ntx) * GT;
  const int t = threadIdx.x, lane = t & 63;
  const int ix = tx0 + (t & 3) + 4 * ((t >> 3) & 3);
  const int iz = tz0 + ((t >> 2) & 1) + 2 * (t >> 5);
  const double c = 0.5 * (N - 1);
  const double rx = ix - c, rz = iz - c;
  // this thread's value of a view: row y0 + t % YB, column c0 + t / YB of the stack
  const int row = y0 + t % YB + (M - N) / 2, wc = t / YB;
  const bool row_ok = y0 + t % YB < N && unsigned(row) < unsigned(M);
  const unsigned row_ofs = unsigned(row) * unsigned(M) * unsigned(ES);
  const size_t view_sz = size_t(M) * M;

  // window origins, one view per lane (FP64, from the tile corners)
  int obase = -64, lane_c0 = 0;
  auto origin = [&](int n) {
    if (n >= obase + 64) {
      obase = n;
      const int v = n + lane;
      if (v < nb) {
        const int t0 = opaque(tx0), z0 = opaque(tz0);
        const double ax = t0 - c, bx = t0 + GT - 1 - c, az = z0 - c, bz = z0 + GT - 1 - c;
        const ViewGeom& g = geom[v];
        lane_c0 = int(floor(fmin(g.u[0] * ax, g.u[0] * bx) + fmin(g.u[2] * az, g.u[2] * bz) + hm));
      }
    }
    return __builtin_amdgcn_readlane(lane_c0, n - obase);
  };
  int corg[2][VB];                                      // origins of the views in flight and in use
  float buf[VB];
  auto fetch = [&](int n0, int (&org)[VB]) {
#pragma unroll
    for (int i = 0; i < VB; ++i) {
      buf[i] = 0.0f;
      org[i] = 0;
      if (n0 + i < nb) {                                // uniform
        org[i] = origin(n0 + i);
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<InT*>(stack + size_t(n0 + i) * view_sz), short(0), int(view_sz * ES), 0x00020000);
        const int cc = org[i] + wc;
        const unsigned ofs = row_ok && unsigned(cc) < unsigned(M) ? row_ofs + unsigned(cc) * unsigned(ES) : kOutOfRange;
        if constexpr (ES == 4) {
          buf[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, int(ofs), 0, 0));
        } else {
          const unsigned short h = __builtin_amdgcn_raw_buffer_load_b16(rs, int(ofs), 0, 0);
          if constexpr (std::is_same<InT, __half>::value) buf[i] = __half2float(__ushort_as_half(h));
          else buf[i] = __uint_as_float(unsigned(h) << 16);
        }
      }
    }
  };
  float acc[YB];
#pragma unroll
  for (int j = 0; j < YB; ++j) acc[j] = 0.0f;
  // coordinates as 1.5 2^20 + value: integer part in the high word, fraction in units of 2^-32 below
  constexpr double kBias = 1572864.0;
  constexpr unsigned kBiasHi = 0x41380000u;
  const int rounds = (nb + VB - 1) / VB;
  fetch(0, corg[0]);
  for (int r = 0; r < rounds; ++r) {
    float (*dst)[W * YB] = win[r & 1];
#pragma unroll
    for (int i = 0; i < VB; ++i) {
      dst[i][t] = buf[i];
      corg[1][i] = corg[0][i];
    }
    __syncthreads();
    if (r + 1 < rounds) fetch((r + 1) * VB, corg[0]);
#pragma unroll
    for (int i = 0; i < VB; ++i) {
      const int n = r * VB + i;
      if (n >= nb) break;                               // uniform
      const ViewGeom& g = geom[n];
      const double fc = g.u[0] * rx + g.u[2] * rz + (hm + kBias);
      const unsigned long long b = __double_as_longlong(fc);
      float tx = float(unsigned(b)) * 0x1p-32f, ux = 1.0f - tx;
      if constexpr (std::is_same<InT, __half>::value) {
        const float inv = 1.0f / scale[n];              // exact: the scale is a power of two
        ux *= inv;
        tx *= inv;
      }
      // voxels past the volume's edge may lie past the window: any column of it serves them
      const unsigned lc = min(unsigned(b >> 32) - (kBiasHi + unsigned(corg[1][i])), unsigned(W - 2));
      const float4* tap = reinterpret_cast<const float4*>(&dst[i][lc * YB]);
#pragma unroll
      for (int h = 0; h < YB / 4; ++h) {
        const float4 a0 = tap[h], a1 = tap[h + YB / 4];
        acc[4 * h + 0] = fmaf(tx, a1.x, fmaf(ux, a0.x, acc[4 * h + 0]));
        acc[4 * h + 1] = fmaf(tx, a1.y, fmaf(ux, a0.y, acc[4 * h + 1]));
        acc[4 * h + 2] = fmaf(tx, a1.z, fmaf(ux, a0.z, acc[4 * h + 2]));
        acc[4 * h + 3] = fmaf(tx, a1.w, fmaf(ux, a0.w, acc[4 * h + 3]));
      }
    }
  }
  if (ix >= N || iz >= N) return;
#pragma unroll
  for (int j = 0; j < YB; ++j) {
    const int iy = y0 + j;
    if (iy < N) {
      float* dst = vol + (size_t(iz) * N + iy) * N + ix;
      *dst = accumulate ? *dst + acc[j] : acc[j];
    }
  }
}

// General view frames with a compact footprint (e.g. single-axis scans with a tilt):
// per view the bounding box of the workgroup's 16 (x) x YB (y) x 16 (z) voxel tile in
// (row, plane, column) coordinates is staged into LDS when it fits in BR x 24 x BOXW;
// the eight trilinear taps are then LDS reads.  Views whose box does not fit (steep
// tilts, directions far from the rotation axis) are gathered from global memory.
constexpr int BX_BR = 12;       // detector rows staged per view

template <int YB, class InT>
__global__ __launch_bounds__(256) void k_grid_box(const InT* __restrict__ stack,
                                                  const ViewGeom* __restrict__ geom,
                                                  const float* __restrict__ scale,
                                                  float* __restrict__ vol, int N, int M, int K,
                                                  int nb, int accumulate, int flat) {
  using B = AxisBox<InT>;
  constexpr int VEC = B::VEC, BOXW = B::BOXW, BOXP = B::BOXP;
  constexpr int BR = BX_BR, BH = AX_BOXH;
  constexpr int QN = BOXW / VEC;
  constexpr int NE = BR * BH * QN;
  constexpr int PER = (NE + 255) / 256;
  __shared__ float box[BR][BH][BOXP];
  const int ntx = (N + GT - 1) / GT;
  const int tiles = ntx * ntx;
  const int wg = blockIdx.x, xcd = wg & 7, k = wg >> 3;
  const int yblk = xcd + 8 * (k / tiles), tile = k % tiles;
  const int y0 = yblk * YB;
  if (y0 >= N) return;                                  // uniform
  const int tx0 = (tile % ntx) * GT, tz0 = (tile / ntx) * GT;
  const int ix = tx0 + (threadIdx.x % GT);
  const int iz = tz0 + (threadIdx.x / GT);
  const bool live = ix < N && iz < N;
  const double c = 0.5 * (N - 1);
  const double rx = ix - c, rz = iz - c;
  const double hm = 0.5 * (M - 1), hk = 0.5 * (K - 1);
  const size_t plane_sz = size_t(K) * M;
  const bool vec = (M % VEC) == 0;
  const double lo[3] = {tx0 - c, y0 - c, tz0 - c};
  const double hi[3] = {tx0 + GT - 1 - c, y0 + YB - 1 - c, tz0 + GT - 1 - c};

  // box of view n: origin (r0, p0, c0) and whether it fits (uniform)
  auto origin = [&](int n, int& r0, int& p0, int& c0) -> bool {
    const ViewGeom& g = geom[n];
    double cmin = hm, cmax = hm, rmin = hm, rmax = hm, pmin = hk, pmax = hk;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      cmin += fmin(g.u[a] * lo[a], g.u[a] * hi[a]);
      cmax += fmax(g.u[a] * lo[a], g.u[a] * hi[a]);
      rmin += fmin(g.v[a] * lo[a], g.v[a] * hi[a]);
      rmax += fmax(g.v[a] * lo[a], g.v[a] * hi[a]);
      pmin += fmin(g.d[a] * lo[a], g.d[a] * hi[a]);
      pmax += fmax(g.d[a] * lo[a], g.d[a] * hi[a]);
    }
    c0 = int(floor(cmin)) & ~(VEC - 1);
    r0 = int(floor(rmin));
    p0 = flat ? 0 : int(floor(pmin));
    // taps reach floor(max)+1; keep one slot of slack for rounding
    return vec && (int(floor(cmax)) + 2 - c0 < BOXW) && (int(floor(rmax)) + 2 - r0 < BR) &&
           (flat || int(floor(pmax)) + 2 - p0 < BH);
  };
  auto fetch = [&](int n, int r0, int p0, int c0, uint4 (&v)[PER], unsigned& valid) {
    const InT* vbase = stack + size_t(n) * plane_sz * M;
    valid = 0u;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = threadIdx.x + 256 * i;
      const int q = e % QN, pl = (e / QN) % BH, j = e / (QN * BH);
      const int row = r0 + j, pp = p0 + pl, cc = c0 + VEC * q;
      const bool ok = e < NE && unsigned(row) < unsigned(M) && unsigned(pp) < unsigned(K) && cc >= 0 && cc < M &&
                      vec;
      valid |= ok ? (1u << i) : 0u;
      const int rowc = min(max(row, 0), M - 1), ppc = min(max(pp, 0), K - 1);
      const int ccc = min(max(cc, 0), M - VEC);
      v[i] = *reinterpret_cast<const uint4*>(stack + size_t(n) * plane_sz * M + (size_t(rowc) * K + ppc) * M +
                                             (vec ? ccc : 0));
      (void)vbase;
    }
  };
  auto stage = [&](const uint4 (&v)[PER], unsigned valid) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = threadIdx.x + 256 * i;
      if (e < NE) {
        const int q = e % QN, pl = (e / QN) % BH, j = e / (QN * BH);
        Chunk16 x;
        x.u = (valid >> i) & 1u ? v[i] : make_uint4(0u, 0u, 0u, 0u);
        float* dst = &box[j][pl][VEC * q];
#pragma unroll
        for (int h = 0; h < VEC; h += 4)
          *reinterpret_cast<float4*>(dst + h) = make_float4(chunk_value<InT>(x, h), chunk_value<InT>(x, h + 1),
                                                            chunk_value<InT>(x, h + 2), chunk_value<InT>(x, h + 3));
      }
    }
  };

  float acc[YB];
#pragma unroll
  for (int j = 0; j < YB; ++j) acc[j] = 0.0f;
  uint4 buf[PER];
  unsigned valid = 0u;
  int r0 = 0, p0 = 0, c0 = 0;
  bool fits = false;
  if (nb > 0) {
    fits = origin(0, r0, p0, c0);
    if (fits) fetch(0, r0, p0, c0, buf, valid);
  }
  for (int n = 0; n < nb; ++n) {
    const bool fits_n = fits;
    const int rr0 = r0, pp0 = p0, cc0 = c0;
    __syncthreads();                                    // previous view's LDS reads are done
    if (fits_n) stage(buf, valid);
    __syncthreads();
    if (n + 1 < nb) {                                   // next view's loads overlap this view's math
      fits = origin(n + 1, r0, p0, c0);
      if (fits) fetch(n + 1, r0, p0, c0, buf, valid);
    }
    if (!live) continue;
    const ViewGeom& g = geom[n];
    const float inv = scale ? 1.0f / scale[n] : 1.0f;   // exact: the scale is a power of two
    const double bc = g.u[0] * rx + g.u[2] * rz + hm;
    const double br = g.v[0] * rx + g.v[2] * rz + hm;
    const double bp = g.d[0] * rx + g.d[2] * rz + hk;
    if (fits_n) {
      // box-local coordinates of the thread's first voxel row in FP64, rounded once; the
      // other rows step by (u_y, v_y, d_y) in FP32 (|local| < 32: error ~1e-6 voxel)
      const double ry0 = y0 - c;
      const float lc0 = float(g.u[1] * ry0 + bc - cc0), lr0 = float(g.v[1] * ry0 + br - rr0);
      const float lp0 = flat ? 0.0f : float(g.d[1] * ry0 + bp - pp0);
      const float uy = float(g.u[1]), vy = float(g.v[1]), dy = flat ? 0.0f : float(g.d[1]);
#pragma unroll
      for (int j = 0; j < YB; ++j) {
        // fmax guards against a rounding-level dip below the box origin
        const float fc = fmaxf(fmaf(float(j), uy, lc0), 0.0f);
        const float fr = fmaxf(fmaf(float(j), vy, lr0), 0.0f);
        const float fp = fmaxf(fmaf(float(j), dy, lp0), 0.0f);
        const float fc0 = floorf(fc), fr0 = floorf(fr), fp0 = floorf(fp);
        const float tc = fc - fc0, tr = fr - fr0, tp = fp - fp0;
        const int lc = int(fc0), lr = int(fr0), lp = int(fp0);
        const int lp1 = flat ? lp : lp + 1;
        const float* a0 = &box[lr][lp][lc];
        const float* a1 = &box[lr][lp1][lc];
        const float* b0 = &box[lr + 1][lp][lc];
        const float* b1 = &box[lr + 1][lp1][lc];
        const float wp1 = flat ? 0.0f : tp, wp0 = 1.0f - wp1;
        const float v0 = a0[0] + tc * (a0[1] - a0[0]);
        const float v1 = a1[0] + tc * (a1[1] - a1[0]);
        const float v2 = b0[0] + tc * (b0[1] - b0[0]);
        const float v3 = b1[0] + tc * (b1[1] - b1[0]);
        acc[j] += inv * ((1.0f - tr) * (wp0 * v0 + wp1 * v1) + tr * (wp0 * v2 + wp1 * v3));
      }
    } else {
      const InT* base = stack + size_t(n) * plane_sz * M;
      // one voxel row per iteration (rare path: keep its registers small)
#pragma unroll 1
      for (int j = 0; j < YB; ++j) {
        const double ry = (y0 + j) - c;
        const double fc = g.u[1] * ry + bc, fr = g.v[1] * ry + br, fp = g.d[1] * ry + bp;
        const double fc0 = floor(fc), fr0 = floor(fr), fp0 = floor(fp);
        const float tc = float(fc - fc0), tr = float(fr - fr0), tp = float(fp - fp0);
        const int c0i = int(fc0), r0i = int(fr0), p0i = int(fp0);
        const float wc0 = (unsigned(c0i) < unsigned(M)) ? 1.0f - tc : 0.0f;
        const float wc1 = (unsigned(c0i + 1) < unsigned(M)) ? tc : 0.0f;
        const float wr0 = (unsigned(r0i) < unsigned(M)) ? 1.0f - tr : 0.0f;
        const float wr1 = (unsigned(r0i + 1) < unsigned(M)) ? tr : 0.0f;
        const float wp0 = flat ? 1.0f : (unsigned(p0i) < unsigned(K)) ? 1.0f - tp : 0.0f;
        const float wp1 = flat ? 0.0f : (unsigned(p0i + 1) < unsigned(K)) ? tp : 0.0f;
        const int c0c = min(max(c0i, 0), M - 1), c1c = min(max(c0i + 1, 0), M - 1);
        const int r0c = min(max(r0i, 0), M - 1), r1c = min(max(r0i + 1, 0), M - 1);
        const int p0c = flat ? 0 : min(max(p0i, 0), K - 1), p1c = flat ? 0 : min(max(p0i + 1, 0), K - 1);
        const InT* a0 = base + (size_t(r0c) * K + p0c) * M;
        const InT* a1 = base + (size_t(r0c) * K + p1c) * M;
        const InT* b0 = base + (size_t(r1c) * K + p0c) * M;
        const InT* b1 = base + (size_t(r1c) * K + p1c) * M;
        const float v0 = wc0 * from_store<InT>(a0[c0c]) + wc1 * from_store<InT>(a0[c1c]);
        const float v1 = wc0 * from_store<InT>(a1[c0c]) + wc1 * from_store<InT>(a1[c1c]);
        const float v2 = wc0 * from_store<InT>(b0[c0c]) + wc1 * from_store<InT>(b0[c1c]);
        const float v3 = wc0 * from_store<InT>(b1[c0c]) + wc1 * from_store<InT>(b1[c1c]);
        const float add = inv * (wr0 * (wp0 * v0 + wp1 * v1) + wr1 * (wp0 * v2 + wp1 * v3));
#pragma unroll
        for (int jj = 0; jj < YB; ++jj) acc[jj] += (jj == j) ? add : 0.0f;
      }
    }
  }
  if (!live) return;
#pragma unroll
  for (int j = 0; j < YB; ++j) {
    const int iy = y0 + j;
    if (iy < N) {
      float* dst = vol + (size_t(iz) * N + iy) * N + ix;
      *dst = accumulate ? *dst + acc[j] : acc[j];
    }
  }
}

// Near-axis general frames (single-axis scans with a tilt, directions close to the rotation
// axis's normal plane): per view, the bounding box of the workgroup's 16 (x) x YB (y) x 16 (z)
// voxel tile in (row, plane, column) coordinates -- BR = YB + 4 detector rows x 24 planes x
// BOXW columns -- is fetched straight into LDS by buffer loads with the LDS destination, as in
// k_grid_axis_dma: chunk-linear boxes, chunks outside the stack zero-filled by the hardware, two
// boxes alternating so that view n + 1 is in flight while view n is interpolated (trilinear:
// eight LDS taps per voxel row; with ONE_BOX a single box, fetched and then interpolated, two
// barriers per view).  Per view the box origin, its extent and whether the footprint
// fits are computed one view per lane (FP32 with a margin, from the tile corners) and read out with
// readlane; only the view's own extent is fetched, and a view whose footprint does not fit is gathered
// for that tile straight from global memory.  Bound by vector issue (FP16, 4 rows: 79 % of the cycles;
// FP64-to-FP32 coordinates of three conversions each took 30 % more instructions) and the fetch path
// (texture data unit busy 88 %, two thirds of that waiting for L2).  The 4-row kernel is held to six waves per SIMD (80
// VGPRs): 256^3 with FP16 stacks over a tilt-jittered scan, per 8-view launch 318 us before, 296 with
// fixed-point coordinates at five waves, 280 at six, 310 at seven (spills).  For directions far
// from the axis, whose footprints often take the global gather, the bound costs time: the
// autotuner sees both.  The 8-row kernel would spill at such a bound.
template <int YB>
constexpr int tilt_waves_per_eu() { return YB == 4 ? 6 : 1; }
template <int YB, class InT, bool ONE_BOX>
__global__ __launch_bounds__(256, tilt_waves_per_eu<YB>()) void k_grid_tilt_dma(const InT* __restrict__ stack,
                                                       const ViewGeom* __restrict__ geom,
                                                       const float* __restrict__ scale,
                                                       float* __restrict__ vol, int N, int M, int K, int nb,
                                                       int accumulate, int flat, double hm, double hk) {
  constexpr int VEC = DmaBox<InT>::VEC, BOXW = DmaBox<InT>::BOXW, QN = BOXW / VEC;
  constexpr int ES = int(sizeof(InT));                  // bytes per stored value
  constexpr int BR = YB + 4, BH = AX_BOXH;              // rows and planes staged per view
  constexpr int QP = ES == 2 ? QN + 1 : QN;             // 16-byte slots per (row, plane): one spare for 16-bit
  constexpr int PITCH = QP * 4;                         // dwords per staged (row, plane)
  constexpr int NE = BR * BH * QP;                      // slots per staged view
  constexpr int PER = (NE + 255) / 256;                 // loads per thread per view
  constexpr int PAD = ES == 2 ? 4 : 0;                  // 16-bit tap pairs may read one dword past a row
  __shared__ __attribute__((aligned(16))) unsigned box0[NE * 4 + PAD];
  __shared__ __attribute__((aligned(16))) unsigned box1[ONE_BOX ? 4 : NE * 4 + PAD];
  const int ntx = (N + GT - 1) / GT;
  const int tiles = ntx * ntx;
  const int wg = blockIdx.x, xcd = wg & 7, k = wg >> 3;
  const int yblk = xcd + 8 * (k / tiles), tile = k % tiles;
  const int y0 = yblk * YB;
  if (y0 >= N) return;                                  // uniform
  const int tx0 = (tile % ntx) * GT, tz0 = (tile / ntx) * GT;
  const int ix = tx0 + (threadIdx.x % GT);
  const int iz = tz0 + (threadIdx.x / GT);
  const bool live = ix < N && iz < N;
  const double c = 0.5 * (N - 1);
  const double rx = ix - c, rz = iz - c, ry0 = y0 - c;
  const size_t view_sz = size_t(K) * M * M;
  const int wbase = (threadIdx.x & ~63) * 4;            // this wave's first dword in a box, per load
  const int lane = threadIdx.x & 63;

  // box origin (column rounded down to a 16-byte chunk), extent and fit of view n, one view per
  // lane; the extent is packed as columns | rows << 10 | planes << 20
  int obase = -64, lane_c0 = 0, lane_r0 = 0, lane_p0 = 0, lane_fit = 0, lane_ext = 0;
  auto origin = [&](int n, int& c0, int& r0, int& p0, int& ext) -> bool {
    if (n >= obase + 64) {
      obase = n;
      const int v = n + lane;
      int cc = 0, rr = 0, pp = 0, ft = 0, ex = 0;
      if (v < nb) {
        const int t0 = opaque(tx0), z0 = opaque(tz0);
        const float cf = float(c);
        const float lo[3] = {float(t0) - cf, float(ry0), float(z0) - cf}, ed[3] = {GT - 1, YB - 1, GT - 1};
        const ViewGeom& g = geom[v];
        // one detector coordinate at a time (fewer registers live at once)
        auto extremes = [&](const double* w, double h0, int& fmn, int& fmx) {
          float mn = float(h0), mx = mn;
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            const float wa = float(w[a]), e = wa * lo[a], f = wa * (lo[a] + ed[a]);
            mn += fminf(e, f);
            mx += fmaxf(e, f);
          }
          fmn = int(floorf(mn - kBoxMargin));
          fmx = int(floorf(mx));
          __builtin_amdgcn_sched_barrier(0);
        };
        int cmn, cmx, rmn, rmx, pmn, pmx;
        extremes(g.u, hm, cmn, cmx);
        extremes(g.v, hm, rmn, rmx);
        extremes(g.d, hk, pmn, pmx);
        cc = cmn & ~(VEC - 1);
        rr = rmn;
        pp = flat ? 0 : pmn;
        // taps reach floor(max) + 1; one slot of slack for the rounding of the extremes
        const int cn = cmx + 3 - cc, rn = rmx + 3 - rr;
        const int pn = flat ? 2 : pmx + 3 - pp;
        ft = cn <= BOXW && rn <= BR && pn <= BH;
        if (ft) ex = ((cn + VEC - 1) & ~(VEC - 1)) | (rn << 10) | (pn << 20);
      }
      lane_c0 = cc;
      lane_r0 = rr;
      lane_p0 = pp;
      lane_fit = ft;
      lane_ext = ex;
    }
    c0 = __builtin_amdgcn_readlane(lane_c0, n - obase);
    r0 = __builtin_amdgcn_readlane(lane_r0, n - obase);
    p0 = __builtin_amdgcn_readlane(lane_p0, n - obase);
    ext = __builtin_amdgcn_readlane(lane_ext, n - obase);
    return __builtin_amdgcn_readlane(lane_fit, n - obase) != 0;
  };
  // per chunk slot: byte offset from the box origin, and its (row, plane, column) in the box
  // (the host launches this kernel only for M a multiple of VEC and views below 2^31 bytes)
  unsigned cfo[PER], slot[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int e = threadIdx.x + 256 * i;
    const int q = e % QP, pl = (e / QP) % BH, j = e / (QP * BH);
    const bool used = e < NE && q < QN;                 // the spare 16-bit slot is never fetched
    slot[i] = slot_pack(used ? j : 127, used ? pl : 0, VEC * q);
    cfo[i] = unsigned((j * K + pl) * M + VEC * q) * unsigned(ES);
  }
  auto load = [&](int n, int c0, int r0, int p0, int ext, unsigned* dst) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<InT*>(stack + size_t(n) * view_sz), short(0), int(view_sz * ES), 0x00020000);
    // slots outside the view's extent fetch nothing (their LDS words are never read)
    const int cw = ext & 1023, rh = (ext >> 10) & 1023, bh = ext >> 20;
    const unsigned se = slot_extent(rh, bh, cw);
    if (r0 >= 0 && r0 + rh <= M && p0 >= 0 && p0 + bh <= K && c0 >= 0 && c0 + cw <= M) {
      const int so = ((r0 * K + p0) * M + c0) * ES;
#pragma unroll
      for (int i = 0; i < PER; ++i)
        if (slot_inside(se, slot[i]))
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)(dst + 1024 * i + wbase), 16, int(cfo[i]), so,
                                                   0, 0);
    } else {
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        if (slot_inside(se, slot[i])) {
          const int sl = opaque(int(slot[i]));
          const int row = r0 + (sl & 255), pp = p0 + (sl >> 8 & 255), cc = c0 + (sl >> 16);
          const bool ok = unsigned(row) < unsigned(M) && unsigned(pp) < unsigned(K) && unsigned(cc) < unsigned(M);
          const unsigned off = ok ? unsigned((row * K + pp) * M + cc) * unsigned(ES) : kOutOfRange;
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)(dst + 1024 * i + wbase), 16, int(off), 0,
                                                   0, 0);
        }
      }
    }
  };

  const unsigned mask = fix_mask();
  float acc[YB];
#pragma unroll
  for (int j = 0; j < YB; ++j) acc[j] = 0.0f;
  int oc0 = 0, or0 = 0, op0 = 0, oc1 = 0, or1 = 0, op1 = 0;   // origins of the views in each buffer
  int oe0 = 0, oe1 = 0;                                       // their extents
  bool of0 = false, of1 = false;                              // their footprints fit
  // wait for this wave's loads and LDS reads, then for every wave
  auto sync = [&]() {
    __builtin_amdgcn_s_waitcnt(7 << 4);                 // vmcnt(0) lgkmcnt(0)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // interpolation of view n from its staged box bx (origin cb, rb, pb; fb: it fits)
  auto interp = [&](const unsigned* bx, int cb, int rb, int pb, bool fb, int n) {
    if (!live) return;
    const ViewGeom& g = geom[n];
    float inv = 1.0f;
    if constexpr (std::is_same<InT, __half>::value) inv = 1.0f / scale[n];   // exact: a power of two
    // flat (one plane): a zero depth direction and hk = 0 put every tap on plane 0 with the
    // second plane's (zero-filled) taps at weight 0
    const double d0 = flat ? 0.0 : g.d[0], d1 = flat ? 0.0 : g.d[1], d2 = flat ? 0.0 : g.d[2];
    if (fb) {
      // box-local coordinates of the first voxel row; the other rows step by (u_y, v_y, d_y)
      unsigned vc = fix_of(g.u[0] * rx + g.u[1] * ry0 + g.u[2] * rz + (hm + kFixBias)) - (unsigned(cb) << 23);
      unsigned vr = fix_of(g.v[0] * rx + g.v[1] * ry0 + g.v[2] * rz + (hm + kFixBias)) - (unsigned(rb) << 23);
      unsigned vp = fix_of(d0 * rx + d1 * ry0 + d2 * rz + (hk + kFixBias)) - (unsigned(pb) << 23);
      const unsigned uy = fix_of(g.u[1] + kFixBias), vy = fix_of(g.v[1] + kFixBias), dy = fix_of(d1 + kFixBias);
#pragma unroll
      for (int j = 0; j < YB; ++j, vc += uy, vr += vy, vp += dy) {
        const unsigned lc = fix_index(vc);
        const float tc = fix_frac(vc, mask), tr = fix_frac(vr, mask), tp = fix_frac(vp, mask);
        // dwords to (row, plane)
        const int o = int(__umul24(fix_index(vr), unsigned(BH * PITCH)) + __umul24(fix_index(vp), unsigned(PITCH)));
        float v[4];                                     // (row, plane) = (lr + a, lp + b) at 2 a + b, along the columns
#pragma unroll
        for (int ab = 0; ab < 4; ++ab) {
          const int oo = o + (ab >> 1) * BH * PITCH + (ab & 1) * PITCH;
          if constexpr (ES == 4) {
            const float* r0 = reinterpret_cast<const float*>(bx) + oo + lc;
            v[ab] = fmaf(tc, r0[1] - r0[0], r0[0]);
          } else {
            const unsigned* r0 = bx + oo + (lc >> 1);
            v[ab] = lerp_pair<InT>(__builtin_amdgcn_alignbit(r0[1], r0[0], (lc & 1u) * 16u), tc);
          }
        }
        const float w0 = fmaf(tp, v[1] - v[0], v[0]), w1 = fmaf(tp, v[3] - v[2], v[2]);
        acc[j] = fmaf(inv, fmaf(tr, w1 - w0, w0), acc[j]);
      }
    } else {
      const InT* base = stack + size_t(n) * view_sz;
      // footprint too large for the box: one voxel row per iteration from global memory
#pragma unroll 1
      for (int j = 0; j < YB; ++j) {
        const double ry = ry0 + j;
        const double fc = g.u[0] * rx + g.u[1] * ry + g.u[2] * rz + hm;
        const double fr = g.v[0] * rx + g.v[1] * ry + g.v[2] * rz + hm;
        const double fp = d0 * rx + d1 * ry + d2 * rz + hk;
        const double fc0 = floor(fc), fr0 = floor(fr), fp0 = floor(fp);
        const float tc = float(fc - fc0), tr = float(fr - fr0), tp = float(fp - fp0);
        const int c0i = int(fc0), r0i = int(fr0), p0i = int(fp0);
        const float wc0 = (unsigned(c0i) < unsigned(M)) ? 1.0f - tc : 0.0f;
        const float wc1 = (unsigned(c0i + 1) < unsigned(M)) ? tc : 0.0f;
        const float wr0 = (unsigned(r0i) < unsigned(M)) ? 1.0f - tr : 0.0f;
        const float wr1 = (unsigned(r0i + 1) < unsigned(M)) ? tr : 0.0f;
        const float wp0 = (unsigned(p0i) < unsigned(K)) ? 1.0f - tp : 0.0f;
        const float wp1 = (unsigned(p0i + 1) < unsigned(K)) ? tp : 0.0f;
        const int c0c = min(max(c0i, 0), M - 1), c1c = min(max(c0i + 1, 0), M - 1);
        const int r0c = min(max(r0i, 0), M - 1), r1c = min(max(r0i + 1, 0), M - 1);
        const int p0c = min(max(p0i, 0), K - 1), p1c = min(max(p0i + 1, 0), K - 1);
        const InT* a0 = base + (size_t(r0c) * K + p0c) * M;
        const InT* a1 = base + (size_t(r0c) * K + p1c) * M;
        const InT* b0 = base + (size_t(r1c) * K + p0c) * M;
        const InT* b1 = base + (size_t(r1c) * K + p1c) * M;
        const float v0 = wc0 * from_store<InT>(a0[c0c]) + wc1 * from_store<InT>(a0[c1c]);
        const float v1 = wc0 * from_store<InT>(a1[c0c]) + wc1 * from_store<InT>(a1[c1c]);
        const float v2 = wc0 * from_store<InT>(b0[c0c]) + wc1 * from_store<InT>(b0[c1c]);
        const float v3 = wc0 * from_store<InT>(b1[c0c]) + wc1 * from_store<InT>(b1[c1c]);
        const float add = inv * (wr0 * (wp0 * v0 + wp1 * v1) + wr1 * (wp0 * v2 + wp1 * v3));
#pragma unroll
        for (int jj = 0; jj < YB; ++jj) acc[jj] += (jj == j) ? add : 0.0f;
      }
    }
  };
  // two boxes: view n + 1 is fetched while view n is interpolated, one barrier per view
  auto step = [&](const unsigned* bx, int& cb, int& rb, int& pb, bool& fb, unsigned* other, int& co, int& ro,
                  int& po, int& eo, bool& fo, int n) {
    if (n >= nb) return;                                // uniform
    sync();
    if (n + 1 < nb) {
      fo = origin(n + 1, co, ro, po, eo);
      if (fo) load(n + 1, co, ro, po, eo, other);
    }
    interp(bx, cb, rb, pb, fb, n);
  };
  if constexpr (ONE_BOX) {
    // one box (half the LDS, so more workgroups per CU hide each other's fetches): fetch,
    // wait, interpolate, two barriers per view
    for (int n = 0; n < nb; ++n) {
      if (n > 0) sync();                                // every wave is done with the box
      of0 = origin(n, oc0, or0, op0, oe0);
      if (of0) load(n, oc0, or0, op0, oe0, box0);
      sync();
      interp(box0, oc0, or0, op0, of0, n);
    }
  } else {
    if (nb > 0) {
      of0 = origin(0, oc0, or0, op0, oe0);
      if (of0) load(0, oc0, or0, op0, oe0, box0);
    }
    for (int n0 = 0; n0 < nb; n0 += 2) {
      step(box0, oc0, or0, op0, of0, box1, oc1, or1, op1, oe1, of1, n0);
      step(box1, oc1, or1, op1, of1, box0, oc0, or0, op0, oe0, of0, n0 + 1);
    }
  }
  if (!live) return;
#pragma unroll
  for (int j = 0; j < YB; ++j) {
    const int iy = y0 + j;
    if (iy < N) {
      float* dst = vol + (size_t(iz) * N + iy) * N + ix;
      *dst = accumulate ? *dst + acc[j] : acc[j];
    }
  }
}

// General view frames, cubic tiles: 8 x 8 x 8 voxels, two per thread (iz and iz + 4).
// The voxel centres of a cube of edge 8 span at most 7 (|a_x| + |a_y| + |a_z|) <= 7 sqrt(3)
// < 12.2 along any unit vector a, so with the taps and the floor of the origin a box of
// 16 rows x 16 planes x CW columns (column start rounded down to a 16-byte boundary) holds
// the footprint for every view: no fallback path, whatever the orientation.
// k_grid_cube stages 16-bit rows of an odd number of values, which start at any halfword, value
// by value through registers.
template <class InT>
struct CubeBox;
template <>
struct CubeBox<__hip_bfloat16> {
  static constexpr int VEC = 8, CW = 24, CP = 24;
};
template <>
struct CubeBox<__half> {
  static constexpr int VEC = 8, CW = 24, CP = 24;
};
constexpr int CB_E = 8;    // voxel tile edge
constexpr int CB_R = 16;   // rows and planes staged per view

// Tile t of the n^3 tiles of the cubic-tile kernels, octant by octant: consecutive tiles, and so
// those of one XCD, lie in a compact block, whose footprint in a view touches fewer cache lines
// than a slab's.
__device__ __forceinline__ void cube_tile(int t, int n, int& tx, int& ty, int& tz) {
  const int h = (n + 1) / 2;
  int sx = h, sy = h, sz = h, ox = 0, oy = 0, oz = 0;
#pragma unroll
  for (int o = 0; o < 8; ++o) {
    ox = o & 1 ? h : 0;
    oy = o & 2 ? h : 0;
    oz = o & 4 ? h : 0;
    sx = o & 1 ? n - h : h;
    sy = o & 2 ? n - h : h;
    sz = o & 4 ? n - h : h;
    if (o == 7 || t < sx * sy * sz) break;
    t -= sx * sy * sz;
  }
  tx = ox + t % sx;
  ty = oy + t / sx % sy;
  tz = oz + t / (sx * sy);
}

template <class InT>
__global__ __launch_bounds__(256) void k_grid_cube(const InT* __restrict__ stack,
                                                   const ViewGeom* __restrict__ geom,
                                                   const float* __restrict__ scale,
                                                   float* __restrict__ vol, int N, int M, int K,
                                                   int nb, int accumulate, int flat) {
  using B = CubeBox<InT>;
  constexpr int VEC = B::VEC, CW = B::CW, CP = B::CP;
  constexpr int QN = CW / VEC;
  constexpr int NE = CB_R * CB_R * QN;
  constexpr int PER = (NE + 255) / 256;
  __shared__ float box[CB_R][CB_R][CP];
  // tiles of one XCD are consecutive in x, then y, then z (neighbours share stack rows in L2)
  const int ntc = (N + CB_E - 1) / CB_E;
  const int tiles = ntc * ntc * ntc;
  const int per = (tiles + 7) / 8;
  const int tile = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (tile >= tiles) return;                           // uniform
  const int tx0 = (tile % ntc) * CB_E, ty0 = ((tile / ntc) % ntc) * CB_E, tz0 = (tile / (ntc * ntc)) * CB_E;
  const int ix = tx0 + (threadIdx.x % CB_E), iy = ty0 + (threadIdx.x / CB_E) % CB_E;
  const int iz0 = tz0 + int(threadIdx.x) / (CB_E * CB_E);
  const bool live0 = ix < N && iy < N && iz0 < N, live1 = ix < N && iy < N && iz0 + 4 < N;
  const double c = 0.5 * (N - 1);
  const double rx = ix - c, ry = iy - c, rz0 = iz0 - c;
  const double hm = 0.5 * (M - 1), hk = 0.5 * (K - 1);
  const size_t plane_sz = size_t(K) * M;
  // (false for every stack that comes here, but a compiler that knows it reorders the loads: 125^3 from 40
  // views 1.18 -> 1.34 ms, 27^3 from 223 views 0.67 -> 0.79)
  const bool vec = (M % VEC) == 0;
  const double lo[3] = {tx0 - c, ty0 - c, tz0 - c};
  const double hi[3] = {tx0 + CB_E - 1 - c, ty0 + CB_E - 1 - c, tz0 + CB_E - 1 - c};

  auto origin = [&](int n, int& r0, int& p0, int& c0) {
    const ViewGeom& g = geom[n];
    double cmin = hm, rmin = hm, pmin = hk;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      cmin += fmin(g.u[a] * lo[a], g.u[a] * hi[a]);
      rmin += fmin(g.v[a] * lo[a], g.v[a] * hi[a]);
      pmin += fmin(g.d[a] * lo[a], g.d[a] * hi[a]);
    }
    c0 = int(floor(cmin)) & ~(VEC - 1);
    r0 = int(floor(rmin));
    p0 = flat ? 0 : int(floor(pmin));
  };
  // The view-independent part of every staged chunk (its row, plane and column offsets in
  // the box and its LDS offset), computed once; per view only the box origin moves.
  int cj[PER], cpl[PER], cq[PER], cdst[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int e = threadIdx.x + 256 * i;
    cq[i] = VEC * (e % QN);
    cpl[i] = (e / QN) % CB_R;
    cj[i] = e < NE ? e / (QN * CB_R) : -1;
    cdst[i] = e < NE ? (cj[i] * CB_R + cpl[i]) * CP + cq[i] : -1;
  }
  auto fetch = [&](int n, int r0, int p0, int c0, uint4 (&v)[PER], unsigned& valid) {
    const InT* vbase = stack + size_t(n) * plane_sz * M;
    valid = 0u;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int row = r0 + cj[i], pp = p0 + cpl[i], cc = c0 + cq[i];
      const bool ok = cj[i] >= 0 && unsigned(row) < unsigned(M) && unsigned(pp) < unsigned(K) && cc >= 0 && cc < M;
      valid |= ok ? (1u << i) : 0u;
      const int rowc = min(max(row, 0), M - 1), ppc = min(max(pp, 0), K - 1);
      if (vec) {
        const unsigned off = unsigned(rowc * K + ppc) * unsigned(M) + unsigned(min(max(cc, 0), M - VEC));
        v[i] = *reinterpret_cast<const uint4*>(vbase + off);
      } else {
        const InT* src = vbase + (size_t(rowc) * K + ppc) * M;
        Chunk16 x;
#pragma unroll
        for (int kk = 0; kk < VEC; ++kk) {
          const int ce = min(max(cc + kk, 0), M - 1);
          const bool ek = unsigned(cc + kk) < unsigned(M);
          x.h[kk] = ek ? reinterpret_cast<const unsigned short*>(src)[ce] : (unsigned short)0;
        }
        v[i] = x.u;
        if (cj[i] >= 0 && unsigned(row) < unsigned(M) && unsigned(pp) < unsigned(K)) valid |= (1u << i);
      }
    }
  };
  auto stage = [&](const uint4 (&v)[PER], unsigned valid) {
    float* boxf = &box[0][0][0];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      if (cdst[i] >= 0) {
        Chunk16 x;
        x.u = (valid >> i) & 1u ? v[i] : make_uint4(0u, 0u, 0u, 0u);
        float* dst = boxf + cdst[i];
#pragma unroll
        for (int h = 0; h < VEC; h += 4)
          *reinterpret_cast<float4*>(dst + h) = make_float4(chunk_value<InT>(x, h), chunk_value<InT>(x, h + 1),
                                                            chunk_value<InT>(x, h + 2), chunk_value<InT>(x, h + 3));
      }
    }
  };

  float acc0 = 0.0f, acc1 = 0.0f;
  uint4 buf[PER];
  unsigned valid = 0u;
  int r0 = 0, p0 = 0, c0 = 0;
  if (nb > 0) {
    origin(0, r0, p0, c0);
    fetch(0, r0, p0, c0, buf, valid);
  }
  for (int n = 0; n < nb; ++n) {
    const int rr0 = r0, pp0 = p0, cc0 = c0;
    __syncthreads();
    stage(buf, valid);
    __syncthreads();
    if (n + 1 < nb) {
      origin(n + 1, r0, p0, c0);
      fetch(n + 1, r0, p0, c0, buf, valid);
    }
    const ViewGeom& g = geom[n];
    const float inv = scale ? 1.0f / scale[n] : 1.0f;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const double rz = rz0 + 4 * h;
      // box-local coordinates (FP64, rounded once); fmax guards a rounding-level dip below the origin
      const float fc = float(fmax(g.u[0] * rx + g.u[1] * ry + g.u[2] * rz + hm - cc0, 0.0));
      const float fr = float(fmax(g.v[0] * rx + g.v[1] * ry + g.v[2] * rz + hm - rr0, 0.0));
      const float fp = flat ? 0.0f : float(fmax(g.d[0] * rx + g.d[1] * ry + g.d[2] * rz + hk - pp0, 0.0));
      const float fc0 = floorf(fc), fr0 = floorf(fr), fp0 = floorf(fp);
      const float tc = fc - fc0, tr = fr - fr0, tp = flat ? 0.0f : fp - fp0;
      const int lc = int(fc0), lr = int(fr0), lp = int(fp0);
      const int lp1 = flat ? lp : lp + 1;
      const float* a0 = &box[lr][lp][lc];
      const float* a1 = &box[lr][lp1][lc];
      const float* b0 = &box[lr + 1][lp][lc];
      const float* b1 = &box[lr + 1][lp1][lc];
      const float v0 = a0[0] + tc * (a0[1] - a0[0]);
      const float v1 = a1[0] + tc * (a1[1] - a1[0]);
      const float v2 = b0[0] + tc * (b0[1] - b0[0]);
      const float v3 = b1[0] + tc * (b1[1] - b1[0]);
      const float add = inv * ((1.0f - tr) * ((1.0f - tp) * v0 + tp * v1) + tr * ((1.0f - tp) * v2 + tp * v3));
      if (h == 0) acc0 += add;
      else acc1 += add;
    }
  }
  if (live0) {
    float* dst = vol + (size_t(iz0) * N + iy) * N + ix;
    *dst = accumulate ? *dst + acc0 : acc0;
  }
  if (live1) {
    float* dst = vol + (size_t(iz0 + 4) * N + iy) * N + ix;
    *dst = accumulate ? *dst + acc1 : acc1;
  }
}

// The cube kernel of every other stack: each view's footprint is fetched straight into LDS by
// buffer loads (no register staging, no per-chunk clamps: what lies outside the stack gets an offset
// past the buffer's range and reads as zeros).  Per view only the footprint's own extent of the box
// is fetched (over random directions about 2.2 times fewer bytes than the whole box), and the
// box origins and extents of 64 views are computed at once, one view per lane.  One box and two
// barriers per view: a second box (view n + 1 in flight while view n is interpolated) halves
// the workgroups per CU and measured slower.
//
// Bound by the fetches' latency and what they miss in L2 (a quarter of its reads; the texture data
// unit is busy 70 % of the time, half of it waiting), and by vector issue (55 %; about 120
// instructions per wave and view): hence FP32 box origins and packed slots (71 VGPRs, so seven
// workgroups per CU, with 94 five), tiles of an XCD in octants (cube_tile), and fixed-point
// coordinates.  96^3, 120 views: 310 us; with slabs, five workgroups and FP64 coordinates 384;
// octants with five workgroups 358; slabs with six 416 (more views in flight than L2 holds).
//
// CH is the fetch, in bytes per lane.  16: rows of whole 16-byte chunks, a box of 16 x 16 x 20
// (16-bit values: 24) whose columns start at a chunk; each staged row is followed by XS spare
// slots that are never fetched: at a row pitch of 344 dwords the tap reads of a wave (an 8 x 8
// voxel slice, rotated into the box) meet 3.5 bank cycles per pair read in a count over random
// directions, against 5.3 at 320, where taps in different rows fall on one bank.  4: rows of
// whole dwords, a box of 16 columns (16-bit values: 18); one load of the view group fetches one
// box row (lane = plane and column), so that the rows may lie at a pitch of 268 or 260 dwords
// (bank cycles within 1 % of the best pitch, against twice as many at 256): 90^3, 60 views
// 185 us, against 524 staged through registers value by value.
//
// G view groups of 256 threads take every G-th view of one tile, each with its own box, and
// their sums are added through LDS in the order of the groups.
template <int ES, int CH>
struct CubeFetch;                                      // ES: bytes per stored value
template <>
struct CubeFetch<4, 16> {
  static constexpr int QN = 5, XS = 6, SR = CB_R * QN + XS, NE = CB_R * SR;   // chunks per (row, plane), spares, slots
  static constexpr int CW = 20, PP = 20, RP = SR * 4, BOX = NE * 4;           // columns; pitches and box, dwords
};
template <>
struct CubeFetch<2, 16> {
  static constexpr int QN = 3, XS = 2, SR = CB_R * QN + XS, NE = CB_R * SR;
  static constexpr int CW = 24, PP = 12, RP = SR * 4, BOX = NE * 4;
};
template <>
struct CubeFetch<4, 4> {
  static constexpr int QN = 16, SR = 256, NE = 256;    // slots of one load
  static constexpr int CW = 16, PP = 16, RP = CB_R * PP + 12, BOX = CB_R * RP;
};
template <>
struct CubeFetch<2, 4> {
  static constexpr int QN = 16, SR = 256, NE = 256;
  static constexpr int CW = 18, PP = 16, RP = CB_R * PP + 4, BOX = CB_R * RP;
};

template <class InT, int CH, int G>
__global__ __launch_bounds__(256 * G) void k_grid_cube_dma(const InT* __restrict__ stack,
                                                           const ViewGeom* __restrict__ geom,
                                                           const float* __restrict__ scale,
                                                           float* __restrict__ vol, int N, int M, int K, int nb,
                                                           int accumulate, int flat) {
  constexpr int ES = int(sizeof(InT)), V = CH / ES;    // bytes per stored value, values per slot
  using F = CubeFetch<ES, CH>;
  __shared__ __attribute__((aligned(16))) unsigned boxes[G * F::BOX];
  const int ntc = (N + CB_E - 1) / CB_E;
  const int tiles = ntc * ntc * ntc;
  const int per = (tiles + 7) / 8;
  const int tile = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (tile >= tiles) return;                           // uniform
  const int grp = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 8), tid = threadIdx.x & 255;
  unsigned* box = boxes + grp * F::BOX;
  int tx0, ty0, tz0;
  cube_tile(tile, ntc, tx0, ty0, tz0);
  tx0 *= CB_E;
  ty0 *= CB_E;
  tz0 *= CB_E;
  const int ix = tx0 + (tid % CB_E), iy = ty0 + (tid / CB_E) % CB_E;
  const int iz0 = tz0 + tid / (CB_E * CB_E);
  const bool live0 = ix < N && iy < N && iz0 < N, live1 = ix < N && iy < N && iz0 + 4 < N;
  const double c = 0.5 * (N - 1);
  const double rx = ix - c, ry = iy - c, rz0 = iz0 - c;
  const double hm = 0.5 * (M - 1), hk = flat ? 0.0 : 0.5 * (K - 1);
  const size_t view_sz = size_t(K) * M * M;
  const int lane = threadIdx.x & 63;

  // Box origin as in k_grid_cube and extent of a view, lane l of every wave for step
  // obase + l of its group; per view the workgroup-uniform values are read out of one lane into
  // scalar registers.  Taps lie at most one past the floor of a voxel's coordinates, and one more
  // row, plane and column absorb a last-bit difference between the corner and the voxel
  // arithmetic (at most 16 rows, planes and columns past the rounding to chunks: a tile's
  // footprint spans < 12.2).
  int obase = -64, lane_o = 0, lane_e = 0;
  auto origin = [&](int step, int& r0, int& p0, int& c0, int& rh, int& ph, int& cw) {
    if (step >= obase + 64) {
      obase = step;
      const int v = (step + lane) * G + grp;
      int o = 0, ex = 0;
      if (v < nb) {
        const float cf = float(c);
        const float lo[3] = {float(opaque(tx0)) - cf, float(opaque(ty0)) - cf, float(opaque(tz0)) - cf};
        const ViewGeom& g = geom[v];
        // one detector coordinate at a time (fewer registers live at once)
        auto extremes = [&](const double* w, double h0, int& fmn, int& fmx) {
          float mn = float(h0), mx = mn;
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            const float wa = float(w[a]), e = wa * lo[a], f = wa * (lo[a] + float(CB_E - 1));
            mn += fminf(e, f);
            mx += fmaxf(e, f);
          }
          fmn = int(floorf(mn - kBoxMargin));
          fmx = int(floorf(mx));
          __builtin_amdgcn_sched_barrier(0);
        };
        int cmn, cmx, rmn, rmx, pmn, pmx;
        extremes(g.u, hm, cmn, cmx);
        extremes(g.v, hm, rmn, rmx);
        extremes(g.d, hk, pmn, pmx);
        const int cc = cmn & ~(V - 1);
        const int rr = rmn;
        const int pp = flat ? 0 : pmn;
        const int ww = min(F::CW, (cmx - cc + 3 + V - 1) & ~(V - 1));
        const int hh = min(CB_R, rmx - rr + 3);
        const int dd = flat ? 2 : min(CB_R, pmx - pp + 3);
        // packed in 12-bit fields, offset by 1024 (rows, planes) and 2048 (columns): a tile
        // corner is at most sqrt(3) (N - 1) / 2 < 887 from the volume centre (N <= 1024), so
        // every origin lies in [-890, 1024 + 887) (M <= 256, K <= 2048)
        o = (rr + 1024) | ((pp + 1024) << 12);
        ex = (cc + 2048) | (ww << 12) | (hh << 18) | (dd << 24);
      }
      lane_o = o;
      lane_e = ex;
    }
    const int o = __builtin_amdgcn_readlane(lane_o, step - obase);
    const int ex = __builtin_amdgcn_readlane(lane_e, step - obase);
    r0 = (o & 4095) - 1024;
    p0 = ((o >> 12) & 4095) - 1024;
    c0 = (ex & 4095) - 2048;
    cw = (ex >> 12) & 63;
    rh = (ex >> 18) & 63;
    ph = (ex >> 24) & 63;
  };
  // (views are below 2^31 bytes, as M <= 256 and K <= 2048; M is a multiple of V); what lies outside the
  // view's extent is not fetched (its LDS words are never read)
  constexpr int PER = CH == 16 ? (F::BOX / 4 + 255) / 256 : 1;
  // 16-byte slots: offsets in the box (spare slots and slots past the box are never fetched)
  // and bytes from the box origin; dword loads: lane = plane and column, one load per row
  unsigned cfo[PER], slot[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int e = CH == 16 ? tid + 256 * i : tid;
    const int row = CH == 16 ? e / F::SR : 0, rem = CH == 16 ? e % F::SR : e;
    const int pl = rem / F::QN, q = rem % F::QN * V;
    const bool used = CH == 4 || (e < F::NE && rem < CB_R * F::QN);
    slot[i] = slot_pack(used ? row : 127, used ? pl : 0, q);
    cfo[i] = unsigned((row * K + pl) * M + q) * unsigned(ES);
  }
  unsigned* dst = box + (tid & ~63) * (CH / 4);           // this wave's first dword of a load
  auto load = [&](int n, int r0, int p0, int c0, int rh, int ph, int cw) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<InT*>(stack + size_t(n) * view_sz), short(0), int(view_sz * ES), 0x00020000);
    const bool inside = r0 >= 0 && r0 + rh <= M && p0 >= 0 && p0 + ph <= K && c0 >= 0 && c0 + cw <= M;
    const unsigned ext = slot_extent(CH == 16 ? rh : 1, ph, cw);
    if constexpr (CH == 16) {
      if (inside) {
        const int so = ((r0 * K + p0) * M + c0) * ES;
#pragma unroll
        for (int i = 0; i < PER; ++i)
          if (slot_inside(ext, slot[i]))
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)(dst + 1024 * i), 16, int(cfo[i]), so, 0, 0);
      } else {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
          if (slot_inside(ext, slot[i])) {
            // c0 and M are multiples of V: a slot is wholly inside or wholly outside the columns
            const int sl = opaque(int(slot[i]));
            const int row = r0 + (sl & 255), pp = p0 + (sl >> 8 & 255), cc = c0 + (sl >> 16);
            const bool ok = unsigned(row) < unsigned(M) && unsigned(pp) < unsigned(K) && unsigned(cc) < unsigned(M);
            const unsigned off = ok ? unsigned((row * K + pp) * M + cc) * unsigned(ES) : kOutOfRange;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)(dst + 1024 * i), 16, int(off), 0, 0, 0);
          }
        }
      }
    } else if (slot_inside(ext, slot[0])) {
      if (inside) {
        int so = ((r0 * K + p0) * M + c0) * ES;
#pragma unroll
        for (int i = 0; i < CB_R; ++i, so += ES * K * M)
          if (i < rh)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)(dst + F::RP * i), 4, int(cfo[0]), so, 0, 0);
      } else {
        const int sl = opaque(int(slot[0]));
        const int pp = p0 + (sl >> 8 & 255), cc = c0 + (sl >> 16);
        const bool ok = unsigned(pp) < unsigned(K) && unsigned(cc) < unsigned(M);
#pragma unroll
        for (int i = 0; i < CB_R; ++i) {
          if (i < rh) {
            const int row = r0 + i;
            const unsigned off = ok && unsigned(row) < unsigned(M) ? unsigned((row * K + pp) * M + cc) * unsigned(ES) : kOutOfRange;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)(dst + F::RP * i), 4, int(off), 0, 0, 0);
          }
        }
      }
    }
  };
  auto sync = [&]() {
    __builtin_amdgcn_s_waitcnt(7 << 4);                // vmcnt(0) lgkmcnt(0): this wave's loads and reads
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  const unsigned mask = fix_mask();
  float acc0 = 0.0f, acc1 = 0.0f;
  const int steps = (nb + G - 1) / G;
  for (int step = 0; step < steps; ++step) {
    const int n = step * G + grp;
    int rr0 = 0, pp0 = 0, cc0 = 0, rh = 0, ph = 0, cw = 0;
    sync();                                            // every wave is done with the box
    if (G == 1 || n < nb) {
      origin(step, rr0, pp0, cc0, rh, ph, cw);
      load(n, rr0, pp0, cc0, rh, ph, cw);
    }
    sync();                                            // every wave's share has landed
    if (G > 1 && n >= nb) break;                       // the last step of this group: no barrier after it
    const ViewGeom& g = geom[n];
    float inv = 1.0f;
    if constexpr (std::is_same<InT, __half>::value) inv = 1.0f / scale[n];   // exact: a power of two
    // flat (one plane): a zero depth coordinate puts every tap on plane 0, with the second
    // plane's (zero-filled) taps at weight 0
    const double d0 = flat ? 0.0 : g.d[0], d1 = flat ? 0.0 : g.d[1], d2 = flat ? 0.0 : g.d[2];
    unsigned vc = fix_of(g.u[0] * rx + g.u[1] * ry + g.u[2] * rz0 + (hm + kFixBias)) - (unsigned(cc0) << 23);
    unsigned vr = fix_of(g.v[0] * rx + g.v[1] * ry + g.v[2] * rz0 + (hm + kFixBias)) - (unsigned(rr0) << 23);
    unsigned vp = fix_of(d0 * rx + d1 * ry + d2 * rz0 + (hk + kFixBias)) - (unsigned(pp0) << 23);
    const unsigned sc = fix_of(4.0 * g.u[2] + kFixBias), sr = fix_of(4.0 * g.v[2] + kFixBias);
    const unsigned sp = fix_of(4.0 * d2 + kFixBias);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float tc = fix_frac(vc, mask), tr = fix_frac(vr, mask), tp = fix_frac(vp, mask);
      const unsigned lc = fix_index(vc);
      const unsigned* o = box + __umul24(fix_index(vr), F::RP) + __umul24(fix_index(vp), F::PP);
      float v[4];                                      // (row, plane) = (lr + a, lp + b) at 2 a + b, along the columns
#pragma unroll
      for (int ab = 0; ab < 4; ++ab) {
        const unsigned* oo = o + (ab >> 1) * F::RP + (ab & 1) * F::PP;
        if constexpr (ES == 4) {
          const float* r0 = reinterpret_cast<const float*>(oo) + lc;
          v[ab] = fmaf(tc, r0[1] - r0[0], r0[0]);
        } else {
          const unsigned* r0 = oo + (lc >> 1);
          v[ab] = lerp_pair<InT>(__builtin_amdgcn_alignbit(r0[1], r0[0], (lc & 1u) * 16u), tc);
        }
      }
      const float w0 = fmaf(tp, v[1] - v[0], v[0]), w1 = fmaf(tp, v[3] - v[2], v[2]);
      const float add = fmaf(tr, w1 - w0, w0);
      if (h == 0) acc0 = fmaf(inv, add, acc0);
      else acc1 = fmaf(inv, add, acc1);
      vc += sc;
      vr += sr;
      vp += sp;
    }
  }
  if constexpr (G > 1) {
    // a group's own box holds its sums: every wave of it has to be done with the taps
    sync();
    if (grp > 0) {
      box[tid] = __float_as_uint(acc0);
      box[256 + tid] = __float_as_uint(acc1);
    }
    sync();
    if (grp > 0) return;
#pragma unroll
    for (int k = 1; k < G; ++k) {
      acc0 += __uint_as_float(boxes[k * F::BOX + tid]);
      acc1 += __uint_as_float(boxes[k * F::BOX + 256 + tid]);
    }
  }
  if (live0) {
    float* dst0 = vol + (size_t(iz0) * N + iy) * N + ix;
    *dst0 = accumulate ? *dst0 + acc0 : acc0;
  }
  if (live1) {
    float* dst1 = vol + (size_t(iz0 + 4) * N + iy) * N + ix;
    *dst1 = accumulate ? *dst1 + acc1 : acc1;
  }
}

// ------------------------------------------------------------------ plan tables (FP64)

__device__ __forceinline__ double2 filter_value(const FilterArgs& fa, const ViewGeom& g,
                                                const double* wv, int ky, int kx, int n) {
  const double qx = signed_q(kx, fa.M, fa.dx), qy = signed_q(ky, fa.M, fa.dx);
  const double q2 = qx * qx + qy * qy;
  double w;
  if (fa.mode == 0) w = g.a * fabs(qx);
  else if (fa.mode == 1) w = 2.0 * sqrt(q2) / double(fa.n_views);
  else w = wv[(size_t(n) * fa.M + ky) * fa.M + kx];
  const double omega = atan(fa.sigma);
  const double cst = fa.lambda / (4.0 * M_PI * sqrt(1.0 + fa.sigma * fa.sigma));
  const double chi = M_PI * fa.lambda * g.R * q2 - omega;
  double sn, cs;
  sincos(chi, &sn, &cs);
  const double hre = sn / (sn * sn + fa.epsilon);
  const double him = fa.ewald ? -cs / (cs * cs + fa.epsilon) : 0.0;
  return make_double2(cst * w * hre, cst * w * him);
}

__global__ void k_filter_table(FilterArgs fa, const ViewGeom* __restrict__ geom,
                               const double* __restrict__ wtab, float4* __restrict__ filt) {
  const size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const size_t per = size_t(fa.M) * fa.M;
  if (i >= per * fa.n_views) return;
  const int n = int(i / per);
  const int ky = int((i % per) / fa.M), kx = int(i % fa.M);
  const ViewGeom g = geom[n];
  const double2 f = filter_value(fa, g, wtab, ky, kx, n);
  const double2 fm = filter_value(fa, g, wtab, (fa.M - ky) % fa.M, (fa.M - kx) % fa.M, n);
  // F_h = (F(k) + conj F(-k))/2, F_a = (F(k) - conj F(-k))/2
  const double hr = 0.5 * (f.x + fm.x), hi = 0.5 * (f.y - fm.y);
  const double ar = 0.5 * (f.x - fm.x), ai = 0.5 * (f.y + fm.y);
  const double inv = 1.0 / (double(fa.M) * double(fa.M));
  // G1 = (1+i) F_h / M^2,  G2 = -(1+i) F_a / M^2
  float4 o;
  o.x = float((hr - hi) * inv);
  o.y = float((hr + hi) * inv);
  o.z = float(-(ar - ai) * inv);
  o.w = float(-(ar + ai) * inv);
  filt[i] = o;
}

// Sampling matrix in 2^-32 fixed point (integer atomics: order independent).
__global__ void k_sampling_splat(FilterArgs fa, const ViewGeom* __restrict__ geom,
                                 unsigned long long* __restrict__ smat) {
  const size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const size_t per = size_t(fa.M) * fa.M;
  if (i >= per * fa.n_views) return;
  const int n = int(i / per);
  const int ky = int((i % per) / fa.M), kx = int(i % fa.M);
  double p[3];
  sample_point(fa, geom[n], ky, kx, p);
  const int N = fa.N, lo = -(N / 2);
  for (int sgn = 0; sgn < 2; ++sgn) {
    double f[3];
    int i0[3];
    double t[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      f[a] = (sgn ? -p[a] : p[a]) - lo;
      const double fl = floor(f[a]);
      i0[a] = int(fl);
      t[a] = f[a] - fl;
    }
    for (int cz = 0; cz < 2; ++cz)
      for (int cy = 0; cy < 2; ++cy)
        for (int cx = 0; cx < 2; ++cx) {
          const int jx = i0[0] + cx, jy = i0[1] + cy, jz = i0[2] + cz;
          if (unsigned(jx) >= unsigned(N) || unsigned(jy) >= unsigned(N) || unsigned(jz) >= unsigned(N))
            continue;
          const double w = (cx ? t[0] : 1.0 - t[0]) * (cy ? t[1] : 1.0 - t[1]) * (cz ? t[2] : 1.0 - t[2]);
          const unsigned long long fx = (unsigned long long)llrint(0.5 * w * kFix);
          atomicAdd(&smat[(size_t(jz) * N + jy) * N + jx], fx);
        }
  }
}

__global__ void k_sampling_weights(FilterArgs fa, const ViewGeom* __restrict__ geom,
                                   const unsigned long long* __restrict__ smat, double* __restrict__ wtab) {
  const size_t i = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
  const size_t per = size_t(fa.M) * fa.M;
  if (i >= per * fa.n_views) return;
  const int n = int(i / per);
  const int ky = int((i % per) / fa.M), kx = int(i % fa.M);
  double p[3];
  sample_point(fa, geom[n], ky, kx, p);
  const int N = fa.N, lo = -(N / 2), hi = (N + 1) / 2 - 1;
  bool inside = true;
  double t[3];
  int i0[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    inside = inside && (p[a] >= lo) && (p[a] <= hi);
    const double f = p[a] - lo;
    const double fl = floor(f);
    i0[a] = int(fl);
    t[a] = f - fl;
  }
  double shat = 0.0;
  for (int cz = 0; cz < 2; ++cz)
    for (int cy = 0; cy < 2; ++cy)
      for (int cx = 0; cx < 2; ++cx) {
        const int jx = i0[0] + cx, jy = i0[1] + cy, jz = i0[2] + cz;
        if (unsigned(jx) >= unsigned(N) || unsigned(jy) >= unsigned(N) || unsigned(jz) >= unsigned(N))
          continue;
        const double w = (cx ? t[0] : 1.0 - t[0]) * (cy ? t[1] : 1.0 - t[1]) * (cz ? t[2] : 1.0 - t[2]);
        shat += w * (double(smat[(size_t(jz) * N + jy) * N + jx]) / kFix);
      }
  const double scale = double(fa.M) * fa.M / (double(N) * N * N * fa.dx);
  wtab[i] = inside ? scale * shat / (shat * shat + fa.eps_sampling) : 0.0;
}

// ------------------------------------------------------------------ launchers
// Size table of the spectra / plane kernels: one group per translation unit.
const FftSize* fft_size(int M) {
  struct Group {
    const FftSize* sizes;
    int count;
  };
  static const Group groups[] = {
      {kFftSizesA, kFftSizesACount}, {kFftSizesB, kFftSizesBCount}, {kFftSizesC, kFftSizesCCount},
      {kFftSizesD, kFftSizesDCount}, {kFftSizesE, kFftSizesECount}, {kFftSizesF, kFftSizesFCount},
      {kFftSizesG, kFftSizesGCount}, {kFftSizesH, kFftSizesHCount}, {kFftSizesI, kFftSizesICount},
      {kFftSizesJ, kFftSizesJCount}};
  for (const Group& g : groups)
    for (int i = 0; i < g.count; ++i)
      if (g.sizes[i].M == M) return &g.sizes[i];
  return nullptr;
}

bool fft_supported(int M) { return fft_size(M) != nullptr; }

int fft_split(int M) {
  const FftSize* f = fft_size(M);
  return f ? f->P : 0;
}

int spectra_groups(int M) { return (M / 2 + 1 + 15) / 16; }

size_t spectra_scratch_bytes(int M) { return size_t((M + 1) / 2) * M * sizeof(float2); }

hipError_t launch_spectra(int M, const float* images, const double2* tw, const float4* filt, float4* q, int* status,
                          double inv_iin, int nb, hipStream_t s, void* scratch, size_t scratch_bytes) {
  if (nb <= 0) return hipSuccess;
  const FftSize* f = fft_size(M);
  if (!f || !f->spectra) return hipErrorInvalidValue;
  return f->spectra(SpectraLaunch{images, tw, filt, q, static_cast<float2*>(scratch),
                                  scratch_bytes / spectra_scratch_bytes(M), status, inv_iin, nullptr, nb, s});
}

hipError_t launch_spectra32(int M, const float* images, const float4* filt, const float2* tw_fwd, const float2* tw_half_fwd,
                            float4* q, int* status, double inv_iin, float* scale, float* l1part, int nb, hipStream_t s) {
  if (nb <= 0) return hipSuccess;
  const FftSize* f = fft_size(M);
  if (!f) return hipErrorInvalidValue;
  return f->spectra32(Spectra32Launch{images, filt, tw_fwd, tw_half_fwd, q, status, inv_iin, scale, l1part, nb, s});
}

hipError_t launch_spectra_complex(int M, const float* images, const double2* tw, const float2* filt, float2* q, int* status,
                                  double inv_iin, int nb, hipStream_t s, void* scratch, size_t scratch_bytes, float* l1) {
  if (nb <= 0) return hipSuccess;
  const FftSize* f = fft_size(M);
  if (!f) return hipErrorInvalidValue;
  return f->spectra_complex(SpectraLaunch{images, tw, filt, q, static_cast<float2*>(scratch),
                                          scratch_bytes / spectra_scratch_bytes(M), status, inv_iin, l1, nb, s});
}

hipError_t launch_planes(int M, int dtype, const float4* q, const float2* prop, const float2* tw_inv,
                         void* stack, int K, int npairs, int nb, const float* scale, hipStream_t s,
                         const float2* tw_half_inv) {
  if (nb <= 0) return hipSuccess;
  const FftSize* f = fft_size(M);
  if (!f) return hipErrorInvalidValue;
  return f->planes(PlanesLaunch{dtype, q, prop, tw_inv, tw_half_inv, stack, K, npairs, nb, scale, s});
}

template <int kYB, class InT>
static hipError_t grid_impl(bool axis_fast, const void* stack, const ViewGeom* geom, const float* scale,
                            float* vol, int N, int M, int K, int nb, int accumulate, int flat, hipStream_t s) {
  const dim3 grid((N + GT - 1) / GT, (N + GT - 1) / GT, (N + kYB - 1) / kYB);
  const InT* st = static_cast<const InT*>(stack);
  if (axis_fast) {
    // flat grid: (x, z) tiles x row blocks, row blocks padded to a multiple of 8 (one XCD each)
    if (size_t(K) * M * M * sizeof(InT) > size_t(0x7fffffff)) return hipErrorInvalidValue;
    const int tiles = int(grid.x * grid.y);
    const auto blocks = [&](int rows) { return dim3(unsigned(tiles * (((N + rows - 1) / rows + 7) / 8 * 8))); };
    if (flat) {
      hipLaunchKernelGGL((k_grid_axis_flat<8, InT>), blocks(8), dim3(256), 0, s, st, geom, scale, vol, N, M, nb,
                         accumulate, 0.5 * (M - 1));
    } else if (M % DmaBox<InT>::VEC == 0) {
      hipLaunchKernelGGL((k_grid_axis_dma<kYB, InT, 16>), blocks(kYB), dim3(256), 0, s, st, geom, scale, vol, N, M, K,
                         nb, accumulate, 0.5 * (M - 1), 0.5 * (K - 1));
    } else if (M % (4 / int(sizeof(InT))) == 0) {
      // rows that are not whole 16-byte chunks: the box is fetched dword by dword, four rows
      // (the slots of eight would take 84 registers)
      hipLaunchKernelGGL((k_grid_axis_dma<4, InT, 4>), blocks(4), dim3(256), 0, s, st, geom, scale, vol, N, M, K, nb,
                         accumulate, 0.5 * (M - 1), 0.5 * (K - 1));
    } else {
      return hipErrorInvalidValue;
    }
  } else if constexpr (kYB >= 4) {
    const int tiles = int(grid.x * grid.y);
    const int yblocks8 = int((grid.z + 7) / 8 * 8);
    hipLaunchKernelGGL((k_grid_box<kYB, InT>), dim3(unsigned(tiles * yblocks8)), dim3(256), 0, s, st, geom,
                       scale, vol, N, M, K, nb, accumulate, flat);
  } else {
    return hipErrorInvalidValue;   // 2 rows per thread: single-axis plans only
  }
  return hipGetLastError();
}

template <int YB>
static hipError_t grid_dtype(bool axis_fast, int dtype, const void* stack, const ViewGeom* geom, const float* scale,
                             float* vol, int N, int M, int K, int nb, int accumulate, int flat, hipStream_t s) {
  switch (dtype) {
    case 0: return grid_impl<YB, float>(axis_fast, stack, geom, nullptr, vol, N, M, K, nb, accumulate, flat, s);
    case 1:
      return grid_impl<YB, __hip_bfloat16>(axis_fast, stack, geom, nullptr, vol, N, M, K, nb, accumulate, flat, s);
    case 2: return grid_impl<YB, __half>(axis_fast, stack, geom, scale, vol, N, M, K, nb, accumulate, flat, s);
    default: return hipErrorInvalidValue;
  }
}

template <class InT>
static hipError_t grid_cube_impl(const InT* stack, const ViewGeom* geom, const float* scale, float* vol, int N, int M,
                                 int K, int nb, int accumulate, int flat, hipStream_t s) {
  constexpr int ES = int(sizeof(InT));
  const int ntc = (N + CB_E - 1) / CB_E;
  const int tiles = ntc * ntc * ntc, per = (tiles + 7) / 8;
  auto go = [&](auto ch, auto groups) {
    constexpr int CH = decltype(ch)::value, G = decltype(groups)::value;
    hipLaunchKernelGGL((k_grid_cube_dma<InT, CH, G>), dim3(unsigned(8 * per)), dim3(256 * G), 0, s, stack, geom, scale,
                       vol, N, M, K, nb, accumulate, flat);
    return hipGetLastError();
  };
  // One tile per workgroup and one view at a time leave a small volume with one wave per SIMD
  // and every fetch exposed.  Up to one tile per CU four view groups share a tile (45^3, 60
  // views: 41 us, two groups 53, one 79), up to two per CU two do (64^3, 100 views: 106 us, one
  // group 134, four 136; 50^3, 60 views: 74, 97, 82); beyond that the tiles fill the chip by
  // themselves (72^3, 100 views: one group 164 us, two 184).
  // But no group without a view: its waves only delay the others' barriers (16^3, one view per
  // launch: 9.4 us with four groups).  The sums are those of four or two groups, bit for bit.
  using std::integral_constant;
  auto pick = [&](auto ch) {
    if (tiles <= 256 && nb > 2) return go(ch, integral_constant<int, 4>{});
    if (tiles <= 512 && nb > 1) return go(ch, integral_constant<int, 2>{});
    return go(ch, integral_constant<int, 1>{});
  };
  // rows of whole 16-byte chunks take the wide fetch (96^3, 120 views: 384 us, by dwords 432)
  if (M * ES % 16 == 0) return pick(integral_constant<int, 16>{});
  if (M * ES % 4 == 0) return pick(integral_constant<int, 4>{});
  if constexpr (ES == 2) {
    hipLaunchKernelGGL(k_grid_cube<InT>, dim3(unsigned(8 * per)), dim3(256), 0, s, stack, geom, scale, vol, N, M, K,
                       nb, accumulate, flat);
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

template <int YB, class InT>
static hipError_t grid_tilt_impl(const void* stack, const ViewGeom* geom, const float* scale, float* vol, int N,
                                 int M, int K, int nb, int accumulate, int flat, hipStream_t s) {
  if (M % DmaBox<InT>::VEC != 0 || size_t(K) * M * M * sizeof(InT) > size_t(0x7fffffff)) return hipErrorInvalidValue;
  const int ntx = (N + GT - 1) / GT;
  const int yblocks8 = ((N + YB - 1) / YB + 7) / 8 * 8;
  // 4 and 8 rows: one box per workgroup, six / four workgroups per CU instead of three / two with
  // two boxes (256^3 FP32, per 8-view launch, with five / four: 376 vs 385 us, 363 vs 446 us); 2 rows
  // keep two boxes
  hipLaunchKernelGGL((k_grid_tilt_dma<YB, InT, YB >= 4>), dim3(unsigned(ntx * ntx * yblocks8)), dim3(256), 0, s,
                     static_cast<const InT*>(stack), geom, scale, vol, N, M, K, nb, accumulate, flat, 0.5 * (M - 1),
                     flat ? 0.0 : 0.5 * (K - 1));
  return hipGetLastError();
}

template <int YB>
static hipError_t grid_tilt_dtype(int dtype, const void* stack, const ViewGeom* geom, const float* scale, float* vol,
                                  int N, int M, int K, int nb, int accumulate, int flat, hipStream_t s) {
  switch (dtype) {
    case 0: return grid_tilt_impl<YB, float>(stack, geom, nullptr, vol, N, M, K, nb, accumulate, flat, s);
    case 1: return grid_tilt_impl<YB, __hip_bfloat16>(stack, geom, nullptr, vol, N, M, K, nb, accumulate, flat, s);
    case 2: return grid_tilt_impl<YB, __half>(stack, geom, scale, vol, N, M, K, nb, accumulate, flat, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_grid(bool axis_fast, int dtype, const void* stack, const ViewGeom* geom, const float* scale,
                       float* vol, int N, int M, int K, int nb, int accumulate, int flat, hipStream_t s, int rows) {
  if (rows == kGridTilt8 && !axis_fast)
    return grid_tilt_dtype<8>(dtype, stack, geom, scale, vol, N, M, K, nb, accumulate, flat, s);
  if (rows == kGridTilt4 && !axis_fast)
    return grid_tilt_dtype<4>(dtype, stack, geom, scale, vol, N, M, K, nb, accumulate, flat, s);
  if (rows == kGridTilt2 && !axis_fast)
    return grid_tilt_dtype<2>(dtype, stack, geom, scale, vol, N, M, K, nb, accumulate, flat, s);
  if (rows == 0 && !axis_fast) {
    switch (dtype) {
      case 0: return grid_cube_impl(static_cast<const float*>(stack), geom, nullptr, vol, N, M, K, nb, accumulate, flat, s);
      case 1: return grid_cube_impl(static_cast<const __hip_bfloat16*>(stack), geom, nullptr, vol, N, M, K, nb, accumulate, flat, s);
      case 2: return grid_cube_impl(static_cast<const __half*>(stack), geom, scale, vol, N, M, K, nb, accumulate, flat, s);
      default: return hipErrorInvalidValue;
    }
  }
  if (rows == 4) return grid_dtype<4>(axis_fast, dtype, stack, geom, scale, vol, N, M, K, nb, accumulate, flat, s);
  if (rows == 2 && axis_fast)
    return grid_dtype<2>(axis_fast, dtype, stack, geom, scale, vol, N, M, K, nb, accumulate, flat, s);
  if (rows == 8) return grid_dtype<8>(axis_fast, dtype, stack, geom, scale, vol, N, M, K, nb, accumulate, flat, s);
  return hipErrorInvalidValue;
}

static const AxisSize* axis_size_of(int M) {
  struct Group {
    const AxisSize* sizes;
    int count;
  };
  static const Group groups[] = {{kAxisSizesA, kAxisSizesACount}, {kAxisSizesB, kAxisSizesBCount},
                                 {kAxisSizesC, kAxisSizesCCount}, {kAxisSizesD, kAxisSizesDCount},
                                 {kAxisSizesE, kAxisSizesECount}};
  for (const Group& g : groups)
    for (int i = 0; i < g.count; ++i)
      if (g.sizes[i].M == M) return &g.sizes[i];
  return nullptr;
}

bool axis_supported(int M, int N, int K) {
  return axis_size_of(M) && N <= M && K <= M && (M - N) % 2 == 0 && (M - K) % 2 == 0;
}

size_t axis_part_bytes(int M, int N) {
  const AxisSize* a = axis_size_of(M);
  return a ? size_t(a->n_slices) * axis_slice_pitch(N) * sizeof(float) : 0;
}

// Where a single-axis reconstruction is faster by plane stacks than by slices (us of a pass by slices /
// by stacks):
//  - the shortest scans of small detectors, which cost their launches and the latency of one workgroup
//    each: one launch more by slices, or two (32^2: one view 15.5 / 13.0, three 16.2 / 15.0, four 15.9 /
//    16.5; 36^2 three 17.0 / 15.3; 64^2 one 21.2 / 18.3, 80^2 one 25.2 / 25.2; rows that are not whole
//    16-byte chunks cost stacks more: 50^2 one 19.8 / 18.3, 54^2 one 18.8 / 20.0).
//  - few planes, whose stacks leave room for fewer partial volumes than would fill the device, so that
//    the blocks are long serial chains (32^2, 2 planes, 30 views: one block of 30, 70 / 47; 128^2, 2
//    planes, 120 views 492 / 235; but 32^2, 4 planes, 30 views: three blocks of 10, 33 / 49).
//  - volumes of a small part of a large detector, M > 128: slices transform all of it for any N and K
//    (192^2, 120 views: 24^3 from 24 planes 1270 / 477, 96^3 from 96 planes 1400 / 1257, 144^3 from 144
//    planes faster by slices; 160^2: 20^3 538 / 382, 40^3 from 40 planes 549 / 568).
static bool stacks_faster(const AxisSize* a, int M, int N, int K, int n, int cus, int blocks, int wanted) {
  if (M <= 72 && size_t(n) * M <= size_t(M % 4 == 0 ? 108 : 50)) return true;
  if (blocks < wanted) {
    // a view of a block takes M / 16 us with complex and M / 28 with real cells, times the workgroups
    // that share a CU; a view by stacks 1.25 us and its share of the gridding and the transforms
    const double view = (M <= 64 ? std::max(M / 16.0, 1.5) : M / 28.0) * ((a->units * blocks + cus - 1) / cus);
    // (a third more where rows are not whole 16-byte chunks: 90^2, 10 planes, 30 views 76 / 86)
    const double stacks = (1.25 + 5e-7 * N * N * N + (M > 128 ? 2.2e-6 : 1.1e-6) * K * M * M) * (M % 4 == 0 ? 1.0 : 1.35);
    if (((n + blocks - 1) / blocks + 1) * view > n * stacks + 3.0) return true;
  }
  const double part = double(K) / M + 0.3 * N * N * N / (double(M) * M * M);
  return M > 128 && n > 4 && part < (M <= 162 ? 0.4 : M <= 180 ? 0.5 : 0.7);
}

int axis_blocks(int M, int N, int K, int n, int cus, size_t room) {
  const AxisSize* a = axis_size_of(M);
  if (!a || room == 0) return 0;
  // Workgroups (units x blocks) run in rounds of at most two per CU, each over its block's views
  // (and about two views' time of set-up); every block adds a partial volume to sum, a fifth of a
  // view's time.  Measured: 128^3 from 180 views takes 337 us with the 4 blocks of this rule (512
  // workgroups), 406 with 2 and 445 with 3; 64^3 from 90 views 36 + 6.6 us (slices + columns) with
  // its 16, 49 + 5.4 with 8 and 35 + 8.0 with 24.  At least three views per block, but down to single views
  // where the workgroups leave CUs free (four views: 36^3 22.9 -> 16.8 us, 64^3 31.2 -> 22.9; with two
  // workgroups per CU one-view blocks lose, 128^3 47.5 -> 53.4).
  const int slots = cus * std::max(1, std::min(2, 160 * 1024 / a->lds));
  int best = 1;
  double least = 0.0;
  for (int b = 1; b <= n; ++b) {
    if (b > std::max(1, n / 3) && 8 * a->units * b > 7 * cus) break;
    const int rounds = (a->units * b + slots - 1) / slots;
    const double cost = rounds * double((n + b - 1) / b + 2) + 0.2 * b;
    if (b == 1 || cost < least) {
      least = cost;
      best = b;
    }
  }
  const int blocks = int(std::min<size_t>(room, size_t(best)));
  return stacks_faster(a, M, N, K, n, cus, blocks, best) ? 0 : blocks;
}

hipError_t launch_axis_spectra(int M, const float* images, const double2* tw, const float4* filt, float4* work, int* status,
                               double inv_iin, int nb, hipStream_t s) {
  const AxisSize* a = axis_size_of(M);
  if (!a) return hipErrorInvalidValue;
  // the slices' half rows (at most M + 1 rows of M/2 + 1) at the front of the views' 16 M^2 bytes,
  // the row pairs' spectra (4 M (M + 1) bytes at most) at their end
  const size_t mm = size_t(M) * M, pairs = size_t((M + 1) / 2) * M;
  float2* z = reinterpret_cast<float2*>(work + size_t(nb) * mm) - size_t(nb) * pairs;
  return a->spectra(SpectraLaunch{images, tw, filt, work, z, size_t(nb), status, inv_iin, nullptr, nb, s});
}

hipError_t launch_axis_slices(int M, const float4* work, const float2* prop, const float2* tw_inv,
                              const ViewGeom* geom, float* part, int N, int K, int npairs, int n, int blocks, hipStream_t s) {
  const AxisSize* a = axis_size_of(M);
  if (!a) return hipErrorInvalidValue;
  return a->slices(AxisLaunch{work, prop, tw_inv, nullptr, geom, part, nullptr, N, K, npairs, n, blocks, s});
}

hipError_t launch_axis_columns(int M, const float* part, const double2* tw, float* vol, int N, int blocks, hipStream_t s) {
  const AxisSize* a = axis_size_of(M);
  if (!a) return hipErrorInvalidValue;
  return a->columns(AxisLaunch{nullptr, nullptr, nullptr, tw, nullptr, const_cast<float*>(part), vol, N, 0, 0, 0, blocks, s});
}

hipError_t launch_filter_table(const FilterArgs& fa, const ViewGeom* geom, const double* wtab, float4* filt,
                               hipStream_t s) {
  const size_t total = size_t(fa.M) * fa.M * fa.n_views;
  hipLaunchKernelGGL(k_filter_table, dim3(unsigned((total + 255) / 256)), dim3(256), 0, s, fa, geom, wtab,
                     filt);
  return hipGetLastError();
}

hipError_t launch_sampling(const FilterArgs& fa, const ViewGeom* geom, unsigned long long* smat,
                           double* wtab, hipStream_t s) {
  const size_t total = size_t(fa.M) * fa.M * fa.n_views;
  const dim3 grid(unsigned((total + 255) / 256));
  hipLaunchKernelGGL(k_sampling_splat, grid, dim3(256), 0, s, fa, geom, smat);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_sampling_weights, grid, dim3(256), 0, s, fa, geom, smat, wtab);
  return hipGetLastError();
}

hipError_t launch_sampling_splat(const FilterArgs& fa, const ViewGeom* geom, unsigned long long* smat,
                                 hipStream_t s) {
  const size_t total = size_t(fa.M) * fa.M * fa.n_views;
  hipLaunchKernelGGL(k_sampling_splat, dim3(unsigned((total + 255) / 256)), dim3(256), 0, s, fa, geom, smat);
  return hipGetLastError();
}

hipError_t launch_spectra_out(const float4* q, float2* out, int M, int nb, hipStream_t s) {
  const size_t count = size_t(M) * M * nb;
  if (count == 0) return hipSuccess;
  hipLaunchKernelGGL(k_spectra_out, dim3(unsigned((count + 255) / 256)), dim3(256), 0, s, q, out, count,
                     float(double(M) * M));
  return hipGetLastError();
}

}  // namespace tomo
