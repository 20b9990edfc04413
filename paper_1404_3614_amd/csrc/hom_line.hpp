// Passes with register four-step transforms of any length M = A * B whose
// factors are in the radix set below (every 2/3/5-smooth length up to 729 but
// 512, 640 and 720), in FP32 or FP64 and for any N <= M: the lengths and
// types that have no compile-time specialisation.
//
// What bounds them is memory traffic and latency, so a line makes one LDS
// round trip per transform (the radix-2/3/4/5 passes of hom_kernels.hip make
// one per prime factor) and enters and leaves through registers: a thread
// computes one A- or B-point DFT with compile-time radix, chosen by a switch
// that is uniform over the block.  A, B, M and N are run-time values, so one
// kernel serves all lengths of a radix class; the class (largest radix 9, 16
// or 27) sets the registers a kernel needs, hence how many waves a SIMD holds.
//
// Measured against the generic passes (one launch, primal and dual running
// side by side): 24 FP32 cells of N = 113 x 135 on 225 x 375, column 324 -> 19
// us, first 44 -> 21, last 40 -> 20 (whole solve 27.4 -> 5.5 ms; 4.7 with the batched set-up); 8 FP64 cells
// of N = 313 on 625^2, column 113 -> 78 us, first 94 -> 60, last 60 -> 47 (25.8
// -> 18.9 ms); one FP64 GaNi cell on 600^2, column 37 -> 19, first 36 -> 19,
// last 30 -> 19 (10.2 -> 6.5 ms); the FP64 bound passes of 32 cells of N = 41^3,
// quadrature 1072 -> 523 us, middle 517 -> 290, first 320 -> 168.
//
// Slots.  A four-step transform leaves thread q's results in the slots it (or
// its successor step) reads, so the steps exchange in place with one barrier
// each: inverse, step 1 thread q < B holds x[B n1 + q] and writes slot (q, k1),
// step 2 thread k1 < A reads the slots (n2, k1) and holds X[k1 + A k2]; a
// forward transform runs the same slots backwards.
#pragma once
#include "hom_regfft.hpp"
#include "hom_rows.hpp"

#include <hip/hip_ext.h>

#include <type_traits>

namespace hom {
namespace ln {

// f(radix) for the run-time radix r (uniform over the block) of a class.
template <int RM, typename F>
__device__ __forceinline__ void with_radix(int r, F&& f) {
#define HOM_RX(n) \
  case n: f(std::integral_constant<int, n>{}); break;
  if constexpr (RM == 9) {
    switch (r) { HOM_RX(1) HOM_RX(2) HOM_RX(3) HOM_RX(4) HOM_RX(5) HOM_RX(6) HOM_RX(8) HOM_RX(9) default: break; }
  } else if constexpr (RM == 16) {
    switch (r) {
      HOM_RX(1) HOM_RX(2) HOM_RX(3) HOM_RX(4) HOM_RX(5) HOM_RX(6) HOM_RX(8) HOM_RX(9) HOM_RX(10) HOM_RX(12) HOM_RX(15)
      HOM_RX(16) default: break;
    }
  } else {
    switch (r) {
      HOM_RX(1) HOM_RX(2) HOM_RX(3) HOM_RX(4) HOM_RX(5) HOM_RX(6) HOM_RX(8) HOM_RX(9) HOM_RX(10) HOM_RX(12) HOM_RX(15)
      HOM_RX(16) HOM_RX(18) HOM_RX(20) HOM_RX(24) HOM_RX(25) HOM_RX(27) default: break;
    }
  }
#undef HOM_RX
}

#define HOM_INL __attribute__((always_inline))

// Position on the length-M axis -> kept index on Z_N, or -1 (H = (N - 1) / 2).
__device__ __forceinline__ int keep(int pos, int N, int M, int H) {
  return pos <= H ? pos : (pos >= M - H ? pos - (M - N) : -1);
}
template <typename R>
__device__ __forceinline__ Cx<R> conj_if(Cx<R> w, bool c) {
  return rf::mk<R>(w.x, c ? -w.y : w.y);
}

// Element i of a table at a 32-bit offset from its (block-uniform) base.
template <typename R>
__device__ __forceinline__ Cx<R> gldx(const Cx<R>* base, unsigned i) {
  if constexpr (sizeof(R) == 4) return gldc(base, i * 8u);
  else return __builtin_bit_cast(Cx<double>, gld<gdbl2>(base, i * 16u));
}

// ============================================================== column pass
// Axis 0 of every element (point, pack) of the row-pass buffer: inverse
// transform with zero padding N -> M, the pointwise work of KIND on the grid,
// forward transform with truncation (KIND COL_COEF, COL_TENSOR, COL_FWD).
//   COL_COEF    coefficient product inside a pack (2D packs hold one load's two
//               components; an isotropic coefficient acts on each field alone)
//   COL_TENSOR  3D symmetric coefficient: a load's components straddle packs,
//               so a block holds every pack of its points
//   COL_QUAD    the FP64 quadrature sums of the bounds, packs together
//   COL_GRID    inverse only, values to U.grid;  COL_FWD forward only, from it
// Lines of a block are its nl elements, one per lane group (l fastest), so
// global rows and LDS slots are read in runs of nl elements.  Workgroup x runs
// on XCD x % 8: each XCD takes a run of consecutive blocks, so the rows' cache
// lines shared by neighbouring blocks and the coefficient shared by the packs
// of a point stay in its L2.
//
// A block has one thread per line and DFT.  FP64, class 27: 8 lines are 128
// bytes of a row, 80 KB of LDS and 221 registers, two blocks of four waves per
// CU; with run-time pitch and hoisted coefficient loads it took 334 registers
// (one block) and 105 us where it now takes 78.  FP32, class 27: 16 lines, 512
// threads, 114 registers.
enum ColKind { COL_COEF = 0, COL_TENSOR = 1, COL_QUAD = 2, COL_GRID = 3, COL_FWD = 4 };

// Elements per block, the LDS pitch of a slot: as many lines as the threads
// allow for the largest radix of the class, known at compile time so that a
// thread's slots are constant LDS offsets.
template <typename R, int RM>
struct ColShape {
  static constexpr int NT = (RM == 27 && sizeof(R) == 4) ? 512 : 256;
  static constexpr int NL = RM == 9 ? 28 : (RM == 16 ? 16 : (sizeof(R) == 4 ? 16 : 8));
  static_assert(NL * RM <= NT, "one thread per line and DFT");
};

// f(n1, base) for the stored rows among the positions B n1 + q, n1 < RA: base
// is the row of Z_N of position B n1 (q is added by the caller), or f0(n1) for
// a dropped position.  Rows on one side of the padding for every q < B take a
// branch that is uniform over the block.
template <int RA, typename F, typename F0>
__device__ __forceinline__ void for_rows(int B, int q, int N, int M, int H, F&& f, F0&& f0) {
#pragma unroll
  for (int n1 = 0; n1 < RA; ++n1) {
    const int lo = B * n1, hi = lo + B - 1;
    if (hi <= H) {
      f(n1, lo);
    } else if (lo >= M - H) {
      f(n1, lo - (M - N));
    } else if (lo > H && hi < M - H) {
      f0(n1);
    } else {
      const int pos = lo + q;
      if (pos <= H) f(n1, lo);
      else if (pos >= M - H) f(n1, lo - (M - N));
      else f0(n1);
    }
  }
}

template <typename R, int RM, int KIND, int NC>
__global__ __launch_bounds__((ColShape<R, RM>::NT)) void k_col_reg(Geo g, const UnitDev* __restrict__ units, int cg) {
  constexpr int NL = ColShape<R, RM>::NL, NT = ColShape<R, RM>::NT;
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double s_red[kBlock / 64];
  Cx<R>* ex = reinterpret_cast<Cx<R>*>(smem);            // [M][NL]
  const UnitDev& U = units[blockIdx.z];
  if (cg) {
    bool any = false;
    for (int l = 0; l < g.L; ++l) any |= (U.sc[l].status == 0);
    if (!any) return;
  }
  constexpr bool WHOLE = KIND == COL_TENSOR || KIND == COL_QUAD;
  const int A = g.rA[0], B = g.rB[0], M = g.M[0], N = g.N[0], H = (N - 1) / 2;
  const int P = g.P, npts = g.M[1] * g.M[2], F = g.L * g.d;
  const int tp = g.rgT;
  const int nb = WHOLE ? (npts + tp - 1) / tp : (g.pmaj ? P * ((npts + NL - 1) / NL) : (npts * P + NL - 1) / NL);
  const int nb8 = (nb + 7) / 8;
  const int cb = (int)(blockIdx.x % 8) * nb8 + (int)(blockIdx.x / 8);
  if (cb >= nb) return;  // uniform over the block
  const int tid = threadIdx.x, l = tid % NL, q = tid / NL;
  int pt, pk;
  bool ok = true;
  if constexpr (WHOLE) {
    ok = l < tp * P;
    const int lw = ok ? l : 0;
    if (g.pmaj) {
      pk = lw / tp;
      pt = cb * tp + (lw - pk * tp);
    } else {
      pt = cb * tp + lw / P;
      pk = lw % P;
    }
  } else if (g.pmaj) {
    pk = cb % P;
    pt = (cb / P) * NL + l;
  } else {
    const int e = cb * NL + l;
    pt = e / P;
    pk = e - pt * P;
  }
  ok = ok && pt < npts;
  const size_t Mtot = (size_t)M * npts;
  Cx<R>* data = reinterpret_cast<Cx<R>*>(g.N[1] > 1 ? U.bufB : U.bufA);
  const size_t rs = g.pmaj ? (size_t)npts : (size_t)npts * P;
  // this thread's element: row i of Z_N at data[i rs + off]
  const size_t off = g.pmaj ? (size_t)pk * N * npts + pt : (size_t)pt * P + pk;
  const size_t offq = off + (size_t)q * rs;
  const Cx<R>* tw = reinterpret_cast<const Cx<R>*>(g.tw[0]);
  const R* coef = reinterpret_cast<const R*>(U.coef);
  const unsigned cq = (unsigned)((size_t)(q < A ? q : 0) * npts + (ok ? pt : 0)) * (unsigned)sizeof(R);
  const bool f0 = 2 * pk < F, f1 = 2 * pk + 1 < F;

  if constexpr (KIND != COL_FWD) {
    with_radix<RM>(A, [&](auto ra) HOM_INL {
      constexpr int RA = decltype(ra)::value;
      if (q < B) {
        Cx<R> v[RA];
        for_rows<RA>(
            B, q, N, M, H, [&](int n1, int row) HOM_INL { v[n1] = ok ? gload(data + (size_t)row * rs, offq) : rf::mk<R>(0, 0); },
            [&](int n1) HOM_INL { v[n1] = rf::mk<R>(0, 0); });
        rf::Dft<R, RA, 1>::run(v);
        Cx<R>* e = ex + q * RA * NL + l;
#pragma unroll
        for (int k1 = 0; k1 < RA; ++k1) e[k1 * NL] = rf::mul(v[k1], conj_if(gldx<R>(tw, (unsigned)(q * k1)), true));
      }
    });
    __syncthreads();
  }
  // step 2: thread q < A holds the grid values x0 = q + A k2 of its element; slot k2 A + q is x0 itself
  with_radix<RM>(B, [&](auto rb) HOM_INL {
    constexpr int RB = decltype(rb)::value;
    if (q < A) {
      Cx<R>* e = ex + q * NL + l;
      const int es = A * NL;
      Cx<R> v[RB];
      if constexpr (KIND == COL_FWD) {
#pragma unroll
        for (int k2 = 0; k2 < RB; ++k2) {
          const size_t gi = (size_t)(q + A * k2) * npts + pt;
          v[k2] = rf::mk<R>((ok && f0) ? (R)gload(U.grid + (size_t)(2 * pk) * Mtot, gi) : (R)0,
                            (ok && f1) ? (R)gload(U.grid + (size_t)(2 * pk + 1) * Mtot, gi) : (R)0);
        }
      } else {
#pragma unroll
        for (int n2 = 0; n2 < RB; ++n2) v[n2] = e[n2 * es];
        rf::Dft<R, RB, 1>::run(v);
      }
      if constexpr (KIND == COL_GRID) {
#pragma unroll
        for (int k2 = 0; k2 < RB; ++k2) {
          const size_t gi = (size_t)(q + A * k2) * npts + pt;
          if (ok && f0) U.grid[(size_t)(2 * pk) * Mtot + gi] = (float)v[k2].x;
          if (ok && f1) U.grid[(size_t)(2 * pk + 1) * Mtot + gi] = (float)v[k2].y;
        }
      } else if constexpr (WHOLE) {
#pragma unroll
        for (int k2 = 0; k2 < RB; ++k2) e[k2 * es] = v[k2];
      } else {
        if constexpr (KIND == COL_COEF) {
          // the loads stay behind the inverse DFT: hoisted, they cost the registers of a second line
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int k2 = 0; k2 < RB; ++k2) {
            const R* ck = coef + (size_t)(A * k2) * npts;  // uniform base, per-thread 32-bit offset
            if constexpr (NC == 1) {
              const R a = gld<R>(ck, cq);
              v[k2] = rf::mk<R>(f0 ? a * v[k2].x : (R)0, f1 ? a * v[k2].y : (R)0);
            } else {  // 2D: xx, yy, xy
              const R a0 = gld<R>(ck, cq), a1 = gld<R>(ck + Mtot, cq), a2 = gld<R>(ck + 2 * Mtot, cq);
              v[k2] = rf::mk<R>(a0 * v[k2].x + a2 * v[k2].y, a2 * v[k2].x + a1 * v[k2].y);
            }
          }
        }
        rf::Dft<R, RB, -1>::run(v);
#pragma unroll
        for (int m2 = 0; m2 < RB; ++m2) e[m2 * es] = rf::mul(v[m2], gldx<R>(tw, (unsigned)(q * m2)));
      }
    }
  });
  if constexpr (KIND == COL_GRID) return;
  __syncthreads();
  if constexpr (WHOLE) {
    double acc[kMaxLoads * kMaxLoads];
#pragma unroll
    for (int i = 0; i < kMaxLoads * kMaxLoads; ++i) acc[i] = 0.0;
    for (int t = tid; t < M * tp; t += NT) {
      const int x0 = t / tp, pi = t - x0 * tp;
      if (cb * tp + pi >= npts) continue;
      const size_t ci = (size_t)x0 * npts + cb * tp + pi;
      R a[6];
#pragma unroll
      for (int c = 0; c < 6; ++c) a[c] = c < g.nc ? gload(coef + c * Mtot, ci) : (R)0;
      R u[2 * kMaxPacks];
#pragma unroll
      for (int k = 0; k < kMaxPacks; ++k) {
        const Cx<R> z = k < P ? ex[x0 * NL + (g.pmaj ? k * tp + pi : pi * P + k)] : rf::mk<R>(0, 0);
        u[2 * k] = z.x;
        u[2 * k + 1] = z.y;
      }
      if constexpr (KIND == COL_QUAD) {
        if (g.d == 2)
          point_quad<R, 2>(g.nc, g.L, a, u, acc);
        else
          point_quad<R, 3>(g.nc, g.L, a, u, acc);
      } else {
        R w[2 * kMaxPacks];
#pragma unroll
        for (int k = 0; k < 2 * kMaxPacks; ++k) w[k] = (R)0;
        point_coef<R, 3>(g.nc, g.L, a, u, w);
#pragma unroll
        for (int k = 0; k < kMaxPacks; ++k)
          if (k < P) ex[x0 * NL + pi * P + k] = rf::mk<R>(w[2 * k], w[2 * k + 1]);
      }
    }
    if constexpr (KIND == COL_QUAD) {
      static_assert(NT == kBlock, "block_sum adds the waves of a kBlock block");
#pragma unroll
      for (int i = 0; i < kMaxLoads * kMaxLoads; ++i) {
        if (i / kMaxLoads >= g.L || i % kMaxLoads >= g.L) continue;  // uniform over the block
        const double s = block_sum(acc[i], s_red);
        if (tid == 0) U.part_q[(size_t)cb * 9 + i] = s;
      }
      return;
    }
    __syncthreads();
    with_radix<RM>(B, [&](auto rb) HOM_INL {
      constexpr int RB = decltype(rb)::value;
      if (q < A) {
        Cx<R>* e = ex + q * NL + l;
        const int es = A * NL;
        Cx<R> v[RB];
#pragma unroll
        for (int n2 = 0; n2 < RB; ++n2) v[n2] = e[n2 * es];
        rf::Dft<R, RB, -1>::run(v);
#pragma unroll
        for (int m2 = 0; m2 < RB; ++m2) e[m2 * es] = rf::mul(v[m2], gldx<R>(tw, (unsigned)(q * m2)));
      }
    });
    __syncthreads();
  }
  with_radix<RM>(A, [&](auto ra) HOM_INL {
    constexpr int RA = decltype(ra)::value;
    if (q < B) {
      const Cx<R>* e = ex + q * RA * NL + l;
      Cx<R> v[RA];
#pragma unroll
      for (int n1 = 0; n1 < RA; ++n1) v[n1] = e[n1 * NL];
      rf::Dft<R, RA, -1>::run(v);
      // X[q + B m1]
      if (ok)
        for_rows<RA>(
            B, q, N, M, H, [&](int m1, int row) HOM_INL { gstore(data + (size_t)row * rs, offq, v[m1]); },
            [&](int) HOM_INL {});
    }
  });
}

// ============================================================== lines along an axis
// Transforms of strided lines without pointwise work: the middle axis of 3D
// passes (zero-padded or truncated), the coefficient set-up, images and GaNi
// coefficients.  Element e of block x is line x nl + l; index i of the
// line is at (i * stride + line offset).  With contiguous lines (stride 1) the
// thread index runs along the line instead of across the lines, so that global
// accesses stay contiguous.
struct LineArgs {
  int A, B, M, nl;     // lines per block
  int N;               // stored length on the truncated side (N = M: plain transform)
  int lines;           // lines per outer index
  int rowwise;         // lines are contiguous (stride 1)
  size_t stride;       // between elements of a line
  size_t lstep;        // between lines
  size_t oin, oout;    // outer strides of input and output
};

// out: an array, or RealOut: only the real parts, in FP64 and (if there is one) an FP32 copy.
using hom::gstore;
struct RealOut {
  double* a64;
  float* a32;
};
__device__ __forceinline__ void gstore(const RealOut& o, size_t i, Cx<double> v) {
  gstore(o.a64, i, v.x);
  if (o.a32) o.a32[i] = (float)v.x;
}
template <typename R, int RM, typename O>
__device__ __forceinline__ void line_body(const LineArgs& a, const Cx<R>* in, O out, const Cx<R>* tw, int inverse,
                                          Cx<R>* ex) {
  const int A = a.A, B = a.B, M = a.M, N = a.N, H = (N - 1) / 2, nl = a.nl;
  const int T = A > B ? A : B;
  const int tid = threadIdx.x;
  const int l = a.rowwise ? tid / T : tid % nl, q = a.rowwise ? tid - l * T : tid / nl;
  const int line = blockIdx.x * nl + l;
  const bool ok = l < nl && line < a.lines;
  const bool full = N == M;
  // slot s of line l
  const int ss = a.rowwise ? 1 : nl, ls = a.rowwise ? M : 1;
  const size_t bi = (size_t)line * a.lstep;
  Cx<R>* e = ex + (size_t)(l < nl ? l : 0) * ls;
  if (inverse) {
    with_radix<RM>(A, [&](auto ra) HOM_INL {
      constexpr int RA = decltype(ra)::value;
      if (ok && q < B) {
        Cx<R> v[RA];
#pragma unroll
        for (int n1 = 0; n1 < RA; ++n1) {
          const int pos = B * n1 + q, i = full ? pos : keep(pos, N, M, H);
          v[n1] = i >= 0 ? gload(in, bi + (size_t)i * a.stride) : rf::mk<R>(0, 0);
        }
        rf::Dft<R, RA, 1>::run(v);
#pragma unroll
        for (int k1 = 0; k1 < RA; ++k1) e[(q * RA + k1) * ss] = rf::mul(v[k1], conj_if(gload(tw, (size_t)(q * k1)), true));
      }
    });
    __syncthreads();
    with_radix<RM>(B, [&](auto rb) HOM_INL {
      constexpr int RB = decltype(rb)::value;
      if (ok && q < A) {
        Cx<R> v[RB];
#pragma unroll
        for (int n2 = 0; n2 < RB; ++n2) v[n2] = e[(n2 * A + q) * ss];
        rf::Dft<R, RB, 1>::run(v);
#pragma unroll
        for (int k2 = 0; k2 < RB; ++k2) gstore(out, bi + (size_t)(q + A * k2) * a.stride, v[k2]);
      }
    });
  } else {
    with_radix<RM>(B, [&](auto rb) HOM_INL {
      constexpr int RB = decltype(rb)::value;
      if (ok && q < A) {
        Cx<R> v[RB];
#pragma unroll
        for (int n2 = 0; n2 < RB; ++n2) v[n2] = gload(in, bi + (size_t)(q + A * n2) * a.stride);
        rf::Dft<R, RB, -1>::run(v);
#pragma unroll
        for (int m2 = 0; m2 < RB; ++m2) e[(m2 * A + q) * ss] = rf::mul(v[m2], gload(tw, (size_t)(q * m2)));
      }
    });
    __syncthreads();
    with_radix<RM>(A, [&](auto ra) HOM_INL {
      constexpr int RA = decltype(ra)::value;
      if (ok && q < B) {
        Cx<R> v[RA];
#pragma unroll
        for (int n1 = 0; n1 < RA; ++n1) v[n1] = e[(q * RA + n1) * ss];
        rf::Dft<R, RA, -1>::run(v);
#pragma unroll
        for (int m1 = 0; m1 < RA; ++m1) {
          const int pos = q + B * m1, i = full ? pos : keep(pos, N, M, H);
          if (i >= 0) gstore(out, bi + (size_t)i * a.stride, v[m1]);
        }
      }
    });
  }
}

// Middle pass of the units (3D, axis 1): grid (element blocks, N0 rows, units).
template <typename R, int RM>
__global__ __launch_bounds__(kBlock) void k_mid_reg(Geo g, const UnitDev* __restrict__ units, LineArgs a, int flags) {
  extern __shared__ __align__(16) unsigned char smem[];
  const UnitDev& U = units[blockIdx.z];
  const int inverse = flags & 1;
  if (flags & MID_CG) {
    bool any = false;
    for (int l = 0; l < g.L; ++l) any |= (U.sc[l].status == 0);
    if (!any) return;
  }
  const Cx<R>* in = reinterpret_cast<const Cx<R>*>(inverse ? U.bufA : U.bufB) + blockIdx.y * a.oin;
  Cx<R>* out = reinterpret_cast<Cx<R>*>(inverse ? U.bufB : U.bufA) + blockIdx.y * a.oout;
  line_body<R, RM>(a, in, out, reinterpret_cast<const Cx<R>*>(g.tw[1]), inverse, reinterpret_cast<Cx<R>*>(smem));
}

// One array in place (images, GaNi coefficients): grid (line blocks, outer).
template <typename R, int RM>
__global__ __launch_bounds__(kBlock) void k_line_reg(Cx<R>* data, LineArgs a, const Cx<R>* __restrict__ tw, int inverse) {
  extern __shared__ __align__(16) unsigned char smem[];
  Cx<R>* d = data + blockIdx.y * a.oin;
  line_body<R, RM>(a, d, d, tw, inverse, reinterpret_cast<Cx<R>*>(smem));
}

// One axis of the coefficient set-up (series k = 0: A, 1: A^-1) of every cell of
// a table, or of one cell passed by value: grid (line blocks, outer, cells).
// The first axis reads the caller's Fourier data and writes the scratch, the
// last one writes the grid values; so a series takes one pass over memory per
// axis (with a copy before and a pass for the real parts after them 83 MB per
// 81^3 series, now 49), and a batch one launch per axis and series instead of
// seven per cell and series.  Measured from new coefficients to bounds: 32 cells
// on 81^3 38.0 -> 35.8 ms, 24 small 2D cells 5.5 -> 5.0 ms.
template <int RM>
__global__ __launch_bounds__(kBlock) void k_line_setup(const CoefJob* __restrict__ jobs, CoefJob one, LineArgs a,
                                                       const Cx<double>* __restrict__ tw, int k, int first, int last) {
  extern __shared__ __align__(16) unsigned char smem[];
  const CoefJob& J = jobs ? jobs[blockIdx.z] : one;
  Cx<double>* ex = reinterpret_cast<Cx<double>*>(smem);
  const Cx<double>* in = first ? (k ? J.B : J.A) : J.scratch;
  if (last)
    line_body<double, RM>(a, in, k ? RealOut{J.b64, J.b32} : RealOut{J.a64, J.a32}, tw, 1, ex);   // one outer index
  else
    line_body<double, RM>(a, in + blockIdx.y * a.oin, J.scratch + blockIdx.y * a.oin, tw, 1, ex);
}

// ============================================================== row passes
// As the specialised row passes (hom_fast.hip) with run-time lengths: rgG row
// pairs per block, in 2D one load per block (grid y), in 3D every load.  Lengths
// with a split always fit LDS (at most 729 * 11 FP64 values).
constexpr int kRowPairsMax = 16;

template <typename R, int RM, int D, int DUAL>
__global__ __launch_bounds__(kBlock) void k_first_reg(Geo g, const UnitDev* __restrict__ units, int mode, int jstep,
                                                      const int* __restrict__ iter_base) {
  constexpr int m = DUAL ? D - 1 : 1, LM = D == 2 ? 1 : kMaxLoads, PM = D == 2 ? 1 : kMaxPacks;
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double s_alpha[kMaxLoads];
  __shared__ int s_act[kMaxLoads];
  __shared__ double s_red[kBlock / 64];
  __shared__ RowInfo s_row[kRowPairsMax];
  const int M = g.M[2], A = g.rA[2], B = g.rB[2], N2 = g.N[2], N1 = g.N[1];
  const int G = g.rgG, L = D == 2 ? 1 : g.L, lo = D == 2 ? (int)blockIdx.y : 0;
  const int P = D == 2 ? 1 : g.P, po = D == 2 ? lo : 0;
  const size_t lstr = g.pmaj ? 1 : (size_t)g.P, pstr = g.pmaj ? (size_t)g.N[0] * N1 * M : 1;
  const UnitDev& U = units[blockIdx.z];
  const int tid = threadIdx.x;
  const int it = iter_base ? (*iter_base + jstep) : 0;
  Cx<R>* tw = reinterpret_cast<Cx<R>*>(smem);            // [M]
  Cx<R>* stage = tw + M;                                 // [2G][P][M], natural positions
  Cx<R>* out = reinterpret_cast<Cx<R>*>(U.bufA);

  // one wave per load: alpha_{it-1} from the <r, C r> partials of the last pass; block 0 records the step
  if (tid < LM * 64) {
    const int w = tid >> 6, lane = tid & 63;
    if (w < L) {
      int act = 1;
      double alpha = 0.0;
      if (mode == FIRST_CG) {
        CgScal* sc = U.sc + lo + w;
        double dl[1] = {0.0};
        wave_sum_rows<1>(U.part_d + (size_t)(lo + w) * g.nbL, 0, g.nbL, dl);
        act = (sc->status == 0);
        if (act && it > 0) {
          const double gam = sc->gamma[(it - 1) & 1];
          double den = dl[0];
          if (it > 1) den = dl[0] - sc->beta[(it - 1) & 1] * gam / sc->alpha[(it - 2) & 1];
          const bool rec = blockIdx.x == 0 && lane == 0;
          if (!(den > 0.0)) {
            act = 0;
            if (rec) {
              sc->status = -3;
              sc->iters = it - 1;
              sc->gamma_last = gam;
            }
          } else {
            alpha = gam / den;
            if (rec) {
              sc->alpha[(it - 1) & 1] = alpha;
              energy_record(sc, sc, it - 1, alpha * gam);
            }
          }
        }
      }
      if (lane == 0) {
        s_alpha[w] = alpha;
        s_act[w] = act;
      }
    }
  }
  if (tid < G) row_info(g, blockIdx.x * G + tid, s_row[tid]);
  const Cx<R>* twg = reinterpret_cast<const Cx<R>*>(g.tw[2]);
  for (int i = tid; i < M; i += kBlock) tw[i] = gload(twg, (size_t)i);
  for (int i = tid; i < 2 * G * P * M; i += kBlock) stage[i] = rf::mk<R>(0, 0);
  __syncthreads();
  if (mode == FIRST_CG) {
    int any = 0;
    for (int l = 0; l < L; ++l) any |= s_act[l];
    if (!any) return;
  }
  // element (line ln of pair gp, pack, position) of the row-pass buffer
  auto at = [&](const RowInfo& ri, int line, int pos, int pk) -> size_t {
    const int i0 = line ? ri.i0B : ri.h0, i1 = line ? ri.i1B : ri.i1A;
    return (((size_t)i0 * N1 + i1) * M + pos) * lstr + (po + pk) * pstr;
  };

  // ---- CG update of the stored entries; packed fields of the rows into the staging area
  double gp[LM];
#pragma unroll
  for (int l = 0; l < LM; ++l) gp[l] = 0.0;
  for (int t = tid; t < G * 2 * N2; t += kBlock) {
    const int gi = t / (2 * N2), rem = t - gi * 2 * N2;
    const int row = rem / N2, i2 = rem - row * N2;
    const RowInfo& ri = s_row[gi];
    if (!ri.valid || (row == 1 && !ri.rowB)) continue;
    const int h0 = ri.h0, i1 = row ? ri.i1B : ri.i1A;
    const double wt = h0 == 0 ? 1.0 : 2.0;
    Cx<double> rv[LM][m];
#pragma unroll
    for (int l = 0; l < LM; ++l) {
#pragma unroll
      for (int c = 0; c < m; ++c) {
        Cx<double> v = cx(0.0, 0.0);
        if (l < L) {
          const size_t idx = ((size_t)(c * g.H0 + h0) * N1 + i1) * N2 + i2;
          if (mode != FIRST_CG) {
            v = gload((const Cx<double>*)U.x[lo + l], idx);
          } else if (s_act[l]) {
            v = gload((const Cx<double>*)U.r[lo + l], idx);
            if (it > 0) {
              const double a = s_alpha[l];
              const Cx<double> xv = gload((const Cx<double>*)U.x[lo + l], idx), pv = gload((const Cx<double>*)U.p[lo + l], idx),
                               sv = gload((const Cx<double>*)U.s[lo + l], idx);
              v = v - sv * a;
              gstore(U.x[lo + l], idx, xv + pv * a);
              gstore(U.r[lo + l], idx, v);
            }
            gp[l] += wt * (v.x * v.x + v.y * v.y);
          }
        }
        rv[l][c] = v;
      }
    }
    if (row == 1) continue;
    const int k2 = fr(i2, N2);
    double Tb[3][2];
    basis_t<D, DUAL>(g, h0, ri.k1, k2, Tb);
    const int posA = padpos(i2, N2, M), posB = padpos(ixn(-k2, N2), N2, M);
#pragma unroll
    for (int pk = 0; pk < PM; ++pk) {
      if (pk >= P) continue;
      Cx<double> X[2];
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int f = 2 * pk + s, lf = f / D, gam = f - (f / D) * D;
        X[s] = cx(0.0, 0.0);
        if (lf < LM) {
          if (lf < L) {
#pragma unroll
            for (int c = 0; c < m; ++c) X[s] = X[s] + rv[lf < LM ? lf : 0][c] * Tb[gam][c];
            if (mode == FIRST_BOUNDS && ri.self && k2 == 0) X[s].x += U.E[lo + lf][gam];
          }
        }
      }
      const Cx<R> zA = rf::mk<R>((R)(X[0].x - X[1].y), (R)(X[0].y + X[1].x));
      const Cx<R> zB = rf::mk<R>((R)(X[0].x + X[1].y), (R)(-X[0].y + X[1].x));
      stage[((size_t)(2 * gi) * P + pk) * M + posA] = zA;
      if (!ri.self) stage[((size_t)(2 * gi + 1) * P + pk) * M + posB] = zB;
    }
  }
  if (mode == FIRST_CG) {
#pragma unroll
    for (int l = 0; l < LM; ++l) {
      if (l >= L) continue;
      const double s = block_sum(gp[l], s_red);
      if (tid == 0) gstore(U.part_g, (size_t)(lo + l) * g.nbF + blockIdx.x, s);
    }
  }
  __syncthreads();

  // ---- inverse four-step transform of every (line, pack)
  const int nlp = 2 * G * P;
  auto live = [&](int lp) -> bool {
    const int ln = lp / P;
    const RowInfo& ri = s_row[ln >> 1];
    return ri.valid && !((ln & 1) && ri.self);
  };
  with_radix<RM>(A, [&](auto ra) HOM_INL {
    constexpr int RA = decltype(ra)::value;
    for (int t = tid; t < nlp * B; t += kBlock) {
      const int lp = t / B, q = t - lp * B;
      if (!live(lp)) continue;
      Cx<R>* e = stage + (size_t)lp * M + q;
      Cx<R> v[RA];
#pragma unroll
      for (int n1 = 0; n1 < RA; ++n1) v[n1] = e[B * n1];
      rf::Dft<R, RA, 1>::run(v);
#pragma unroll
      for (int k1 = 0; k1 < RA; ++k1) e[B * k1] = rf::mul(v[k1], conj_if(tw[q * k1], true));
    }
  });
  __syncthreads();
  with_radix<RM>(B, [&](auto rb) HOM_INL {
    constexpr int RB = decltype(rb)::value;
    for (int t = tid; t < nlp * A; t += kBlock) {
      const int lp = t / A, q = t - lp * A;
      if (!live(lp)) continue;
      Cx<R>* e = stage + (size_t)lp * M + q * RB;
      Cx<R> v[RB];
#pragma unroll
      for (int n2 = 0; n2 < RB; ++n2) v[n2] = e[n2];
      rf::Dft<R, RB, 1>::run(v);
      if constexpr (D == 2) {
        const RowInfo& ri = s_row[lp >> 1];
        const size_t base = at(ri, lp & 1, q, 0);
#pragma unroll
        for (int k2 = 0; k2 < RB; ++k2) gstore(out, base + (size_t)(A * k2) * lstr, v[k2]);
      } else {
        // packs of a position are interleaved in HBM: results stay in this thread's slots and are
        // written below with all packs of a position back to back
#pragma unroll
        for (int k2 = 0; k2 < RB; ++k2) e[k2] = v[k2];
      }
    }
  });
  if constexpr (D == 3) {
    __syncthreads();
    for (int t = tid; t < 2 * G * M * P; t += kBlock) {
      const int pk = t % P, r = t / P, ln = r / M, pos = r - ln * M;
      const RowInfo& ri = s_row[ln >> 1];
      if (!ri.valid || ((ln & 1) && ri.self)) continue;
      const int k2 = pos / A, k1 = pos - k2 * A;
      gstore(out, at(ri, ln & 1, pos, pk), stage[((size_t)ln * P + pk) * M + k1 * B + k2]);
    }
  }
}

template <typename R, int RM, int D, int DUAL>
__global__ __launch_bounds__(kBlock) void k_last_reg(Geo g, const UnitDev* __restrict__ units, int mode, int jstep,
                                                     const int* __restrict__ iter_base) {
  constexpr int m = DUAL ? D - 1 : 1, LM = D == 2 ? 1 : kMaxLoads;
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double s_beta[kMaxLoads];
  __shared__ int s_act[kMaxLoads];
  __shared__ double s_red[kBlock / 64];
  __shared__ RowInfo s_row[kRowPairsMax];
  const int M = g.M[2], A = g.rA[2], B = g.rB[2], N2 = g.N[2], N1 = g.N[1];
  const int G = g.rgG, L = D == 2 ? 1 : g.L, lo = D == 2 ? (int)blockIdx.y : 0;
  const int P = D == 2 ? 1 : g.P, po = D == 2 ? lo : 0;
  const size_t lstr = g.pmaj ? 1 : (size_t)g.P, pstr = g.pmaj ? (size_t)g.N[0] * N1 * M : 1;
  const UnitDev& U = units[blockIdx.z];
  const int tid = threadIdx.x;
  const int it = iter_base ? (*iter_base + jstep) : 0;
  Cx<R>* tw = reinterpret_cast<Cx<R>*>(smem);            // [M]
  Cx<R>* stage = tw + M;                                 // [2G][P][M]
  const Cx<R>* in = reinterpret_cast<const Cx<R>*>(U.bufA);

  // one wave per load: gamma_it from the first-pass partials, stop test, beta_it; block 0 records them
  if (tid < LM * 64) {
    const int w = tid >> 6, lane = tid & 63;
    if (w < L) {
      int act = 1;
      double beta = 0.0;
      if (mode == LAST_CG) {
        CgScal* sc = U.sc + lo + w;
        double gs[1] = {0.0};
        wave_sum_rows<1>(U.part_g + (size_t)(lo + w) * g.nbF, 0, g.nbF, gs);
        act = (sc->status == 0);
        if (act) {
          const double gam = gs[0];
          const bool bad = !(gam == gam) || gam > 1e300;
          const bool rec = blockIdx.x == 0 && lane == 0;
          const bool conv = stop_test(sc, rec ? sc : nullptr, it, gam);
          if (bad || conv || it >= sc->maxit) {
            act = 0;
            if (rec) {
              sc->status = bad ? -1 : (conv ? 1 : 2);
              sc->iters = it;
              sc->gamma_last = gam;
              if (it == 0) sc->gamma0 = gam;
            }
          } else {
            beta = (it == 0) ? 0.0 : gam / sc->gamma[(it - 1) & 1];
            if (rec) {
              sc->gamma[it & 1] = gam;
              sc->beta[it & 1] = beta;
              if (it == 0) sc->gamma0 = gam;
            }
          }
        }
      }
      if (lane == 0) {
        s_beta[w] = beta;
        s_act[w] = act;
      }
    }
  }
  if (tid < G) row_info(g, blockIdx.x * G + tid, s_row[tid]);
  const Cx<R>* twg = reinterpret_cast<const Cx<R>*>(g.tw[2]);
  for (int i = tid; i < M; i += kBlock) tw[i] = gload(twg, (size_t)i);
  __syncthreads();
  {
    int any = 0;
    for (int l = 0; l < L; ++l) any |= s_act[l];
    if (!any) return;
  }
  auto at = [&](const RowInfo& ri, int line, int pos, int pk) -> size_t {
    const int i0 = line ? ri.i0B : ri.h0, i1 = line ? ri.i1B : ri.i1A;
    return (((size_t)i0 * N1 + i1) * M + pos) * lstr + (po + pk) * pstr;
  };

  // ---- forward four-step transform of every (line, pack), natural order in the staging area
  const int nlp = 2 * G * P;
  with_radix<RM>(B, [&](auto rb) HOM_INL {
    constexpr int RB = decltype(rb)::value;
    for (int t = tid; t < nlp * A; t += kBlock) {
      // 3D: packs fastest (they are interleaved in HBM); 2D has one pack per block
      int lp, q;
      if constexpr (D == 3) {
        const int pk = t % P, r = t / P, ln = r / A;
        q = r - ln * A;
        lp = ln * P + pk;
      } else {
        lp = t / A;
        q = t - lp * A;
      }
      const int ln = lp / P;
      const RowInfo& ri = s_row[ln >> 1];
      if (!ri.valid || ((ln & 1) && ri.self)) continue;
      const size_t base = at(ri, ln & 1, q, lp - ln * P);
      Cx<R> v[RB];
#pragma unroll
      for (int n2 = 0; n2 < RB; ++n2) v[n2] = gload(in, base + (size_t)(A * n2) * lstr);
      rf::Dft<R, RB, -1>::run(v);
      Cx<R>* e = stage + (size_t)lp * M + q * RB;
#pragma unroll
      for (int m2 = 0; m2 < RB; ++m2) e[m2] = rf::mul(v[m2], tw[q * m2]);
    }
  });
  __syncthreads();
  with_radix<RM>(A, [&](auto ra) HOM_INL {
    constexpr int RA = decltype(ra)::value;
    for (int t = tid; t < nlp * B; t += kBlock) {
      const int lp = t / B, q = t - lp * B, ln = lp / P;
      const RowInfo& ri = s_row[ln >> 1];
      if (!ri.valid || ((ln & 1) && ri.self)) continue;
      Cx<R>* e = stage + (size_t)lp * M + q;
      Cx<R> v[RA];
#pragma unroll
      for (int n1 = 0; n1 < RA; ++n1) v[n1] = e[B * n1];
      rf::Dft<R, RA, -1>::run(v);
      // X[q + B m1] takes the slots this thread read
#pragma unroll
      for (int m1 = 0; m1 < RA; ++m1) e[B * m1] = v[m1];
    }
  });
  __syncthreads();

  // ---- epilogue: unpack, project (T^T), CG direction update, <r, C r>
  double dp[LM];
#pragma unroll
  for (int l = 0; l < LM; ++l) dp[l] = 0.0;
  const double sc_m = g.invM * 0.5;
  for (int t = tid; t < G * 2 * N2; t += kBlock) {
    const int gi = t / (2 * N2), rem = t - gi * 2 * N2;
    const int row = rem / N2, i2 = rem - row * N2;
    const RowInfo& re = s_row[gi];
    if (!re.valid || (row == 1 && !re.rowB)) continue;
    const int k2 = fr(i2, N2);
    const int lineK = re.self ? 0 : row, lineM = re.self ? 0 : 1 - row;
    const int jK = padpos(i2, N2, M), jM = padpos(ixn(-k2, N2), N2, M);
    const int kk0 = row ? 0 : re.h0, kk1 = row ? -re.k1 : re.k1;
    const int ii1 = row ? re.i1B : re.i1A;
    const double wt = (re.h0 == 0) ? 1.0 : 2.0;
    double Tb[3][2];
    basis_t<D, DUAL>(g, kk0, kk1, k2, Tb);
    auto z_at = [&](int line, int pos, int pk) -> Cx<R> {
      return stage[((size_t)(2 * gi + line) * P + pk) * M + pos];
    };
#pragma unroll
    for (int l = 0; l < LM; ++l) {
      if (l >= L || (mode == LAST_CG && !s_act[l])) continue;
      Cx<double> rv[m], pv[m], sv[m], bv[m];
#pragma unroll
      for (int c = 0; c < m; ++c) {
        const size_t idx = ((size_t)(c * g.H0 + kk0) * N1 + ii1) * N2 + i2;
        if (mode == LAST_CG) {
          rv[c] = gload((const Cx<double>*)U.r[lo + l], idx);
          if (it > 0) {
            pv[c] = gload((const Cx<double>*)U.p[lo + l], idx);
            sv[c] = gload((const Cx<double>*)U.s[lo + l], idx);
          }
        } else if (mode == LAST_RESID) {
          bv[c] = gload((const Cx<double>*)U.b[lo + l], idx);
        }
      }
      Cx<double> wv[D];
#pragma unroll
      for (int gam = 0; gam < D; ++gam) {
        const int f = l * D + gam, pk = f >> 1;
        const Cx<R> za = z_at(lineK, jK, pk), zb = z_at(lineM, jM, pk);
        if ((f & 1) == 0)
          wv[gam] = cx(((double)za.x + (double)zb.x) * sc_m, ((double)za.y - (double)zb.y) * sc_m);
        else
          wv[gam] = cx(((double)za.y + (double)zb.y) * sc_m, -((double)za.x - (double)zb.x) * sc_m);
      }
#pragma unroll
      for (int c = 0; c < m; ++c) {
        Cx<double> w = cx(0.0, 0.0);
#pragma unroll
        for (int gam = 0; gam < D; ++gam) w = w + wv[gam] * Tb[gam][c];
        const size_t idx = ((size_t)(c * g.H0 + kk0) * N1 + ii1) * N2 + i2;
        double e;
        if (mode == LAST_CG) {
          const double b = s_beta[l];
          if (it == 0) {
            gstore(U.p[lo + l], idx, rv[c]);
            gstore(U.s[lo + l], idx, w);
          } else {
            gstore(U.p[lo + l], idx, rv[c] + pv[c] * b);
            gstore(U.s[lo + l], idx, w + sv[c] * b);
          }
          e = wt * (rv[c].x * w.x + rv[c].y * w.y);
        } else if (mode == LAST_RESID) {
          const Cx<double> rn = bv[c] - w;
          gstore(U.r[lo + l], idx, rn);
          e = wt * (rn.x * rn.x + rn.y * rn.y);
        } else {
          gstore(U.s[lo + l], idx, w);
          e = wt * (w.x * w.x + w.y * w.y);
        }
        dp[l] += e;
      }
    }
  }
#pragma unroll
  for (int l = 0; l < LM; ++l) {
    if (l >= L) continue;
    const double s = block_sum(dp[l], s_red);
    if (tid == 0) gstore(U.part_d, (size_t)(lo + l) * g.nbL + blockIdx.x, s);
  }
}

// ============================================================== launches
template <int NT = kBlock, typename K, typename... Args>
static hipError_t launch_line(K kern, dim3 grid, size_t lds, hipStream_t st, Args... args) {
  if (lds > kLdsMax) return hipErrorInvalidValue;
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  if (g_ext_timing.on)
    hipExtLaunchKernelGGL(kern, grid, dim3(NT), lds, st, g_ext_timing.start, g_ext_timing.stop, 0, args...);
  else
    hipLaunchKernelGGL(kern, grid, dim3(NT), lds, st, args...);
  return hipGetLastError();
}

// CALL(class) for the radix class of a split (A, B).
#define HOM_RCLASS(A, B, CALL)                          \
  do {                                                  \
    const int rm_ = (A) > (B) ? (A) : (B);              \
    if (rm_ <= 9) return CALL(9);                       \
    if (rm_ <= 16) return CALL(16);                     \
    return CALL(27);                                    \
  } while (0)

template <typename R, int RM, int KIND>
static hipError_t run_col(const Geo& g, const UnitDev* units, int n, int cg, hipStream_t st) {
  constexpr bool whole = KIND == COL_TENSOR || KIND == COL_QUAD;
  constexpr int NL = ColShape<R, RM>::NL, NT = ColShape<R, RM>::NT;
  const int npts = g.M[1] * g.M[2];
  const int nb = whole ? (npts + g.rgT - 1) / g.rgT
                       : (g.pmaj ? g.P * ((npts + NL - 1) / NL) : (npts * g.P + NL - 1) / NL);
  const dim3 grid(8 * ((nb + 7) / 8), 1, n);
  const size_t lds = (size_t)g.M[0] * NL * sizeof(Cx<R>);
  if constexpr (KIND == COL_COEF) {
    if (g.nc > 1) return launch_line<NT>(k_col_reg<R, RM, KIND, 3>, grid, lds, st, g, units, cg);
  }
  return launch_line<NT>(k_col_reg<R, RM, KIND, 1>, grid, lds, st, g, units, cg);
}

template <typename R, int KIND>
static hipError_t run_col_class(const Geo& g, const UnitDev* units, int n, int cg, hipStream_t st) {
#define HOM_C(RM) run_col<R, RM, KIND>(g, units, n, cg, st)
  HOM_RCLASS(g.rA[0], g.rB[0], HOM_C);
#undef HOM_C
}

template <typename R>
static size_t row_lds(const Geo& g) {
  return (size_t)g.M[2] * (1 + 2 * g.rgG * (g.d == 2 ? 1 : g.P)) * sizeof(Cx<R>);
}

template <typename R, int RM, int D, int DUAL>
static hipError_t run_row_reg(bool first, const Geo& g, const UnitDev* units, int n, int mode, int jstep, const int* ib,
                              hipStream_t st) {
  const dim3 grid((g.Q + g.rgG - 1) / g.rgG, D == 2 ? g.L : 1, n);
  if (first) return launch_line(k_first_reg<R, RM, D, DUAL>, grid, row_lds<R>(g), st, g, units, mode, jstep, ib);
  return launch_line(k_last_reg<R, RM, D, DUAL>, grid, row_lds<R>(g), st, g, units, mode, jstep, ib);
}

template <typename R, int D, int DUAL>
static hipError_t run_row_class(bool first, const Geo& g, const UnitDev* units, int n, int mode, int jstep, const int* ib,
                                hipStream_t st) {
#define HOM_C(RM) run_row_reg<R, RM, D, DUAL>(first, g, units, n, mode, jstep, ib, st)
  HOM_RCLASS(g.rA[2], g.rB[2], HOM_C);
#undef HOM_C
}

template <typename R>
bool reg_row(bool first, const Geo& g, const UnitDev* units, int n, int mode, int jstep, const int* ib, hipStream_t st,
             hipError_t* err) {
  if (!g.rA[2]) return false;
  if (g.d == 2)
    *err = g.dual ? run_row_class<R, 2, 1>(first, g, units, n, mode, jstep, ib, st)
                  : run_row_class<R, 2, 0>(first, g, units, n, mode, jstep, ib, st);
  else
    *err = g.dual ? run_row_class<R, 3, 1>(first, g, units, n, mode, jstep, ib, st)
                  : run_row_class<R, 3, 0>(first, g, units, n, mode, jstep, ib, st);
  return true;
}

template <typename R>
bool reg_mid(const Geo& g, const UnitDev* units, int n, int flags, hipStream_t st, hipError_t* err) {
  if (!g.rA[1]) return false;
  LineArgs a{};
  a.A = g.rA[1];
  a.B = g.rB[1];
  a.M = g.M[1];
  a.N = g.N[1];
  a.lines = g.M[2] * g.P;
  a.stride = (size_t)a.lines;
  a.lstep = 1;
  a.nl = g.rgM;
  const size_t big = (size_t)a.M * a.lines, small = (size_t)a.N * a.lines;
  a.oin = (flags & 1) ? small : big;
  a.oout = (flags & 1) ? big : small;
  const dim3 grid((a.lines + a.nl - 1) / a.nl, g.N[0], n);
  const size_t lds = (size_t)a.M * a.nl * sizeof(Cx<R>);
  auto go = [&]() -> hipError_t {
#define HOM_C(RM) launch_line(k_mid_reg<R, RM>, grid, lds, st, g, units, a, flags)
    HOM_RCLASS(a.A, a.B, HOM_C);
#undef HOM_C
  };
  *err = go();
  return true;
}

// Operator modes of launch_apply; the bound quadrature and the grid transfers run in FP64 only.
template <typename R>
bool reg_col(const Geo& g, const UnitDev* units, int n, int mode, hipStream_t st, hipError_t* err) {
  if (!g.rA[0]) return false;
  if (mode == APPLY_COEF || mode == APPLY_COEF_CG) {
    const int cg = mode == APPLY_COEF_CG ? 1 : 0;
    *err = (g.d == 3 && g.nc > 1) ? run_col_class<R, COL_TENSOR>(g, units, n, cg, st)
                                  : run_col_class<R, COL_COEF>(g, units, n, cg, st);
    return true;
  }
  if constexpr (sizeof(R) == 8) {
    if (mode == APPLY_QUAD) *err = run_col_class<R, COL_QUAD>(g, units, n, 0, st);
    else if (mode == APPLY_GRID) *err = run_col_class<R, COL_GRID>(g, units, n, 0, st);
    else *err = run_col_class<R, COL_FWD>(g, units, n, 0, st);
    return true;
  }
  return false;
}

// Lines of length Lm of an array [outer][Lm][inner]; false without a split or past the grid's limits.
template <typename R>
static bool array_lines(int outer, int Lm, int inner, LineArgs* a, dim3* grid, size_t* lds) {
  *a = LineArgs{};
  if (!reg_split(Lm, &a->A, &a->B)) return false;
  a->M = a->N = Lm;
  const int T = a->A > a->B ? a->A : a->B;
  if (inner == 1) {
    a->lines = outer;
    a->rowwise = 1;
    a->stride = 1;
    a->lstep = Lm;
    outer = 1;
  } else {
    a->lines = inner;
    a->stride = inner;
    a->lstep = 1;
    a->oin = a->oout = (size_t)Lm * inner;
  }
  if (outer > 65535) return false;
  a->nl = kBlock / T;
  while (a->nl > 1 && (size_t)Lm * a->nl * sizeof(Cx<R>) > 64 * 1024) --a->nl;
  if (a->nl > a->lines) a->nl = a->lines;
  *grid = dim3((a->lines + a->nl - 1) / a->nl, outer);
  *lds = (size_t)Lm * a->nl * sizeof(Cx<R>);
  return true;
}

template <typename R>
bool reg_line(Cx<R>* data, int outer, int Lm, int inner, const Cx<R>* tw, int inverse, hipStream_t st, hipError_t* err) {
  LineArgs a;
  dim3 grid;
  size_t lds;
  if (!array_lines<R>(outer, Lm, inner, &a, &grid, &lds)) return false;
  auto go = [&]() -> hipError_t {
#define HOM_C(RM) launch_line(k_line_reg<R, RM>, grid, lds, st, data, a, tw, inverse)
    HOM_RCLASS(a.A, a.B, HOM_C);
#undef HOM_C
  };
  *err = go();
  return true;
}

}  // namespace ln
}  // namespace hom
