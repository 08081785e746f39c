// Device bodies of the coarse correction of the two-level preconditioner
// (eq:two-level-preconditioners, def:algebraic-perfact-coarse-space), shared by
// the coarse kernels and by the launches that carry them as extra workgroups
// (the dense GEMM carries R_0 r, the clipped-class correction A_0^{-1} c; a
// batch's too).
#pragma once
#include "k_common.h"

namespace ddeig {

// c_sub = phi_class . R_sub r  (R_0 r of def:algebraic-perfact-coarse-space):
// one workgroup per subdomain.  Thread t takes the box elements t + kBlock q
// (natural order; the grid line from a multiply-high division), 8 at a time
// with all 16 loads issued before the products; the products are added in q
// order, then the threads in a fixed order.  sh: kBlock / 64 + 1 doubles of LDS.
__device__ __forceinline__ void coarse_rhs_body(const Geo& g, const PcgState* __restrict__ st,
                                                const double* __restrict__ r,
                                                const TypeDev* __restrict__ types,
                                                const SubDev* __restrict__ subs,
                                                double* __restrict__ crhs, int bid, double* sh) {
  if (st != nullptr && st->done) return;
  const SubDev sd = subs[bid];
  const TypeDev td = types[sd.type];
  const int m0 = td.m[0], m1 = td.m[1];
  const int m2 = td.m[2], mtot = m0 * m1 * m2;
  constexpr int U = 8;
  double acc = 0.0;
  for (int e0 = threadIdx.x; e0 < mtot; e0 += U * kBlock) {
    double ph[U], rv[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const int e = e0 + q * kBlock;
      ph[q] = rv[q] = 0.0;
      if (e < mtot) {
        const int line = (int)fdiv((unsigned)e, td.fm0);
        const int u0 = e - line * m0;
        const int u2 = m2 > 1 ? line / m1 : 0, u1 = line - u2 * m1;
        ph[q] = td.phi[e];
        rv[q] = r[(sd.o[0] + u0) + (long)g.N[0] * ((sd.o[1] + u1) + (long)g.N[1] * (sd.o[2] + u2))];
      }
    }
#pragma unroll
    for (int q = 0; q < U; ++q) acc += ph[q] * rv[q];
  }
  const double sum = block_sum_in<kBlock>(acc, sh);
  if (threadIdx.x == 0) crhs[bid] = sum;
}

// The coarse right-hand side (R_0 r)_i of one subdomain by one wave, in the
// order of coarse_rhs_body's workgroup of kBlock threads: lane l keeps the
// partial sums of that workgroup's threads l + 64 w (w < kBlock / 64), takes
// each through the same shuffle tree and adds the wave sums to 0 in w order,
// so the two give identical bits.  A batch has thousands of subdomains; a
// wave each needs no workgroup barrier.
__device__ __forceinline__ void coarse_rhs_wave(const Geo& g, const PcgState* __restrict__ st,
                                                const double* __restrict__ r,
                                                const TypeDev* __restrict__ types,
                                                const SubDev* __restrict__ subs,
                                                double* __restrict__ crhs, int sid) {
  constexpr int U = 8, NW = kBlock / 64;
  if (st != nullptr && st->done) return;
  const int lane = threadIdx.x & 63;
  const SubDev sd = subs[sid];
  const TypeDev td = types[sd.type];
  const int m0 = td.m[0], m1 = td.m[1];
  const int m2 = td.m[2], mtot = m0 * m1 * m2;
  double acc[NW];
#pragma unroll
  for (int w = 0; w < NW; ++w) acc[w] = 0.0;
  for (int base = 0; base < mtot; base += U * kBlock) {
    // every load of the pass first (the steps past the subdomain's end add
    // only zeros and are skipped), then the sums in the workgroup's order
    double ph[U][NW], rv[U][NW];
#pragma unroll
    for (int q = 0; q < U; ++q)
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const int e = base + q * kBlock + 64 * w + lane;
        ph[q][w] = rv[q][w] = 0.0;
        if (base + q * kBlock < mtot && e < mtot) {
          const int line = (int)fdiv((unsigned)e, td.fm0);
          const int u0 = e - line * m0;
          const int u2 = m2 > 1 ? line / m1 : 0, u1 = line - u2 * m1;
          ph[q][w] = td.phi[e];
          rv[q][w] = r[(sd.o[0] + u0) +
                       (long)g.N[0] * ((sd.o[1] + u1) + (long)g.N[1] * (sd.o[2] + u2))];
        }
      }
#pragma unroll
    for (int q = 0; q < U; ++q)
#pragma unroll
      for (int w = 0; w < NW; ++w) acc[w] += ph[q][w] * rv[q][w];
  }
  double t = 0.0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    double v = acc[w];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    t += v;
  }
  if (lane == 0) crhs[sid] = t;
}

// y0 = A0^{-1} c with the dense symmetric inverse: one wave64 per row, lanes
// stride the row (coalesced), fixed-order shuffle reduction.
__device__ __forceinline__ void coarse_solve_body(int N, const PcgState* __restrict__ st,
                                                  const double* __restrict__ A0inv,
                                                  const double* __restrict__ c,
                                                  double* __restrict__ y, int bid) {
  if (st != nullptr && st->done) return;
  const int lane = threadIdx.x & 63;
  const int row = bid * (kBlock / 64) + (threadIdx.x >> 6);
  if (row >= N) return;
  double acc = 0.0;
  for (int j = lane; j < N; j += 64) acc += A0inv[(long)row * N + j] * c[j];
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
  if (lane == 0) y[row] = acc;
}

}  // namespace ddeig
