// Restriction, extension and coarse space of the two-level additive Schwarz
// preconditioner (§2.2 eq:dd-preconditioners, eq:two-level-preconditioners,
// §2.3 def:algebraic-perfact-coarse-space, §3 eq:twoLevelASMPreconditioner).
//
// Subdomains are the L^p unit cells extended by delta element layers in every
// expanding direction (§3, §4.1): along an expanding axis, cell c (1-based)
// owns the node indices [(c-1) n_e - delta + 1, c n_e + delta - 1] clipped to
// [1, L n_e - 1]; fixed directions are not split.  With 2 delta <= n_e a node
// lies in at most two cells per axis.  The extension sums, for every node, the
// local solutions of the subdomains covering it in a fixed order (no atomics).
#include "k_common.h"
#include "k_coarse.h"

#include <type_traits>

namespace ddeig {

// 1-based cells covering node index gi (1-based) along one expanding axis.
__device__ inline void covering(int gi, int ne, int L, int delta, int& clo, int& chi) {
  // g <= c ne + delta - 1  <=>  c >= (g - delta + 1) / ne
  const int num = gi - delta + 1;
  clo = num <= 0 ? 1 : (num + ne - 1) / ne;
  chi = (gi + delta - 1) / ne + 1;
  if (clo < 1) clo = 1;
  if (chi > L) chi = L;
}

// The same with the multiply-high division by n_e (num + n_e < 2^31).
__device__ inline void covering(int gi, const Geo& g, int delta, int& clo, int& chi) {
  clo = max(1, (int)fdiv((unsigned)max(gi - delta + g.ne, 0), g.fne));
  chi = min(g.L, (int)fdiv((unsigned)(gi + delta - 1), g.fne) + 1);
}

// Distance from node coordinate (index gi, in units of h) to the faces of
// cell c's box along one axis that are not on the global boundary; INT_MAX if none.
__device__ inline int face_dist(int gi, int c, int ne, int L, int delta) {
  int dmin = 0x7fffffff;
  if (c > 1) {
    const int lo = (c - 1) * ne - delta;  // face at ((c-1) n_e - delta) h
    dmin = min(dmin, gi - lo);
  }
  if (c < L) {
    const int hi = c * ne + delta;
    dmin = min(dmin, hi - gi);
  }
  return dmin;
}

// Partition-of-unity weight of subdomain with cell index c at the node with
// 0-based unknown indices i.  pu = 0: 1 / #covering subdomains (§2.2);
// pu = 1: distance-based d_c / sum_c' d_c' (§4.1.2) with the distance to the
// interior faces of the box (the minimum over axes of perpendicular distances).
__device__ inline double pu_weight(const Geo& g, int delta, int pu, const int* c, const int* i) {
  if (pu == 0) {
    double w = 1.0;
    for (int a = 0; a < g.p; ++a) {
      int clo, chi;
      covering(i[a] + 1, g.ne, g.L, delta, clo, chi);
      w /= (double)(chi - clo + 1);
    }
    return w;
  }
  int lo[2] = {1, 1}, hi[2] = {1, 1};
  for (int a = 0; a < g.p; ++a) covering(i[a] + 1, g.ne, g.L, delta, lo[a], hi[a]);
  auto dist = [&](const int* cc) {
    int dm = 0x7fffffff;
    for (int a = 0; a < g.p; ++a) dm = min(dm, face_dist(i[a] + 1, cc[a], g.ne, g.L, delta));
    return dm;
  };
  const int dc = dist(c);
  if (dc == 0x7fffffff) return 1.0;  // a single subdomain: no interior faces
  double tot = 0.0;
  for (int c1 = lo[1]; c1 <= hi[1]; ++c1)
    for (int c0 = lo[0]; c0 <= hi[0]; ++c0) {
      const int cc[2] = {c0, c1};
      tot += (double)dist(cc);
    }
  return (double)dc / tot;
}

__device__ inline int sub_index(const Geo& g, const int* c) {
  return g.p == 1 ? c[0] - 1 : (c[0] - 1) + g.L * (c[1] - 1);
}

// Partition-of-unity weight of cell c at a node from the per-axis covering
// tables: the product of the per-axis factors, except for the distance-based
// weights with two expanding axes, which are not separable (pu_weight).
__device__ inline double cover_weight(const Geo& g, int delta, int pu, const XCover* const* xc,
                                      const int* c, const int* i, const int* which) {
  if (pu == 1 && g.p == 2) return pu_weight(g, delta, pu, c, i);
  double w = xc[0][i[0]].w[which[0]];
  if (g.p == 2) w *= xc[1][i[1]].w[which[1]];
  return w;
}

// ---- dense local solves: restriction and extension with arithmetic addressing
//
// With dense local solves the batch row of a subdomain is its id and every
// subdomain's box sits inside the unclipped box of its cell, so the batch
// index of a node follows from the node and cell indices alone: along an
// expanding axis the unclipped box of cell c starts at node (c - 1) n_e -
// delta, giving the box-local index i + delta - (c - 1) n_e.  The kernels
// below therefore issue all of a node's loads at once (no table look-ups in
// between); the covering cells come from covering() and the partition-of-unity
// weights from the same per-axis tables as in the generic kernels.
// Covering cells of a node: slot q = q0 + 2 q1 (q1 = 0 for one expanding
// axis) is cell (clo0 + q0, clo1 + q1) when that exists.  Out-of-range slots
// are clamped to an existing cell so that their loads stay valid and can be
// issued unconditionally; `val` masks their contributions.
template <int PX>
struct Cover {
  static constexpr int NC = PX == 1 ? 2 : 4;
  int clo0, chi0, clo1, chi1;
  __device__ Cover(const Geo& g, int delta, const int* i) {
    clo1 = chi1 = 1;
    covering(i[0] + 1, g, delta, clo0, chi0);
    if (PX == 2) covering(i[1] + 1, g, delta, clo1, chi1);
  }
  __device__ bool val(int q) const { return clo0 + (q & 1) <= chi0 && clo1 + (q >> 1) <= chi1; }
  __device__ int c0(int q) const { return min(clo0 + (q & 1), chi0); }
  __device__ int c1(int q) const { return min(clo1 + (q >> 1), chi1); }
};

// pu_weight of the covering cells of a node with two expanding axes (of slots that
// exist), every cell's distance formed once.  The extension takes each weight for
// the coarse term and, RAS, for the local solution; formed for each of the two and
// each cell anew, every time with all the distances for their sum, they made it
// keep one workgroup to a CU (71 registers) and cost 23 us: 225 subdomains of 18 x
// 18 x 15 in bf16, an application of two-level RAS 89.3 us, 65.1 so (63.5 with equal
// weights); additive 79.5 -> 66.1.
__device__ __forceinline__ void cover_weights(const Geo& g, int delta, int pu, const Cover<2>& cv,
                                              const int* i, double (&w)[4]) {
  if (pu == 0) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      w[q] = (cv.clo0 < cv.chi0 ? 0.5 : 1.0) * (cv.clo1 < cv.chi1 ? 0.5 : 1.0);
    return;
  }
  int d[4];
  double tot = 0.0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    d[q] = min(face_dist(i[0] + 1, cv.c0(q), g.ne, g.L, delta),
               face_dist(i[1] + 1, cv.c1(q), g.ne, g.L, delta));
    if (cv.val(q)) tot += (double)d[q];
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)  // (a single subdomain has no interior faces)
    w[q] = d[q] == 0x7fffffff ? 1.0 : (double)d[q] / tot;
}

// One item of the node-parallel dense kernels: 256 consecutive nodes of one grid
// line, a thread each.  The item is the same for the four waves that share it,
// so its part of every address is scalar and a lane adds a 32-bit byte offset.
// The kernels move 52 MB (restriction with the CG update) and 30 MB (extension)
// at 1,032,129 unknowns, 10.5 and 6 us at the card's copy rate; with divisions
// and 64-bit addresses per thread, eight waves a SIMD spent as long on issuing
// instructions as on memory, and the extension spilled at its 64 registers:
// 12.4 -> 11.9 us and 11.0 -> 9.3 us (32 instances of 16..256 subdomains,
// n_e = 32: 45.0 -> 43.4 and 33.6 -> 29.3 us).
struct LineItem {
  bool live;     // false: past the last item (the last one stands in for its loads)
  int s0, i1, i2;
  long line;
  __device__ LineItem(const Geo& g, unsigned it, unsigned items) {
    live = it < items;
    it = min(it, items - 1);
    line = fdiv(it, g.fseg);
    s0 = (int)(it - (unsigned)line * g.fseg.d) * kBlock;
    i2 = g.D == 3 ? (int)fdiv((unsigned)line, g.fN1) : 0;
    i1 = (int)line - i2 * g.N[1];
  }
};

// Batch positions of a lane's node: position(q) = base(q1) + lane(q0) for the
// covering cells q = q0 + 2 q1.  Along an axis the position moves by ld - n_e
// (axis 0) from a cell to the next; the first lane's first cell gives the base.
template <int PX>
struct DensePos {
  long base[PX];
  unsigned lane[2];
  int cw;
  __device__ DensePos(const Geo& g, int delta, const DenseArgs& da, const LineItem& t, int tl,
                      const Cover<PX>& cv) {
    cw = __builtin_amdgcn_readfirstlane(cv.clo0);
    const int step = da.ld - g.ne;
#pragma unroll
    for (int q1 = 0; q1 < PX; ++q1) {
      const int c1 = cv.c1(2 * q1);
      const int u1 = PX == 2 ? t.i1 + delta - (c1 - 1) * g.ne : t.i1;
      base[q1] = (long)(cw - 1) * step + t.s0 + delta + (PX == 2 ? (long)g.L * (c1 - 1) * da.ld : 0L) +
                 (long)da.hm0 * (u1 + (long)da.hm1 * t.i2);
    }
#pragma unroll
    for (int q0 = 0; q0 < 2; ++q0) lane[q0] = (unsigned)((cv.c0(q0) - cw) * step + tl);
  }
};

template <class T>
__device__ __forceinline__ T& at_bytes(T* p, unsigned off) {
  typedef std::conditional_t<std::is_const_v<T>, const char, char> byte_t;
  return *reinterpret_cast<T*>(reinterpret_cast<byte_t*>(p) + off);
}

// Scatter r into the subdomain batches (box natural order): node-parallel over
// row segments of kBlock x1 positions, four segments per workgroup of kBig
// threads; every node writes its copy into each covering subdomain (at most
// 2^p), so reads of r and writes of a batch row are both coalesced.  The
// covering cells come from the node index, the place in a subdomain's batch from
// one record per subdomain (SubBase): through a table per grid line, the
// subdomain's class and the class's fields in LDS it took 8.5 us, 7.1 us so, and
// the extension 17.0 and 11.0 us (256 subdomains, 1,032,129 unknowns).  With
// xr.on the node first takes the CG update of iteration k (x += alpha p,
// r -= alpha q, written back) and the kernel leaves the partials of ||r||^2
// in rr.
template <int PX>
__global__ void __launch_bounds__(kBig) k_restrict(Geo g, int delta, PcgState* __restrict__ st,
                                                   XrArgs xr, Red rr, double* __restrict__ r,
                                                   const SubBase* __restrict__ sb) {
  if (st != nullptr && st->done) return;
  double alpha = 0.0;
  if (xr.on == 1) {
    const double gamma = sum_partials<kBig>(xr.gam.part, xr.gam.np);
    if (!(gamma > 0.0)) {
      if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->done = 2;
        st->iters = xr.k - 1;
      }
      return;
    }
    alpha = st->rho[(xr.k - 1) & 1] / gamma;
  }
  const int N0 = g.N[0];
  const unsigned items = g.fseg.d * (unsigned)(g.N[1] * g.N[2]);
  const int sub = __builtin_amdgcn_readfirstlane(threadIdx.x / kBlock), tx = threadIdx.x % kBlock;
  double acc = 0.0;
  constexpr unsigned IPB = kBig / kBlock;
  for (unsigned grp = blockIdx.x; grp * IPB < items; grp += gridDim.x) {
    const LineItem t(g, grp * IPB + sub, items);
    const int tl = min(tx, N0 - 1 - t.s0);  // (lanes past the line: its last node)
    if (!t.live || tl < tx) continue;
    const long k0 = t.s0 + N0 * t.line;
    const unsigned o = 8u * tl;
    const int i[3] = {t.s0 + tl, t.i1, t.i2};
    const Cover<PX> cv(g, delta, i);
    const int cw = __builtin_amdgcn_readfirstlane(cv.clo0);
    SubBase b[Cover<PX>::NC];
#pragma unroll
    for (int q = 0; q < Cover<PX>::NC; ++q)
      b[q] = at_bytes(sb + (cw - 1 + (PX == 2 ? (long)g.L * (cv.c1(q) - 1) : 0L)),
                      (unsigned)sizeof(SubBase) * (cv.c0(q) - cw));
    double rv = at_bytes(r + k0, o);
    if (xr.on) {
      rv -= alpha * at_bytes(xr.q + k0, o);
      at_bytes(xr.x + k0, o) += alpha * at_bytes(xr.p + k0, o);
      at_bytes(r + k0, o) = rv;
      acc += rv * rv;
    }
#pragma unroll
    for (int q = 0; q < Cover<PX>::NC; ++q)
      if (cv.val(q)) b[q].p[b[q].at(i)] = rv;
  }
  if (xr.on) write_partial<kBig>(acc, rr.part);
}

// Bodies of the node-parallel kernels take the block index `bid` and the
// block count `nblk` of their problem (blockIdx.x / gridDim.x of a single
// problem, or the block's index and its instance's block count in a grouped
// launch).
template <int PX>
__device__ __forceinline__ void restrict_dense_body(const Geo& g, int delta,
                                                    PcgState* __restrict__ st, const XrArgs& xr,
                                                    const Red& rr, double* __restrict__ r,
                                                    const DenseArgs& da, int bid, int nblk) {
  if (st != nullptr && st->done) return;
  double alpha = 0.0;
  if (xr.on == 1) {
    const double gamma = sum_partials<kBig>(xr.gam.part, xr.gam.np);
    if (!(gamma > 0.0)) {
      if (bid == 0 && threadIdx.x == 0) {
        st->done = 2;
        st->iters = xr.k - 1;
      }
      return;
    }
    alpha = st->rho[(xr.k - 1) & 1] / gamma;
  }
  const int N0 = g.N[0];
  const unsigned items = g.fseg.d * (unsigned)(g.N[1] * g.N[2]);
  const int sub = __builtin_amdgcn_readfirstlane(threadIdx.x / kBlock), tx = threadIdx.x % kBlock;
  double acc = 0.0;
  // two nodes per thread and pass (items it and it + IPB), all their loads
  // issued before either is updated: the grid (node_grid_dense) fits on the
  // chip in one round
  constexpr unsigned IPB = kBig / kBlock;
  for (unsigned grp = bid; grp * 2 * IPB < items; grp += nblk) {
    const LineItem t[2] = {LineItem(g, grp * 2 * IPB + sub, items),
                           LineItem(g, grp * 2 * IPB + IPB + sub, items)};
    int tl[2];
    double rv[2], qv[2], pv[2], xv[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const long k0 = t[u].s0 + N0 * t[u].line;
      tl[u] = min(tx, N0 - 1 - t[u].s0);  // (lanes past the line: its last node)
      const unsigned o = 8u * tl[u];
      rv[u] = at_bytes((xr.on == 2 ? xr.q : r) + k0, o);
      if (xr.on == 1) {
        qv[u] = at_bytes(xr.q + k0, o);
        pv[u] = at_bytes(xr.p + k0, o);
        xv[u] = at_bytes(xr.x + k0, o);
      }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (!t[u].live || tl[u] < tx) continue;
      const long k0 = t[u].s0 + N0 * t[u].line;
      const unsigned o = 8u * tl[u];
      double rvv = rv[u];
      if (xr.on == 1) {
        rvv -= alpha * qv[u];
        at_bytes(xr.x + k0, o) = xv[u] + alpha * pv[u];
        at_bytes(r + k0, o) = rvv;
        acc += rvv * rvv;
      } else if (xr.on == 2) {
        at_bytes(xr.x + k0, o) = 0.0;
        at_bytes(r + k0, o) = rvv;
        acc += rvv * rvv;
      }
      const __bf16 hi = to_bf16(rvv);
      const __bf16 lo = to_bf16(rvv - (double)hi);
      const int i[3] = {t[u].s0 + tl[u], t[u].i1, t[u].i2};
      const Cover<PX> cv(g, delta, i);
      const DensePos<PX> pos(g, delta, da, t[u], tl[u], cv);
#pragma unroll
      for (int q = 0; q < Cover<PX>::NC; ++q) {
        if (!cv.val(q)) continue;
        at_bytes(da.Rh + pos.base[q >> 1], 2u * pos.lane[q & 1]) = hi;
        if (da.Rl != nullptr) at_bytes(da.Rl + pos.base[q >> 1], 2u * pos.lane[q & 1]) = lo;
      }
    }
  }
  if (xr.on) write_partial_at<kBig>(acc, rr.part, bid);
}

template <int PX>
__global__ void __launch_bounds__(kBig) k_restrict_dense(Geo g, int delta, PcgState* __restrict__ st,
                                                         XrArgs xr, Red rr, double* __restrict__ r,
                                                         DenseArgs da) {
  restrict_dense_body<PX>(g, delta, st, xr, rr, r, da, blockIdx.x, gridDim.x);
}

// z = sum_c R_c^T y_c + psi_ext cf (cf from k_coarse_field when coarse != 0).
// RAS weights every local solution by the partition of unity,
// z = sum_c R_c^T D_c y_c (+ the coarse term): the restricted additive Schwarz
// extension of eq:dd-preconditioners, from the same per-axis covering tables.
// INL forms the coarse field at the node from y0 itself (cf then points to
// y0): sum_c D_c y0_c over the covering cells in slot order, the arithmetic of
// k_coarse_field.
template <int PX, int KS, bool RAS = false, bool INL = false, int NPT = 1>
__device__ __forceinline__ void extend_dense_body(const Geo& g, int delta, int coarse,
                                                  PcgState* __restrict__ st, const CheckArgs& chk,
                                                  const DenseArgs& da,
                                                  const double* __restrict__ psi,
                                                  const double* __restrict__ cf,
                                                  const double* __restrict__ r,
                                                  double* __restrict__ z, int use_dot,
                                                  const Red& dot, int bid, int nblk, int pu = 0,
                                                  const XCover* __restrict__ xc0 = nullptr) {
  constexpr int NC = Cover<PX>::NC;
  if (st != nullptr && st->done) return;
  if (chk.on) {
    const double rn2 = sum_partials<kBig>(chk.rr.part, chk.rr.np);
    const bool conv = rn2 <= st->tol2, last = chk.k >= chk.maxit;
    if (bid == 0 && threadIdx.x == 0) {
      st->relres = sqrt(rn2 / st->r0n2);
      if (chk.hist && chk.k < chk.hist_cap) chk.hist[chk.k] = st->relres;
      st->iters = chk.k;
      if (conv) st->done = 1;
      else if (last) st->done = 4;
    }
    if (conv || last) return;
  }
  double acc = 0.0;
  const int N0 = g.N[0];
  const unsigned items = g.fseg.d * (unsigned)(g.N[1] * g.N[2]);
  const int sub = __builtin_amdgcn_readfirstlane(threadIdx.x / kBlock), tx = threadIdx.x % kBlock;
  // NPT nodes per thread and pass (items it + u IPB): every load of them
  // first, then their sums
  constexpr unsigned IPB = kBig / kBlock;
  for (unsigned grp = bid; grp * NPT * IPB < items; grp += nblk) {
    bool okn[NPT], two[NPT];
    unsigned on[NPT];
    double wan[NPT][2], yan[NPT][INL ? NC : 1], rkn[NPT], psn[NPT];
    float zsn[NPT][NC][KS];
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
      const LineItem t(g, grp * NPT * IPB + u * IPB + sub, items);
      const int tl = min(tx, N0 - 1 - t.s0);  // (lanes past the line: its last node)
      okn[u] = t.live && tl == tx;
      on[u] = 8u * tl;
      const int i[3] = {t.s0 + tl, t.i1, t.i2};
      const Cover<PX> cv(g, delta, i);
      const DensePos<PX> pos(g, delta, da, t, tl, cv);
      two[u] = cv.val(1);
      psn[u] = 0.0;
      // the weights of one expanding axis (equal ones need no table)
      if (PX == 1 && (RAS || (INL && coarse))) {
        wan[u][0] = wan[u][1] = two[u] ? 0.5 : 1.0;
        if (pu != 0) {
          const double* w = &xc0[t.s0].w[0];
          wan[u][0] = at_bytes(w, (unsigned)sizeof(XCover) * tl);
          wan[u][1] = at_bytes(w + 1, (unsigned)sizeof(XCover) * tl);
        }
      }
      if (coarse) {
        // cell-local table node: x dims (i + 1) mod n_e
        const int j0 = i[0] + 1 - g.ne * (int)fdiv((unsigned)(i[0] + 1), g.fne);
        const int j1 = PX == 2 ? t.i1 + 1 - g.ne * (int)fdiv((unsigned)(t.i1 + 1), g.fne) : t.i1;
        psn[u] = at_bytes(psi + (long)g.P[0] * (j1 + (long)g.P[1] * t.i2), 8u * j0);
        if constexpr (INL) {
#pragma unroll
          for (int q = 0; q < NC; ++q)
            yan[u][q] = at_bytes(cf + (pos.cw - 1 + (PX == 2 ? (long)g.L * (cv.c1(q) - 1) : 0L)),
                                 8u * (cv.c0(q) - pos.cw));
        } else {
          yan[u][0] = at_bytes(cf + (PX == 1 ? (long)t.s0 : t.s0 + (long)N0 * t.i1), on[u]);
        }
      }
#pragma unroll
      for (int q = 0; q < NC; ++q) {
        // (a line of one cell along axis 1: the same for the whole wave)
        if (PX == 2 && q >= 2 && cv.clo1 == cv.chi1) continue;
#pragma unroll
        for (int sp = 0; sp < KS; ++sp)
          zsn[u][q][sp] = at_bytes(da.Z + (sp * da.zsplit + pos.base[q >> 1]), 4u * pos.lane[q & 1]);
      }
      rkn[u] = at_bytes(r + (t.s0 + N0 * t.line), on[u]);
    }
#pragma unroll
    for (int u = 0; u < NPT; ++u) {
    if (!okn[u]) continue;
    const LineItem t(g, grp * NPT * IPB + u * IPB + sub, items);
    const int i[3] = {t.s0 + tx, t.i1, t.i2};
    // (one expanding axis: both cells exist, or the second stands in for none)
    const Cover<PX> cv(g, delta, i);
    auto val = [&](int q) { return PX == 1 ? q == 0 || two[u] : cv.val(q); };
    float (&zs)[NC][KS] = zsn[u];
    const double rk = rkn[u];
    double ps = psn[u], zc = 0.0, w[NC];
    if constexpr (PX == 2 && (RAS || INL)) cover_weights(g, delta, pu, cv, i, w);
    else if constexpr (RAS || INL) { w[0] = wan[u][0]; w[1] = wan[u][1]; }
    if (coarse) {
      if constexpr (INL && PX == 1) {
        zc = w[0] * yan[u][0];
        if (two[u]) zc = fma(w[1], yan[u][1], zc);
      } else if constexpr (INL) {
#pragma unroll
        for (int q = 0; q < NC; ++q)
          if (cv.val(q)) zc += w[q] * yan[u][q];
      } else {
        zc = yan[u][0];
      }
    }
    // ... then the sums, cells in slot order and splits in split order
    double zl = 0.0;
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      if (!val(q)) continue;
      float zq = 0.0f;
#pragma unroll
      for (int sp = 0; sp < KS; ++sp) zq += zs[q][sp];
      if constexpr (RAS) zl += w[q] * (double)zq;
      else zl += (double)zq;
    }
    // one rounding for the coarse term, whatever the compiler knows of `coarse`
    const double zv = coarse ? fma(ps, zc, zl) : zl;
    at_bytes(z + (t.s0 + N0 * t.line), on[u]) = zv;
    acc += rk * zv;
    }
  }
  if (use_dot) write_partial_at<kBig>(acc, dot.part, bid);
}

template <int PX, int KS, bool RAS, bool INL>
__global__ void __launch_bounds__(kBig) k_extend_dense(Geo g, int delta, int coarse,
                                                       PcgState* __restrict__ st, CheckArgs chk,
                                                       DenseArgs da, const double* __restrict__ psi,
                                                       const double* __restrict__ cf,
                                                       const double* __restrict__ r,
                                                       double* __restrict__ z, int use_dot, Red dot,
                                                       int pu, const XCover* __restrict__ xc0) {
  extend_dense_body<PX, KS, RAS, INL>(g, delta, coarse, st, chk, da, psi, cf, r, z, use_dot, dot,
                                      blockIdx.x, gridDim.x, pu, xc0);
}

// One expanding axis: two nodes per thread on node_grid_dense's grid, at most
// 64 VGPRs so that two 1024-thread workgroups fit on a CU (one round).
template <int KS, bool RAS, bool INL>
__global__ void __launch_bounds__(kBig) __attribute__((amdgpu_waves_per_eu(8)))
k_extend_dense_p1(Geo g, int delta, int coarse,
                                                       PcgState* __restrict__ st, CheckArgs chk,
                                                       DenseArgs da, const double* __restrict__ psi,
                                                       const double* __restrict__ cf,
                                                       const double* __restrict__ r,
                                                       double* __restrict__ z, int use_dot, Red dot,
                                                       int pu, const XCover* __restrict__ xc0) {
  extend_dense_body<1, KS, RAS, INL, 2>(g, delta, coarse, st, chk, da, psi, cf, r, z, use_dot, dot,
                                      blockIdx.x, gridDim.x, pu, xc0);
}

DenseArgs dense_args(const ddeig_problem* P) {
  const DenseHost& H = P->dh;
  return DenseArgs{H.Rh, H.Rl, H.Z, (long)H.mp * H.ld, H.ld, P->ksplit, H.box.m[0], H.box.m[1]};
}

// Workgroups of the node-parallel kernels: four row segments per workgroup,
// at most kMaxRed workgroups (partial-sum capacity).
int node_grid(const Geo& g) {
  const long segs = (g.N[0] + kBlock - 1) / kBlock;
  const long items = segs * g.N[1] * g.N[2];
  const long groups = (items + kBig / kBlock - 1) / (kBig / kBlock);
  return (int)std::max<long>(1, std::min<long>(groups, kMaxRed));
}

// The dense restriction and (one expanding axis, additive) extension take two
// items per thread and pass; a batch uses the same count per instance, so its
// partial sums match the single problem's bit for bit.
int node_grid_dense(const Geo& g) {
  const long segs = (g.N[0] + kBlock - 1) / kBlock;
  const long items = segs * g.N[1] * g.N[2];
  const long groups = (items + 2 * (kBig / kBlock) - 1) / (2 * (kBig / kBlock));
  return (int)std::max<long>(1, std::min<long>(groups, kMaxRed));
}

void launch_restrict(const ddeig_problem* P, double* r, PcgState* st, const XrArgs& xr, Red* rr,
                     hipStream_t s) {
  const int blocks = P->opt.local_prec >= 2 ? node_grid_dense(P->g) : node_grid(P->g);
  const Red none{nullptr, 0, nullptr};
  if (xr.on) rr->np = blocks;
  if (P->opt.local_prec >= 2) {
    if (P->g.p == 1)
      hipLaunchKernelGGL(k_restrict_dense<1>, dim3(blocks), dim3(kBig), 0, s, P->g, P->delta, st,
                         xr, xr.on ? *rr : none, r, dense_args(P));
    else
      hipLaunchKernelGGL(k_restrict_dense<2>, dim3(blocks), dim3(kBig), 0, s, P->g, P->delta, st,
                         xr, xr.on ? *rr : none, r, dense_args(P));
  } else {
    auto kern = P->g.p == 1 ? k_restrict<1> : k_restrict<2>;
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(kBig), 0, s, P->g, P->delta, st, xr,
                       xr.on ? *rr : none, r, P->dSubBase);
  }
}

__global__ void __launch_bounds__(kBlock) k_coarse_rhs(Geo g, const PcgState* __restrict__ st,
                                                       const double* __restrict__ r,
                                                       const TypeDev* __restrict__ types,
                                                       const SubDev* __restrict__ subs,
                                                       double* __restrict__ crhs) {
  __shared__ double sh[kBlock / 64 + 1];
  coarse_rhs_body(g, st, r, types, subs, crhs, blockIdx.x, sh);
}

void launch_coarse_rhs(const ddeig_problem* P, const double* r, const PcgState* st,
                       hipStream_t s) {
  hipLaunchKernelGGL(k_coarse_rhs, dim3(P->nsub), dim3(kBlock), 0, s, P->g, st, r, P->dTypes,
                     P->dSubs, P->crhs);
}

// phi of every class from its first member's box: D_c(k) psi_ext(k).
__global__ void k_coarse_phi(Geo g, int delta, int pu, const TypeDev* __restrict__ types,
                             const SubDev* __restrict__ subs, const int* __restrict__ first,
                             const XCover* __restrict__ xc0, const XCover* __restrict__ xc1,
                             const double* __restrict__ psi, double* const* __restrict__ phis) {
  const int t = blockIdx.y;
  const TypeDev td = types[t];
  const SubDev sd = subs[first[t]];
  const XCover* xc[2] = {xc0, xc1};
  const int m0 = td.m[0], m1 = td.m[1];
  const int mtot = m0 * m1 * td.m[2];
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < mtot; e += gridDim.x * blockDim.x) {
    const int line = e / m0, u0 = e - line * m0;
    const int u2 = line / m1, u1 = line - u2 * m1;
    const int i[3] = {sd.o[0] + u0, sd.o[1] + u1, sd.o[2] + u2};
    int which[2] = {0, 0};
    for (int a = 0; a < g.p; ++a) which[a] = xc[a][i[a]].c[0] == sd.c[a] ? 0 : 1;
    phis[t][e] = cover_weight(g, delta, pu, xc, sd.c, i, which) *
                 psi[table_node(g, i[0], i[1], i[2])];
  }
}

void launch_coarse_phi(const ddeig_problem* P, hipStream_t s) {
  const int nt = (int)P->types.size();
  hipLaunchKernelGGL(k_coarse_phi, dim3(64, nt), dim3(kBlock), 0, s, P->g, P->delta, P->opt.pu,
                     P->dTypes, P->dSubs, P->dFirst, P->dXC[0], P->dXC[1], P->psi, P->dPhis);
}

__global__ void k_coarse_solve(int N, const PcgState* __restrict__ st,
                               const double* __restrict__ A0inv, const double* __restrict__ c,
                               double* __restrict__ y) {
  coarse_solve_body(N, st, A0inv, c, y, blockIdx.x);
}

void launch_coarse_solve(const ddeig_problem* P, const PcgState* st, hipStream_t s) {
  const int rows_per_block = kBlock / 64;
  hipLaunchKernelGGL(k_coarse_solve, dim3((P->nsub + rows_per_block - 1) / rows_per_block),
                     dim3(kBlock), 0, s, P->nsub, st, P->A0inv, P->crhs, P->cy);
}

// The coarse correction R_0^T y0 at a node is psi_ext(node) times
// sum_c D_c(node) y0_c over the covering cells c, and both the covering cells
// and the weights depend only on the node's expanding indices.  This kernel
// forms that sum once per expanding-index point (i0, or (i0, i1) for two
// expanding axes), cells in slot order, so the extension reads one value.
template <int PX>
__device__ __forceinline__ void coarse_field_body(const Geo& g, int delta, int pu,
                                                  const PcgState* __restrict__ st,
                                                  const XCover* __restrict__ xc0,
                                                  const XCover* __restrict__ xc1,
                                                  const double* __restrict__ y0,
                                                  double* __restrict__ cf, int bid, int nblk) {
  if (st != nullptr && st->done) return;
  const XCover* xc[2] = {xc0, xc1};
  const long npts = PX == 1 ? (long)g.N[0] : (long)g.N[0] * g.N[1];
  for (long idx = bid * (long)blockDim.x + threadIdx.x; idx < npts;
       idx += (long)nblk * blockDim.x) {
    const int i[3] = {(int)(idx % g.N[0]), PX == 2 ? (int)(idx / g.N[0]) : 0, 0};
    const Cover<PX> cv(g, delta, i);
    double zc = 0.0;
#pragma unroll
    for (int q = 0; q < Cover<PX>::NC; ++q) {
      if (!cv.val(q)) continue;
      const int c[3] = {cv.c0(q), PX == 2 ? cv.c1(q) : 0, 0};
      const int which[2] = {q & 1, q >> 1};
      zc += cover_weight(g, delta, pu, xc, c, i, which) * y0[(c[0] - 1) + g.L * (cv.c1(q) - 1)];
    }
    cf[idx] = zc;
  }
}

template <int PX>
__global__ void k_coarse_field(Geo g, int delta, int pu, const PcgState* __restrict__ st,
                               const XCover* __restrict__ xc0, const XCover* __restrict__ xc1,
                               const double* __restrict__ y0, double* __restrict__ cf) {
  coarse_field_body<PX>(g, delta, pu, st, xc0, xc1, y0, cf, blockIdx.x, gridDim.x);
}

void launch_coarse_field(const ddeig_problem* P, const PcgState* st, hipStream_t s) {
  const long npts = P->g.p == 1 ? (long)P->g.N[0] : (long)P->g.N[0] * P->g.N[1];
  const int blocks = (int)std::min<long>((npts + kBlock - 1) / kBlock, 4096);
  if (P->g.p == 1)
    hipLaunchKernelGGL(k_coarse_field<1>, dim3(blocks), dim3(kBlock), 0, s, P->g, P->delta,
                       P->opt.pu, st, P->dXC[0], P->dXC[1], P->cy, P->cfield);
  else
    hipLaunchKernelGGL(k_coarse_field<2>, dim3(blocks), dim3(kBlock), 0, s, P->g, P->delta,
                       P->opt.pu, st, P->dXC[0], P->dXC[1], P->cy, P->cfield);
}

// z = sum_c R_c^T y_c (+ R_0^T y0), partials of r.z.  Work items are row
// segments of kBlock x1 positions, four per workgroup of kBig threads; the
// covering cells of a node and their values come as in the restriction (covering,
// SubBase), distance-based weights of one axis from its table, and the cells are
// summed in a fixed order.
// With chk.on the kernel first applies the stopping test of PCG iteration k,
// ||r_k|| <= rtol ||r_0|| (§4.1), records the history and, once CG stops,
// does nothing else (every later kernel of the iteration sees `done`).
template <int PX>
__global__ void __launch_bounds__(kBig) k_extend(Geo g, int delta, int pu, int coarse, int ras,
                                                 PcgState* __restrict__ st, CheckArgs chk,
                                                 const SubBase* __restrict__ sb,
                                                 const XCover* __restrict__ xc0,
                                                 const double* __restrict__ psi,
                                                 const double* __restrict__ y0,
                                                 const double* __restrict__ r,
                                                 double* __restrict__ z, int use_dot, Red dot) {
  constexpr int NC = Cover<PX>::NC;
  if (st != nullptr && st->done) return;
  if (chk.on) {
    const double rn2 = sum_partials<kBig>(chk.rr.part, chk.rr.np);
    const bool conv = rn2 <= st->tol2, last = chk.k >= chk.maxit;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      st->relres = sqrt(rn2 / st->r0n2);
      if (chk.hist && chk.k < chk.hist_cap) chk.hist[chk.k] = st->relres;
      st->iters = chk.k;
      if (conv) st->done = 1;
      else if (last) st->done = 4;
    }
    if (conv || last) return;
  }
  double acc = 0.0;
  const int N0 = g.N[0];
  const unsigned items = g.fseg.d * (unsigned)(g.N[1] * g.N[2]);
  const int sub = __builtin_amdgcn_readfirstlane(threadIdx.x / kBlock), tx = threadIdx.x % kBlock;
  constexpr unsigned IPB = kBig / kBlock;
  for (unsigned grp = blockIdx.x; grp * IPB < items; grp += gridDim.x) {
    const LineItem t(g, grp * IPB + sub, items);
    const int tl = min(tx, N0 - 1 - t.s0);  // (lanes past the line: its last node)
    if (!t.live || tl < tx) continue;
    const long k0 = t.s0 + N0 * t.line;
    const int i[3] = {t.s0 + tl, t.i1, t.i2};
    const Cover<PX> cv(g, delta, i);
    const int cw = __builtin_amdgcn_readfirstlane(cv.clo0);
    // the records and whatever does not hang on them, then the local solutions
    SubBase b[NC];
    double wc[NC], yc[NC], zi[NC], ps = 0.0;
    const bool weigh = coarse || ras;
    if constexpr (PX == 2) {
      cover_weights(g, delta, weigh ? pu : 0, cv, i, wc);
    } else {
      // (equal weights need no table)
      wc[0] = wc[1] = cv.clo0 < cv.chi0 ? 0.5 : 1.0;
      if (pu != 0 && weigh) {
        const double* w = &xc0[t.s0].w[0];
        wc[0] = at_bytes(w, (unsigned)sizeof(XCover) * tl);
        wc[1] = at_bytes(w + 1, (unsigned)sizeof(XCover) * tl);
      }
    }
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      const long sw = cw - 1 + (PX == 2 ? (long)g.L * (cv.c1(q) - 1) : 0L);
      const unsigned sl = (unsigned)(cv.c0(q) - cw);
      b[q] = at_bytes(sb + sw, (unsigned)sizeof(SubBase) * sl);
      yc[q] = coarse ? at_bytes(y0 + sw, 8u * sl) : 0.0;
    }
    const double rk = at_bytes(r + k0, 8u * tl);
    if (coarse) {
      // cell-local table node: x dims (i + 1) mod n_e
      const int j0 = i[0] + 1 - g.ne * (int)fdiv((unsigned)(i[0] + 1), g.fne);
      const int j1 = PX == 2 ? t.i1 + 1 - g.ne * (int)fdiv((unsigned)(t.i1 + 1), g.fne) : t.i1;
      ps = at_bytes(psi + (long)g.P[0] * (j1 + (long)g.P[1] * t.i2), 8u * j0);
    }
#pragma unroll
    for (int q = 0; q < NC; ++q) zi[q] = b[q].p[b[q].at(i)];
    double zl = 0.0, zc = 0.0;
#pragma unroll
    for (int q = 0; q < NC; ++q) {
      if (!cv.val(q)) continue;
      zl += ras ? wc[q] * zi[q] : zi[q];
      zc += wc[q] * yc[q];
    }
    double zv = zl;
    if (coarse) zv += ps * zc;
    at_bytes(z + k0, 8u * tl) = zv;
    acc += rk * zv;
  }
  if (use_dot) write_partial<kBig>(acc, dot.part);
}

template <bool RAS, bool INL>
static auto dense_extend_kernel(int p, int ks) {
  if (p == 1 && !RAS)  // (the RAS weights would spill at 64 VGPRs)
    return ks == 1 ? k_extend_dense_p1<1, RAS, INL>
                   : (ks == 2 ? k_extend_dense_p1<2, RAS, INL> : k_extend_dense_p1<3, RAS, INL>);
  if (p == 1)
    return ks == 1 ? k_extend_dense<1, 1, RAS, INL>
                   : (ks == 2 ? k_extend_dense<1, 2, RAS, INL> : k_extend_dense<1, 3, RAS, INL>);
  return ks == 1 ? k_extend_dense<2, 1, RAS, INL>
                 : (ks == 2 ? k_extend_dense<2, 2, RAS, INL> : k_extend_dense<2, 3, RAS, INL>);
}

// inline_field: the coarse field is formed in the extension from y0 (P->cy)
// instead of read from k_coarse_field's output (dense local solves only).
void launch_extend(const ddeig_problem* P, const double* r, double* z, int coarse, Red* dot,
                   PcgState* st, const CheckArgs& chk, hipStream_t s, int ras, int inline_field) {
  const int blocks = P->opt.local_prec >= 2 && P->g.p == 1 && !ras ? node_grid_dense(P->g)
                                                                   : node_grid(P->g);
  const Red none{nullptr, 0, nullptr};
  if (dot) dot->np = blocks;
  if (P->opt.local_prec >= 2) {
    // the K split is 1..3 by construction (assemble)
    const bool inl = coarse && inline_field;
    auto kern = ras ? (inl ? dense_extend_kernel<true, true>(P->g.p, P->ksplit)
                           : dense_extend_kernel<true, false>(P->g.p, P->ksplit))
                    : (inl ? dense_extend_kernel<false, true>(P->g.p, P->ksplit)
                           : dense_extend_kernel<false, false>(P->g.p, P->ksplit));
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(kBig), 0, s, P->g, P->delta, coarse, st, chk,
                       dense_args(P), P->psi, inl ? P->cy : P->cfield, r, z, dot ? 1 : 0,
                       dot ? *dot : none, P->opt.pu, P->dXC[0]);
    return;
  }
  auto kern = P->g.p == 1 ? k_extend<1> : k_extend<2>;
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(kBig), 0, s, P->g, P->delta, P->opt.pu, coarse, ras, st,
                     chk, P->dSubBase, P->dXC[0], P->psi, P->cy, r, z, dot ? 1 : 0,
                     dot ? *dot : none);
}

// The coarse correction alone, z = R_0^T y0 = psi_ext * cf at every node
// (cf from k_coarse_field), with the partials of r.z when use_dot: the
// correction step of eq:two-level-stationary-ras-mult-cc.
__global__ void __launch_bounds__(kBlock) k_coarse_extend(Geo g, const PcgState* __restrict__ st,
                                                          const double* __restrict__ psi,
                                                          const double* __restrict__ cf,
                                                          const double* __restrict__ r,
                                                          double* __restrict__ z, int use_dot,
                                                          Red dot) {
  if (st != nullptr && st->done) return;
  double acc = 0.0;
  for (long k = blockIdx.x * (long)kBlock + threadIdx.x; k < g.n; k += (long)gridDim.x * kBlock) {
    int i0, i1, i2;
    unflatten(g, k, i0, i1, i2);
    const double v = psi[table_node(g, i0, i1, i2)] * cf[g.p == 1 ? (long)i0 : i0 + (long)g.N[0] * i1];
    z[k] = v;
    acc += r[k] * v;
  }
  if (use_dot) write_partial(acc, dot.part);
}

void launch_coarse_extend(const ddeig_problem* P, const double* r, double* z, Red* dot,
                          const PcgState* st, hipStream_t s) {
  const int blocks = (int)std::max<long>(1, std::min<long>((P->g.n + kBlock - 1) / kBlock, kMaxRed));
  const Red none{nullptr, 0, nullptr};
  if (dot) dot->np = blocks;
  hipLaunchKernelGGL(k_coarse_extend, dim3(blocks), dim3(kBlock), 0, s, P->g, st, P->psi,
                     P->cfield, r, z, dot ? 1 : 0, dot ? *dot : none);
}

// A0[c][d] = phi_d^T A_sigma phi_c for neighbouring cells (one workgroup per
// pair), phi_c = D_c psi_ext on the box of c (the classes' phi, column c of
// R_0^T) and 0 elsewhere.  A node of box d takes the 3^D taps that reach box c.
// With the weight and psi_ext formed again at every tap: 288 us at 256 cells of
// 71 x 63 nodes and 1490 us at 256 of 18 x 18 x 15; 36 and 142 us so.
template <int D>
__global__ void __launch_bounds__(kBlock) k_coarse_matrix(Geo g, const double* __restrict__ T,
                                                          const TypeDev* __restrict__ types,
                                                          const SubDev* __restrict__ subs,
                                                          double* __restrict__ A0) {
  constexpr int NT = D == 2 ? 9 : 27;
  const int N = gridDim.x;
  const int cid = blockIdx.x;
  const int nb = blockIdx.y;  // neighbour offset in {-1,0,1}^p
  const SubDev sc = subs[cid];
  const int dc[2] = {nb % 3 - 1, nb / 3 - 1};
  const int cd[3] = {sc.c[0] + dc[0], g.p == 2 ? sc.c[1] + dc[1] : 0, 0};
  if (g.p == 1 && dc[1] != -1) return;  // only nb in {0,1,2} for p = 1
  for (int a = 0; a < g.p; ++a)
    if (cd[a] < 1 || cd[a] > g.L) return;
  const int did = sub_index(g, cd);
  const SubDev sdd = subs[did];
  const TypeDev& tc = types[sc.type];
  const TypeDev& tdd = types[sdd.type];
  const int m0 = tdd.m[0], m1 = tdd.m[1], mtot = m0 * m1 * tdd.m[2];
  const int c0 = tc.m[0], c1 = tc.m[1], c2 = tc.m[2];
  const double* __restrict__ phic = tc.phi;
  double acc = 0.0;
  for (int e = threadIdx.x; e < mtot; e += kBlock) {
    const int line = (int)fdiv((unsigned)e, tdd.fm0), u2 = D == 3 ? line / m1 : 0;
    const int i[3] = {sdd.o[0] + e - line * m0, sdd.o[1] + line - u2 * m1, sdd.o[2] + u2};
    // the node's place in box c, along each axis
    const int v0 = i[0] - sc.o[0], v1 = i[1] - sc.o[1], v2 = i[2] - sc.o[2];
    if (v0 < -1 || v0 > c0 || v1 < -1 || v1 > c1 || (D == 3 && (v2 < -1 || v2 > c2))) continue;
    const long tn = table_node(g, i[0], i[1], i[2]);
    double co[NT], ph[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int w0 = v0 + t % 3 - 1, w1 = v1 + t / 3 % 3 - 1, w2 = D == 3 ? v2 + t / 9 - 1 : 0;
      const bool in = w0 >= 0 && w0 < c0 && w1 >= 0 && w1 < c1 && (D == 2 || (w2 >= 0 && w2 < c2));
      co[t] = T[t * g.tsize + tn];
      ph[t] = in ? phic[w0 + c0 * (w1 + (D == 3 ? c1 * w2 : 0))] : 0.0;
    }
    double aphi = 0.0;
#pragma unroll
    for (int t = 0; t < NT; ++t) aphi += co[t] * ph[t];
    acc += tdd.phi[e] * aphi;
  }
  const double s = block_sum(acc);
  if (threadIdx.x == 0) A0[(long)cid * N + did] = s;
}

__global__ void k_symmetrise(double* A, int N) {
  const long nn = (long)N * N;
  for (long idx = blockIdx.x * (long)blockDim.x + threadIdx.x; idx < nn;
       idx += (long)gridDim.x * blockDim.x) {
    const int i = (int)(idx / N), j = (int)(idx % N);
    if (j > i) {
      const double v = 0.5 * (A[idx] + A[(long)j * N + i]);
      A[idx] = v;
      A[(long)j * N + i] = v;
    }
  }
}

void launch_symmetrise(double* A, int N, hipStream_t s) {
  const long nn = (long)N * N;
  const int blocks = (int)std::min<long>((nn + kBlock - 1) / kBlock, 4096);
  hipLaunchKernelGGL(k_symmetrise, dim3(blocks), dim3(kBlock), 0, s, A, N);
}

void build_coarse_matrix(ddeig_problem* P, double* A0, hipStream_t s) {
  const int N = P->nsub;
  check_hip(hipMemsetAsync(A0, 0, sizeof(double) * (size_t)N * N, s), "memset A0");
  const int nnb = P->g.p == 1 ? 3 : 9;
  // for p = 1 the neighbour offsets are encoded as nb = 0,1,2 with dc[1] = -1
  auto kern = P->g.D == 2 ? k_coarse_matrix<2> : k_coarse_matrix<3>;
  hipLaunchKernelGGL(kern, dim3(N, nnb), dim3(kBlock), 0, s, P->g, P->tabAs, P->dTypes, P->dSubs, A0);
  launch_symmetrise(A0, N, s);
}

// Grouped kernels of PCG iteration k over the instances of a batch (2-D,
// one expanding axis, dense local solves): block b runs block map[b].y of
// instance map[b].x with that instance's operands, CG state and partials.
__global__ void __launch_bounds__(kBig) k_b_restrict(const InstDev* __restrict__ I,
                                                     const int2* __restrict__ map, int k) {
  const int2 m = map[blockIdx.x];
  const InstDev& d = I[m.x];
  const XrArgs xr{1, k, d.gam, d.x, d.pp[k & 1], d.q};
  restrict_dense_body<1>(d.g, d.delta, d.st, xr, d.rr, d.r, d.da, m.y, d.nb_node);
}

// PCG from x_0 = 0 with b = w (the batch's inverse iteration): r_0 = w,
// x_0 = 0, the partials of ||r_0||^2 and the restriction of r_0, for the
// instances with act[j] != 0 (their CG state is set afterwards).
__global__ void __launch_bounds__(kBig) k_b_restrict_start(const InstDev* __restrict__ I,
                                                           const int2* __restrict__ map,
                                                           const int* __restrict__ act) {
  const int2 m = map[blockIdx.x];
  if (!act[m.x]) return;
  const InstDev& d = I[m.x];
  const XrArgs xr{2, 0, d.rr, d.x, nullptr, d.w};
  restrict_dense_body<1>(d.g, d.delta, nullptr, xr, d.rr, d.r, d.da, m.y, d.nb_node);
}

__global__ void k_b_pcg_init(const InstDev* __restrict__ I, const int* __restrict__ act,
                             double rtol) {
  const int j = blockIdx.x;
  if (!act[j]) return;
  pcg_init_body(I[j].st, rtol, I[j].rr, I[j].hist, 0.0);
}

// Inverse-iteration normalisation (as k_ipm_normalise) of every instance with
// act[j] != 0: x_new = sign(1^T M u) u / sqrt(u^T M u) into xo, and the
// partials of ||x_new - x||_M^2 = (x_new - x)^T (scale Mu - b) (Mu in z, b in w).
__global__ void __launch_bounds__(kBig) k_b_normalise(const InstDev* __restrict__ I,
                                                      const int2* __restrict__ map,
                                                      const int* __restrict__ act) {
  const int2 m = map[blockIdx.x];
  if (!act[m.x]) return;
  const InstDev& d = I[m.x];
  const double ssum = sum_partials<kBig>(d.nm_sum.part, d.nm_sum.np);
  const double uu = sum_partials<kBig>(d.nm_uMu.part, d.nm_uMu.np);
  const double sc = (ssum < 0.0 ? -1.0 : 1.0) / sqrt(uu);
  const long n = d.g.n;
  double acc = 0.0;
  for (long i = m.y * (long)kBig + threadIdx.x; i < n; i += (long)d.nb_node * kBig) {
    const double xn = sc * d.x[i];
    const double dd = xn - d.xo[i];
    acc += dd * (sc * d.z[i] - d.w[i]);
    d.xo[i] = xn;
  }
  write_partial_at<kBig>(acc, d.nm_dx.part, m.y);
}

// res[2 j] = ||x_new - x||_M^2, res[2 j + 1] = x_new^T A_sigma x_new (act[j] != 0).
__global__ void k_b_finish_norm(const InstDev* __restrict__ I, const int* __restrict__ act,
                                double* __restrict__ res) {
  const int j = blockIdx.x;
  if (!act[j]) return;
  const double dx = sum_partials(I[j].nm_dx.part, I[j].nm_dx.np);
  const double xq = sum_partials(I[j].nm_xq.part, I[j].nm_xq.np);
  if (threadIdx.x == 0) {
    res[2 * j] = dx;
    res[2 * j + 1] = xq;
  }
}

template <int KS>
// Two nodes per thread on node_grid_dense's grid, as the single problem's
// extension; check = 0 at the start of CG (z_0 and the partials of r_0.z_0 only).
__global__ void __launch_bounds__(kBig) __attribute__((amdgpu_waves_per_eu(8)))
k_b_extend(const InstDev* __restrict__ I, const int2* __restrict__ map, int k, int maxit,
           int check) {
  const int2 m = map[blockIdx.x];
  const InstDev& d = I[m.x];
  const CheckArgs chk{check, k, maxit, d.hist_cap, d.rr, d.hist};
  extend_dense_body<1, KS, false, true, 2>(d.g, d.delta, 1, d.st, chk, d.da, d.psi, d.cy, d.r, d.z,
                                           1, d.rz, m.y, d.nb_node, d.pu, d.xc0);
}

// Copies every instance's CG state into out[] (the host reads them with one
// copy); with mark_done the states are first set to finished (5), so that an
// instance whose solve is not started stays idle in the grouped kernels.
__global__ void k_b_states(const InstDev* __restrict__ I, int n, PcgState* __restrict__ out,
                           int mark_done) {
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < n; j += gridDim.x * blockDim.x) {
    PcgState* st = I[j].st;
    if (mark_done) st->done = 5;
    out[j] = *st;
  }
}

void launch_b_restrict(const InstDev* I, const BlockMap& bm, int k, hipStream_t s) {
  hipLaunchKernelGGL(k_b_restrict, dim3(bm.nblocks), dim3(kBig), 0, s, I, bm.map, k);
}

void launch_b_extend(const InstDev* I, const BlockMap& bm, int k, int maxit, int ksplit,
                     hipStream_t s, int check) {
  auto kern = ksplit == 1 ? k_b_extend<1> : (ksplit == 2 ? k_b_extend<2> : k_b_extend<3>);
  hipLaunchKernelGGL(kern, dim3(bm.nblocks), dim3(kBig), 0, s, I, bm.map, k, maxit, check);
}

void launch_b_restrict_start(const InstDev* I, const BlockMap& bm, const int* act, hipStream_t s) {
  hipLaunchKernelGGL(k_b_restrict_start, dim3(bm.nblocks), dim3(kBig), 0, s, I, bm.map, act);
}

void launch_b_pcg_init(const InstDev* I, int n, const int* act, double rtol, hipStream_t s) {
  hipLaunchKernelGGL(k_b_pcg_init, dim3(n), dim3(kBlock), 0, s, I, act, rtol);
}

void launch_b_normalise(const InstDev* I, const BlockMap& bm, const int* act, hipStream_t s) {
  hipLaunchKernelGGL(k_b_normalise, dim3(bm.nblocks), dim3(kBig), 0, s, I, bm.map, act);
}

void launch_b_finish_norm(const InstDev* I, int n, const int* act, double* res, hipStream_t s) {
  hipLaunchKernelGGL(k_b_finish_norm, dim3(n), dim3(kBlock), 0, s, I, act, res);
}

void launch_b_states(const InstDev* I, int n, PcgState* out, int mark_done, hipStream_t s) {
  hipLaunchKernelGGL(k_b_states, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, s, I, n, out,
                     mark_done);
}

}  // namespace ddeig
