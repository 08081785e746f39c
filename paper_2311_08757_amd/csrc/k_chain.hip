// Block-tridiagonal ("chain") factorisation and solves of box operators.
//
// The local matrices A_sigma,i = R_i A_sigma R_i^T of §3
// (eq:twoLevelASMPreconditioner) and the cell operator of
// eq:weak-form-cell-problem are the stencil operator restricted to a box of
// unknowns.  Ordered slice by slice along the last (fixed, Dirichlet) grid
// direction they are block tridiagonal: diagonal blocks D_i (couplings inside
// slice i, with the periodic wrap of the cell problem inside the slice) and
// sub-diagonal blocks E_i (slice i to slice i-1).  Block elimination gives
//   S_0 = D_0,  S_i = D_i - E_i S_{i-1}^{-1} E_i^T,  W_i = S_i^{-1},
// and a solve is
//   forward   t_i = W_i (b_i - E_i t_{i-1}),
//   backward  x_{n-1} = t_{n-1},  x_i = t_i - W_i E_{i+1}^T x_{i+1}.
// From both ends (FactorJobs) the slices after the middle one, h = n / 2, are
// eliminated upwards in the same way and slice h takes both neighbours; a solve runs
// inwards on either side, through h, and outwards again.
// E_i and D_i are never stored: they are read from the period-cell table.
// W_i is stored dense (b x b), where row solves read it in their order (RowsLayout);
// it is symmetric, so W_i[s][r] is read with r running over the threads, which
// coalesces.
#include "k_common.h"

#include <mutex>
#include <set>
#include <utility>

namespace ddeig {

// Allows a kernel `bytes` of dynamic LDS, the most that it is ever launched with.
// The limit belongs to the kernel on a device, not to a problem: set to each
// launch's own size, two problems on two threads could lower it under each other
// between the call and the launch.  So it is set once, before the first launch.
static void allow_lds(int device, const void* kern, size_t bytes) {
  static std::mutex mu;
  static std::set<std::pair<int, const void*>> done;
  std::lock_guard<std::mutex> lk(mu);
  if (done.count({device, kern})) return;
  check_hip(hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes),
            "dynamic LDS");
  done.insert({device, kern});
}

// In-slice neighbour of box-local u (slice coordinates a < D-1) along tap d.
__device__ inline bool slice_nbr(const Box& bx, int D, const int* u, const int* d, int& rn) {
  int idx = 0, stride = 1;
  for (int a = 0; a < D - 1; ++a) {
    int w = u[a] + d[a];
    if (bx.per[a]) w = (w + bx.m[a]) % bx.m[a];
    else if (w < 0 || w >= bx.m[a]) return false;
    idx += w * stride;
    stride *= bx.m[a];
  }
  rn = idx;
  return true;
}

__device__ inline void slice_coords(const Box& bx, int D, int r, int* u) {
  u[0] = 0; u[1] = 0; u[2] = 0;
  for (int a = 0; a < D - 1; ++a) {
    u[a] = r % bx.m[a];
    r /= bx.m[a];
  }
}

__device__ inline long box_tnode(const Geo& g, const Box& bx, const int* u) {
  return table_node(g, bx.o[0] + u[0], bx.o[1] + u[1], bx.o[2] + u[2]);
}

// ---- factorisation
//
// S_i = D_i - E_i W_{i-1} E_i^T and W_i = S_i^{-1} by Gauss-Jordan elimination
// without pivoting (the leading minors are positive; a non-positive pivot sets
// the flag).  Slices depend on each other, so the work is nch dependent
// inversions; everything below serves the length of that chain.
//  * 2-D slices of at most kFacMaxB unknowns (k_chain_factor2d): one workgroup
//    per class runs the whole chain, with the matrix in registers (16 x 16
//    threads, NA x NA entries each) and one barrier per kFacP pivots.  Four
//    waves, one per SIMD: the instructions around the update (broadcast reads,
//    reciprocals, selects) are per wave, and they, not the update, set the pace
//    (16 waves of fewer entries each took 1.2 us a pivot, one pivot per barrier
//    0.62, four 0.49 with the Schur complement: 2.2 ms for 63 slices of 71).
//    Chains whose row solves go from both ends (rows_both) are factored from
//    both, a workgroup each, the middle slices in a second launch: 2.19 -> 0.99
//    ms there.
//  * larger slices: the Schur complement by one workgroup per row
//    (k_schur_row), the inversion in pivot blocks of kGjNb (two launches per
//    block: the inverse of the diagonal block times its row panel, then the
//    rank-kGjNb update of the rest), for all classes at once.
// One launch per pivot took 2.9 us a pivot (6.1 us at b = 1085): 13.7 ms for
// a 63-slice chain of b = 71 and 217 ms for a 31-slice one of b = 1085.
constexpr int kFacMaxB = 128;
constexpr int kRowsMaxB = 128;
constexpr int kFacG = 16;  // thread grid: kFacG x kFacG = kBlock
static_assert(kFacG * kFacG == kBlock, "square thread grid");

// Matrices factored together; one chain from slice 0 (dir 0), or two: the upper
// half 0..h-1 (dir 0), the lower one nch-1..h+1 (dir 1), h = nch / 2, and the
// middle (step kFacMid of the dir 0 jobs).
constexpr int kFacMid = -1;
constexpr int kFacJobs = 2 * kMaxTypes;
struct FactorJobs {
  Box bx[kFacJobs];
  double* W[kFacJobs];
  int dir[kFacJobs];
  int both;
  // slice of job j in a step, or -1
  __host__ __device__ int slice(int j, int step) const {
    const int n = bx[j].nch, h = n / 2;
    if (!both) return step < n ? step : -1;
    if (step == kFacMid) return dir[j] ? -1 : h;
    const int i = dir[j] ? n - 1 - step : step;
    return (dir[j] ? i > h : i < h) ? i : -1;
  }
};

// Layout of the factors that the row solves read (chain_rows): the columns in 8
// parts of chunk = ceil(b / 8), 8 row pairs per wave: lane 8 part + q of a wave
// holds the pair (2 rp, 2 rp + 1), rp = 8 wave + q, of the columns s =
// part chunk + k; a load of a wave is 1 KB of consecutive memory: pair
// ((i nw + wave) chunk + k) 64 + lane of slice i.  Entries of no row or column
// stay zero.
struct RowsLayout {
  int nw, chunk;  // waves, columns per part
  __host__ __device__ explicit RowsLayout(int b) : nw((b + 15) / 16), chunk((b + 7) / 8) {}
  __host__ __device__ int slice() const { return nw * chunk * 64; }  // pairs per slice
  __host__ __device__ int at(int s, int r) const {                   // entry of column s, row r
    const int rp = r >> 1, part = s / chunk, k = s - part * chunk;
    return (((rp >> 3) * chunk + k) * 64 + part * 8 + (rp & 7)) * 2 + (r & 1);
  }
};

// 1 / x for a positive, normal x: the hardware estimate (2^-24) and three Newton
// steps with fused multiply-adds.  Two bring it within an ulp, and from there the
// third rounds correctly (P. Markstein, IBM J. Res. Dev. 34, 1990; an x of all ones
// alone can end an ulp off), as the division does that is a third longer in the
// pivot chain.
__device__ __forceinline__ double fast_rcp(double x) {
  double y = __builtin_amdgcn_rcp(x);
#pragma unroll
  for (int q = 0; q < 3; ++q) y = __builtin_fma(y, __builtin_fma(-x, y, 1.0), y);
  return y;
}

// Gauss-Jordan inversion of a b x b matrix spread over a workgroup, kFacP
// pivots at a time: thread (ti, tj) holds entries (ti + 16 x, tj + 16 y).
// rowb (kFacP x 16 NA) and colb (16 NA x kFacP), in two copies, hold the rows
// and columns of the pivot block before its step.  Rows and columns handed to
// LDS are zeroed in the registers; with X the inverse of the diagonal block
// (formed by every thread), rs = X r, rs_j = X_j for the block's columns and
// c_i = -(unit vector) for its rows, one update a -= c rs forms all of the new
// matrix.  Rows past b act as unit pivots.  Returns false (for the whole
// workgroup) at a non-positive pivot.
constexpr int kFacP = 4;
template <int NA>
__device__ __forceinline__ bool gj_registers(double (&a)[NA][NA], int b, int ti, int tj,
                                             double* __restrict__ rowb, double* __restrict__ colb) {
  constexpr int LD = kFacG * NA;
  // rows and columns 16 kb + kl .. + 3 of the current matrix into copy `c`
  auto publish = [&](int kb, int kl, int c) {
    double* rn = rowb + c * kFacP * LD;
    double* cn = colb + c * kFacP * LD;
    const unsigned pi = (unsigned)(ti - kl), pj = (unsigned)(tj - kl);
    if (pj < (unsigned)kFacP) {
#pragma unroll
      for (int x = 0; x < NA; ++x) cn[(ti + kFacG * x) * kFacP + pj] = a[x][kb];
    }
    if (pi < (unsigned)kFacP) {
#pragma unroll
      for (int y = 0; y < NA; ++y) rn[pi * LD + tj + kFacG * y] = a[kb][y];
    }
#pragma unroll
    for (int x = 0; x < NA; ++x) a[x][kb] = pj < (unsigned)kFacP ? 0.0 : a[x][kb];
#pragma unroll
    for (int y = 0; y < NA; ++y) a[kb][y] = pi < (unsigned)kFacP ? 0.0 : a[kb][y];
  };
  publish(0, 0, 0);
  __syncthreads();
#pragma unroll
  for (int kb = 0; kb < NA; ++kb) {
    for (int kl = 0; kl < kFacG; kl += kFacP) {
      const int k = kFacG * kb + kl, cp = (kl / kFacP) & 1;
      if (k >= b) return true;
      const double* rk = rowb + cp * kFacP * LD;
      const double* ck = colb + cp * kFacP * LD;
      double X[kFacP][kFacP], r[kFacP][NA], c[NA][kFacP];
#pragma unroll
      for (int p = 0; p < kFacP; ++p)
#pragma unroll
        for (int q = 0; q < kFacP; ++q) X[p][q] = rk[p * LD + k + q];
#pragma unroll
      for (int x = 0; x < NA; ++x)
#pragma unroll
        for (int p = 0; p < kFacP; ++p) {
          r[p][x] = rk[p * LD + tj + kFacG * x];
          c[x][p] = ck[(ti + kFacG * x) * kFacP + p];
        }
      bool ok = true;
#pragma unroll
      for (int p = 0; p < kFacP; ++p) {
        const double piv = k + p < b ? X[p][p] : 1.0;
        ok = ok && piv > 0.0;
        const double ip = fast_rcp(piv);
        X[p][p] = 1.0;
#pragma unroll
        for (int q = 0; q < kFacP; ++q) X[p][q] *= ip;
#pragma unroll
        for (int i = 0; i < kFacP; ++i) {
          if (i == p) continue;
          const double f = X[i][p];
          X[i][p] = 0.0;
#pragma unroll
          for (int q = 0; q < kFacP; ++q) X[i][q] -= f * X[p][q];
        }
      }
      if (!ok) return false;
      const int pi = ti - kl, pj = tj - kl;
#pragma unroll
      for (int y = 0; y < NA; ++y) {
        double t[kFacP];
#pragma unroll
        for (int p = 0; p < kFacP; ++p) {
          t[p] = X[p][0] * r[0][y];
#pragma unroll
          for (int q = 1; q < kFacP; ++q) t[p] += X[p][q] * r[q][y];
        }
#pragma unroll
        for (int p = 0; p < kFacP; ++p) r[p][y] = t[p];
      }
#pragma unroll
      for (int p = 0; p < kFacP; ++p)
#pragma unroll
        for (int q = 0; q < kFacP; ++q) {
          if (pj == q) r[p][kb] = X[p][q];
          if (pi == q) c[kb][p] = p == q ? -1.0 : 0.0;
        }
#pragma unroll
      for (int x = 0; x < NA; ++x)
#pragma unroll
        for (int y = 0; y < NA; ++y)
#pragma unroll
          for (int p = 0; p < kFacP; ++p) a[x][y] -= c[x][p] * r[p][y];
      if (kl + kFacP < kFacG) publish(kb, kl + kFacP, cp ^ 1);
      else if (kb + 1 < NA) publish(kb + 1 < NA ? kb + 1 : kb, 0, cp ^ 1);
      __syncthreads();
    }
  }
  return true;
}

// The chain of a 2-D class (along y, slices along x, couplings d0 = -1..1), or
// one half of it (FactorJobs), in one workgroup; the last inverse stays in LDS
// for the next slice, and the next slice's 6 b coefficients are loaded while the
// current one is inverted.  MID: the middle slices of the two-ended jobs, from
// the inverses on either side.
template <int NA, bool MID>
__global__ void __launch_bounds__(kBlock) k_chain_factor2d(Geo g, const double* __restrict__ T,
                                                           FactorJobs jobs, int rows,
                                                           int* __restrict__ flag) {
  constexpr int LD = kFacG * NA;
  constexpr int NT = MID ? 9 : 6;                        // taps per node
  constexpr int NC = (NT * LD + kBlock - 1) / kBlock;    // coefficients per thread
  extern __shared__ double wp[];  // b x b, two of them with MID
  // cf: the taps to the last slice of every node of the slice, its own (D_i),
  // and with MID those to the slice after
  __shared__ __align__(16) double row[2 * kFacP * LD], col[2 * kFacP * LD];
  __shared__ double cf[NC * kBlock];
  const int job = blockIdx.x, dir = jobs.dir[job];
  const Box bx = jobs.bx[job];
  double* __restrict__ W = jobs.W[job];
  const int b = bx.b, per = bx.per[0];
  const int ti = threadIdx.x / kFacG, tj = threadIdx.x % kFacG;
  const RowsLayout l(b);
  const long wslice = rows ? 2 * l.slice() : b * b;
  // neighbour u + d - 1 in the slice; one that does not exist points at the
  // node itself and has coefficient zero
  auto nbr = [&](int u, int d) {
    const int v = u + d - 1;
    return v < 0 ? (per ? b - 1 : u) : v >= b ? (per ? 0 : u) : v;
  };
  const int mid = MID ? jobs.slice(job, kFacMid) : 0;
  if (MID) {
    for (int q = threadIdx.x; q < 2 * b * b; q += kBlock) {
      const int i = q < b * b ? mid - 1 : mid + 1, rc = q < b * b ? q : q - b * b;
      wp[q] = i >= 0 && i < bx.nch ? W[i * wslice + (rows ? l.at(rc / b, rc % b) : rc)] : 0.0;
    }
  }
  const double* Tc[NC];
  bool cload[NC];
  double cnext[NC];
  int i = MID ? mid : jobs.slice(job, 0);
  if (i < 0) return;
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const int idx = threadIdx.x + q * kBlock, ct = idx / LD, cu = idx % LD, v = cu + ct % 3 - 1;
    const int tap = !MID && dir && ct < 3 ? ct + 6 : ct;
    cload[q] = ct < NT && cu < b && (per || (v >= 0 && v < b));
    Tc[q] = T + (cload[q] ? tap * g.tsize + (bx.o[0] + cu + 1 + g.ne) % g.ne : 0);
    cnext[q] = cload[q] ? Tc[q][(long)g.P[0] * (bx.o[1] + i)] : 0.0;
  }
  for (int step = 0; i >= 0; ++step) {
#pragma unroll
    for (int q = 0; q < NC; ++q) cf[threadIdx.x + q * kBlock] = cnext[q];
    __syncthreads();
    const int inext = MID ? -1 : jobs.slice(job, step + 1);
#pragma unroll
    for (int q = 0; q < NC; ++q)
      if (cload[q] && inext >= 0) cnext[q] = Tc[q][(long)g.P[0] * (bx.o[1] + inext)];
    // (opaque copies: the entries' addresses hoisted out of the slice loop would spill)
    int vi = ti, vj = tj;
    asm volatile("" : "+v"(vi), "+v"(vj));
    double a[NA][NA];
#pragma unroll
    for (int x = 0; x < NA; ++x)
#pragma unroll
      for (int y = 0; y < NA; ++y) {
        const int r = vi + kFacG * x, c = vj + kFacG * y;
        // (E W E^T)_rc of a neighbouring slice's inverse
        auto schur = [&](const double* wn, const double* e) {
          double corr = 0.0;
#pragma unroll
          for (int d1 = 0; d1 < 3; ++d1) {
            const double* wr = wn + nbr(r, d1) * b;
            double inner = 0.0;
#pragma unroll
            for (int d2 = 0; d2 < 3; ++d2) inner += e[d2 * LD + c] * wr[nbr(c, d2)];
            corr += e[d1 * LD + r] * inner;
          }
          return corr;
        };
        double v = 0.0;
        if (r < b && c < b) {
#pragma unroll
          for (int d = 0; d < 3; ++d)
            if (nbr(r, d) == c) v += cf[(3 + d) * LD + r];
          if (MID) v -= schur(wp, cf) + schur(wp + b * b, cf + 6 * LD);
          else if (step > 0) v -= schur(wp, cf);
        }
        a[x][y] = v;
      }
    if (!gj_registers<NA>(a, b, ti, tj, row, col)) {
      if (threadIdx.x == 0) atomicOr(flag, 1);
      return;
    }
    // (every read of the previous slice's wp and cf lies before the elimination's barriers)
    double* Wi = W + i * wslice;
#pragma unroll
    for (int x = 0; x < NA; ++x)
#pragma unroll
      for (int y = 0; y < NA; ++y) {
        const int r = ti + kFacG * x, c = tj + kFacG * y;
        if (r < b && c < b) {
          Wi[rows ? l.at(r, c) : r * b + c] = a[x][y];  // (symmetric)
          if (!MID) wp[r * b + c] = a[x][y];
        }
      }
    i = inext;
  }
}

// A single inversion of at most kFacMaxB unknowns in one workgroup.
template <int NA>
__global__ void __launch_bounds__(kBlock) k_gj_small(double* __restrict__ A, int b,
                                                    int* __restrict__ flag) {
  __shared__ __align__(16) double row[2 * kFacP * kFacG * NA], col[2 * kFacP * kFacG * NA];
  const int ti = threadIdx.x / kFacG, tj = threadIdx.x % kFacG;
  double a[NA][NA];
#pragma unroll
  for (int x = 0; x < NA; ++x)
#pragma unroll
    for (int y = 0; y < NA; ++y) {
      const int i = ti + kFacG * x, j = tj + kFacG * y;
      a[x][y] = i < b && j < b ? A[(long)i * b + j] : 0.0;
    }
  if (!gj_registers<NA>(a, b, ti, tj, row, col)) {
    if (threadIdx.x == 0) atomicOr(flag, 1);
    return;
  }
#pragma unroll
  for (int x = 0; x < NA; ++x)
#pragma unroll
    for (int y = 0; y < NA; ++y) {
      const int i = ti + kFacG * x, j = tj + kFacG * y;
      if (i < b && j < b) A[(long)i * b + j] = a[x][y];
    }
}

// S_i of every job, one workgroup per (row, job): row r of E_i W_{i-1} is
// formed once in LDS from 3^(D-1) coalesced rows of W_{i-1}, then every entry
// of the row takes its 3^(D-1) couplings from LDS (the product entry by entry
// would read W_{i-1} 9^(D-1) times: 420 us a slice at b = 1085).
constexpr int kSchurTaps = 9;
__global__ void __launch_bounds__(kBlock) k_schur_row(Geo g, FactorJobs jobs, int step,
                                                      const double* __restrict__ T) {
  extern __shared__ double u[];  // b
  const Box bx = jobs.bx[blockIdx.y];
  const int b = bx.b, D = g.D, last = D - 1, r = blockIdx.x;
  const int i = jobs.slice(blockIdx.y, step);
  if (r >= b || i < 0) return;
  const int ntap = D == 2 ? 3 : 9;  // taps of one slice offset, in tap order
  const long bb = (long)b * b;
  double* __restrict__ S = jobs.W[blockIdx.y] + (long)i * bb + (long)r * b;
  int ur[3];
  slice_coords(bx, D, r, ur);
  ur[last] = i;
  const long tr = box_tnode(g, bx, ur);
  auto offs = [&](int t, int* d) {
    d[0] = t % 3 - 1;
    d[1] = D == 3 ? t / 3 - 1 : 0;
    d[2] = 0;
  };
  for (int s = threadIdx.x; s < b; s += kBlock) {
    double v = 0.0;
    for (int t = 0; t < ntap; ++t) {
      int d[3], n;
      offs(t, d);
      if (slice_nbr(bx, D, ur, d, n) && n == s) v += T[(ntap + t) * g.tsize + tr];
    }
    S[s] = v;
  }
  // the eliminated neighbours: slice i - 1 of an upper chain, i + 1 of a lower
  // one, both of the middle
  const bool mid = step == kFacMid, low = jobs.dir[blockIdx.y] != 0;
  for (int side = 0; side < 2; ++side) {
    if (!mid && side != (low ? 1 : 0)) continue;
    const int j = side ? i + 1 : i - 1;
    if (j < 0 || j >= bx.nch) continue;
    const long tap0 = side ? 2 * ntap : 0;  // the taps towards slice j
    const double* Wp = jobs.W[blockIdx.y] + (long)j * bb;
    double e[kSchurTaps];
    long at[kSchurTaps];
#pragma unroll
    for (int t = 0; t < kSchurTaps; ++t) {
      e[t] = 0.0;
      at[t] = (long)r * b;
      int d[3], n1;
      offs(t, d);
      if (t < ntap && slice_nbr(bx, D, ur, d, n1)) {
        e[t] = T[(tap0 + t) * g.tsize + tr];
        at[t] = (long)n1 * b;
      }
    }
    __syncthreads();  // (u of the other side has been read)
    for (int s = threadIdx.x; s < b; s += kBlock) {
      double v = 0.0;
#pragma unroll
      for (int t = 0; t < kSchurTaps; ++t) v += e[t] * Wp[at[t] + s];
      u[s] = v;
    }
    __syncthreads();
    for (int s = threadIdx.x; s < b; s += kBlock) {
      int us[3];
      slice_coords(bx, D, s, us);
      us[last] = i;
      const long ts = box_tnode(g, bx, us);
      double corr = 0.0;
      for (int t = 0; t < ntap; ++t) {
        int d[3], n;
        offs(t, d);
        if (slice_nbr(bx, D, us, d, n)) corr += T[(tap0 + t) * g.tsize + ts] * u[n];
      }
      S[s] -= corr;
    }
  }
}

// Blocked Gauss-Jordan, pivot block [k0, k0 + nb) of every job (grid y).  The
// panel kernel inverts the diagonal block (every workgroup for itself, in
// registers) and writes, for its kGjTile rows and columns, the row panel
// R = D^{-1} A_kj (with R_kk = D^{-1}) and a copy of the column panel C = A_ik;
// the update kernel then applies A_ij -= C_i R_j, A_ik = -C_i D^{-1},
// A_kj = R_j.  Buffers per job: R (kGjNb x b), then C (b x kGjNb).
constexpr int kGjNb = 32, kGjTile = 64;

__global__ void __launch_bounds__(kBlock) k_gj_panel(FactorJobs jobs, int step, int k0,
                                                     double* __restrict__ buf, long bstride,
                                                     int* __restrict__ flag) {
  constexpr int NA = kGjNb / kFacG;
  __shared__ __align__(16) double row[2 * kFacP * kGjNb], col[2 * kFacP * kGjNb];
  __shared__ double D[kGjNb][kGjNb + 1], P[kGjNb][kGjTile + 1];
  const Box bx = jobs.bx[blockIdx.y];
  const int b = bx.b;
  const int c0 = blockIdx.x * kGjTile;
  const int i = jobs.slice(blockIdx.y, step);
  if (k0 >= b || c0 >= b || i < 0) return;
  const int nb = min(kGjNb, b - k0);
  const double* __restrict__ A = jobs.W[blockIdx.y] + (long)i * b * b;
  double* __restrict__ R = buf + blockIdx.y * bstride;
  double* __restrict__ C = R + (long)kGjNb * b;
  const int ti = threadIdx.x / kFacG, tj = threadIdx.x % kFacG;
  double a[NA][NA];
#pragma unroll
  for (int x = 0; x < NA; ++x)
#pragma unroll
    for (int y = 0; y < NA; ++y) {
      const int r = ti + kFacG * x, c = tj + kFacG * y;
      a[x][y] = r < nb && c < nb ? A[(long)(k0 + r) * b + k0 + c] : 0.0;
    }
  // this workgroup's columns of the row panel, and rows of the column panel
#pragma unroll
  for (int q = threadIdx.x; q < kGjNb * kGjTile; q += kBlock) {
    const int k = q / kGjTile, j = q % kGjTile;
    P[k][j] = k < nb && c0 + j < b ? A[(long)(k0 + k) * b + c0 + j] : 0.0;
    const int kk = q % kGjNb, r = c0 + q / kGjNb;
    if (r < b) C[(long)r * kGjNb + kk] = kk < nb ? A[(long)r * b + k0 + kk] : 0.0;
  }
  if (!gj_registers<NA>(a, nb, ti, tj, row, col)) {
    if (threadIdx.x == 0) atomicOr(flag, 1);
    return;
  }
#pragma unroll
  for (int x = 0; x < NA; ++x)
#pragma unroll
    for (int y = 0; y < NA; ++y) {
      const int r = ti + kFacG * x, c = tj + kFacG * y;
      D[r][c] = r < nb && c < nb ? a[x][y] : 0.0;
    }
  __syncthreads();
#pragma unroll
  for (int q = threadIdx.x; q < kGjNb * kGjTile; q += kBlock) {
    const int r = q / kGjTile, jl = q % kGjTile, j = c0 + jl;
    double v = 0.0;
    if (j >= k0 && j < k0 + nb) {
      v = D[r][j - k0];
    } else {
#pragma unroll 8
      for (int k = 0; k < kGjNb; ++k) v += D[r][k] * P[k][jl];
    }
    if (j < b) R[(long)r * b + j] = v;
  }
}

__global__ void __launch_bounds__(kBlock) k_gj_update(FactorJobs jobs, int step, int k0,
                                                      const double* __restrict__ buf, long bstride) {
  __shared__ double Cs[kGjNb][kGjTile + 2], Rs[kGjNb][kGjTile + 2];
  const Box bx = jobs.bx[blockIdx.z];
  const int b = bx.b;
  const int i0 = blockIdx.y * kGjTile, j0 = blockIdx.x * kGjTile;
  const int i = jobs.slice(blockIdx.z, step);
  if (k0 >= b || i0 >= b || j0 >= b || i < 0) return;
  const int nb = min(kGjNb, b - k0);
  double* __restrict__ A = jobs.W[blockIdx.z] + (long)i * b * b;
  const double* __restrict__ R = buf + blockIdx.z * bstride;
  const double* __restrict__ C = R + (long)kGjNb * b;
  for (int q = threadIdx.x; q < kGjNb * kGjTile; q += kBlock) {
    const int k = q / kGjTile, j = q % kGjTile;
    Rs[k][j] = j0 + j < b ? R[(long)k * b + j0 + j] : 0.0;
    const int kk = q % kGjNb, r = q / kGjNb;
    Cs[kk][r] = i0 + r < b ? C[(long)(i0 + r) * kGjNb + kk] : 0.0;
  }
  // thread: rows 4 ty .. + 3, columns tx + 16 y
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
  double acc[4][4];
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      const int r = i0 + 4 * ty + x, j = j0 + tx + 16 * y;
      const bool kj = j >= k0 && j < k0 + nb;
      acc[x][y] = r < b && j < b && !kj ? A[(long)r * b + j] : 0.0;
    }
  __syncthreads();
#pragma unroll 8
  for (int k = 0; k < kGjNb; ++k) {
    double c[4], r[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      c[x] = Cs[k][4 * ty + x];
      r[x] = Rs[k][tx + 16 * x];
    }
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int y = 0; y < 4; ++y) acc[x][y] -= c[x] * r[y];
  }
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      const int r = i0 + 4 * ty + x, j = j0 + tx + 16 * y;
      if (r >= b || j >= b) continue;
      const bool ki = r >= k0 && r < k0 + nb;
      A[(long)r * b + j] = ki ? Rs[r - k0][tx + 16 * y] : acc[x][y];
    }
}

// Inverts every job's slice of a step in pivot blocks.
static void gj_blocked(ddeig_problem* P, const FactorJobs& jobs, int njobs, int bmax, int step,
                       hipStream_t s) {
  const long stride = 2L * kGjNb * P->gj_stride;
  const int nt = (bmax + kGjTile - 1) / kGjTile;
  for (int k0 = 0; k0 < bmax; k0 += kGjNb) {
    hipLaunchKernelGGL(k_gj_panel, dim3(nt, njobs), dim3(kBlock), 0, s, jobs, step, k0, P->gjbuf,
                       stride, P->flag);
    hipLaunchKernelGGL(k_gj_update, dim3(nt, nt, njobs), dim3(kBlock), 0, s, jobs, step, k0,
                       P->gjbuf, stride);
  }
}

long gj_buffer_doubles(int bmax, int njobs) { return 2L * kGjNb * bmax * njobs; }

void launch_gj_invert(ddeig_problem* P, double* A, int b, hipStream_t s) {
  if (b <= kFacMaxB) {
    auto kern = b <= 32 ? k_gj_small<2> : b <= 64 ? k_gj_small<4> : b <= 80 ? k_gj_small<5> : k_gj_small<8>;
    hipLaunchKernelGGL(kern, dim3(1), dim3(kBlock), 0, s, A, b, P->flag);
    return;
  }
  FactorJobs jobs{};
  jobs.bx[0].b = b;
  jobs.bx[0].nch = 1;
  jobs.W[0] = A;
  gj_blocked(P, jobs, 1, b, 0, s);
}

// Row solves (chain_rows) of slices of b, nch of them: the LDS copy of the
// right-hand side has to fit, and one wave holds a slice.
constexpr size_t kRowsLds = 128 * 1024;
constexpr size_t kRowsLdsMax = kRowsLds + kRowsMaxB * sizeof(double);  // (a line more for an even count)
static size_t rows_lds(int b, int nch) {
  return ((size_t)b * (nch | 1) + 2 * 64 + 2) * sizeof(double);
}
static bool rows_ok(int b, int nch) {
  return b <= kRowsMaxB && ((size_t)b * nch + 2 * 64 + 2) * sizeof(double) <= kRowsLds;
}

// Whether the row solves of a box and their FP64 factor eliminate from both
// ends: half the dependent steps, twice the waves, of which a CU holds those of
// 80 rows.
constexpr int kRowsBothB = 80;  // (k_chain_factor2d<5, true> at most)
bool rows_both(int D, int b, int nch) { return D == 2 && rows_ok(b, nch) && b <= kRowsBothB; }

// Entries of a 2-D or 3-D box's factor, in either layout; bmax, nchmax: over the
// problem's classes (one kernel serves them all).
size_t factor_entries(int D, const Box& bx, int bmax, int nchmax) {
  if (D == 2 && rows_ok(bmax, nchmax)) return (size_t)bx.nch * 2 * RowsLayout(bx.b).slice();
  return (size_t)bx.nch * bx.b * bx.b;
}

// The chains of all boxes (their W pointers alongside); as many at once as the
// pivot buffers hold.
void chain_factor(ddeig_problem* P, const std::vector<Box>& boxes, const std::vector<double*>& Ws,
                  const double* tab, hipStream_t s, bool both_ends) {
  int bmax = 0, nch = 0;
  for (const Box& bx : boxes) {
    bmax = std::max(bmax, bx.b);
    nch = std::max(nch, bx.nch);
  }
  const bool small = P->g.D == 2 && bmax <= kFacMaxB;
  const int rows = P->g.D == 2 && rows_ok(bmax, nch);
  const int nd = both_ends ? 2 : 1;
  const size_t at_once = small ? (size_t)(kFacJobs / nd) : std::max<size_t>(1, std::min(kFacJobs, P->gj_jobs) / nd);
  if (rows)  // (its entries of no row or column stay zero)
    for (size_t j = 0; j < boxes.size(); ++j)
      check_hip(hipMemsetAsync(Ws[j], 0, factor_entries(2, boxes[j], bmax, nch) * sizeof(double), s),
                "clear factor");
  for (size_t j0 = 0; j0 < boxes.size(); j0 += at_once) {
    const int nb = (int)std::min(at_once, boxes.size() - j0), nj = nb * nd;
    FactorJobs jobs{};
    jobs.both = both_ends ? 1 : 0;
    for (int j = 0; j < nj; ++j) {
      jobs.bx[j] = boxes[j0 + j % nb];
      jobs.W[j] = Ws[j0 + j % nb];
      jobs.dir[j] = j / nb;
    }
    if (small) {
      const int na = bmax <= 32 ? 2 : bmax <= 48 ? 3 : bmax <= 64 ? 4 : bmax <= 80 ? 5 : 8;
#define FACTOR_PICK(MID)                                                            \
  (na == 2   ? k_chain_factor2d<2, MID>                                             \
   : na == 3 ? k_chain_factor2d<3, MID>                                             \
   : na == 4 ? k_chain_factor2d<4, MID> : k_chain_factor2d<5, MID>)
      for (int m = 0; m < nd; ++m) {  // the chains, then the slices between two halves
        auto kern = m ? FACTOR_PICK(true) : na <= 5 ? FACTOR_PICK(false) : k_chain_factor2d<8, false>;
        const size_t lds = (size_t)(m + 1) * bmax * bmax * sizeof(double);
        allow_lds(P->device, reinterpret_cast<const void*>(kern),
                  (size_t)(m + 1) * (kFacG * na) * (kFacG * na) * sizeof(double));
        hipLaunchKernelGGL(kern, dim3(m ? nb : nj), dim3(kBlock), lds, s, P->g, tab, jobs, rows,
                           P->flag);
      }
#undef FACTOR_PICK
      continue;
    }
    auto step = [&](int i, int n) {
      hipLaunchKernelGGL(k_schur_row, dim3(bmax, n), dim3(kBlock), (size_t)bmax * sizeof(double), s,
                         P->g, jobs, i, tab);
      gj_blocked(P, jobs, n, bmax, i, s);
    };
    for (int i = 0; i < (both_ends ? nch / 2 : nch); ++i) step(i, nj);
    if (both_ends) step(kFacMid, nb);
  }
}

// One workgroup solves one right-hand side v (nch * b values, slice-major,
// overwritten by the solution).  sh holds 2 b doubles of LDS.
template <typename WT>
__device__ void chain_solve_block(const Geo& g, const Box& bx, const double* __restrict__ T,
                                  const WT* __restrict__ W, double* __restrict__ v, double* sh) {
  const int b = bx.b, nch = bx.nch, D = g.D, last = D - 1;
  double* gb = sh;
  double* tb = sh + b;
  const long bb = (long)b * b;
  // forward sweep
  for (int i = 0; i < nch; ++i) {
    for (int r = threadIdx.x; r < b; r += blockDim.x) {
      double val = v[(long)i * b + r];
      if (i > 0) {
        int u[3];
        slice_coords(bx, D, r, u);
        u[last] = i;
        const long tn = box_tnode(g, bx, u);
        for (int t = 0; t < g.ntaps; ++t) {
          int d[3];
          tap_offsets(t, g.ntaps, d[0], d[1], d[2]);
          if (d[last] != -1) continue;
          int rn;
          if (slice_nbr(bx, D, u, d, rn)) val -= T[t * g.tsize + tn] * tb[rn];
        }
      }
      gb[r] = val;
    }
    __syncthreads();
    const WT* Wi = W + (long)i * bb;
    for (int r = threadIdx.x; r < b; r += blockDim.x) {
      double acc = 0.0;
      for (int s2 = 0; s2 < b; ++s2) acc += (double)Wi[(long)s2 * b + r] * gb[s2];
      v[(long)i * b + r] = acc;
      tb[r] = acc;
    }
    __syncthreads();
  }
  // backward sweep; tb holds x_{i+1}
  for (int i = nch - 2; i >= 0; --i) {
    for (int r = threadIdx.x; r < b; r += blockDim.x) {
      int u[3];
      slice_coords(bx, D, r, u);
      u[last] = i;
      const long tn = box_tnode(g, bx, u);
      double val = 0.0;
      for (int t = 0; t < g.ntaps; ++t) {
        int d[3];
        tap_offsets(t, g.ntaps, d[0], d[1], d[2]);
        if (d[last] != 1) continue;
        int rn;
        if (slice_nbr(bx, D, u, d, rn)) val += T[t * g.tsize + tn] * tb[rn];
      }
      gb[r] = val;
    }
    __syncthreads();
    const WT* Wi = W + (long)i * bb;
    for (int r = threadIdx.x; r < b; r += blockDim.x) {
      double acc = 0.0;
      for (int s2 = 0; s2 < b; ++s2) acc += (double)Wi[(long)s2 * b + r] * gb[s2];
      const double x = v[(long)i * b + r] - acc;
      v[(long)i * b + r] = x;
      tb[r] = x;
    }
    __syncthreads();
  }
}

// ---- chain solves of one box with wide slices (3-D boxes, 2-D ones of more than
// kRowsMaxB unknowns), one launch per sweep step over all CUs (one workgroup
// for the whole solve took 1 ms a step at b = 992).
//
// The couplings of slice i with slice i - 1 (d = -1) or i + 1 (d = +1): the
// right-hand side of row k without b_i.  All loads are issued before any is
// used (a neighbour that does not exist is row k itself, masked): loaded one by
// one behind their tests they made a step 36 us at b = 992.
__device__ __forceinline__ double slice_coupling(const Geo& g, const Box& bx,
                                                 const double* __restrict__ T, int i, int k, int d,
                                                 const double* __restrict__ nb) {
  const int D = g.D, m0 = bx.m[0], m1 = D == 3 ? bx.m[1] : 1;
  const int u1 = k / m0, u0 = k - u1 * m0;
  int u[3] = {u0, u1, 0};
  u[D - 1] = i;
  const int ntap = D == 2 ? 3 : 9;
  const double* Tk = T + box_tnode(g, bx, u) + (d < 0 ? 0 : 2 * ntap) * g.tsize;
  double c[9], v[9];
#pragma unroll
  for (int t = 0; t < 9; ++t) {
    int w0 = u0 + t % 3 - 1, w1 = D == 3 ? u1 + t / 3 - 1 : 0;
    if (bx.per[0]) w0 = w0 < 0 ? w0 + m0 : w0 >= m0 ? w0 - m0 : w0;
    if (D == 3 && bx.per[1]) w1 = w1 < 0 ? w1 + m1 : w1 >= m1 ? w1 - m1 : w1;
    const bool in = t < ntap && w0 >= 0 && w0 < m0 && w1 >= 0 && w1 < m1;
    const double ct = Tk[min(t, ntap - 1) * g.tsize], vt = nb[in ? w0 + m0 * w1 : k];
    c[t] = in ? ct : 0.0;
    v[t] = vt;
  }
  double s = 0.0;
#pragma unroll
  for (int t = 0; t < 9; ++t) s += c[t] * v[t];
  return s;
}

// One right-hand side: workgroup = 4 rows of W_i, one per wave, whose entries
// (up to kWideKeep per lane) are loaded before anything is waited for.  Every
// workgroup forms the slice's g for itself in LDS (the slice before it is the
// last launch's output); forward t_i = W_i (b_i - E_i t_{i-1}) into out, backward
// x_i = t_i - W_i E_{i+1}^T x_{i+1}.  bi: b_i (forward); ti: t_i (backward).
constexpr int kWideRows = kBlock / 64, kWideKeep = 18;
template <bool FWD>
__global__ void __launch_bounds__(kBlock) k_wide_row(Geo g, Box bx, const double* __restrict__ T,
                                                     const double* __restrict__ W, int i,
                                                     const double* __restrict__ bi,
                                                     const double* __restrict__ nb,
                                                     const double* __restrict__ ti,
                                                     double* __restrict__ out) {
  extern __shared__ double gs[];  // b
  const int b = bx.b, lane = threadIdx.x & 63;
  const int r = min((int)blockIdx.x * kWideRows + ((int)threadIdx.x >> 6), b - 1);
  const double* Wr = W + ((long)i * b + r) * b;
  double w[kWideKeep];
#pragma unroll
  for (int q = 0; q < kWideKeep; ++q) w[q] = Wr[min(lane + 64 * q, b - 1)];
  const double t = FWD ? 0.0 : ti[r];
  for (int k = threadIdx.x; k < b; k += kBlock) {
    const double c = FWD && i == 0 ? 0.0 : slice_coupling(g, bx, T, i, k, FWD ? -1 : 1, nb);
    gs[k] = FWD ? bi[k] - c : c;
  }
  __syncthreads();
  double acc = 0.0;
#pragma unroll
  for (int q = 0; q < kWideKeep; ++q) {
    const int k = lane + 64 * q;
    acc += k < b ? w[q] * gs[k] : 0.0;
  }
  for (int k = lane + 64 * kWideKeep; k < b; k += 64) acc += Wr[k] * gs[k];
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
  // (the waves past the last row repeat it: same value)
  if (lane == 0) out[r] = FWD ? acc : t - acc;
}

// The columns of the identity, x[col] (nch b values each): 64 x 64 tiles of
// (rows of the slice, columns), 4 x 4 entries per thread, g formed while it is
// staged (the unit entry needs no memory).  A forward tile whose columns all
// start in a later slice is zero.
constexpr int kWideT = 64, kWideK = 32;
template <bool FWD>
__global__ void __launch_bounds__(kBlock) k_wide_tile(Geo g, Box bx, const double* __restrict__ T,
                                                      const double* __restrict__ W, int i, int ncol,
                                                      double* __restrict__ x) {
  __shared__ double Ws[kWideK][kWideT], Gs[kWideK][kWideT + 1];
  const int b = bx.b, r0 = blockIdx.x * kWideT, c0 = blockIdx.y * kWideT;
  const long m = (long)bx.nch * b;
  const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;  // rows r0 + tx + 16 y, columns c0 + ty + 16 z
  double acc[4][4] = {};
  if (!FWD || c0 < (i + 1) * b) {
    const double* Wi = W + (long)i * b * b;
    for (int k0 = 0; k0 < b; k0 += kWideK) {
#pragma unroll
      for (int q = 0; q < kWideK * kWideT / kBlock; ++q) {
        const int idx = threadIdx.x + q * kBlock;
        const int k = k0 + idx / kWideT, r = r0 + idx % kWideT;
        Ws[idx / kWideT][idx % kWideT] = k < b && r < b ? Wi[(long)k * b + r] : 0.0;
        const int kk = k0 + idx % kWideK, c = c0 + idx / kWideK;
        double v = 0.0;
        if (kk < b && c < ncol) {
          if (!FWD || i > 0)
            v = slice_coupling(g, bx, T, i, kk, FWD ? -1 : 1, x + c * m + (long)(FWD ? i - 1 : i + 1) * b);
          if (FWD) v = (c == i * b + kk ? 1.0 : 0.0) - v;
        }
        Gs[idx % kWideK][idx / kWideK] = v;
      }
      __syncthreads();
#pragma unroll 8
      for (int k = 0; k < kWideK; ++k) {
        double w[4], v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          w[q] = Ws[k][tx + 16 * q];
          v[q] = Gs[k][ty + 16 * q];
        }
#pragma unroll
        for (int z = 0; z < 4; ++z)
#pragma unroll
          for (int y = 0; y < 4; ++y) acc[z][y] += w[y] * v[z];
      }
      __syncthreads();
    }
  }
#pragma unroll
  for (int z = 0; z < 4; ++z)
#pragma unroll
    for (int y = 0; y < 4; ++y) {
      const int r = r0 + tx + 16 * y, c = c0 + ty + 16 * z;
      if (r >= b || c >= ncol) continue;
      double* o = x + c * m + (long)i * b + r;
      *o = FWD ? acc[z][y] : *o - acc[z][y];
    }
}

bool launch_rows_box(const ddeig_problem* P, const Box& bx, const double* tab, const double* W,
                     double* v, int nrhs, int identity, hipStream_t s);

// v <- A^{-1} v for one right-hand side; tmp: nch b values
void launch_chain_solve(const ddeig_problem* P, const Box& bx, const double* tab, const double* W,
                        double* v, double* tmp, hipStream_t s) {
  if (launch_rows_box(P, bx, tab, W, v, 1, 0, s)) return;
  const int b = bx.b, n = bx.nch;
  const size_t lds = (size_t)b * sizeof(double);
  const dim3 grid((b + kWideRows - 1) / kWideRows);
  for (int i = 0; i < n; ++i)
    hipLaunchKernelGGL(k_wide_row<true>, grid, dim3(kBlock), lds, s, P->g, bx, tab, W, i,
                       v + (long)i * b, i > 0 ? tmp + (long)(i - 1) * b : nullptr, nullptr,
                       tmp + (long)i * b);
  launch_copy(v + (long)(n - 1) * b, tmp + (long)(n - 1) * b, b, s);
  for (int i = n - 2; i >= 0; --i)
    hipLaunchKernelGGL(k_wide_row<false>, grid, dim3(kBlock), lds, s, P->g, bx, tab, W, i, nullptr,
                       v + (long)(i + 1) * b, tmp + (long)i * b, v + (long)i * b);
}

// x <- A^{-1} (all nch b columns)
void launch_chain_inverse(const ddeig_problem* P, const Box& bx, const double* tab, const double* W,
                          double* x, hipStream_t s) {
  const int m = bx.nch * bx.b;
  if (launch_rows_box(P, bx, tab, W, x, m, 1, s)) return;
  const dim3 grid((bx.b + kWideT - 1) / kWideT, (m + kWideT - 1) / kWideT);
  for (int i = 0; i < bx.nch; ++i)
    hipLaunchKernelGGL(k_wide_tile<true>, grid, dim3(kBlock), 0, s, P->g, bx, tab, W, i, m, x);
  for (int i = bx.nch - 2; i >= 0; --i)
    hipLaunchKernelGGL(k_wide_tile<false>, grid, dim3(kBlock), 0, s, P->g, bx, tab, W, i, m, x);
}

// All local subdomain solves of the level-1 preconditioner in one launch:
// workgroup = subdomain, solved with its class's shared factor.
template <typename WT>
__global__ void __launch_bounds__(kBlock) k_local_solves(Geo g, const double* __restrict__ T,
                                                         const TypeDev* __restrict__ types,
                                                         const SubDev* __restrict__ subs,
                                                         const PcgState* __restrict__ st) {
  extern __shared__ double sh[];
  if (st != nullptr && st->done) return;
  const SubDev sd = subs[blockIdx.x];
  const TypeDev td = types[sd.type];
  Box bx;
  for (int a = 0; a < 3; ++a) {
    bx.o[a] = sd.o[a];
    bx.m[a] = td.m[a];
    bx.per[a] = 0;
  }
  bx.b = td.b;
  bx.nch = td.nch;
  const WT* W;
  if constexpr (sizeof(WT) == 4) W = reinterpret_cast<const WT*>(td.W32);
  else W = reinterpret_cast<const WT*>(td.W);
  chain_solve_block<WT>(g, bx, T, W, td.batch + (long)sd.slot * td.nch * td.b, sh);
}

// ---- batched chain solves
//
// All members of a class share the factors W_i, so a sweep step is the same
// for every member: forward t_i = W_i (b_i - E_i t_{i-1}), backward
// x_i = t_i - W_i E_{i+1}^T x_{i+1}.  A step is three launches:
//   k_chain_rhs: the right-hand sides g of every member (the coupling taps
//     from the table), thread per row, into a buffer [member][row];
//   k_chain_mm: workgroup (row tile of 64 rows, K chunk, member group of up
//     to 64 members of one class) stages its K chunk of g in LDS and
//     multiplies it by rows [r0, r0 + 64) of W_i restricted to the chunk
//     (lane = row, reading W_i by columns since it is symmetric, which
//     coalesces; wave = 16 members); the partial products go to a buffer
//     [K chunk][member][row];
//   k_chain_fin: adds the K-chunk partials of each (member, row) in chunk
//     order and writes t_i (forward) or x_i = t_i - (sum) (backward).
// W_i is read once per member group and step, and a step has row tiles x
// K chunks x groups workgroups.  Arithmetic in WT (FP64, or FP32 for
// local_prec 1) with the right-hand sides formed in FP64.  3-D boxes only
// (chain along the last dim, slices of the first two).
template <typename WT>
struct ChainCfg {
  static constexpr int RT = 64;                         // rows per workgroup
  static constexpr int KC = 64;                         // K chunk (16 or 32 KB of LDS)
  static constexpr int MG = 64;                         // members per group
};

// The right-hand sides g of step i for every member of a job, once per step:
// row r of member m into G[(mg0 + m) * bmax + r] (thread per row).
template <typename WT, bool FWD>
__global__ void __launch_bounds__(kBlock) k_chain_rhs(Geo g, const double* __restrict__ T,
                                                      const TypeDev* __restrict__ types,
                                                      const ChainJob* __restrict__ jobs, int i,
                                                      int bmax, WT* __restrict__ G,
                                                      const PcgState* __restrict__ st) {
  if (st != nullptr && st->done) return;
  const ChainJob jb = jobs[blockIdx.y];
  const TypeDev td = types[jb.type];
  const int b = td.b, nch = td.nch;
  const int r = blockIdx.x * kBlock + threadIdx.x;
  if (r >= b || (int)blockIdx.z >= jb.nm) return;
  const long mstride = (long)nch * b;
  const int m0 = td.m[0], m1 = td.m[1];
  const bool couple = FWD ? i > 0 : true;
  const int j = FWD ? i - 1 : i + 1;
  const double* nb = FWD ? td.tbatch : td.batch;
  // the 9 taps with d2 = -1 (forward) or +1 (backward), in tap order
  const int u1 = r / m0, u0 = r - u1 * m0;
  const long tn = table_node(g, td.o[0] + u0, td.o[1] + u1, td.o[2] + i);
  const int d2 = FWD ? -1 : 1;
  double c[9];
  int nbr[9];
#pragma unroll
  for (int t9 = 0; t9 < 9; ++t9) {
    const int d0 = t9 % 3 - 1, d1 = t9 / 3 - 1;
    const int w0 = u0 + d0, w1 = u1 + d1;
    const bool in = couple && w0 >= 0 && w0 < m0 && w1 >= 0 && w1 < m1;
    c[t9] = in ? T[(t9 + 9 * (d2 + 1)) * g.tsize + tn] : 0.0;
    nbr[t9] = in ? w0 + m0 * w1 : r;
  }
  const int m = blockIdx.z;  // the member (grid z covers a job's members)
  const long base = (long)(jb.m0 + m) * mstride;
  double acc = FWD ? td.batch[base + (long)i * b + r] : 0.0;
  if (couple) {
    const double* nbs = nb + base + (long)j * b;
#pragma unroll
    for (int t9 = 0; t9 < 9; ++t9) acc += (FWD ? -c[t9] : c[t9]) * nbs[nbr[t9]];
  }
  G[(long)(jb.mg0 + m) * bmax + r] = (WT)acc;
}

template <typename WT>
__global__ void __launch_bounds__(kBlock) k_chain_mm(const TypeDev* __restrict__ types,
                                                     const ChainJob* __restrict__ jobs, int i,
                                                     int mtot, int bmax,
                                                     const WT* __restrict__ G,
                                                     WT* __restrict__ part,
                                                     const PcgState* __restrict__ st) {
  using C = ChainCfg<WT>;
  __shared__ __attribute__((aligned(16))) WT gs[C::KC][C::MG];
  if (st != nullptr && st->done) return;
  const ChainJob jb = jobs[blockIdx.z];
  const TypeDev td = types[jb.type];
  const int b = td.b;
  const int r0 = blockIdx.x * C::RT, k0 = blockIdx.y * C::KC;
  if (r0 >= b || k0 >= b) return;
  const int kn = min(C::KC, b - k0);
  // the chunk of the right-hand sides (row fastest: coalesced reads)
  for (int idx = threadIdx.x; idx < kn * C::MG; idx += kBlock) {
    const int m = idx / kn, k = idx - m * kn;
    gs[k][m] = m < jb.nm ? G[(long)(jb.mg0 + m) * bmax + k0 + k] : (WT)0;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int r = r0 + lane;
  constexpr int MW = C::MG / (kBlock / 64);  // members per wave
  WT acc[MW];
#pragma unroll
  for (int q = 0; q < MW; ++q) acc[q] = (WT)0;
  if (r < b && wv * MW < jb.nm) {
    const WT* Wi = (sizeof(WT) == 4 ? reinterpret_cast<const WT*>(td.W32)
                                    : reinterpret_cast<const WT*>(td.W)) +
                   (long)i * b * b + (long)k0 * b + r;
    constexpr int KB = 32;  // loads of W_i in flight per lane
    for (int kk = 0; kk < kn; kk += KB) {
      WT w[KB];
#pragma unroll
      for (int q = 0; q < KB; ++q) w[q] = kk + q < kn ? Wi[(long)(kk + q) * b] : (WT)0;
#pragma unroll
      for (int q = 0; q < KB; ++q) {
        // (past the chunk w[q] = 0 multiplies the chunk's last, written, row);
        // the wave's MW values of the row are read 16 bytes at a time (every
        // lane reads the same address: a broadcast)
        typedef __attribute__((__vector_size__(16))) WT wvec;
        constexpr int VW = 16 / sizeof(WT);
        const wvec* gk = reinterpret_cast<const wvec*>(&gs[min(kk + q, kn - 1)][wv * MW]);
#pragma unroll
        for (int v4 = 0; v4 < MW / VW; ++v4) {
          const wvec gv = gk[v4];
#pragma unroll
          for (int e = 0; e < VW; ++e) acc[v4 * VW + e] += w[q] * gv[e];
        }
      }
    }
  }
  if (r >= b) return;
#pragma unroll
  for (int mm = 0; mm < MW; ++mm) {
    const int m = wv * MW + mm;
    if (m < jb.nm) part[((long)blockIdx.y * mtot + jb.mg0 + m) * bmax + r] = acc[mm];
  }
}

// t_i = sum of the K-chunk partials (forward), x_i = t_i - sum (backward),
// x_{n-1} = t_{n-1} (copy, the first backward step).
template <typename WT, bool FWD>
__global__ void __launch_bounds__(kBlock) k_chain_fin(const TypeDev* __restrict__ types,
                                                      const ChainJob* __restrict__ jobs, int i,
                                                      int mtot, int bmax,
                                                      const WT* __restrict__ part, int copy,
                                                      const PcgState* __restrict__ st) {
  if (st != nullptr && st->done) return;
  const ChainJob jb = jobs[blockIdx.y];
  const TypeDev td = types[jb.type];
  const int b = td.b;
  const int r = blockIdx.x * kBlock + threadIdx.x;
  const int m = blockIdx.z;  // the member (grid z covers a job's members)
  if (r >= b || m >= jb.nm) return;
  const int nkc = (b + ChainCfg<WT>::KC - 1) / ChainCfg<WT>::KC;
  const long mstride = (long)td.nch * b;
  const long at = (long)(jb.m0 + m) * mstride + (long)i * b + r;
  if (copy) {
    td.batch[at] = td.tbatch[at];
    return;
  }
  double v = 0.0;
  for (int kc = 0; kc < nkc; ++kc) v += (double)part[((long)kc * mtot + jb.mg0 + m) * bmax + r];
  if (FWD) td.tbatch[at] = v;
  else td.batch[at] = td.tbatch[at] - v;
}

// Members per group of the batched chain solves and the partial buffer size.
int chain_group_members() { return ChainCfg<double>::MG; }

size_t chain_part_bytes(int bmax, int mtot, int fp32) {
  // the K-chunk partials, then the right-hand sides
  const int kc = fp32 ? ChainCfg<float>::KC : ChainCfg<double>::KC;
  return (size_t)((bmax + kc - 1) / kc + 1) * mtot * bmax * (fp32 ? sizeof(float) : sizeof(double));
}

template <typename WT>
static void chain_sweeps(const ddeig_problem* P, const PcgState* st, hipStream_t s) {
  using C = ChainCfg<WT>;
  const int nch = P->types[0].box.nch;
  const int bmax = P->chain_bmax, mtot = P->chain_mtot;
  const int nkc = (bmax + C::KC - 1) / C::KC;
  WT* part = reinterpret_cast<WT*>(P->chain_part);
  WT* G = part + (long)nkc * mtot * bmax;
  const dim3 gmm((bmax + C::RT - 1) / C::RT, nkc, P->nchainjobs);
  const dim3 gnode((bmax + kBlock - 1) / kBlock, P->nchainjobs, C::MG);
  for (int i = 0; i < nch; ++i) {
    hipLaunchKernelGGL((k_chain_rhs<WT, true>), gnode, dim3(kBlock), 0, s, P->g, P->tabAs,
                       P->dTypes, P->dChainJobs, i, bmax, G, st);
    hipLaunchKernelGGL((k_chain_mm<WT>), gmm, dim3(kBlock), 0, s, P->dTypes, P->dChainJobs, i,
                       mtot, bmax, G, part, st);
    hipLaunchKernelGGL((k_chain_fin<WT, true>), gnode, dim3(kBlock), 0, s, P->dTypes,
                       P->dChainJobs, i, mtot, bmax, part, 0, st);
  }
  hipLaunchKernelGGL((k_chain_fin<WT, false>), gnode, dim3(kBlock), 0, s, P->dTypes,
                     P->dChainJobs, nch - 1, mtot, bmax, part, 1, st);
  for (int i = nch - 2; i >= 0; --i) {
    hipLaunchKernelGGL((k_chain_rhs<WT, false>), gnode, dim3(kBlock), 0, s, P->g, P->tabAs,
                       P->dTypes, P->dChainJobs, i, bmax, G, st);
    hipLaunchKernelGGL((k_chain_mm<WT>), gmm, dim3(kBlock), 0, s, P->dTypes, P->dChainJobs, i,
                       mtot, bmax, G, part, st);
    hipLaunchKernelGGL((k_chain_fin<WT, false>), gnode, dim3(kBlock), 0, s, P->dTypes,
                       P->dChainJobs, i, mtot, bmax, part, 0, st);
  }
}

void launch_chain_batched(const ddeig_problem* P, const PcgState* st, hipStream_t s) {
  if (P->opt.local_prec == 1) chain_sweeps<float>(P, st, s);
  else chain_sweeps<double>(P, st, s);
}

bool local_solves_fast_ok(const ddeig_problem* P);
void launch_local_solves_fast(const ddeig_problem* P, const PcgState* st, hipStream_t s,
                              bool coarse);
bool launch_local_solves_staged(const ddeig_problem* P, const PcgState* st, hipStream_t s);

void launch_local_solves(const ddeig_problem* P, const PcgState* st, hipStream_t s,
                         const double* coarse_r) {
  if (P->opt.local_prec >= 2) {
    // one batch of all subdomains: MFMA tiles, or the streaming kernel for a
    // handful of rows (one of the two has no work); coarse_r (nullable): the
    // GEMM launch also forms R_0 coarse_r
    launch_dense_gemm(P, st, s, coarse_r);
    launch_dense_gemv(P, st, s);
    return;
  }
  if (local_solves_fast_ok(P)) {
    launch_local_solves_fast(P, st, s, coarse_r != nullptr);
    return;
  }
  if (P->nchainjobs > 0) {
    if (P->chain_mfma) launch_chain_mfma(P, st, s);
    else launch_chain_batched(P, st, s);
    return;
  }
  if (launch_local_solves_staged(P, st, s)) return;
  const size_t lds = 2 * (size_t)P->maxb * sizeof(double);
  if (P->opt.local_prec == 1)
    hipLaunchKernelGGL(k_local_solves<float>, dim3(P->nsub), dim3(kBlock), lds, s, P->g,
                       P->tabAs, P->dTypes, P->dSubs, st);
  else
    hipLaunchKernelGGL(k_local_solves<double>, dim3(P->nsub), dim3(kBlock), lds, s, P->g,
                       P->tabAs, P->dTypes, P->dSubs, st);
}

}  // namespace ddeig

namespace ddeig {

// ---- chain solves of 2-D boxes: slices along x of at most kRowsMaxB unknowns,
// chain along y, one workgroup per right-hand side.
//
// A sweep from one end is 2 nch - 1 dependent steps t = W_i g, g = b_i - E_i t_{i-1} (or
// E_{i+1}^T x_{i+1}), so a step's latency is the time of the solve.  It is a
// chain of instructions (a wave issues one every 4 to 5 cycles) and LDS round
// trips, so it is split to keep what the chain waits for short:
//  - wave 0 forms g, two rows per lane, from the last slice in LDS; couplings
//    and b_i are in its registers by then;
//  - a lane of the other waves multiplies its part's columns of g by its pair of
//    rows of W_i (RowsLayout), the 8 parts of a row are added across the wave,
//    and the lane that ends up with a row writes it to the slice in LDS.  They
//    load W of the slice after next while wave 0 forms g.
// The right-hand side and the sweep's vectors stay in LDS throughout: no global
// store, and no load whose latency a step waits for.  At b = 71: W_i staged
// through LDS with three barriers a step 2.2 us; partial sums passed through LDS
// 0.96; every wave forming g for itself (one barrier) 0.60, at b = 35 0.46; this
// 0.60 and 0.36.  From both ends (BOTH) a step takes two slices: 1.09 us and
// 0.26 us, half as many; at b = 71 the 90 KB of W it reads, 21 TB/s over the 256
// workgroups, are what it waits for (256 subdomains of 63 lines: 285 -> 84 -> 76
// us; 32 of 31 lines of 35: 20.9 -> 16.6 us).
// In 2-D the couplings are the taps (-1..1, -1), i.e. table taps 0..2
// (forward), and (-1..1, +1), taps 6..8 (backward).
template <typename WT>
struct Pair;
template <>
struct Pair<double> {
  typedef double __attribute__((ext_vector_type(2))) type;
};
template <>
struct Pair<float> {
  typedef float __attribute__((ext_vector_type(2))) type;
};

// The values of a and b of all 8 parts added: lanes 0..31 receive the sums of
// a, lanes 32..63 those of b.
__device__ __forceinline__ double part_sum2(double a, double b) {
  typedef unsigned __attribute__((ext_vector_type(2))) u2;
  auto join = [](unsigned lo, unsigned hi) { return __builtin_bit_cast(double, u2{lo, hi}); };
  const u2 ua = __builtin_bit_cast(u2, a), ub = __builtin_bit_cast(u2, b);
  // lanes 0..31: a of both halves, lanes 32..63: b of both halves
  auto l = __builtin_amdgcn_permlane32_swap(ua.x, ub.x, false, false);
  auto h = __builtin_amdgcn_permlane32_swap(ua.y, ub.y, false, false);
  double v = join(l[0], h[0]) + join(l[1], h[1]);
  u2 u = __builtin_bit_cast(u2, v);
  l = __builtin_amdgcn_permlane16_swap(u.x, u.x, false, false);
  h = __builtin_amdgcn_permlane16_swap(u.y, u.y, false, false);
  v = join(l[0], h[0]) + join(l[1], h[1]);
  u = __builtin_bit_cast(u2, v);
  // row_ror:8
  return v + join(__builtin_amdgcn_update_dpp(0, u.x, 0x128, 0xf, 0xf, false),
                  __builtin_amdgcn_update_dpp(0, u.y, 0x128, 0xf, 0xf, false));
}

// o0, o1: origin of the box; per: periodic in x.  col >= 0: the right-hand side
// is column col of the identity (v is not read, and the sweep starts at its
// slice's step).  tbuf: rows_lds(b, nch) bytes of LDS.  csum (nullable): receives
// phi . v, of the right-hand side (col < 0).
// Step st = 0 .. 2 h works on slice min(st, 2 h - st); BOTH: h = nch / 2 and the
// mirrored slice 2 h minus that one is worked on at the same time by waves of
// its own (an even nch has no slice 2 h; its W reads as zero).  Otherwise h = nch - 1.
template <typename WT, int KM, bool BOTH>
__device__ __forceinline__ void chain_rows(const Geo& g, const double* __restrict__ T,
                                           const WT* __restrict__ W, double* __restrict__ v, int b,
                                           int nch, int o0, int o1, bool per, int col,
                                           double* __restrict__ tbuf,
                                           const double* __restrict__ phi = nullptr,
                                           double* __restrict__ csum = nullptr) {
  typedef typename Pair<WT>::type wpair;
  constexpr int GS = KM | 1;  // stride of a part's columns of g (odd: distinct banks)
  constexpr int NS = BOTH ? 2 : 1;
  __shared__ double gsh[NS][8 * GS + 1];  // g, and a slot for rows that do not exist
  const int tid = threadIdx.x, lane = tid & 63, nth = blockDim.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const RowsLayout l(b);
  const int h = BOTH ? nch / 2 : nch - 1;
  const int i0 = col < 0 ? 0 : col / b;
  const int st0 = min(i0, 2 * h - i0), end = 2 * h + 1;  // the steps are [st0, end)
  // waves 0 .. NS - 1 form g, the rest multiply, those of the mirrored side last
  const int side = !BOTH ? 0 : wave < NS ? wave : (wave - NS >= l.nw ? 1 : 0);
  // the slice of step st (past the last step: any slice)
  auto slice = [&](int st) {
    const int u = max(min(st, 2 * h - st), 0);
    return __builtin_amdgcn_readfirstlane(side ? 2 * h - u : u);
  };
  // one row in front of the slices and 64 rows behind them are read, not used
  double* tb = tbuf + 1;
  const int dump = (BOTH ? nch | 1 : nch) * b;
  double pv = 0.0;
  if (csum != nullptr) {
    for (int q = tid; q < nch * b; q += nth) {
      const double x = v[q];
      tb[q] = x;
      pv += phi[q] * x;
    }
  } else {
    for (int q = tid; q < nch * b; q += nth) tb[q] = col < 0 ? v[q] : (q == col ? 1.0 : 0.0);
  }
  for (int q = nch * b + tid; q < dump + 2 * 64; q += nth) tb[q] = 0.0;
  if (tid == 0) tbuf[0] = 0.0;
  for (int q = tid; q < NS * (8 * GS + 1); q += nth) gsh[0][q] = 0.0;
  __syncthreads();
  // (the steps past the last that the unrolling by three needs change nothing: a
  // break inside the loops would spoil the compiler's load counters)
  if (wave < NS) {
    // rows r0, r0 + 1 of this lane, the columns that hold their neighbours, and
    // their places in g
    const int r0 = 2 * lane, r1 = r0 + 1;
    const int nl = per && r0 == 0 ? b - 1 : r0 - 1;  // left of r0
    const int nm = per && r0 == b - 1 ? 0 : r1;      // right of r0, and r1 itself
    const int nr = per && r1 == b - 1 ? 0 : r0 + 2;  // right of r1
    auto place = [&](int r) { return r < b ? r / l.chunk * GS + r % l.chunk : 8 * GS; };
    double* g0p = gsh[side] + place(r0);
    double* g1p = gsh[side] + place(r1);
    // couplings of a step: three taps of each row (zero without a neighbour)
    const auto rt = __builtin_amdgcn_make_buffer_rsrc((void*)T, (short)0, (int)(9 * g.tsize * 8),
                                                      0x00020000);
    int coff[6];
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      const int u = t < 3 ? r0 : r1, d = t % 3, n = u + d - 1;
      const bool in = u < b && (per || (n >= 0 && n < b));
      // (an offset past the table reads as zero)
      coff[t] = (int)(in ? d * g.tsize + (o0 + u + 1 + g.ne) % g.ne : 9 * g.tsize) * 8;
    }
    const int cline = g.P[0] * 8, cback = (int)(6 * g.tsize * 8);
    struct Coup {
      double e[6];
    };
    // couplings of slice i to the slice before it, or after it
    auto loadc = [&](int i, bool after) {
      Coup c;
#pragma unroll
      for (int t = 0; t < 6; ++t)
        c.e[t] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(
                                                rt, coff[t], (o1 + i) * cline + (after ? cback : 0), 0));
      return c;
    };
    // (a side meets the slice it has solved last)
    auto after = [&](int st) { return (st > h) != (side != 0); };
    int sp = slice(st0), s0 = sp, s1 = slice(st0 + 1), s2 = slice(st0 + 2), s3 = slice(st0 + 3);
    // (the first step has no couplings)
    Coup ca{}, cb = loadc(s1, after(st0 + 1)), cc = loadc(s2, after(st0 + 2));
    const Coup cm = BOTH ? loadc(h, true) : Coup{};
    double v0 = tb[s0 * b + r0], v1 = tb[s0 * b + r1];
    // h of the lane's rows from the slice at tp
    auto couple = [&](const double* tp, const Coup& c, double& h0, double& h1) {
      const double tl = tp[nl], t0 = tp[r0], t1 = tp[nm], tr = tp[nr];
      h0 = c.e[0] * tl;
      h1 = c.e[3] * t0;
      h0 += c.e[1] * t0;
      h1 += c.e[4] * t1;
      h0 += c.e[2] * t1;
      h1 += c.e[5] * tr;
    };
    // step st: couplings in c, replaced by those of step st + 3
    auto step = [&](int st, Coup& c) {
      const double sg = st <= h ? -1.0 : 1.0;  // g = b_i - E t, or E^T x
      double h0, h1;
      couple(tb + sp * b, c, h0, h1);
      if (BOTH && st == h) {  // the middle slice takes both neighbours
        double m0, m1;
        couple(tb + min(h + 1, nch) * b, cm, m0, m1);
        if (h + 1 < nch) {
          h0 += m0;
          h1 += m1;
        }
      }
      *g0p = v0 + sg * h0;
      *g1p = v1 + sg * h1;
      __syncthreads();
      c = loadc(s3, after(st + 3));
      v0 = tb[s1 * b + r0];
      v1 = tb[s1 * b + r1];
      if (st + 1 > h) v0 = v1 = 0.0;
      sp = s0;
      s0 = s1;
      s1 = s2;
      s2 = s3;
      s3 = slice(st + 4);
      __syncthreads();
    };
    for (int st = st0; st < end; st += 3) {
      step(st, ca);
      step(st + 1, cb);
      step(st + 2, cc);
    }
  } else {
    const int w0 = wave - NS - (side ? l.nw : 0), q = lane & 7;
    // this lane's pairs of W.  Loads past a part's columns read the next wave's
    // or slice's entries, or zero past the end: those terms meet a zero of g;
    // lanes without rows read nothing.
    constexpr int WB = (int)sizeof(wpair);
    const int sbytes = l.slice() * WB;
    const auto rw = __builtin_amdgcn_make_buffer_rsrc((void*)W, (short)0, nch * sbytes, 0x00020000);
    const int wlane = w0 < l.nw && 16 * w0 + 2 * q < b ? (w0 * l.chunk * 64 + lane) * WB : nch * sbytes;
    auto loadw = [&](wpair (&w)[KM], int i) {
      const int base = i * sbytes;
#pragma unroll
      for (int k = 0; k < KM; ++k) {
        constexpr int reach = 4096 / (64 * WB);  // loads an immediate offset reaches
        // (a scalar offset past the buffer's end would wrap in its bounds check)
        const int imm = k % reach * 64 * WB, off = min(base + k / reach * 4096, nch * sbytes);
        if constexpr (sizeof(WT) == 8)
          w[k] = __builtin_bit_cast(wpair, __builtin_amdgcn_raw_buffer_load_b128(rw, wlane + imm, off, 0));
        else
          w[k] = __builtin_bit_cast(wpair, __builtin_amdgcn_raw_buffer_load_b64(rw, wlane + imm, off, 0));
      }
    };
    const double* gl = gsh[side] + (lane >> 3) * GS;
    // the row that part_sum2 leaves in this lane
    const int own = 16 * w0 + 2 * q + (lane >> 5);
    const bool owner = (lane & 24) == 0 && own < b;
    int s0 = slice(st0), s1 = slice(st0 + 1), s2 = slice(st0 + 2);
    wpair wa[KM], wb[KM], wc[KM];
    loadw(wa, s0);
    loadw(wb, s1);
    // step st: W in w; loads W of step st + 2 into wn.  (In the middle step the
    // mirrored side has no slice of its own.)
    auto step = [&](int st, const wpair (&w)[KM], wpair (&wn)[KM]) {
      loadw(wn, s2);
      const double told = tb[s0 * b + own];
      double* out = tb + (owner && st < end && !(side && st == h) ? s0 * b + own : dump);
      s0 = s1;
      s1 = s2;
      s2 = slice(st + 3);
      __syncthreads();
      double a0 = 0.0, a1 = 0.0;
#pragma unroll
      for (int k = 0; k < KM; ++k) {
        a0 += (double)w[k].x * gl[k];
        a1 += (double)w[k].y * gl[k];
      }
      const double t = part_sum2(a0, a1);
      *out = st <= h ? t : told - t;
      __syncthreads();
    };
    for (int st = st0; st < end; st += 3) {
      step(st, wa, wc);
      step(st + 1, wb, wa);
      step(st + 2, wc, wb);
    }
  }
  for (int q = tid; q < nch * b; q += nth) v[q] = tb[q];
  if (csum != nullptr) {
    for (int off = 32; off > 0; off >>= 1) pv += __shfl_down(pv, off, 64);
    if (lane == 0) gsh[0][wave] = pv;
    __syncthreads();
    if (tid == 0) {
      double t = 0.0;
      for (int i = 0; i < nth / 64; ++i) t += gsh[0][i];
      *csum = t;
    }
  }
}

// The level-1 preconditioner's local solves: workgroup = subdomain, with its
// class's factor.  With crhs a workgroup also forms its entry of the coarse
// right-hand side, phi . R_i r, from the copy of R_i r that it reads anyway.  As
// a kernel of its own that was 4 to 10 us on a second stream beside the solves,
// and ordering the two streams cost more than the solves gained: 256 boxes of
// 63 x 71, an application 107.1 -> 100.2 us; 32 boxes of 31 x 35, a solve with
// its gradient 15.3 -> 12.2 ms.
template <typename WT, int NT, int KM, bool BOTH>
__global__ void __launch_bounds__(NT) k_rows_local(Geo g, const double* __restrict__ T,
                                                   const TypeDev* __restrict__ types,
                                                   const SubDev* __restrict__ subs,
                                                   const PcgState* __restrict__ st,
                                                   double* __restrict__ crhs) {
  extern __shared__ double tb[];
  if (st != nullptr && st->done) return;
  const SubDev sd = subs[blockIdx.x];
  const TypeDev& td = types[sd.type];
  const WT* W;
  if constexpr (sizeof(WT) == 4) W = reinterpret_cast<const WT*>(td.W32);
  else W = reinterpret_cast<const WT*>(td.W);
  chain_rows<WT, KM, BOTH>(g, T, W, td.batch + (long)sd.slot * td.nch * td.b, td.b, td.nch,
                           sd.o[0], sd.o[1], false, -1, tb, td.phi,
                           crhs != nullptr ? crhs + blockIdx.x : nullptr);
}

// Right-hand sides of one box (FP64 factors): workgroup = right-hand side;
// columns of the identity start in their own slice.
template <int NT, int KM, bool BOTH>
__global__ void __launch_bounds__(NT) k_rows_box(Geo g, Box bx, const double* __restrict__ T,
                                                 const double* __restrict__ W,
                                                 double* __restrict__ v, int identity) {
  extern __shared__ double tb[];
  const long m = (long)bx.nch * bx.b;
  const int col = identity ? (int)blockIdx.x : -1;
  chain_rows<double, KM, BOTH>(g, T, W, v + blockIdx.x * m, bx.b, bx.nch, bx.o[0], bx.o[1],
                               bx.per[0] != 0, col, tb);
}

// The kernel for slices of at most b: columns per part (b / 8 rounded up), and
// threads (per side a wave that forms g and a wave per 16 rows).  In FP64 the widest,
// 97 to 128 unknowns, spills 46 of its registers: 16 subdomains of 119 lines of 127,
// 762 us an application (95 wide, 89 lines: 164), k_local_solves 7.3 ms.
#define ROWS_PICK_WIDE(KERN, b, ...) \
  ((b) <= 96 ? KERN<__VA_ARGS__ 448, 12, false> : KERN<__VA_ARGS__ 576, 16, false>)
#define ROWS_PICK(KERN, b, ...)                                                         \
  ((b) <= 24   ? KERN<__VA_ARGS__ 192, 3, false>                                        \
   : (b) <= 40 ? KERN<__VA_ARGS__ 256, 5, false>                                        \
   : (b) <= 56 ? KERN<__VA_ARGS__ 320, 7, false>                                        \
   : (b) <= 64 ? KERN<__VA_ARGS__ 320, 8, false>                                        \
   : (b) <= 72 ? KERN<__VA_ARGS__ 384, 9, false>                                        \
   : (b) <= 80 ? KERN<__VA_ARGS__ 384, 10, false> : ROWS_PICK_WIDE(KERN, b, __VA_ARGS__))
#define ROWS_PICK_BOTH(KERN, b, ...)                                                    \
  ((b) <= 24   ? KERN<__VA_ARGS__ 384, 3, true>                                         \
   : (b) <= 40 ? KERN<__VA_ARGS__ 512, 5, true>                                         \
   : (b) <= 56 ? KERN<__VA_ARGS__ 640, 7, true>                                         \
   : (b) <= 64 ? KERN<__VA_ARGS__ 640, 8, true>                                         \
   : (b) <= 72 ? KERN<__VA_ARGS__ 768, 9, true> : KERN<__VA_ARGS__ 768, 10, true>)
#define ROWS_COMMA ,

template <typename K>
static void rows_launch(const ddeig_problem* P, K kern, bool both, int b, int nch, size_t& lds,
                        int& nt) {
  lds = rows_lds(b, nch);
  nt = 64 * (RowsLayout(b).nw + 1) * (both ? 2 : 1);
  allow_lds(P->device, reinterpret_cast<const void*>(kern), kRowsLdsMax);
}

bool launch_rows_box(const ddeig_problem* P, const Box& bx, const double* tab, const double* W,
                     double* v, int nrhs, int identity, hipStream_t s) {
  if (P->g.D != 2 || !rows_ok(bx.b, bx.nch)) return false;
  const bool both = rows_both(P->g.D, bx.b, bx.nch);
  // (every box of at most kRowsBothB is solved from both ends)
  auto kern = both ? ROWS_PICK_BOTH(k_rows_box, bx.b) : ROWS_PICK_WIDE(k_rows_box, bx.b);
  size_t lds;
  int nt;
  rows_launch(P, kern, both, bx.b, bx.nch, lds, nt);
  hipLaunchKernelGGL(kern, dim3(nrhs), dim3(nt), lds, s, P->g, bx, tab, W, v, identity);
  return true;
}

static void class_extents(const ddeig_problem* P, int& b, int& nch) {
  b = nch = 0;
  for (const auto& t : P->types) {
    b = std::max(b, t.box.b);
    nch = std::max(nch, t.box.nch);
  }
}

// Local solves of 2-D slices of at most kFastB unknowns whose chain is longer than
// the row solves' LDS copy (rows_ok), from one end, workgroup = subdomain.  W_i
// (rows of b values) is staged in LDS with double buffering; while step i computes
// from LDS, every thread already holds its share of W_{i+1} (W_{i-1} in the backward
// sweep), the next slice of the right-hand side and the next coupling coefficients
// in registers.  Each row's dot product is split over np = floor(256 / b) thread
// groups and the parts are added in a fixed order.  The couplings to the neighbouring
// slice are table taps 0..2 (forward) and 6..8 (backward), with in-slice neighbours
// r - 1, r, r + 1.  64 subdomains of 255 lines of 71 unknowns in FP64: 1.16 ms an
// application, with k_local_solves 9.03 ms; 16 of 511 lines of 35 1.49 ms, 9.08.
constexpr int kFastB = 72;
constexpr int kFastRegs = (kFastB * kFastB + kBlock - 1) / kBlock;
template <typename WT>
__device__ inline double dot_part(const WT* __restrict__ wc, const double* __restrict__ gv, int b,
                                  int r, int s0, int s1) {
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  int s = s0;
  for (; s + 3 < s1; s += 4) {
    a0 += (double)wc[s * b + r] * gv[s];
    a1 += (double)wc[(s + 1) * b + r] * gv[s + 1];
    a2 += (double)wc[(s + 2) * b + r] * gv[s + 2];
    a3 += (double)wc[(s + 3) * b + r] * gv[s + 3];
  }
  for (; s < s1; ++s) a0 += (double)wc[s * b + r] * gv[s];
  return (a0 + a1) + (a2 + a3);
}
template <typename WT>
__global__ void __launch_bounds__(kBlock) k_local_solves_2d(Geo g, const double* __restrict__ T,
                                                            const TypeDev* __restrict__ types,
                                                            const SubDev* __restrict__ subs,
                                                            const PcgState* __restrict__ st) {
  __shared__ WT wbuf[2][kFastB * kFastB];
  __shared__ double gb[kFastB];
  __shared__ double tb[kFastB];
  __shared__ double red[kBlock];
  if (st != nullptr && st->done) return;
  const SubDev sd = subs[blockIdx.x];
  const TypeDev td = types[sd.type];
  const int b = td.b, nch = td.nch;
  const int bb = b * b;
  const int tid = threadIdx.x;
  const int np = kBlock / b;  // thread groups per row
  const int chunk = (b + np - 1) / np;
  const int part = tid / b, rr = tid - part * b;
  const bool dot_thread = part < np;
  const int s0 = min(b, part * chunk), s1 = min(b, s0 + chunk);
  const WT* __restrict__ W;
  if constexpr (sizeof(WT) == 4) W = reinterpret_cast<const WT*>(td.W32);
  else W = reinterpret_cast<const WT*>(td.W);
  double* __restrict__ v = td.batch + (long)sd.slot * nch * b;
  const bool row = tid < b;
  const int jx = row ? (sd.o[0] + tid + 1) % g.ne : 0;
  const bool has_l = tid > 0, has_r = tid + 1 < b;
  WT pre[kFastRegs];
  for (int j = tid; j < bb; j += kBlock) wbuf[0][j] = W[j];
  double vnext = row ? v[tid] : 0.0;
  double cn0 = 0.0, cn1 = 0.0, cn2 = 0.0;
  __syncthreads();
  // forward sweep: t_i = W_i (b_i - E_i t_{i-1})
  for (int i = 0; i < nch; ++i) {
    const double vi = vnext, c0 = cn0, c1 = cn1, c2 = cn2;
    if (i + 1 < nch) {
      const WT* Wn = W + (long)(i + 1) * bb;
#pragma unroll
      for (int j = 0; j < kFastRegs; ++j) {
        const int idx = tid + j * kBlock;
        if (idx < bb) pre[j] = Wn[idx];
      }
      if (row) {
        vnext = v[(long)(i + 1) * b + tid];
        const long tn = jx + (long)g.P[0] * (sd.o[1] + i + 1);
        cn0 = T[0 * g.tsize + tn];
        cn1 = T[1 * g.tsize + tn];
        cn2 = T[2 * g.tsize + tn];
      }
    }
    if (row) {
      double val = vi;
      if (i > 0) {
        if (has_l) val -= c0 * tb[tid - 1];
        val -= c1 * tb[tid];
        if (has_r) val -= c2 * tb[tid + 1];
      }
      gb[tid] = val;
    }
    __syncthreads();
    if (dot_thread) red[tid] = dot_part(wbuf[i & 1], gb, b, rr, s0, s1);
    __syncthreads();
    if (row) {
      double acc = red[tid];
      for (int pp = 1; pp < np; ++pp) acc += red[pp * b + tid];
      v[(long)i * b + tid] = acc;
      tb[tid] = acc;
    }
    if (i + 1 < nch) {
#pragma unroll
      for (int j = 0; j < kFastRegs; ++j) {
        const int idx = tid + j * kBlock;
        if (idx < bb) wbuf[(i + 1) & 1][idx] = pre[j];
      }
    }
    __syncthreads();
  }
  // backward sweep: x_i = t_i - W_i E_{i+1}^T x_{i+1}; W_{nch-2} is still in wbuf[nch & 1]
  if (nch >= 2 && row) {
    const long tn = jx + (long)g.P[0] * (sd.o[1] + nch - 2);
    cn0 = T[6 * g.tsize + tn];
    cn1 = T[7 * g.tsize + tn];
    cn2 = T[8 * g.tsize + tn];
    vnext = v[(long)(nch - 2) * b + tid];
  }
  for (int i = nch - 2; i >= 0; --i) {
    const double vi = vnext, c0 = cn0, c1 = cn1, c2 = cn2;
    if (i >= 1) {
      const WT* Wn = W + (long)(i - 1) * bb;
#pragma unroll
      for (int j = 0; j < kFastRegs; ++j) {
        const int idx = tid + j * kBlock;
        if (idx < bb) pre[j] = Wn[idx];
      }
      if (row) {
        vnext = v[(long)(i - 1) * b + tid];
        const long tn = jx + (long)g.P[0] * (sd.o[1] + i - 1);
        cn0 = T[6 * g.tsize + tn];
        cn1 = T[7 * g.tsize + tn];
        cn2 = T[8 * g.tsize + tn];
      }
    }
    if (row) {
      double val = c1 * tb[tid];
      if (has_l) val += c0 * tb[tid - 1];
      if (has_r) val += c2 * tb[tid + 1];
      gb[tid] = val;
    }
    __syncthreads();
    if (dot_thread) red[tid] = dot_part(wbuf[i & 1], gb, b, rr, s0, s1);
    __syncthreads();
    if (row) {
      double acc = red[tid];
      for (int pp = 1; pp < np; ++pp) acc += red[pp * b + tid];
      const double x = vi - acc;
      v[(long)i * b + tid] = x;
      tb[tid] = x;
    }
    if (i >= 1) {
#pragma unroll
      for (int j = 0; j < kFastRegs; ++j) {
        const int idx = tid + j * kBlock;
        if (idx < bb) wbuf[(i - 1) & 1][idx] = pre[j];
      }
    }
    __syncthreads();
  }
}

bool launch_local_solves_staged(const ddeig_problem* P, const PcgState* st, hipStream_t s) {
  int b, nch;
  class_extents(P, b, nch);
  if (P->g.D != 2 || b > kFastB) return false;
  auto kern = P->opt.local_prec == 1 ? k_local_solves_2d<float> : k_local_solves_2d<double>;
  hipLaunchKernelGGL(kern, dim3(P->nsub), dim3(kBlock), 0, s, P->g, P->tabAs, P->dTypes, P->dSubs, st);
  return true;
}

// Row solves of the classes: FP64 factors from both ends, FP32 factors from one (their
// solves from both ends have not been built or measured).
bool classes_both(const ddeig_problem* P) {
  int b, nch;
  class_extents(P, b, nch);
  return P->opt.local_prec != 1 && rows_both(P->g.D, b, nch);
}

bool local_solves_fast_ok(const ddeig_problem* P) {
  int b, nch;
  class_extents(P, b, nch);
  return P->g.D == 2 && rows_ok(b, nch);
}

template <typename WT>
static void launch_rows_local(const ddeig_problem* P, const PcgState* st, double* crhs,
                              hipStream_t s) {
  int b, nch, nt;
  size_t lds;
  class_extents(P, b, nch);
  const bool both = classes_both(P);
  auto kern = ROWS_PICK_WIDE(k_rows_local, b, WT ROWS_COMMA);
  if constexpr (sizeof(WT) == 8) {
    if (both) kern = ROWS_PICK_BOTH(k_rows_local, b, WT ROWS_COMMA);
  } else {
    kern = ROWS_PICK(k_rows_local, b, WT ROWS_COMMA);
  }
  rows_launch(P, kern, both, b, nch, lds, nt);
  hipLaunchKernelGGL(kern, dim3(P->nsub), dim3(nt), lds, s, P->g, P->tabAs, P->dTypes, P->dSubs, st,
                     crhs);
}

void launch_local_solves_fast(const ddeig_problem* P, const PcgState* st, hipStream_t s,
                              bool coarse) {
  double* crhs = coarse ? P->crhs : nullptr;
  if (P->opt.local_prec == 1) launch_rows_local<float>(P, st, crhs, s);
  else launch_rows_local<double>(P, st, crhs, s);
}

// The coarse right-hand side rides in the local solves when they are row solves.
bool rows_coarse(const ddeig_problem* P) {
  return P->opt.coarse && P->opt.local_prec < 2 && local_solves_fast_ok(P);
}

}  // namespace ddeig
