// Batched block-chain local solves of 3-D boxes with FP32 factors on MFMA.
//
// The local matrices A_sigma,i of §3 (eq:twoLevelASMPreconditioner) are block
// tridiagonal along the last (fixed) direction.  They are eliminated from both
// ends towards slice h = n / 2 (k_chain.hip): for the upper chain (i < h)
// W_i = S_i^{-1} with S_i = D_i - E_i W_{i-1} E_i^T, for the lower one (i > h)
// the same with slice i + 1, and slice h takes both.  A solve is
//   inwards   t_i = W_i (b_i - coupling of i with the slice before it),
//   middle    x_h = W_h (b_h - both couplings),
//   outwards  x_i = t_i - W_i (coupling of i with the slice nearer to h).
// The two chains run in the same launches, so a solve is n dependent steps
// instead of 2 n - 1 (a step is bound by its latency: with one chain, 61 steps
// of 31 slices took 16 us each at 16 subdomains, 31 steps of two 22 us).
// All members of a class share W_i, so each step is one product of W_i
// (b x b, FP32) with the right-hand sides of all members of the class.  A step
// is two launches:
//   k_cm_rhs: finishes the previous step (t or x of the neighbouring slice, as
//     the fixed-order sum of the previous product's K-chunk partials, less t
//     outwards), stores it for the workgroup's own rows, and forms this step's
//     right-hand sides g from it with the coupling taps of the period-cell
//     table.  The previous step's values are gathered into LDS for the
//     workgroup's rows and a halo of one slice line on each side, which covers
//     every coupling tap.
//   k_cm_mm: the product W_i g on v_mfma_f32_32x32x2f32: workgroup = 128 rows
//     x 64 members x one K chunk of 8 NK rows of W_i.  W_i comes straight from
//     memory into the A operand: a lane loads 4 consecutive entries of its row
//     k of W_i (W_i is symmetric, so its rows are the columns of the operand)
//     and they feed four 32-row tiles, whose rows interleave; each wave takes a
//     quarter of the chunk, with all of its loads in flight at once, and the
//     four sums are added through LDS, in FP64.  NK (9, 18 or 34) is the largest that
//     leaves about a workgroup per CU: the launch is a stream of W_i (26 MB a
//     step for three classes of b = 1085, two chains).
// One more launch finishes the outermost slices.  The right-hand sides are
// formed and the partials (sums of at most 72 products) added and kept in FP64;
// W_i, g and the products are FP32 (FP32 accumulation on the matrix cores).  W_i
// staged through LDS in chunks of 72 rows took 14.8 us a step (1.8 TB/s) and the
// right-hand sides 6.9; streamed, on 16-wide tiles, which 14 members fill, 8.4 us (3.1
// TB/s; on 32-wide ones 10.2), and with a quarter of the partials and one descriptor
// load 4.3 us.
#include "k_common.h"

namespace ddeig {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(2 * sizeof(double)))) double f64x2;

constexpr int kCmRows = 128;    // output rows per product workgroup
constexpr int kCmMembers = 64;  // members per job: two 32-wide MFMA tiles per wave
constexpr int kCmRb = 256;      // rows per right-hand-side workgroup
constexpr int kCmHalo = 256;    // largest halo (one slice line + 1) of the rhs kernel
constexpr int kCmMaxB = 2304;   // largest slice
constexpr int kCmMaxKc = 18;    // most K chunks (of 72, up to slices of 1280: cm_nk)
constexpr int kCmPad = 272;     // the longest K chunk: G rows end in as many zeros
constexpr int kCmLdr = kCmRows + 4;  // LDS row of a member's partial sums

// What the step kernels read of a job and of one of its members, in one load.
struct CmJob {
  const float* W;  // factors of the class, rows of ldw values
  int b, ldw, nch, dir, nm, slot0;
};
struct CmMember {
  double *batch, *tbatch;  // this member's nch b values
  int b, nch, m0, m1, o[3], dir;
};

// FP64 factors (rows of b values) -> FP32 rows of ldw values, zero padded.
__global__ void k_pad_float(const double* __restrict__ src, float* __restrict__ dst, long rows,
                            int b, int ldw) {
  const long tot = rows * ldw;
  for (long idx = blockIdx.x * (long)blockDim.x + threadIdx.x; idx < tot;
       idx += (long)gridDim.x * blockDim.x) {
    const long r = idx / ldw;
    const int c = (int)(idx - r * ldw);
    dst[idx] = c < b ? (float)src[r * b + c] : 0.0f;
  }
}

void launch_pad_float(const double* src, float* dst, long rows, int b, int ldw, hipStream_t s) {
  const long tot = rows * ldw;
  const int blocks = (int)std::min<long>((tot + kBlock - 1) / kBlock, 8192);
  if (blocks > 0)
    hipLaunchKernelGGL(k_pad_float, dim3(blocks), dim3(kBlock), 0, s, src, dst, rows, b, ldw);
}

int chain_mfma_members() { return kCmMembers; }

bool chain_mfma_ok(int b, int m0) {
  return m0 + 1 <= kCmHalo && b >= 1 && b <= kCmMaxB;
}

// Previous step's value of row r of a member (slot): the sum of the nkc K-chunk
// partials of its class (at most MAXK) in chunk order, subtracted from t (sub !=
// nullptr).  Every load is issued before the first add (clamped addresses,
// masked values), so their latencies overlap; MAXK (the batch's largest chunk
// count rounded up) bounds the loads.
template <int MAXK>
__device__ inline double cm_prev(const double* __restrict__ part, int nkc, int mtot, int bmax,
                                 int slot, int r, const double* sub) {
  double v[MAXK];
#pragma unroll
  for (int kc = 0; kc < MAXK; ++kc)
    v[kc] = part[((long)min(kc, nkc - 1) * mtot + slot) * bmax + r];
  double acc = 0.0;
#pragma unroll
  for (int kc = 0; kc < MAXK; ++kc)
    if (kc < nkc) acc += v[kc];
  return sub != nullptr ? *sub - acc : acc;
}

// The parts of a solve: inwards step k, the middle, outwards step k.
enum { kCmIn = 0, kCmMid = 1, kCmOut = 2 };

// Slice of a job in step k of a part, or -1 when its chain has none.
__device__ __forceinline__ int cm_slice(int mode, int k, int n, int dir) {
  const int h = n / 2;
  if (mode == kCmMid) return dir ? -1 : h;
  if (mode == kCmIn) {
    const int i = dir ? n - 1 - k : k;
    return (dir ? i > h : i < h) ? i : -1;
  }
  const int i = dir ? h + 1 + k : h - 1 - k;
  return i >= 0 && i < n ? i : -1;
}

// The slot (a subdomain's chain) of a workgroup: numbered along y, and on along z
// past the 65535 that y has room for (32768 subdomains and more).
constexpr int kCmMaxY = 65535;
__device__ __forceinline__ int cm_slot() { return blockIdx.y + kCmMaxY * blockIdx.z; }
static dim3 cm_grid(int blocks, int mtot) {
  return dim3(blocks, std::min(mtot, kCmMaxY), (mtot + kCmMaxY - 1) / kCmMaxY);
}

// Right-hand sides of a step.  Grid: (row blocks, slots).  The values of the
// neighbouring slice j are t_j inwards (into tbatch), and x_j = t_j - partials
// outwards (into batch; x_h, the middle's product, is the neighbour of both
// chains' first outward step and stored by the upper one).
template <int MODE, int MAXK>
__global__ void __launch_bounds__(kBlock) k_cm_rhs(Geo g, const double* __restrict__ T,
                                                   const CmMember* __restrict__ mem, int k, int kc,
                                                   int mtot, int pstr, int gstr,
                                                   const double* __restrict__ part,
                                                   float* __restrict__ G,
                                                   const PcgState* __restrict__ st) {
  constexpr int NP = kCmRb + 2 * kCmHalo;
  constexpr int NS = MODE == kCmMid ? 2 : 1;  // neighbours
  __shared__ double prev[NS][NP];
  const int slot = cm_slot(), half = mtot / 2;  // (lower chains: + half)
  if (slot >= mtot) return;
  const CmMember md = mem[slot];
  if (st != nullptr && st->done) return;
  const int b = md.b, nch = md.nch;
  const int i = cm_slice(MODE, k, nch, md.dir);
  const int R0 = blockIdx.x * kCmRb;
  if (i < 0 || R0 >= b) return;
  const int nkc = (b + kc - 1) / kc;
  const int m0 = md.m0, m1 = md.m1;
  const int H = m0 + 1;
  // d2 of each neighbour and whether there is one
  const int d2s[2] = {MODE == kCmMid ? -1 : ((MODE == kCmIn) == (md.dir == 0) ? -1 : 1), 1};
  const bool on[2] = {MODE == kCmMid ? i > 0 : (MODE == kCmOut || k > 0), i + 1 < nch};
  // this thread's couplings and b_i, loaded before the neighbour is gathered
  const int r = R0 + threadIdx.x;
  const int rc = min(r, b - 1), u1 = rc / m0, u0 = rc - u1 * m0;
  const long tn = table_node(g, md.o[0] + u0, md.o[1] + u1, md.o[2] + i);
  double c[NS][9];
#pragma unroll
  for (int sd = 0; sd < NS; ++sd)
#pragma unroll
    for (int t = 0; t < 9; ++t) c[sd][t] = T[(t + 9 * (d2s[sd] + 1)) * g.tsize + tn];
  double acc = MODE == kCmOut ? 0.0 : md.batch[(long)i * b + rc];
  const int lo = max(R0 - H, 0), hi = min(R0 + kCmRb + H, b);
#pragma unroll
  for (int sd = 0; sd < NS; ++sd) {
    if (!on[sd]) continue;
    const int j = i + d2s[sd];
    const bool mid = MODE == kCmOut && k == 0;  // the neighbour is slice h
    const int ps = MODE == kCmMid ? slot + sd * half : (mid && md.dir ? slot - half : slot);
    for (int q = lo + threadIdx.x; q < hi; q += kBlock) {
      double v;
      if (MODE != kCmOut || mid) {
        v = cm_prev<MAXK>(part, nkc, mtot, pstr, ps, q, nullptr);
      } else {
        const double t = md.tbatch[(long)j * b + q];
        v = cm_prev<MAXK>(part, nkc, mtot, pstr, ps, q, &t);
      }
      prev[sd][q - (R0 - H)] = v;
      if (q >= R0 && q < R0 + kCmRb && !(mid && md.dir))
        (MODE == kCmOut ? md.batch : md.tbatch)[(long)j * b + q] = v;
    }
  }
  __syncthreads();
  if (r >= b) return;
#pragma unroll
  for (int sd = 0; sd < NS; ++sd) {
    if (!on[sd]) continue;
    double s = 0.0;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int w0 = u0 + t % 3 - 1, w1 = u1 + t / 3 - 1;
      if (w0 < 0 || w0 >= m0 || w1 < 0 || w1 >= m1) continue;
      s += c[sd][t] * prev[sd][w0 + m0 * w1 - (R0 - H)];
    }
    acc += MODE == kCmOut ? s : -s;
  }
  G[(long)slot * gstr + r] = (float)acc;
}

// Four rows' sums of the four waves (rows at .. at + 3; the waves' sums lie stride
// apart), FP32 sums of at most 72 products each, added in FP64 and kept so: a chunk's
// partial in FP32 would hold up to 272 products.
__device__ __forceinline__ void cm_add4(const float* red, int stride, int at, double* out) {
  double v[4] = {};
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const f32x4 w = *reinterpret_cast<const f32x4*>(&red[p * stride + at]);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += (double)w[e];
  }
  reinterpret_cast<f64x2*>(out)[0] = f64x2{v[0], v[1]};
  reinterpret_cast<f64x2*>(out)[1] = f64x2{v[2], v[3]};
}

// Partial product of a step: rows [R0, R0 + 128) x the job's members x K chunk
// [K0, K0 + 8 NK) of W_i g, into part[chunk][slot][row].  The half-wave kh of
// wave w takes k = K0 + (2 w + kh) NK + q, q < NK.
template <int NK>
__global__ void __launch_bounds__(kBlock) k_cm_mm(const CmJob* __restrict__ jobs, int mode, int k,
                                                  int mtot, int pstr, int gstr,
                                                  const float* __restrict__ G,
                                                  double* __restrict__ part,
                                                  const PcgState* __restrict__ st) {
  __shared__ __attribute__((aligned(16))) float red[4][32 * kCmLdr];
  const CmJob jb = jobs[blockIdx.z];
  if (st != nullptr && st->done) return;
  const int b = jb.b, ldw = jb.ldw;
  const int R0 = blockIdx.x * kCmRows, K0 = blockIdx.y * (8 * NK);
  const int i = cm_slice(mode, k, jb.nch, jb.dir);
  if (i < 0 || R0 >= b || K0 >= b) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int kh = lane >> 5, l32 = lane & 31;
  const int kb = K0 + (2 * w + kh) * NK;
  // rows of W_i past b read as zero (the resource ends with the slice); columns
  // past ldw are other rows' entries and end in output rows that are not stored
  const auto rw = __builtin_amdgcn_make_buffer_rsrc((void*)(jb.W + (long)i * b * ldw), (short)0,
                                                    b * ldw * 4, 0x00020000);
  f32x4 wv[NK];
#pragma unroll
  for (int q = 0; q < NK; ++q)
    wv[q] = __builtin_bit_cast(
        f32x4, __builtin_amdgcn_raw_buffer_load_b128(rw, ((kb + q) * ldw + R0 + 4 * l32) * 4, 0, 0));
  for (int mt = 0; mt < jb.nm; mt += 32) {
    // g of member mt + l32 (a lane without one repeats the last; its column of
    // the product is not stored); rows past b hold zeros
    const float* gp = G + (long)(jb.slot0 + min(mt + l32, jb.nm - 1)) * gstr + kb;
    typedef __attribute__((address_space(1))) const float* gptr;
    float gv[NK];
#pragma unroll
    for (int q = 0; q < NK; ++q) gv[q] = ((gptr)gp)[q];
    f32x16 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[t][e] = 0.0f;
#pragma unroll
    for (int q = 0; q < NK; ++q)
#pragma unroll
      for (int t = 0; t < 4; ++t)
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv[q][t], gv[q], acc[t], 0, 0, 0);
    // accumulator layout: lane l, element e holds A row 8 (e / 4) + 4 (l / 32) +
    // e % 4, which is row 4 of that + t of the workgroup, and member l % 32
    if (mt > 0) __syncthreads();
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int row = 8 * (e >> 2) + 4 * kh + (e & 3);
      *reinterpret_cast<f32x4*>(&red[w][l32 * kCmLdr + 4 * row]) =
          f32x4{acc[0][e], acc[1][e], acc[2][e], acc[3][e]};
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 32 * kCmRows / 4 / kBlock; ++q) {
      const int idx = tid + q * kBlock, j = idx / (kCmRows / 4), c4 = 4 * (idx % (kCmRows / 4));
      if (mt + j >= jb.nm || R0 + c4 >= pstr) continue;
      cm_add4(red[0], 32 * kCmLdr, j * kCmLdr + c4,
              &part[((long)blockIdx.y * mtot + jb.slot0 + mt + j) * pstr + R0 + c4]);
    }
  }
}

// The same product for jobs of at most 16 members, on v_mfma_f32_16x16x4f32
// (half the matrix instructions' time: a wave's share at NK = 34 is 3.6 us on
// 32-wide tiles).  Quarter-wave kq of wave w takes k = K0 + (4 w + kq) NQ + q,
// q < NQ = NK / 2; a lane's two loads of a row feed 16-row tiles (h, t) whose
// row m is row 64 h + 4 m + t of the workgroup.
template <int NK>
__global__ void __launch_bounds__(kBlock) k_cm_mm16(const CmJob* __restrict__ jobs, int mode, int k,
                                                    int mtot, int pstr, int gstr,
                                                    const float* __restrict__ G,
                                                    double* __restrict__ part,
                                                    const PcgState* __restrict__ st) {
  static_assert(NK % 2 == 0, "whole quarter-wave shares");
  constexpr int NQ = NK / 2;
  __shared__ __attribute__((aligned(16))) float red[4][16 * kCmLdr];
  const CmJob jb = jobs[blockIdx.z];
  if (st != nullptr && st->done) return;
  const int b = jb.b, ldw = jb.ldw;
  const int R0 = blockIdx.x * kCmRows, K0 = blockIdx.y * (8 * NK);
  const int i = cm_slice(mode, k, jb.nch, jb.dir);
  if (i < 0 || R0 >= b || K0 >= b) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int kq = lane >> 4, l16 = lane & 15;
  const int kb = K0 + (4 * w + kq) * NQ;
  const auto rw = __builtin_amdgcn_make_buffer_rsrc((void*)(jb.W + (long)i * b * ldw), (short)0,
                                                    b * ldw * 4, 0x00020000);
  f32x4 wv[NQ][2];
#pragma unroll
  for (int q = 0; q < NQ; ++q)
#pragma unroll
    for (int h = 0; h < 2; ++h)
      wv[q][h] = __builtin_bit_cast(
          f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                     rw, ((kb + q) * ldw + R0 + 64 * h + 4 * l16) * 4, 0, 0));
  typedef __attribute__((address_space(1))) const float* gptr;
  const float* gp = G + (long)(jb.slot0 + min(l16, jb.nm - 1)) * gstr + kb;
  float gv[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) gv[q] = ((gptr)gp)[q];
  __builtin_amdgcn_sched_barrier(0);  // every load issued before the first product
  f32x4 acc[2][4];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[h][t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int q = 0; q < NQ; ++q)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int t = 0; t < 4; ++t)
        acc[h][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[q][h][t], gv[q], acc[h][t], 0, 0, 0);
  // accumulator layout: lane l, element e holds tile row 4 (l / 16) + e, member l % 16
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      *reinterpret_cast<f32x4*>(&red[w][l16 * kCmLdr + 64 * h + 4 * (4 * kq + e)]) =
          f32x4{acc[h][0][e], acc[h][1][e], acc[h][2][e], acc[h][3][e]};
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 16 * kCmRows / 4 / kBlock; ++q) {
    const int idx = tid + q * kBlock, j = idx / (kCmRows / 4), c4 = 4 * (idx % (kCmRows / 4));
    if (j >= jb.nm || R0 + c4 >= pstr) continue;
    cm_add4(red[0], 16 * kCmLdr, j * kCmLdr + c4,
            &part[((long)blockIdx.y * mtot + jb.slot0 + j) * pstr + R0 + c4]);
  }
}

// The outermost slice of every chain: x = t - (partials), or x_0 = (partials)
// for a chain of one slice.  Grid: (row blocks, slots).
template <int MAXK>
__global__ void __launch_bounds__(kBlock) k_cm_fin(const CmMember* __restrict__ mem, int kc,
                                                   int mtot, int pstr,
                                                   const double* __restrict__ part,
                                                   const PcgState* __restrict__ st) {
  const int slot = cm_slot();
  if (slot >= mtot) return;
  const CmMember md = mem[slot];
  if (st != nullptr && st->done) return;
  const int b = md.b, h = md.nch / 2;
  if (md.dir && h + 1 >= md.nch) return;  // no lower chain
  const int nkc = (b + kc - 1) / kc;
  const int r = blockIdx.x * kBlock + threadIdx.x;
  if (r >= b) return;
  const long at = (long)(md.dir ? md.nch - 1 : 0) * b + r;
  if (md.nch == 1) {
    md.batch[at] = cm_prev<MAXK>(part, nkc, mtot, pstr, slot, r, nullptr);
  } else {
    const double t = md.tbatch[at];
    md.batch[at] = cm_prev<MAXK>(part, nkc, mtot, pstr, slot, r, &t);
  }
}

// Strides and sizes: partial rows of whole groups of four, G rows of b values and the
// zeros that a last K chunk reads.
static int cm_pstr(int bmax) { return (bmax + 3) / 4 * 4; }
static int cm_gstr(int bmax) { return bmax + kCmPad; }

// Rows of W_i per half-wave: the largest K chunk (8 NK rows) that leaves about
// three quarters of the CUs a workgroup, so that the partials are few.  An
// application, one level, with NK 34 / 18 / 9 everywhere: two subdomains with slices
// of 1023 unknowns 374 / 348 / 390 us, 20 of 768 358 / 298 / 343, 24 of 621 333 / 277 /
// 284, 16 of 437 220 / 198 / 187 (the rule: 18, 18, 9 and 9).
static int cm_nk(int bmax, int njobs) {
  const int tiles = (bmax + kCmRows - 1) / kCmRows * njobs;
  for (int nk : {34, 18})
    if (tiles * ((bmax + 8 * nk - 1) / (8 * nk)) >= 192) return nk;
  return 9;
}

// The members' and jobs' descriptors, the partial buffer and G (zeros behind
// every row of G).
size_t chain_mfma_bytes(int bmax, int mtot, int njobs, size_t* job_off, size_t* part_off) {
  size_t off = (size_t)mtot * sizeof(CmMember);
  *job_off = off;
  off += (size_t)njobs * sizeof(CmJob);
  off = (off + 255) / 256 * 256;
  *part_off = off;
  const int nk = cm_nk(bmax, njobs), nkc = (bmax + 8 * nk - 1) / (8 * nk);
  return off + (size_t)nkc * mtot * cm_pstr(bmax) * sizeof(double) +
         (size_t)mtot * cm_gstr(bmax) * sizeof(float);
}

// Fills the descriptors at the head of the chain buffer and clears G behind the
// partials.
void chain_mfma_setup(ddeig_problem* P, const std::vector<TypeDev>& types,
                      const std::vector<ChainJob>& jobs, hipStream_t s) {
  std::vector<CmJob> cj;
  std::vector<CmMember> cm(P->chain_mtot);
  P->chain_nm = 0;
  for (const ChainJob& j : jobs) {
    const TypeDev& t = types[j.type];
    P->chain_nm = std::max(P->chain_nm, j.nm);
    cj.push_back(CmJob{t.W32, t.b, t.ldw, t.nch, j.dir, j.nm, j.mg0});
    for (int m = 0; m < j.nm; ++m) {
      const long at = (long)(j.m0 + m) * t.nch * t.b;
      cm[j.mg0 + m] = CmMember{t.batch + at, t.tbatch + at, t.b, t.nch, t.m[0], t.m[1],
                               {t.o[0], t.o[1], t.o[2]}, j.dir};
    }
  }
  size_t joff, poff;
  const size_t bytes =
      chain_mfma_bytes(P->chain_bmax, P->chain_mtot, (int)jobs.size(), &joff, &poff);
  unsigned char* base = static_cast<unsigned char*>(P->chain_part);
  check_hip(hipMemcpyAsync(base, cm.data(), sizeof(CmMember) * cm.size(), hipMemcpyHostToDevice, s),
            "copy chain members");
  check_hip(hipMemcpyAsync(base + joff, cj.data(), sizeof(CmJob) * cj.size(), hipMemcpyHostToDevice,
                           s), "copy chain jobs");
  const size_t gbytes = (size_t)P->chain_mtot * cm_gstr(P->chain_bmax) * sizeof(float);
  check_hip(hipMemsetAsync(base + bytes - gbytes, 0, gbytes, s), "clear right-hand sides");
  check_hip(hipStreamSynchronize(s), "chain descriptors");
}

template <int NK, int MAXK>
static void cm_solve(const ddeig_problem* P, const PcgState* st, hipStream_t s) {
  const int nch = P->types[0].box.nch, h = nch / 2;
  const int bmax = P->chain_bmax, mtot = P->chain_mtot, njobs = P->nchainjobs;
  constexpr int kc = 8 * NK;
  const int nkc = (bmax + kc - 1) / kc, pstr = cm_pstr(bmax), gstr = cm_gstr(bmax);
  size_t joff, poff;
  chain_mfma_bytes(bmax, mtot, njobs, &joff, &poff);
  unsigned char* base = static_cast<unsigned char*>(P->chain_part);
  const CmMember* mem = reinterpret_cast<const CmMember*>(base);
  const CmJob* jobs = reinterpret_cast<const CmJob*>(base + joff);
  double* part = reinterpret_cast<double*>(base + poff);
  float* G = reinterpret_cast<float*>(part + (long)nkc * mtot * pstr);
  const dim3 grow = cm_grid((bmax + kCmRb - 1) / kCmRb, mtot);
  constexpr int kMaxZ = 65535;  // jobs of a product launch (grid z)
  auto mm = k_cm_mm<NK>;
  if constexpr (NK % 2 == 0)
    if (P->chain_nm <= 16) mm = k_cm_mm16<NK>;
  auto step = [&](int mode, int k, auto rhs) {
    hipLaunchKernelGGL(rhs, grow, dim3(kBlock), 0, s, P->g, P->tabAs, mem, k, kc, mtot, pstr, gstr,
                       part, G, st);
    for (int j0 = 0; j0 < njobs; j0 += kMaxZ)
      hipLaunchKernelGGL(mm, dim3((bmax + kCmRows - 1) / kCmRows, nkc, std::min(njobs - j0, kMaxZ)),
                         dim3(kBlock), 0, s, jobs + j0, mode, k, mtot, pstr, gstr, G, part, st);
  };
  for (int k = 0; k < h; ++k) step(kCmIn, k, k_cm_rhs<kCmIn, MAXK>);
  step(kCmMid, 0, k_cm_rhs<kCmMid, MAXK>);
  for (int k = 0; k < h; ++k) step(kCmOut, k, k_cm_rhs<kCmOut, MAXK>);
  hipLaunchKernelGGL(k_cm_fin<MAXK>, grow, dim3(kBlock), 0, s, mem, kc, mtot, pstr, part, st);
}

// The solves of every class (all classes share nch).
void launch_chain_mfma(const ddeig_problem* P, const PcgState* st, hipStream_t s) {
  const int nk = cm_nk(P->chain_bmax, P->nchainjobs);
  const int nkc = (P->chain_bmax + 8 * nk - 1) / (8 * nk);
  if (nk == 34) nkc <= 4 ? cm_solve<34, 4>(P, st, s) : cm_solve<34, 9>(P, st, s);
  else if (nk == 18) nkc <= 8 ? cm_solve<18, 8>(P, st, s) : cm_solve<18, 16>(P, st, s);
  else nkc <= 8 ? cm_solve<9, 8>(P, st, s) : nkc <= 16 ? cm_solve<9, 16>(P, st, s)
                                                       : cm_solve<9, kCmMaxKc>(P, st, s);
}

}  // namespace ddeig
