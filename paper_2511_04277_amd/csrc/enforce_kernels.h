// Enforcement kernels (thesis Sec. 3.5.5) shared by the single-instance and
// batched entry points.  See enforce.hip for the algorithm.
#pragma once

#include <algorithm>
#include <atomic>
#include <cstdlib>

#include "common.h"

namespace rad {
namespace {

constexpr int ET = 64;          // tile edge (doubles)
constexpr int ETP = ET + 1;     // padded LDS row (conflict-free transpose)
// 8 waves of 8 tile rows each: at 4 waves per SIMD (two workgroups per
// CU) the sweep keeps twice the loads in flight of a 4-wave shape
constexpr int ENF_THREADS = 512;
constexpr int ENW = ENF_THREADS / 64;  // waves per sweep workgroup

struct EnfCtrl {
  int status;        // device-raised status (0 ok, negative error)
  int converged;     // 1 once the tolerance is met
  int iters;         // iterations executed
  int done;          // finalize blocks of the current iteration that finished
  double last_defect, last_recip;
};


// What the workgroups of the resident kernel exchange, in words: row sums
// (two iterations in turn x row block x column block x 64), closure scales and
// row blocks' states (four iterations in turn), then three maxima, a counter and
// the verdict.
constexpr int ENF_RES_TILES = 31;  // most 64-row blocks of a resident model: 496 tile pairs
// Workgroups of a resident kernel on a CU, and the waves per SIMD that its
// registers are held to (72 each).  All its workgroups have to find a place
// beside whatever other streams run, and the waves that are placed first stay
// where they were put, between waves that end: registers (512 a SIMD) and LDS
// come in contiguous pieces of 8 and 1280, so what is free may be in holes.
// A workgroup's two waves on a SIMD fit beside any one other of its kind: three
// waves with a hole of less than 72 on either side of each are 3 x 72 + 4 x 64 =
// 472 < 512 (with 80 registers 3 x 80 + 4 x 72 = 528: not so), and 38 KB of LDS
// beside another 38 KB anywhere in 160.  A third does not: a CU that ran two
// workgroups of 152 registers and 70 KB (gemm_lds32 in FP64) keeps two, and a
// grid that needs a third on some CUs then waits for ever.
constexpr int ENF_RES_PER_CU = 2;
constexpr int ENF_RES_WAVES = 7;
// One iteration is streamed: it saves nothing that would pay for the exchange's
// set-up.  84 faces, one and two iterations: 22 and 33 us streamed, 23 and 28 on
// chip; 1984 faces: 38 and 57, 46 and 56.  A batch's groups are launched one after
// another, and four more of them take an iteration more to win (16 models in five
// groups, two and three iterations: 164 and 225 us streamed, 183 and 220 on chip).
constexpr int ENF_RES_ITERS = 2;
// Polls (about a microsecond each) until a waiting wave gives up.
constexpr int ENF_PATIENCE = 1 << 20;
typedef unsigned long long EnfWord;
__host__ __device__ constexpr long enf_xch_words(long t) { return 2 * t * t * ET + 4 * t * ET + 4 * t + 5; }

// One enforcement problem as the kernels see it.
struct EnfInst {
  double* F;
  long ldf;
  int n, t;                 // faces, 64-wide tiles per side
  long pairs;               // t (t + 1) / 2 tile pairs
  const double* area;
  const double* inv_area;   // 1 / A_i (workspace)
  const double* nrays;      // null for kappa = 1/2
  int mode;
  int nt;                   // sweeps use nontemporal accesses
  double* scale;            // 1 / s_i of the last closure step
  double* partial;          // (t + 1) x n partial row sums
  double* blkmax;           // 2 per tile pair: max |eta_ij - eta_ji|, max eta
  double* finred;           // 3 per finalize block: closure defect, the two maxima
  EnfCtrl* ctrl;
  EnfWord* xch;             // resident kernel only: enf_xch_words(t)
  int patience;             // and how often a wave asks for a word before it gives up
};

constexpr int ERW = ET / ENW;  // tile rows per wave
static_assert(2 + 2 * ENW <= ET, "the row partials and maxima reuse rows of the tile buffer");

// Element col of a row whose base pointer is wave-uniform: the byte offset
// is a 32-bit lane value, so loads and stores take the scalar-base form and
// one offset register serves every row.
// (readfirstlane pins the row pointer to scalar registers, so the compiler
// cannot fold the lane offset into a per-row vector address).
// The pointer is rebuilt in the global address space: a generic (flat)
// pointer would make every access a flat instruction with a 64-bit address
// per lane, which costs two registers per load in flight.
typedef __attribute__((address_space(1))) char gchar;
typedef __attribute__((address_space(1))) double gdouble;
__device__ __forceinline__ gchar* uniform_ptr(const double* p) {
  const unsigned long long v = reinterpret_cast<unsigned long long>(p);
  const unsigned lo = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(v));
  const unsigned hi = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(v >> 32));
  return reinterpret_cast<gchar*>((static_cast<unsigned long long>(hi) << 32) | lo);
}
// NT: nontemporal, past the last-level cache (see enf_nontemporal).
template <bool NT = true>
__device__ __forceinline__ double row_ld(const double* row, unsigned col) {
  const gdouble* p = reinterpret_cast<const gdouble*>(uniform_ptr(row) + col * 8u);
  return NT ? __builtin_nontemporal_load(p) : *p;
}
template <bool NT = true>
__device__ __forceinline__ void row_st(double* row, unsigned col, double v) {
  gdouble* p = reinterpret_cast<gdouble*>(uniform_ptr(row) + col * 8u);
  if (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// Whether sweeps over matrices of bytes in total go past the last-level cache
// (256 MB).  Up to about its size F stays there between sweeps: 105 -> 85 us an
// iteration at n = 5200 (216 MB, rows on 128-byte lines), 68 -> 59 us at 4048.
// Rows off the 128-byte lines share a line between two tiles, which
// nontemporal accesses fetch and write twice: 704 -> 615 us at n = 12288 and
// 320 -> 268 us at 8192 without them.  Aligned and larger, they win: 238 us
// against 252 at 8192, 523 against 546 at 12288.
inline bool enf_nontemporal(const double* F, long ldf, double bytes) {
  return reinterpret_cast<uintptr_t>(F) % 128 == 0 && ldf % 16 == 0 && bytes > 256.0e6;
}

// kappa of eq. 3.25 from the pair (f_ij, f_ji) and c = A^2 / N of both faces:
// kappa = b / (a + b), a = c_i (1 - f_ij) f_ji, b = c_j (1 - f_ji) f_ij (the
// variances of eq. 3.23 multiplied by F_ij F_ji); 1/2 when both vanish.
// The quotient uses the hardware reciprocal refined by two Newton steps.
// Every operation rounds as written (no contraction into fused multiply-adds
// beyond the two explicit Newton steps), so the result does not depend on how
// the compiler schedules the surrounding code.
__device__ __forceinline__ double kappa_c(double fij, double fji, double ci, double cj) {
#pragma clang fp contract(off)
  const double a = ci * (1.0 - fij) * fji;
  const double b = cj * (1.0 - fji) * fij;
  const double s = a + b;
  double r = __builtin_amdgcn_rcp(s);
  r = r * __builtin_fma(-s, r, 2.0);
  r = r * __builtin_fma(-s, r, 2.0);
  return s > 0.0 ? b * r : 0.5;
}

// This thread's lane, formed anew: what is made from it stays out of registers
// until it is needed (made from threadIdx it would be hoisted out of a loop).
__device__ __forceinline__ int fresh_lane() {
  unsigned z = 0;
  __asm__ volatile("" : "+v"(z));
  return static_cast<int>(__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, z)));
}

// One iteration of a tile pair held in registers: own tile (I, J) in a, partner
// tile (J, I) in b (see enf_sweep_tile); rowc holds the rows' constants and the
// previous closure scale.  put() is called once the new own tile is in a and
// the new partner tile in sB; sums() in wave 0 at the end, with the sums of
// own row l and of partner row l in lane l and the pair's maxima in lane 0.
// WIDE: registers to spare, so the pairs of a thread are computed side by side
// (their chains of dependent operations bind a workgroup alone on its CU).
// MAXIMA: the workgroup's maxima go to sums; otherwise rmax and emax are left
// per thread.
template <bool DIAG, bool EDGE, bool HALF, bool WIDE, bool MAXIMA, class Put, class Sums>
__device__ __forceinline__ void enf_pair_step(const EnfInst& in, int I, int J, int w, double (&a)[ERW],
                                              const double (&b)[ERW], double (*sB)[ETP], double (*rowc)[ET], int& bad,
                                              double& rmax, double& emax, Put put, Sums sums) {
#pragma clang fp contract(off)
  const int n = in.n;
  const bool half = HALF;
  const int r0 = I * ET, c0 = J * ET;
  const int l = WIDE || MAXIMA ? threadIdx.x & 63 : fresh_lane();
  const int jg = c0 + l;
  const int ig = r0 + l;
  // scaled by the positive finite 1 / s (1 on the first sweep); negative or
  // non-finite inputs stay so and are caught where the pair is formed
#pragma unroll
  for (int k = 0; k < ERW; ++k) {
    const int i = r0 + w + ENW * k;
    double v = a[k];
    if (EDGE && !(i < n && jg < n)) v = 0.0;
    a[k] = v * rowc[3][w + ENW * k];
  }
  // partner tile into LDS: sB[jl][il] = F(c0 + jl, r0 + il)
  if (!DIAG) {
#pragma unroll
    for (int k = 0; k < ERW; ++k) {
      const int jr = c0 + w + ENW * k;
      double v = b[k];
      if (EDGE && !(jr < n && ig < n)) v = 0.0;
      sB[w + ENW * k][l] = v * rowc[7][w + ENW * k];
    }
  } else {
#pragma unroll
    for (int k = 0; k < ERW; ++k) sB[w + ENW * k][l] = a[k];
  }
  __syncthreads();

  // reciprocity on each unordered pair {i, j}, i != j, exactly once
  double sb = 0.0;
  rmax = emax = 0.0;
  // constants of row c0 + l (the partner's row; on a diagonal tile the own rows)
  double aj = rowc[DIAG ? 0 : 4][l], iaj = rowc[DIAG ? 1 : 5][l];
  double cj = rowc[DIAG ? 2 : 6][l];
#pragma unroll
  for (int k = 0; k < ERW; ++k) {
    const int il = w + ENW * k;
    if (!WIDE && !MAXIMA) {  // read for every pair: no registers to keep them
      const int lj = fresh_lane();
      aj = rowc[DIAG ? 0 : 4][lj];
      iaj = rowc[DIAG ? 1 : 5][lj];
      cj = rowc[DIAG ? 2 : 6][lj];
    }
    const double ai = rowc[0][il];
    if (DIAG) {
      if (l == il) {                               // the diagonal keeps its value
        emax = fmax(emax, ai * a[k]);
        bad |= !(a[k] >= 0.0) || !(a[k] <= 1.0e300);
      }
      if (l <= il) continue;                       // handled by the owner of (l, il)
    }
    const double iai = rowc[1][il];
    const double fij = a[k], fji = sB[l][il];
    bad |= !(fij >= 0.0) || !(fij <= 1.0e300) || !(fji >= 0.0) || !(fji <= 1.0e300);
    const double eij = ai * fij, eji = aj * fji;
    rmax = fmax(rmax, fabs(eij - eji));
    emax = fmax(emax, fmax(eij, eji));
    const double kp = half ? 0.5 : kappa_c(fij, fji, rowc[2][il], cj);
    const double eh = kp * eij + (1.0 - kp) * eji;
    const double bji = eh * iaj;
    a[k] = eh * iai;
    sB[l][il] = bji;
    sb += bji;
    // fold this pair into the running maxima and the error flag now: left to
    // itself the compiler keeps every pair's terms live and reduces them as a
    // tree after the loop, which doubles the registers of the kernel
    if (!WIDE) __asm__ volatile("" : "+v"(rmax), "+v"(emax), "+v"(bad), "+v"(sb));
  }
  __syncthreads();
  if (DIAG) {
#pragma unroll
    for (int k = 0; k < ERW; ++k)
      if (l < w + ENW * k) a[k] = sB[w + ENW * k][l];  // written by the owner of the mirror
  }

  put();
  __syncthreads();
  // own tile transposed into LDS, then each thread sums ERW entries of row l
#pragma unroll
  for (int k = 0; k < ERW; ++k) sB[l][w + ENW * k] = a[k];
  if constexpr (MAXIMA)
    for (int off = 32; off > 0; off >>= 1) {
      rmax = fmax(rmax, __shfl_xor(rmax, off));
      emax = fmax(emax, __shfl_xor(emax, off));
    }
  __syncthreads();
  double sa = 0.0;
#pragma unroll
  for (int k = 0; k < ERW; ++k) sa += sB[w + ENW * k][l];
  __syncthreads();
  // the transposed tile has been summed: LDS rows 2.. take this wave's
  // partial sums of the partner's row l and of the own row l, rows 0 and 1
  // the wave maxima
  sB[2 + w][l] = sb;
  sB[2 + ENW + w][l] = sa;
  if (MAXIMA && l == 0) {
    sB[0][w] = rmax;
    sB[1][w] = emax;
  }
  __syncthreads();
  if (w == 0) {
    double s_own = 0.0, s_par = 0.0;
#pragma unroll
    for (int q = 0; q < ENW; ++q) {
      s_own += sB[2 + ENW + q][l];
      s_par += sB[2 + q][l];
    }
    if constexpr (MAXIMA) {
      double x = 0.0, y = 0.0;
      if (l == 0) {
        x = sB[0][0];
        y = sB[1][0];
        for (int q = 1; q < ENW; ++q) {
          x = fmax(x, sB[0][q]);
          y = fmax(y, sB[1][q]);
        }
      }
      sums(s_own, s_par, x, y);
    } else {
      sums(s_own, s_par);
    }
  }
}

// One workgroup per tile pair (I, J), I <= J, of 64 x 64 tiles.  Lane l of
// wave w holds column l of tile rows w, w + ENW, ..., so every load and
// store instruction of a wave moves one contiguous 512-byte tile row.  The
// partner tile (J, I) is staged through LDS (65-double rows), where each
// unordered pair {i, j} meets its mirror; the previous iteration's closure
// scale 1 / s_i is applied on load.  The thread that updates pair (i, j)
// also produces the partner's entry (j, i), and its ERW pairs all lie in one
// partner row, so the partner's row sums are formed in registers; the own
// tile's rows are summed after a transpose through the same LDS buffer.
// All sums run in a fixed order (bitwise reproducible).  DIAG: I == J (each
// unordered pair once, the diagonal kept, the space column carried along);
// EDGE: the tile pair crosses n (clamped loads, masked stores).
template <bool DIAG, bool EDGE, bool HALF, bool NT>
__device__ __forceinline__ void enf_sweep_tile(const EnfInst& in, long pair, int I, int J, int first,
                                               double (*sB)[ETP], double (*rowc)[ET]) {
#pragma clang fp contract(off)
  double* __restrict__ F = in.F;
  const long ldf = in.ldf;
  const int n = in.n;
  const double* __restrict__ area = in.area;
  const double* __restrict__ inv_area = in.inv_area;
  const double* __restrict__ nrays = in.nrays;
  const bool half = HALF;
  const double* __restrict__ inv_scale = in.scale;
  const int r0 = I * ET, c0 = J * ET;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
  int bad = 0;

  // The tiles' loads go out first, so that their latency covers the loads
  // of the per-row constants below.  Own tile (I, J): a[k] = F(r0 + w +
  // ENW k, c0 + l); partner tile (J, I): b[k] = F(c0 + w + ENW k, r0 + l).
  // Row pointers are wave-uniform and the lane adds its column, so loads
  // use a scalar base.
  const int jg = c0 + l;
  const int jgc = (EDGE && jg >= n) ? n - 1 : jg;
  const int ig = r0 + l;
  const int igc = (EDGE && ig >= n) ? n - 1 : ig;
  double a[ERW], b[ERW];
#pragma unroll
  for (int k = 0; k < ERW; ++k) {
    const int i = r0 + w + ENW * k;
    const int ic = (EDGE && i >= n) ? n - 1 : i;
    a[k] = row_ld<NT>(F + static_cast<long>(ic) * ldf, jgc);
  }
  if (!DIAG) {
#pragma unroll
    for (int k = 0; k < ERW; ++k) {
      const int jr = c0 + w + ENW * k;
      const int jrc = (EDGE && jr >= n) ? n - 1 : jr;
      b[k] = row_ld<NT>(F + static_cast<long>(jrc) * ldf, igc);
    }
  }
  // per-row constants: area, 1 / area, A^2 / N and the previous closure
  // scale 1 / s of the own tile's rows (rowc[0..3]) and of the partner
  // tile's rows (rowc[4..7])
  if (tid < (DIAG ? ET : 2 * ET)) {
    const int q = tid < ET ? 0 : 4;
    const int base = tid < ET ? r0 : c0;
    const int rl = tid & (ET - 1);
    const int i = (EDGE && base + rl >= n) ? n - 1 : base + rl;
    const double ai = area[i];
    rowc[q + 0][rl] = ai;
    rowc[q + 1][rl] = inv_area[i];
    rowc[q + 2][rl] = half ? 0.0 : ai * ai / nrays[i];
    rowc[q + 3][rl] = first ? 1.0 : inv_scale[i];
  }
  __syncthreads();
  double rmax, emax;
  enf_pair_step<DIAG, EDGE, HALF, false, true>(
      in, I, J, w, a, b, sB, rowc, bad, rmax, emax,
      [&]() {
        // own tile back to F
#pragma unroll
        for (int k = 0; k < ERW; ++k) {
          const int i = r0 + w + ENW * k;
          if (!EDGE || (i < n && jg < n)) row_st<NT>(F + static_cast<long>(i) * ldf, jg, a[k]);
        }
        if (!DIAG) {  // partner tile back to F
#pragma unroll
          for (int k = 0; k < ERW; ++k) {
            const int jr = c0 + w + ENW * k;
            if (!EDGE || (jr < n && ig < n)) row_st<NT>(F + static_cast<long>(jr) * ldf, ig, sB[w + ENW * k][l]);
          }
        }
      },
      [&](double s_own, double s_par, double x, double y) {
        double* __restrict__ partial = in.partial;
        if (!EDGE || r0 + l < n) partial[static_cast<long>(J) * n + r0 + l] = s_own;
        if (!DIAG && (!EDGE || c0 + l < n)) partial[static_cast<long>(I) * n + c0 + l] = s_par;
        if (DIAG && (!EDGE || r0 + l < n)) {  // the space column of the tile's rows rides with the diagonal tile
          double* sp = F + static_cast<long>(r0 + l) * ldf + n;
          double v = *sp;
          bad |= !(v >= 0.0) || !(v <= 1.0e300);
          v *= rowc[3][l];
          *sp = v;
          partial[static_cast<long>(in.t) * n + r0 + l] = v;
        }
        if (l == 0) {
          in.blkmax[2 * pair] = x;
          in.blkmax[2 * pair + 1] = y;
        }
      });
  if (bad) raise_status(&in.ctrl->status, RAD_ENONFINITE);
}

template <bool HALF, bool NT>
__device__ __forceinline__ void enf_sweep_pair(const EnfInst& in, long pair, int I, int J, int first,
                                               double (*sB)[ETP], double (*rowc)[ET]) {
  const bool edge = (J + 1) * ET > in.n;
  if (I == J) {
    if (edge) enf_sweep_tile<true, true, HALF, NT>(in, pair, I, J, first, sB, rowc);
    else enf_sweep_tile<true, false, HALF, NT>(in, pair, I, J, first, sB, rowc);
  } else {
    if (edge) enf_sweep_tile<false, true, HALF, NT>(in, pair, I, J, first, sB, rowc);
    else enf_sweep_tile<false, false, HALF, NT>(in, pair, I, J, first, sB, rowc);
  }
}

__device__ __forceinline__ void enf_sweep_body(const EnfInst& in, long pair, int first) {
  if (in.ctrl->converged || in.ctrl->status < 0) return;
  __shared__ double sB[ET][ETP];
  __shared__ double rowc[8][ET];  // per-row constants of the own and the partner tile
  int I, J;
  pair_from_index(pair, in.t, I, J);
  I = __builtin_amdgcn_readfirstlane(I);  // workgroup-uniform: keeps tile addressing scalar
  J = __builtin_amdgcn_readfirstlane(J);
  if (in.mode == RAD_KAPPA_HALF) {
    if (in.nt) enf_sweep_pair<true, true>(in, pair, I, J, first, sB, rowc);
    else enf_sweep_pair<true, false>(in, pair, I, J, first, sB, rowc);
  } else {
    if (in.nt) enf_sweep_pair<false, true>(in, pair, I, J, first, sB, rowc);
    else enf_sweep_pair<false, false>(in, pair, I, J, first, sB, rowc);
  }
}

// Tile pairs in row order (I, I), (I, I + 1), ...: consecutive pairs share
// the own tiles' rows, so each XCD takes a contiguous range of them and the
// cache lines two neighbouring tiles share meet in one L2.
__global__ void __launch_bounds__(ENF_THREADS, 6) enf_sweep(EnfInst in, int first) {
  enf_sweep_body(in, xcd_contiguous(blockIdx.x, gridDim.x), first);
}

// index of the last entry of start[0..count) that is <= v
__device__ __forceinline__ int find_segment(const long* __restrict__ start, int count, long v) {
  int lo = 0, hi = count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (start[mid] <= v) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Block map of a batched grid: block b works for instance inst on its local
// block local (one load per block instead of a binary search over the
// instance offsets, whose dependent loads delayed every block's start).
struct EnfBlk {
  int inst, local;
};

// all instances of a batch in one grid: map[b] names the instance and its tile pair
__global__ void __launch_bounds__(ENF_THREADS, 6)
enf_sweep_batched(const EnfInst* __restrict__ ins, const EnfBlk* __restrict__ map, int first) {
  const EnfBlk m = map[blockIdx.x];
  enf_sweep_body(ins[m.inst], m.local, first);
}

// finalize blocks (FIN_ROWS rows each), declared ahead of the decide step
constexpr int FIN_LANES = 8;
constexpr int FIN_ROWS = 256 / FIN_LANES;  // rows per 256-thread block

// Iteration count, closure defect, reciprocity error and the stop flag from
// the finalize blocks' maxima, run by the instance's last finalize block.
__device__ __forceinline__ void enf_decide_body(const EnfInst& in, double tol) {
  EnfCtrl* ctrl = in.ctrl;
  const int nf = (in.n + FIN_ROWS - 1) / FIN_ROWS;
  const int status = agent_load(&ctrl->status);
  double d = 0.0, rm = 0.0, em = 0.0;
  for (int b = threadIdx.x; b < nf; b += blockDim.x) {
    d = fmax(d, agent_load(in.finred + 3 * b));
    rm = fmax(rm, agent_load(in.finred + 3 * b + 1));
    em = fmax(em, agent_load(in.finred + 3 * b + 2));
  }
  if (status < 0) return;
  __shared__ double fr[3][4];
  for (int off = 32; off > 0; off >>= 1) {
    d = fmax(d, __shfl_xor(d, off));
    rm = fmax(rm, __shfl_xor(rm, off));
    em = fmax(em, __shfl_xor(em, off));
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    fr[0][w] = d;
    fr[1][w] = rm;
    fr[2][w] = em;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int q = 1; q < 4; ++q) {
      d = fmax(d, fr[0][q]);
      rm = fmax(rm, fr[1][q]);
      em = fmax(em, fr[2][q]);
    }
    d = fmax(d, fr[0][0]);
    rm = fmax(rm, fr[1][0]);
    em = fmax(em, fr[2][0]);
    ctrl->iters += 1;
    ctrl->last_defect = d;
    ctrl->last_recip = em > 0.0 ? rm / em : 0.0;
    if (tol > 0.0 && d <= tol) ctrl->converged = 1;
  }
}

// Row sums s_i of the (t + 1) partials of each row: part p = 0..7 of a row
// sums every 8th partial (q = p, p + 8, ...) in order, then the eight parts
// combine as ((0 + 1) + (2 + 3)) + ((4 + 5) + (6 + 7)) (fixed order).  Thread
// t takes part t / 32 of row t % 32, so each load instruction of a wave reads
// two 256-byte runs of consecutive rows of one partial.  Each block's maxima
// go to finred; the block that finishes last (a counter in the control block,
// one atomic per block) reduces them and decides.  A launch is a chain of round
// trips, so everything a block reads is requested at once, and the maxima
// pass through the memory that all XCDs share by themselves: fences around the
// counter, which write back and drop whole caches, and loads in turn made a
// launch take 11 us at n = 8192 and 16 us in a batch of 16 models (8.5 and 6.3).
__device__ __forceinline__ void enf_finalize_body(const EnfInst& in, int blk, int nblocks, double tol) {
  const int n = in.n, t = in.t;
  const double* __restrict__ partial = in.partial;
  double* __restrict__ scale = in.scale;  // receives 1 / s_i
  const double* __restrict__ blkmax = in.blkmax;
  const long nblk = in.pairs;
  EnfCtrl* ctrl = in.ctrl;
  __shared__ double ps[FIN_LANES][FIN_ROWS];
  const int part = threadIdx.x / FIN_ROWS;
  const int r = threadIdx.x % FIN_ROWS;
  const int i = blk * FIN_ROWS + r;
  const bool stop = ctrl->converged || ctrl->status < 0;
  const double* __restrict__ col = partial + min(i, n - 1);
  double rm = 0.0, em = 0.0, s = 0.0;
  const long tid = static_cast<long>(blk) * blockDim.x + threadIdx.x;
  for (long b = tid; b < nblk; b += static_cast<long>(nblocks) * blockDim.x) {
    rm = fmax(rm, blkmax[2 * b]);
    em = fmax(em, blkmax[2 * b + 1]);
  }
  for (int q = part; q <= t; q += 8 * FIN_LANES) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = col[static_cast<long>(min(q + u * FIN_LANES, t)) * n];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (q + u * FIN_LANES <= t) s += v[u];
  }
  if (stop) return;
  ps[part][r] = s;
  __syncthreads();
  double d = 0.0;
  if (part == 0 && i < n) {
    s = ((ps[0][r] + ps[1][r]) + (ps[2][r] + ps[3][r])) + ((ps[4][r] + ps[5][r]) + (ps[6][r] + ps[7][r]));
    if (!(s > 0.0)) raise_status(&ctrl->status, RAD_EZEROROW);
    scale[i] = 1.0 / s;
    d = fabs(s - 1.0);
  }
  // block maxima to finred
  __shared__ double fr[3][4];
  for (int off = 32; off > 0; off >>= 1) {
    d = fmax(d, __shfl_xor(d, off));
    rm = fmax(rm, __shfl_xor(rm, off));
    em = fmax(em, __shfl_xor(em, off));
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    fr[0][w] = d;
    fr[1][w] = rm;
    fr[2][w] = em;
  }
  __syncthreads();
  __shared__ int last;
  if (threadIdx.x == 0) {
    for (int c = 0; c < 3; ++c) {
      double x = fr[c][0];
      for (int q = 1; q < 4; ++q) x = fmax(x, fr[c][q]);
      agent_store(in.finred + 3 * static_cast<long>(blk) + c, x);
    }
    agent_settle();  // the maxima are there before the block counts itself done
    last = atomicAdd(&ctrl->done, 1) == nblocks - 1;
  }
  __syncthreads();
  if (last) {
    if (threadIdx.x == 0) ctrl->done = 0;
    enf_decide_body(in, tol);
  }
}

inline long fin_blocks(int64_t n) { return ceil_div(n, FIN_ROWS); }

__global__ void __launch_bounds__(256) enf_finalize(EnfInst in, double tol) {
  enf_finalize_body(in, blockIdx.x, gridDim.x, tol);
}

// map[b]: the instance and FIN_ROWS-row block of block b
__global__ void __launch_bounds__(256)
enf_finalize_batched(const EnfInst* __restrict__ ins, const EnfBlk* __restrict__ map, double tol) {
  const EnfBlk m = map[blockIdx.x];
  const EnfInst& in = ins[m.inst];
  enf_finalize_body(in, m.local, (in.n + FIN_ROWS - 1) / FIN_ROWS, tol);
}


// ---- all iterations in one launch, F on chip ---------------------------------
// A pair's two tiles fit the registers of its workgroup, so a model whose tile
// pairs are all resident at once (two workgroups per CU: n <= 1984 on 256
// CUs) is read and written once, and between iterations only row sums travel:
// a workgroup stores its rows' partial sums, the diagonal workgroup of a row
// block adds the block's t + 1 sums and stores the closure scales and the
// block's state, and every workgroup goes on once it has its two blocks' scales
// and all t states.  Bound by the latency of that exchange through the memory
// that all XCDs share, so the data are their own signal: a word holds ENF_EMPTY
// until its value is stored, and a reader loads until it is not.  Two one-way
// trips an iteration; with counters that announce the data there were five
// dependent round trips (n = 1081: 10.5 us an iteration, now 6.4; n = 1900: 16.5, now
// 9.5; n = 1985 streamed: 21).
//
// Buffers are used in turn and emptied by the diagonal workgroup of their row
// block.  Row sums (two in turn): it empties what it has read at iteration k, and
// that is done before it stores the scales of k + 1 (a wave's wait for its loads
// covers its earlier stores), which every writer of iteration k + 2 has seen.
// Scales and states (four): having read the sums of iteration k, whose writers
// have all seen every state of k - 1 and so every workgroup those of k - 2, it
// empties those of k - 2 for iteration k + 2, before it stores those of k + 1.
//
// A workgroup that waits holds its place, and every word that it waits for is
// stored by a workgroup of the same launch, in the same iteration, whether or not
// an error was seen.  The workgroups may start at very different times, so nothing
// but those words ends one: each takes part in every iteration that any of them
// enters.  An error, of the input or a bad area found by an earlier launch, travels
// in the words (ENF_ERROR and the states), every workgroup leaves after the same
// iteration, and the status is raised only then (a workgroup that left on a status
// raised in this launch would leave the others waiting).
//
// Resident grids of a process take turns (ResidentTurn), so a workgroup shares its
// CU with others of its own launch and with kernels that end by themselves; why
// every one gets a place beside those is at ENF_RES_PER_CU.  Ordinary launches:
// the runtime gives cooperative ones a hardware queue beside the four of a process,
// after which everything in several streams is slower (two streams of solves at
// 2000 faces 757 -> 1320 us a call, four at 900 faces 248 -> 616).
//
// Should some not get a place all the same (another process on the GPU), every
// wait ends: a wave whose patience is out declares the launch given up, unless it
// is done.  It is done once a workgroup is through with its last iteration: then
// all sums, scales and states of that have been stored, so the waits for them
// end too.  Nothing outside the exchange is written before that verdict, and
// enf_alone after it does what was given up.  Same operations in the same order
// as enf_sweep, enf_finalize and enf_apply_scale, so the same bits.
constexpr EnfWord ENF_NAN = 0x7ff8000000000000ull;    // any NaN that is stored
constexpr EnfWord ENF_EMPTY = 0x7ff8c0ffee000001ull;  // so no sum or scale is one of these
constexpr EnfWord ENF_ERROR = 0x7ff8c0ffee000002ull;  // in place of a sum: an input error was seen
// state of a row block; ENF_FAILED: ENF_ERROR in its sums, ENF_NOSUM: a row sums to zero
enum : EnfWord { ENF_OPEN = 0, ENF_CLOSED = 1, ENF_FAILED = 2, ENF_NOSUM = 3 };

__device__ __forceinline__ EnfWord enf_word(double x) {
  return x == x ? static_cast<EnfWord>(__double_as_longlong(x)) : ENF_NAN;
}
__device__ __forceinline__ double enf_value(EnfWord v) { return __longlong_as_double(static_cast<long long>(v)); }

// The verdict of a launch: whether its workgroups write their results.
enum : EnfWord { ENF_RUNNING = 0, ENF_DONE = 1, ENF_GIVEN_UP = 2 };
constexpr int ENF_GAVE_UP = 1;  // why a workgroup stops; otherwise an error code

// A whole wave asks after each poll in vain whether to leave.
__device__ __forceinline__ bool enf_gives_up(EnfWord* verdict, int polls, int patience) {
  if (polls < patience && (polls & 63) != 63) return false;
  EnfWord v = ENF_RUNNING;
  if (polls < patience)
    v = agent_load(verdict);
  else if (fresh_lane() == 0)
    v = atomicCAS(verdict, ENF_RUNNING, ENF_GIVEN_UP);
  const int old = __builtin_amdgcn_readfirstlane(static_cast<int>(v));
  return polls < patience ? old == static_cast<int>(ENF_GIVEN_UP) : old != static_cast<int>(ENF_DONE);
}

// One word per lane of a whole wave, once no lane's is empty; false: given up.
__device__ __forceinline__ bool enf_await(const EnfWord* p, EnfWord& v, EnfWord* verdict, int patience) {
  v = agent_load(p);
  for (int polls = 0; __ballot(v == ENF_EMPTY) != 0; ++polls) {
    if (enf_gives_up(verdict, polls, patience)) return false;
    __builtin_amdgcn_s_sleep(1);
    v = agent_load(p);
  }
  return true;
}

// the maximum over the 16 lanes of a row, by rotations within the row (lane
// permutations of the vector pipe; through the LDS, six steps of both maxima of a
// step took 0.45 us of an iteration)
template <int R>
__device__ __forceinline__ double max_rotated(double x) {
  const unsigned long long v = static_cast<unsigned long long>(__double_as_longlong(x));
  const unsigned lo = __builtin_amdgcn_update_dpp(0, static_cast<unsigned>(v), 0x120 + R, 0xf, 0xf, true);  // row_ror:R
  const unsigned hi = __builtin_amdgcn_update_dpp(0, static_cast<unsigned>(v >> 32), 0x120 + R, 0xf, 0xf, true);
  return fmax(x, __longlong_as_double(static_cast<long long>(static_cast<unsigned long long>(hi) << 32 | lo)));
}
__device__ __forceinline__ double max_of_16(double x) {
  return max_rotated<1>(max_rotated<2>(max_rotated<4>(max_rotated<8>(x))));
}

// What lives on between iterations is here, but for the tiles: the kernel is
// held to 72 registers.
struct ResidentShared {
  double sB[ET][ETP];
  double rowc[8][ET];   // see enf_pair_step; of a diagonal tile [4]: its own row sums, [5]: the space column,
                        // [6] and [7]: the rows' closure defects, of two iterations in turn
  double most[2][2][ENW][4];  // of two iterations in turn: both maxima, of 16 threads each
  struct alignas(16) {
    int closed, code, gave_up;  // all row blocks closed; the code if any failed; this workgroup gave up
  } now;
  int refused, error;  // a bad area; that, or an input error that this workgroup has seen
};

template <bool DIAG, bool EDGE, bool HALF, bool WIDE>
__device__ __forceinline__ void enf_resident_tile(const EnfInst& in, int I, int J, int w, double tol, int max_iter,
                                                  ResidentShared& sh) {
#pragma clang fp contract(off)
  double(*const sB)[ETP] = sh.sB;
  double(*const rowc)[ET] = sh.rowc;
  const long ldf = in.ldf;
  const int n = in.n, t = in.t;
  const int r0 = I * ET, c0 = J * ET;
  const int lane = fresh_lane();
  const int jgc = EDGE ? min(c0 + lane, n - 1) : c0 + lane, igc = EDGE ? min(r0 + lane, n - 1) : r0 + lane;
  EnfWord* const xpart = in.xch;
  EnfWord* const xscale = xpart + 2L * t * t * ET;
  EnfWord* const xstate = xscale + 4L * t * ET;
  EnfWord* const xmax = xstate + 4L * t;
  // slot of row block r, column block c in iteration k
  auto slot = [&](int k, int r, int c) { return xpart + ((static_cast<long>(k & 1) * t + r) * t + c) * ET; };
  double a[ERW], b[ERW];
#pragma unroll
  for (int k = 0; k < ERW; ++k) {
    const int i = r0 + w + ENW * k;
    a[k] = row_ld(in.F + static_cast<long>((EDGE && i >= n) ? n - 1 : i) * ldf, jgc);
  }
#pragma unroll
  for (int k = 0; k < ERW; ++k) {
    const int jr = c0 + w + ENW * k;
    b[k] = DIAG ? 0.0 : row_ld(in.F + static_cast<long>((EDGE && jr >= n) ? n - 1 : jr) * ldf, igc);
  }
  if (DIAG && w == 0) rowc[5][lane] = in.F[static_cast<long>(igc) * ldf + n];  // the space column's entries
  const int crow = (w == 0 ? r0 : c0) + lane, cq = w == 0 ? 0 : 4;  // the row of this thread's constants
  const int crc = (EDGE && crow >= n) ? n - 1 : crow;
  if (w < (DIAG ? 1 : 2)) {
    const double ai = in.area[crc];
    rowc[cq + 0][lane] = ai;
    rowc[cq + 1][lane] = in.inv_area[crc];
    rowc[cq + 2][lane] = HALF ? 0.0 : ai * ai / in.nrays[crc];
    rowc[cq + 3][lane] = 1.0;
  }
  if (w == 0 && lane == 0) {
    sh.refused = agent_load(&in.ctrl->status) < 0;  // a bad area, found by an earlier launch
    sh.error = sh.refused;
    sh.now.gave_up = 0;
  }
  __syncthreads();
  int iters = 0, converged = 0, stop = 0;
  while (iters < max_iter && !converged) {
    int bad = 0;
    double rmax, emax;
    enf_pair_step<DIAG, EDGE, HALF, WIDE, false>(
        in, I, J, w, a, b, sB, rowc, bad, rmax, emax,
        [&]() {
          const int l = fresh_lane();
          if (!DIAG)
#pragma unroll
            for (int k = 0; k < ERW; ++k) b[k] = sB[w + ENW * k][l];
          if (__ballot(bad) != 0 && l == 0) sh.error = 1;
        },
        [&](double s_own, double s_par) {
          const int l = fresh_lane(), ig = r0 + l;
          if (DIAG) {
            const double space = rowc[5][l];
            if (!EDGE || ig < n) bad |= !(space >= 0.0) || !(space <= 1.0e300);
            if (__ballot(bad) != 0 && l == 0) sh.error = 1;
            rowc[4][l] = s_own;
            rowc[5][l] = space * rowc[3][l];
          } else {
            const bool e = sh.error != 0;
            agent_store(slot(iters, I, J) + l, e ? ENF_ERROR : enf_word(s_own));
            agent_store(slot(iters, J, I) + l, e ? ENF_ERROR : enf_word(s_par));
          }
        });
    const int l = fresh_lane(), ig = r0 + l;
    rmax = max_of_16(rmax);
    emax = max_of_16(emax);
    if (l % 16 == 0) {
      sh.most[iters & 1][0][w][l / 16] = rmax;
      sh.most[iters & 1][1][w][l / 16] = emax;
    }
    if (DIAG) {
      // wave w sums every 8th partial sum of row l, the last one the space column's
      __syncthreads();
      static_assert(ENW == FIN_LANES, "wave w sums part w of every row");
      double s = 0.0;
      bool e = false;
      constexpr int NU = ENF_RES_TILES / ENW + 1;  // all sums of a part at once: t <= ENF_RES_TILES
      EnfWord v[NU];
      for (int polls = 0;; ++polls) {
        bool wait = false;
#pragma unroll
        for (int u = 0; u < NU; ++u) {
          const int c = w + ENW * u;
          v[u] = c < t && c != I ? agent_load(slot(iters, I, c) + l) : 0;
          wait |= v[u] == ENF_EMPTY;
        }
        if (__ballot(wait) == 0) break;
        if (enf_gives_up(xmax + 4, polls, in.patience)) {
          if (l == 0) sh.now.gave_up = 1;
          break;
        }
      }
      agent_settle();
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const int c = w + ENW * u;
        if (c < t && c != I) agent_store(slot(iters, I, c) + l, ENF_EMPTY);
        e |= v[u] == ENF_ERROR;
        if (c <= t) s += c == I ? rowc[4][l] : c == t ? rowc[5][l] : enf_value(v[u]);
      }
      sB[2 + 2 * ENW + w][l] = s;
      if (__ballot(e) != 0 && l == 0) sh.error = 1;
      __syncthreads();
      if (w == 0) {  // (after giving up these mean nothing, and are not used)
        const double(*p)[ETP] = sB + 2 + 2 * ENW;
        s = ((p[0][l] + p[1][l]) + (p[2][l] + p[3][l])) + ((p[4][l] + p[5][l]) + (p[6][l] + p[7][l]));
        const bool row = !EDGE || ig < n;
        const bool failed = sh.error != 0;
        const bool zero = row && !(s > 0.0) && !failed;  // after an input error a sum means nothing
        const double d = row ? fabs(s - 1.0) : 0.0;
        rowc[6 + (iters & 1)][l] = d;
        const double sc = row && s > 0.0 ? 1.0 / s : 1.0;
        const EnfWord state = failed                       ? ENF_FAILED
                              : __ballot(zero) != 0        ? ENF_NOSUM
                              : __ballot(!(d <= tol)) == 0 ? ENF_CLOSED
                                                           : ENF_OPEN;
        agent_settle();
        agent_store(xscale + ((iters & 3) * static_cast<long>(t) + I) * ET + l, enf_word(sc));
        if (l == 0) agent_store(xstate + (iters & 3) * static_cast<long>(t) + I, state);
        const int e2 = (iters + 2) & 3;
        agent_store(xscale + (e2 * static_cast<long>(t) + I) * ET + l, ENF_EMPTY);
        if (l == 0) agent_store(xstate + e2 * static_cast<long>(t) + I, ENF_EMPTY);
        rowc[3][l] = sc;
      }
    } else if (w < 2) {
      const long r = (iters & 3) * static_cast<long>(t) + (w == 0 ? I : J);
      EnfWord v;
      if (!enf_await(xscale + r * ET + l, v, xmax + 4, in.patience) && l == 0) sh.now.gave_up = 1;
      rowc[w == 0 ? 3 : 7][l] = enf_value(v);
    }
    if (w == 2) {
      EnfWord st;
      if (!enf_await(xstate + (iters & 3) * static_cast<long>(t) + min(l, t - 1), st, xmax + 4, in.patience) && l == 0)
        sh.now.gave_up = 1;
      // the streamed sweep sees a bad entry anywhere before any row's sum
      const bool all = __ballot(st != ENF_CLOSED) == 0, bad_entry = __ballot(st == ENF_FAILED) != 0;
      const bool no_sum = __ballot(st == ENF_NOSUM) != 0;
      if (l == 0) {
        sh.now.closed = all;
        sh.now.code = bad_entry ? RAD_ENONFINITE : no_sum ? RAD_EZEROROW : 0;
      }
    }
    __syncthreads();
    const auto now = sh.now;
    stop = __builtin_amdgcn_readfirstlane(now.gave_up) ? ENF_GAVE_UP : __builtin_amdgcn_readfirstlane(now.code);
    if (stop) break;
    ++iters;
    converged = tol > 0.0 && __builtin_amdgcn_readfirstlane(now.closed);
  }
  const int l = fresh_lane(), jg = c0 + l, ig = r0 + l;
  if (stop == ENF_GAVE_UP || __builtin_amdgcn_readfirstlane(sh.refused)) return;
  if (w == 0 && l == 0) sh.now.gave_up = atomicCAS(xmax + 4, ENF_RUNNING, ENF_DONE) == ENF_GIVEN_UP;
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(sh.now.gave_up)) return;
  if (stop && w == 0 && fresh_lane() == 0) raise_status(&in.ctrl->status, stop);
  // the maxima of the last iteration that was completed (an error ends one
  // without); the workgroup that adds its own last reports
  const int last = (iters - 1) & 1;
  if (w == 0) {
    double x = DIAG ? rowc[6 + last][l] : 0.0;
    for (int off = 32; off > 0; off >>= 1) x = fmax(x, __shfl_xor(x, off));
    if (l == 1 || l == 2) {
      x = 0.0;
      for (int q = 0; q < ENW; ++q)
        for (int g = 0; g < 4; ++g) x = fmax(x, sh.most[last][l - 1][q][g]);
    }
    if (l < 3 && iters > 0) atomicMax(xmax + l, static_cast<EnfWord>(__double_as_longlong(x)));
  }
  agent_settle();
  if (w == 0 && l == 0 && atomicAdd(xmax + 3, 1ull) + 1 == static_cast<EnfWord>(in.pairs)) {
    const double em = enf_value(agent_load(xmax + 2));
    in.ctrl->iters = iters;
    in.ctrl->converged = converged;
    in.ctrl->last_defect = enf_value(agent_load(xmax));
    in.ctrl->last_recip = em > 0.0 ? enf_value(agent_load(xmax + 1)) / em : 0.0;
  }
  if (stop || iters == 0) return;
  // F once, with the last closure scale (rowc[3], rowc[7])
#pragma unroll
  for (int k = 0; k < ERW; ++k) {
    const int i = r0 + w + ENW * k;
    if (!EDGE || (i < n && jg < n)) row_st(in.F + static_cast<long>(i) * ldf, jg, a[k] * rowc[3][w + ENW * k]);
  }
  if (!DIAG)
#pragma unroll
    for (int k = 0; k < ERW; ++k) {
      const int jr = c0 + w + ENW * k;
      if (!EDGE || (jr < n && ig < n)) row_st(in.F + static_cast<long>(jr) * ldf, ig, b[k] * rowc[7][w + ENW * k]);
    }
  if (DIAG && w == 0 && (!EDGE || ig < n)) in.F[static_cast<long>(ig) * ldf + n] = rowc[5][l] * rowc[3][l];
}

template <bool HALF, bool WIDE>
__device__ __forceinline__ void enf_resident_pair(const EnfInst& in, int I, int J, int w, double tol, int max_iter,
                                                  ResidentShared& sh) {
  const bool edge = (J + 1) * ET > in.n;
  if (I == J) {
    if (edge) enf_resident_tile<true, true, HALF, WIDE>(in, I, J, w, tol, max_iter, sh);
    else enf_resident_tile<true, false, HALF, WIDE>(in, I, J, w, tol, max_iter, sh);
  } else {
    if (edge) enf_resident_tile<false, true, HALF, WIDE>(in, I, J, w, tol, max_iter, sh);
    else enf_resident_tile<false, false, HALF, WIDE>(in, I, J, w, tol, max_iter, sh);
  }
}

template <bool WIDE>
__device__ __forceinline__ void enf_resident_body(const EnfInst& in, long pair, double tol, int max_iter,
                                                  ResidentShared& sh) {
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int I, J;
  pair_from_index(pair, in.t, I, J);
  I = __builtin_amdgcn_readfirstlane(I);
  J = __builtin_amdgcn_readfirstlane(J);
  if (in.mode == RAD_KAPPA_HALF) enf_resident_pair<true, WIDE>(in, I, J, w, tol, max_iter, sh);
  else enf_resident_pair<false, WIDE>(in, I, J, w, tol, max_iter, sh);
}
// one workgroup per CU
__global__ void __launch_bounds__(ENF_THREADS, 2) enf_resident_wide(EnfInst in, double tol, int max_iter) {
  __shared__ ResidentShared sh;
  enf_resident_body<true>(in, blockIdx.x, tol, max_iter, sh);
}
// ENF_RES_PER_CU workgroups per CU
__global__ void __launch_bounds__(ENF_THREADS, ENF_RES_WAVES) enf_resident(EnfInst in, double tol, int max_iter) {
  __shared__ ResidentShared sh;
  enf_resident_body<false>(in, blockIdx.x, tol, max_iter, sh);
}

// Several models in one launch, each with an exchange of its own:
// map[b] names the instance and the tile pair of workgroup b.
__global__ void __launch_bounds__(ENF_THREADS, ENF_RES_WAVES)
enf_resident_batched(const EnfInst* __restrict__ ins, const EnfBlk* __restrict__ map, double tol, int max_iter) {
  __shared__ ResidentShared sh;
  const EnfBlk m = map[blockIdx.x];
  const EnfInst in = ins[m.inst];
  enf_resident_body<false>(in, m.local, tol, max_iter, sh);
}

__device__ __forceinline__ void enf_init_body(EnfCtrl* ctrl) {
  {
    ctrl->status = 0;
    ctrl->converged = 0;
    ctrl->iters = 0;
    ctrl->done = 0;
    ctrl->last_defect = ctrl->last_recip = 0.0;
  }
}

// One tile (n <= 64), one workgroup: F stays in its registers for all
// iterations and the exchange in its LDS.  An iteration is one serial chain, so
// it is kept short: each thread holds whole unordered pairs {i, j} (four at
// n = 64, one up to n = 32; both entries), with no transposes, a ballot decides
// on convergence, and the maxima of the statistics are reduced after the last
// iteration only.  0.83 us an iteration at n = 32, 1.6 at n = 64 (3.9 and
// 4.9 with the streamed sweep's tile step).  Every product and the order of
// every sum are the sweep's and the finalize's, so the bits are.  The control
// block and the areas' check, launches of their own elsewhere, are here too.
constexpr int ESP = ET * (ET - 1) / 2 / ENF_THREADS + 1;  // pairs per thread, at most

template <bool HALF>
__device__ __forceinline__ void enf_single_body(const EnfInst& in, double tol, int max_iter, double (*sF)[ETP],
                                                double (*part)[ET], double (*rowc)[ET], int* flags) {
#pragma clang fp contract(off)
  const long ldf = in.ldf;
  const int n = in.n, tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
  if (tid == 0) enf_init_body(in.ctrl);
  const bool own = tid < n;  // this thread has a row's diagonal and space entries
  bool bad_area = false;
  double diag = 0.0, space = 0.0;
  if (own) {
    const double ai = in.area[tid];
    bad_area = !(ai > 0.0 && ai <= 1.0e300);
    rowc[0][tid] = ai;
    rowc[1][tid] = 1.0 / ai;
    rowc[2][tid] = HALF ? 0.0 : ai * ai / in.nrays[tid];
    rowc[3][tid] = 1.0;
    diag = in.F[static_cast<long>(tid) * ldf + tid];
    space = in.F[static_cast<long>(tid) * ldf + n];
  }
  const int npair = n * (n - 1) / 2;
  int pi[ESP], pj[ESP];
  double fij[ESP], fji[ESP];
#pragma unroll
  for (int m = 0; m < ESP; ++m) {
    // row-wise: pair p of rows i < j; rows n - 1, n - 2, .. hold n - 1, n - 2, .. pairs from the end
    const int p = tid + ENF_THREADS * m, back = npair - 1 - min(p, npair - 1);
    int r = static_cast<int>((sqrtf(8.0f * static_cast<float>(max(back, 0)) + 1.0f) - 1.0f) * 0.5f);
    r += (r + 1) * (r + 2) / 2 <= back;
    r -= r * (r + 1) / 2 > back;
    pi[m] = max(n - 2 - r, 0);
    pj[m] = n - 1 - max(back - r * (r + 1) / 2, 0);
    fij[m] = fji[m] = 0.0;
    if (p < npair) {
      fij[m] = in.F[static_cast<long>(pi[m]) * ldf + pj[m]];
      fji[m] = in.F[static_cast<long>(pj[m]) * ldf + pi[m]];
    }
  }
  if (tid < 3) flags[tid] = 0;
  if (__syncthreads_or(bad_area)) {
    if (tid == 0) raise_status(&in.ctrl->status, RAD_EINVAL);
    return;
  }
  const double area = own ? rowc[0][tid] : 0.0;
  int iters = 0, converged = 0, stop = 0;
  double rmax = 0.0, emax = 0.0, d = 0.0;
  double rlast = 0.0, elast = 0.0, dlast = 0.0;  // of the last iteration without an error
  while (iters < max_iter && !converged) {
    // of this iteration: a wave ahead may be in the next while another reads it
    int* error = flags + 1 + (iters & 1);
    bool bad = false;
    rmax = 0.0;
    emax = 0.0;
    if (own) {
      const double sc = rowc[3][tid];
      diag *= sc;  // the diagonal keeps its value
      space *= sc;
      bad = !(diag >= 0.0) || !(diag <= 1.0e300) || !(space >= 0.0) || !(space <= 1.0e300);
      emax = area * diag;
      sF[tid][tid] = diag;
    }
#pragma unroll
    for (int m = 0; m < ESP; ++m) {
      if (tid + ENF_THREADS * m >= npair) break;
      const int i = pi[m], j = pj[m];
      const double x = fij[m] * rowc[3][i], y = fji[m] * rowc[3][j];
      bad |= !(x >= 0.0) || !(x <= 1.0e300) || !(y >= 0.0) || !(y <= 1.0e300);
      const double eij = rowc[0][i] * x, eji = rowc[0][j] * y;
      rmax = fmax(rmax, fabs(eij - eji));
      emax = fmax(emax, fmax(eij, eji));
      const double kp = HALF ? 0.5 : kappa_c(x, y, rowc[2][i], rowc[2][j]);
      const double eh = kp * eij + (1.0 - kp) * eji;
      fij[m] = eh * rowc[1][i];
      fji[m] = eh * rowc[1][j];
      sF[i][j] = fij[m];
      sF[j][i] = fji[m];
    }
    if (__ballot(bad) != 0 && l == 0) *error = RAD_ENONFINITE;
    __syncthreads();
    double s = 0.0;  // every 8th entry of row l, from w
    if (l < n)
      for (int c = w; c < n; c += ENW) s += sF[l][c];
    part[w][l] = s;
    __syncthreads();
    if (w == 0) {
      s = 0.0;
#pragma unroll
      for (int q = 0; q < ENW; ++q) s += part[q][l];
      s += space;
      const bool zero = own && !(s > 0.0);
      d = own ? fabs(s - 1.0) : 0.0;
      if (own) rowc[3][l] = 1.0 / s;
      const bool all = __ballot(d <= tol) == ~0ull;
      if (__ballot(zero) != 0 && l == 0 && *error == 0) *error = RAD_EZEROROW;
      if (l == 0) flags[0] = tol > 0.0 && all;
    }
    __syncthreads();
    stop = *error;
    if (stop != 0) {
      if (tid == 0) raise_status(&in.ctrl->status, stop);
      break;
    }
    ++iters;
    converged = flags[0];
    rlast = rmax;
    elast = emax;
    dlast = d;
  }
  for (int off = 32; off > 0; off >>= 1) {
    rlast = fmax(rlast, __shfl_xor(rlast, off));
    elast = fmax(elast, __shfl_xor(elast, off));
    dlast = fmax(dlast, __shfl_xor(dlast, off));
  }
  __syncthreads();  // part has been read
  if (l == 0) {
    part[0][w] = rlast;
    part[1][w] = elast;
  }
  __syncthreads();
  if (tid == 0 && iters > 0) {
    for (int q = 1; q < ENW; ++q) {
      rlast = fmax(rlast, part[0][q]);
      elast = fmax(elast, part[1][q]);
    }
    in.ctrl->iters = iters;
    in.ctrl->converged = converged;
    in.ctrl->last_defect = dlast;
    in.ctrl->last_recip = elast > 0.0 ? rlast / elast : 0.0;
  }
  if (stop != 0 || iters == 0) return;
#pragma unroll
  for (int m = 0; m < ESP; ++m)
    if (tid + ENF_THREADS * m < npair) {
      in.F[static_cast<long>(pi[m]) * ldf + pj[m]] = fij[m] * rowc[3][pi[m]];
      in.F[static_cast<long>(pj[m]) * ldf + pi[m]] = fji[m] * rowc[3][pj[m]];
    }
  if (own) {
    in.F[static_cast<long>(tid) * ldf + tid] = diag * rowc[3][tid];
    in.F[static_cast<long>(tid) * ldf + n] = space * rowc[3][tid];
  }
}

__global__ void __launch_bounds__(ENF_THREADS, 2) enf_single(EnfInst in, double tol, int max_iter) {
  __shared__ double sF[ET][ETP];
  __shared__ double part[ENW][ET], rowc[4][ET];
  __shared__ int flags[3];  // converged, the error of two iterations in turn
  if (in.mode == RAD_KAPPA_HALF)
    enf_single_body<true>(in, tol, max_iter, sF, part, rowc, flags);
  else
    enf_single_body<false>(in, tol, max_iter, sF, part, rowc, flags);
}

__device__ __forceinline__ void enf_apply_scale_body(const EnfInst& in, long row) {
  if (in.ctrl->status < 0 || in.ctrl->iters == 0) return;
  const double s = in.scale[row];  // 1 / row sum
  double* p = in.F + row * in.ldf;
  for (int j = threadIdx.x; j <= in.n; j += blockDim.x) p[j] = p[j] * s;
}

__global__ void __launch_bounds__(256) enf_apply_scale(EnfInst in) { enf_apply_scale_body(in, blockIdx.x); }

// An enforcement that a resident launch gave up: the streamed steps one after
// another in one workgroup, which waits for nobody.  Reached when the GPU is
// shared with something that holds places for ever; otherwise a launch that
// leaves at once.
template <bool HALF>
__device__ __forceinline__ void enf_alone_body(const EnfInst& in, double tol, int max_iter, ResidentShared& sh,
                                               double (*red)[3]) {
  EnfCtrl* ctrl = in.ctrl;
  const int n = in.n, t = in.t, tid = threadIdx.x;
  auto status = [&]() {
    __threadfence();
    __syncthreads();
    const int st = agent_load(&ctrl->status);
    __syncthreads();
    return st;
  };
  if (status() < 0) return;
  for (int it = 0; it < max_iter; ++it) {
    for (long p = 0; p < in.pairs; ++p) {
      int I, J;
      pair_from_index(p, t, I, J);
      I = __builtin_amdgcn_readfirstlane(I);
      J = __builtin_amdgcn_readfirstlane(J);
      enf_sweep_pair<HALF, false>(in, p, I, J, it == 0, sh.sB, sh.rowc);
      __syncthreads();
    }
    if (status() < 0) return;
    double d = 0.0, rm = 0.0, em = 0.0;
    for (int i = tid; i < n; i += ENF_THREADS) {
      double s[FIN_LANES];
#pragma unroll
      for (int p = 0; p < FIN_LANES; ++p) {
        s[p] = 0.0;
        for (int q = p; q <= t; q += FIN_LANES) s[p] += in.partial[static_cast<long>(q) * n + i];
      }
      const double sum = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
      if (!(sum > 0.0)) raise_status(&ctrl->status, RAD_EZEROROW);
      in.scale[i] = 1.0 / sum;
      d = fmax(d, fabs(sum - 1.0));
    }
    for (long b = tid; b < in.pairs; b += ENF_THREADS) {
      rm = fmax(rm, in.blkmax[2 * b]);
      em = fmax(em, in.blkmax[2 * b + 1]);
    }
    red[tid][0] = d;
    red[tid][1] = rm;
    red[tid][2] = em;
    if (status() < 0) return;
    for (int half = ENF_THREADS / 2; half > 0; half /= 2) {
      if (tid < half)
        for (int c = 0; c < 3; ++c) red[tid][c] = fmax(red[tid][c], red[tid + half][c]);
      __syncthreads();
    }
    const bool converged = tol > 0.0 && red[0][0] <= tol;
    if (tid == 0) {
      ctrl->iters = it + 1;
      ctrl->last_defect = red[0][0];
      ctrl->last_recip = red[0][2] > 0.0 ? red[0][1] / red[0][2] : 0.0;
      ctrl->converged = converged;
    }
    __syncthreads();
    if (converged) break;
  }
  __threadfence();
  __syncthreads();
  for (int row = 0; row < n; ++row) enf_apply_scale_body(in, row);
}
__device__ __forceinline__ void enf_alone_instance(const EnfInst& in, double tol, int max_iter) {
  __shared__ ResidentShared sh;
  __shared__ double red[ENF_THREADS][3];
  if (agent_load(in.xch + enf_xch_words(in.t) - 1) != ENF_GIVEN_UP) return;
  if (in.mode == RAD_KAPPA_HALF) enf_alone_body<true>(in, tol, max_iter, sh, red);
  else enf_alone_body<false>(in, tol, max_iter, sh, red);
}
__global__ void __launch_bounds__(ENF_THREADS) enf_alone(EnfInst in, double tol, int max_iter) {
  enf_alone_instance(in, tol, max_iter);
}
__global__ void __launch_bounds__(ENF_THREADS)
enf_alone_batched(const EnfInst* __restrict__ ins, double tol, int max_iter) {
  enf_alone_instance(ins[blockIdx.x], tol, max_iter);
}

// rows [row_start[k], row_start[k+1]) are instance k's
__global__ void __launch_bounds__(256)
enf_apply_scale_batched(const EnfInst* __restrict__ ins, const long* __restrict__ row_start, int count) {
  const long row = row_start[0] + blockIdx.x;
  const int k = find_segment(row_start, count, row);
  enf_apply_scale_body(ins[k], row - row_start[k]);
}

__device__ __forceinline__ void enf_inv_area_body(const EnfInst& in, int i) {
  if (i >= in.n) return;
  const double a = in.area[i];
  if (!(a > 0.0 && a <= 1.0e300)) raise_status(&in.ctrl->status, RAD_EINVAL);
  const_cast<double*>(in.inv_area)[i] = 1.0 / a;
}

__global__ void __launch_bounds__(256) enf_inv_area(EnfInst in) {
  enf_inv_area_body(in, blockIdx.x * blockDim.x + threadIdx.x);
}

// an empty exchange, ahead of the resident kernel
__device__ __forceinline__ void enf_exchange_init(const EnfInst& in, long block, long blocks) {
  const long words = enf_xch_words(in.t);
  for (long k = block * blockDim.x + threadIdx.x; k < words; k += blocks * blockDim.x)
    in.xch[k] = k < words - 5 ? ENF_EMPTY : 0;
}
__global__ void __launch_bounds__(256) enf_resident_init(EnfInst in) {
  enf_inv_area_body(in, blockIdx.x * blockDim.x + threadIdx.x);
  enf_exchange_init(in, blockIdx.x, gridDim.x);
}
constexpr int ENF_XCH_BLOCKS = 16;  // per instance
__global__ void __launch_bounds__(256) enf_exchange_init_batched(const EnfInst* __restrict__ ins) {
  enf_exchange_init(ins[blockIdx.x / ENF_XCH_BLOCKS], blockIdx.x % ENF_XCH_BLOCKS, ENF_XCH_BLOCKS);
}

// blocks [blk_start[k], blk_start[k+1]) cover the faces of instance k (256 per block)
__global__ void __launch_bounds__(256)
enf_inv_area_batched(const EnfInst* __restrict__ ins, const long* __restrict__ blk_start, int count) {
  const int k = find_segment(blk_start, count, blockIdx.x);
  enf_inv_area_body(ins[k], static_cast<int>(blockIdx.x - blk_start[k]) * blockDim.x + threadIdx.x);
}

__global__ void enf_init(EnfCtrl* ctrl) {
  if (threadIdx.x == 0) enf_init_body(ctrl);
}

__global__ void enf_init_batched(const EnfInst* __restrict__ ins, int count) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < count) enf_init_body(ins[k].ctrl);
}

// Workgroups of a kernel that the current device holds at once, at most per_cu on
// a CU (0: unknown); cache: one slot per device.
inline long resident_workgroups(const void* kernel, int per_cu, std::atomic<long> (&cache)[64]) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
  long v = cache[dev].load(std::memory_order_relaxed);  // count + 1; 0: not looked up yet
  if (v == 0) {
    int cus = 0, per = 0;
    const bool ok =
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, ENF_THREADS, 0) == hipSuccess;
    if (!ok) (void)hipGetLastError();
    v = 1 + (ok ? static_cast<long>(cus) * std::min(per, per_cu) : 0L);
    cache[dev].store(v, std::memory_order_relaxed);
  }
  return v - 1;
}

// ENF_PATIENCE, or what the environment says (the tests: nobody is waited for).
inline int resident_patience() {
  const char* e = std::getenv("RAD_RESIDENT_PATIENCE");
  return e ? std::atoi(e) : ENF_PATIENCE;
}

// Whether the stream is being captured (or cannot be asked): replays would not
// take turns with other resident grids.
inline bool stream_capturing(hipStream_t s) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &st) != hipSuccess) {
    (void)hipGetLastError();
    return true;
  }
  return st != hipStreamCaptureStatusNone;
}

}  // namespace
}  // namespace rad
