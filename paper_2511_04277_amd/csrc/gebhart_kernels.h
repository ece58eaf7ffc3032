// Kernels and layouts of the open-system Gebhart solve, shared by the
// single-instance and batched entry points.  See gebhart.hip.
#pragma once

#include "common.h"
#include "gemm.h"

#include <algorithm>
#include <cmath>

namespace rad {
namespace {

constexpr int NB = 128;          // diagonal block (Gauss-Jordan inverse)
constexpr int NB2 = 1024;        // panel width of the two-level updates

template <class T>
constexpr long pad_elems() { return 128 / static_cast<long>(sizeof(T)); }

// ---------------------------------------------------------------- layout ----
// Factor buffer: K's LDU factors in place (np x ldk), the inverted 128 x 128
// diagonal blocks, and per 1024-wide panel p the inverses of the panel's
// diagonal block of U (W_p, upper) and of L (V_p, unit lower), NB2 x ldw each.
struct FactorLayout {
  int64_t n, np, P;
  long ldk;
  int P2;
  long ldw;
  size_t kf_off, dinv_off, w_off, v_off, bytes;
};

template <class T>
FactorLayout factor_layout(int64_t n) {
  FactorLayout f;
  f.n = n;
  f.np = ceil_div(n, NB) * NB;
  f.P = f.np / NB;
  f.ldk = static_cast<long>(f.np + pad_elems<T>());
  f.P2 = static_cast<int>(ceil_div(f.np, NB2));
  f.ldw = NB2 + pad_elems<T>();
  f.kf_off = 0;
  f.dinv_off = align_up(static_cast<size_t>(f.np) * f.ldk * sizeof(T), 256);
  f.w_off = f.dinv_off + align_up(static_cast<size_t>(f.P) * NB * NB * sizeof(T), 256);
  const size_t wbytes = align_up(static_cast<size_t>(f.P2) * NB2 * f.ldw * sizeof(T), 256);
  f.v_off = f.w_off + wbytes;
  f.bytes = f.v_off + wbytes;
  return f;
}

// scratch of the panel-inverse products: one b x ldt block per (panel, pair,
// matrix) at every level (b <= NB2 / 2)
inline long tri_ldt(long pad) { return NB2 / 2 + pad; }
inline size_t tri_tmp_elems(int P2, long pad) { return static_cast<size_t>(P2) * NB2 * tri_ldt(pad); }

// right-hand-side buffers: columns padded to a multiple of 128 plus 128 bytes
inline long rhs_ld(int64_t n, long pad) { return static_cast<long>(ceil_div(n + 1, 128) * 128 + pad); }

// Block forward substitution over a panel's nb diagonal blocks, step k = 1 ..
// nb - 1: with p the largest power of two that divides k, the p block rows from
// k on take the p blocks before k.  Every block row meets all blocks above it, in
// products of K = p NB: as many as with one block at a time, but half the block
// rows are read and written (12 for 28 of a whole panel), which is what a wide
// product with K = NB is bound by.
struct ForwardStep {
  int row, rows, col, cols;  // rows [row, row + rows) -= L[rows][col, col + cols) times rows [col, col + cols)
};
inline ForwardStep forward_step(int k, int nb) {
  const int p = k & -k;
  return ForwardStep{k * NB, std::min(p, nb - k) * NB, (k - p) * NB, p * NB};
}

struct Scalars {
  int status;
  int arrivals;      // corner tiles of update_invert launches (a multiple of their number between them)
  double max_r;      // max |residual|
  double max_d;      // max |correction|
  double red[2];     // REF check outputs
};

template <class T>
struct Fact {
  T* kf;
  long ldk;
  T* dinv;
  int n, np, P;
  T* W;       // panel inverses of U (P2 x NB2 x ldw)
  T* V;       // panel inverses of L
  long ldw;
  int P2;
};

template <class T>
Fact<T> make_fact(void* base, const FactorLayout& l) {
  Fact<T> f;
  f.kf = reinterpret_cast<T*>(static_cast<char*>(base) + l.kf_off);
  f.ldk = l.ldk;
  f.dinv = reinterpret_cast<T*>(static_cast<char*>(base) + l.dinv_off);
  f.n = static_cast<int>(l.n);
  f.np = static_cast<int>(l.np);
  f.P = static_cast<int>(l.P);
  f.W = reinterpret_cast<T*>(static_cast<char*>(base) + l.w_off);
  f.V = reinterpret_cast<T*>(static_cast<char*>(base) + l.v_off);
  f.ldw = l.ldw;
  f.P2 = l.P2;
  return f;
}

// ---------------------------------------------------------------- kernels ---
__global__ void scalars_init(Scalars* sc) {
  if (threadIdx.x == 0) {
    sc->status = 0;
    sc->arrivals = 0;
    sc->max_r = 0.0;
    sc->max_d = 0.0;
    sc->red[0] = sc->red[1] = 0.0;
  }
}

__global__ void scalars_init_partial(Scalars* sc) {
  if (threadIdx.x == 0) {
    sc->max_r = 0.0;
    sc->max_d = 0.0;
  }
}

// the same reset, then the range checks of a call's optical properties (one
// workgroup; the reset is at the level where the checks' atomics act)
__global__ void __launch_bounds__(1024)
check_optical(const double* __restrict__ eps, const double* __restrict__ rho, int n, Scalars* sc) {
  if (threadIdx.x == 0) {
    agent_store(&sc->status, 0);
    sc->arrivals = 0;
    sc->max_r = 0.0;
    sc->max_d = 0.0;
    sc->red[0] = sc->red[1] = 0.0;
    agent_settle();
  }
  __syncthreads();
  constexpr int U = 4;
  bool bad = false;
  for (int i0 = threadIdx.x; i0 < n; i0 += 1024 * U) {
    double e[U], r[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = min(i0 + 1024 * u, n - 1);
      e[u] = eps ? eps[i] : 0.5;
      r[u] = rho[i];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) bad |= !(e[u] >= 0.0 && e[u] <= 1.0 && r[u] >= 0.0 && r[u] <= 1.0);
  }
  if (bad) raise_status(&sc->status, RAD_ENONFINITE);
}

// Row i of K (padded with identity) and of E (padded with zeros) in precision
// T; returns whether the row has a bad entry.  Bound by memory; six columns of a
// thread are in flight (n = 4096: 111 -> 87 us for 0.4 GB; 8192: 355 us, 4.5 TB/s).
template <class T>
__device__ __forceinline__ bool geb_form_row(const double* __restrict__ F, long ldf, int n,
                                             const double* __restrict__ eps, const double* __restrict__ rho,
                                             T* __restrict__ KF, long ldk, int np, T* __restrict__ Y, long ldy, int i) {
  constexpr int U = 6;
  const double* frow = F + static_cast<long>(min(i, n - 1)) * ldf;
  T* krow = KF + static_cast<long>(i) * ldk;
  T* yrow = Y + static_cast<long>(i) * ldy;
  bool bad = false;
  const int jend = static_cast<int>(ldk > ldy ? ldk : ldy);
  for (int j0 = threadIdx.x; j0 < jend; j0 += 256 * U) {
    double f[U], r[U], e[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = j0 + 256 * u, jr = min(j, n - 1);
      f[u] = frow[min(j, n)];
      r[u] = rho[jr];
      e[u] = eps[jr];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = j0 + 256 * u;
      double kv = (i == j) ? 1.0 : 0.0;
      double yv = 0.0;
      if (i < n && j <= n) {
        bad |= !(f[u] >= 0.0 && f[u] <= 1.0e300);
        if (j < n) {
          kv = kv - f[u] * r[u];
          yv = f[u] * e[u];
        } else {
          yv = f[u];  // space column: no emissivity factor (eq. B.6)
        }
      }
      if (j < ldk) krow[j] = (j < np) ? static_cast<T>(kv) : T(0);
      if (j < ldy) yrow[j] = static_cast<T>(yv);
    }
  }
  return bad;
}

// one workgroup per row of the padded size
template <class T>
__global__ void __launch_bounds__(256)
geb_form(const double* __restrict__ F, long ldf, int n, const double* __restrict__ eps,
         const double* __restrict__ rho, T* __restrict__ KF, long ldk, int np,
         T* __restrict__ Y, long ldy, Scalars* sc) {
  if (geb_form_row(F, ldf, n, eps, rho, KF, ldk, np, Y, ldy, blockIdx.x)) raise_status(&sc->status, RAD_ENONFINITE);
}

// Radiation-only steady balance (eq. 3.12-3.14 with GR_ij = sigma w_i Y_ij,
// eq. 4.2) in x = T^4, each free row divided by sigma w_i:
//   free i:  (s_i - Y_ii) x_i - sum_{j != i} Y_ij x_j = Q_i / (sigma w_i) + Y_i,space x_space,
//            s_i = sum_{j <= n} Y_ij (the row sum, space included);
//   fixed i: x_i = T_i^4.
// One workgroup per row of the padded matrix; rows past n are identity rows.
__global__ void __launch_bounds__(256)
ss_form(const double* __restrict__ Y, long ldy, int n, const double* __restrict__ w,
        const double* __restrict__ Q, long ldq, int m, const double* __restrict__ tfix, double xs, double sigma,
        double* __restrict__ KF, long ldk, int np, double* __restrict__ R, long ldr, Scalars* sc) {
  __shared__ double red[4];
  const int i = blockIdx.x;
  const bool real = i < n;
  const double t = (real && tfix) ? tfix[i] : 0.0;
  const bool fixed = t > 0.0;
  const bool row = real && !fixed;
  const double* yrow = Y + static_cast<long>(i) * ldy;
  int bad = 0;
  double s = 0.0;
  constexpr int U = 8;  // loads of a thread in flight; the sum stays in order
  if (row)
    for (int j0 = threadIdx.x; j0 <= n; j0 += 256 * U) {
      double v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = yrow[min(j0 + 256 * u, n)];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (j0 + 256 * u <= n) {
          bad |= !(v[u] >= 0.0 && v[u] <= 1.0e300);
          s += v[u];
        }
    }
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  s = (red[0] + red[1]) + (red[2] + red[3]);
  const double wi = real ? w[i] : 1.0;
  if (threadIdx.x == 0 && real) {
    bad |= !(wi > 0.0 && wi <= 1.0e300);
    bad |= !(t >= 0.0 && t <= 1.0e300);
  }
  double* krow = KF + static_cast<long>(i) * ldk;
  for (int j0 = threadIdx.x; j0 < ldk; j0 += 256 * U) {
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = row ? yrow[min(j0 + 256 * u, n)] : 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = j0 + 256 * u;
      const double kv = row && j < n ? (i == j ? s - v[u] : -v[u]) : (i == j ? 1.0 : 0.0);
      if (j < ldk) krow[j] = j < np ? kv : 0.0;
    }
  }
  double* rrow = R + static_cast<long>(i) * ldr;
  const double ysp = row ? yrow[n] : 0.0;
  for (int c = threadIdx.x; c < m; c += 256) {  // the solve carries m columns
    double rv = 0.0;
    if (real) {
      if (fixed) {
        rv = (t * t) * (t * t);
      } else {
        const double qv = Q[static_cast<long>(i) * ldq + c];
        bad |= !(qv >= -1.0e300 && qv <= 1.0e300);
        rv = qv / (sigma * wi) + ysp * xs;
      }
    }
    rrow[c] = rv;
  }
  if (bad) raise_status(&sc->status, RAD_ENONFINITE);
}

// T = x^(1/4) for free nodes (x <= 0: no real temperature balances the
// given heat input, reported as RAD_ENONFINITE), the prescribed T otherwise.
__global__ void __launch_bounds__(256)
ss_output(const double* __restrict__ top, long ldtop, const double* __restrict__ X, long ldx, int n, int m,
          const double* __restrict__ tfix,
          double* __restrict__ T, long ldt, Scalars* sc) {
  const long q = static_cast<long>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (q >= static_cast<long>(n) * m) return;
  const int i = static_cast<int>(q / m), c = static_cast<int>(q % m);
  const double tf = tfix ? tfix[i] : 0.0;
  double out = tf;
  if (!(tf > 0.0)) {
    const double x = i < NB2 ? top[static_cast<long>(i) * ldtop + c] : X[static_cast<long>(i) * ldx + c];
    if (x > 0.0 && x <= 1.0e300) {
      out = sqrt(sqrt(x));
    } else {
      out = __builtin_nan("");
      raise_status(&sc->status, RAD_ENONFINITE);
    }
  }
  T[static_cast<long>(i) * ldt + c] = out;
}

// ---- least-squares optimum enforcer (eq. 3.41-3.52 with NNR / SPVA) ------
// The projection of F onto {closure rows sum to 1, W_i F_ik = W_k F_ki} over
// the active entries (a_ik = 1) is F_hat = F - A^T y with (A A^T) y = A F - b.
// A A^T has a diagonal closure block (n_i = active entries of row i), a
// diagonal reciprocity block (d_ik = W_i^2 a_ik + W_k^2 a_ki per pair) and a
// coupling with two entries per pair, so eliminating the pair multipliers
// leaves an n x n system for the closure multipliers lambda:
//   S_ii = n_i - sum_{k != i} a_ik W_i^2 / d_ik,  S_ik = a_ik a_ki W_i W_k / d_ik,
//   S lambda = (sum_j a_ij F_ij - 1) - sum_{k != i} a_ik W_i rho_ik / d_ik,
//   rho_ik = W_i a_ik F_ik - W_k a_ki F_ki;
// then F_hat_ik = F_ik - lambda_i - W_i nu_ik with the pair multiplier
//   nu_ik = (rho_ik - a_ik W_i lambda_i + a_ki W_k lambda_k) / d_ik
// (k != i, k < n), and F_hat_ik = F_ik - lambda_i on the diagonal and the
// space column.  A row with no active entry gets lambda_i = 0.

// mask (n x (n+1), ld n+1): 1 = active; SPVA drops the zeros of the input
__global__ void __launch_bounds__(256)
lsq_mask_init(const double* __restrict__ F, long ldf, int n, int spva, uint8_t* __restrict__ mask,
              Scalars* sc) {
  const int i = blockIdx.y;
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k > n) return;
  const double v = F[static_cast<long>(i) * ldf + k];
  if (!(v >= -1.0e300 && v <= 1.0e300)) raise_status(&sc->status, RAD_ENONFINITE);
  mask[static_cast<long>(i) * (n + 1) + k] = (spva && v == 0.0) ? 0 : 1;
}

// Both kernels below take 16 rows i per workgroup and walk the columns k in
// chunks of 64: the rows' own entries F_ik and a_ik are read as contiguous
// 512-byte row pieces, and the partner entries F_ki, a_ki of the chunk (64
// rows of 16 contiguous entries each) are staged in LDS, so no access is
// strided.  Thread t works on rows w + 4j (w = t / 64, j = 0..3) of the block
// and column t % 64 of each chunk.
constexpr int LSQ_RB = 16;  // rows per workgroup
constexpr int LSQ_KC = 64;  // columns per chunk

// the chunk's partner entries F_ki, a_ki (k in [k0, k0 + 64), i in the block)
__device__ __forceinline__ void lsq_stage_partner(const double* __restrict__ F, long ldf,
                                                  const uint8_t* __restrict__ mask, long ldm, int n, int i0, int k0,
                                                  double (*pf)[LSQ_RB + 1], uint8_t (*pm)[LSQ_RB + 1]) {
#pragma unroll
  for (int q = 0; q < LSQ_KC * LSQ_RB / 256; ++q) {
    const int e = threadIdx.x + 256 * q;
    const int kk = e / LSQ_RB, ii = e % LSQ_RB;
    const int k = k0 + kk, i = i0 + ii;
    const bool in = k < n && i < n;
    pf[kk][ii] = in ? F[static_cast<long>(k) * ldf + i] : 0.0;
    pm[kk][ii] = in ? mask[static_cast<long>(k) * ldm + i] : 0;
  }
}

__global__ void __launch_bounds__(256)
lsq_schur(const double* __restrict__ F, long ldf, int n, const double* __restrict__ W,
          const uint8_t* __restrict__ mask, double* __restrict__ KF, long ldk, int np,
          double* __restrict__ Y, long ldy) {
  __shared__ double pf[LSQ_KC][LSQ_RB + 1];
  __shared__ uint8_t pm[LSQ_KC][LSQ_RB + 1];
  const int i0 = blockIdx.x * LSQ_RB;
  const int t = threadIdx.x, l = t & 63, w = t >> 6;
  const long ldm = n + 1;
  double cnt[4], rsum[4], sub[4], tt[4], wi[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int i = i0 + w + 4 * j;
    cnt[j] = rsum[j] = sub[j] = tt[j] = 0.0;
    wi[j] = i < n ? W[i] : 0.0;
  }
  if (i0 < n) {
    // a chunk's entries (the rows' own, and the partners' as in
    // lsq_stage_partner) are in flight while the chunk before it is summed, for
    // there is less than one workgroup per CU to cover them; addresses clamped
    // into the matrix (n = 2845: 140 -> 78 us, of which 10 for columns of Y
    // that no solve reads)
    constexpr int NP = LSQ_KC * LSQ_RB / 256;
    double fn[4], pn[NP], wn;
    uint8_t an[4], qn[NP];
    auto load = [&](int k0) {
      const int k = min(k0 + l, n);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const long i = min(i0 + w + 4 * j, n - 1);
        an[j] = mask[i * ldm + k];
        fn[j] = F[i * ldf + k];
      }
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        const int e = t + 256 * q;
        const long kk = min(k0 + e / LSQ_RB, n - 1);
        const int i = min(i0 + e % LSQ_RB, n - 1);
        pn[q] = F[kk * ldf + i];
        qn[q] = mask[kk * ldm + i];
      }
      wn = W[min(k, n - 1)];
    };
    load(0);
    for (int k0 = 0; k0 <= n; k0 += LSQ_KC) {
      const int k = k0 + l;
      int am[4];
      double fv[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        am[j] = an[j];
        fv[j] = fn[j];
      }
      const double wk = k < n ? wn : 0.0;
      __syncthreads();  // the previous chunk's partner reads are done
#pragma unroll
      for (int q = 0; q < NP; ++q) {
        const int e = t + 256 * q;
        const bool in = k0 + e / LSQ_RB < n && i0 + e % LSQ_RB < n;
        pf[e / LSQ_RB][e % LSQ_RB] = in ? pn[q] : 0.0;
        pm[e / LSQ_RB][e % LSQ_RB] = in ? qn[q] : 0;
      }
      __syncthreads();
      if (k0 + LSQ_KC <= n) load(k0 + LSQ_KC);
      if (k > n) continue;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int ii = w + 4 * j, i = i0 + ii;
        if (i >= n) continue;
        const int aik = am[j];
        const double fik = fv[j];
        cnt[j] += aik;
        rsum[j] += aik ? fik : 0.0;
        if (k < n && k != i) {
          double sik = 0.0;
          const int aki = pm[l][ii];
          const double d = wi[j] * wi[j] * aik + wk * wk * aki;
          if (d > 0.0) {
            const double rho = (aik ? wi[j] * fik : 0.0) - (aki ? wk * pf[l][ii] : 0.0);
            if (aik) {
              sub[j] += wi[j] * wi[j] / d;
              tt[j] += wi[j] * rho / d;
            }
            if (aik && aki) sik = wi[j] * wk / d;
          }
          KF[static_cast<long>(i) * ldk + k] = sik;
        }
      }
    }
  }
  // row sums over the 64 lanes of the wave (fixed order)
#pragma unroll
  for (int j = 0; j < 4; ++j)
    for (int off = 32; off > 0; off >>= 1) {
      cnt[j] += __shfl_xor(cnt[j], off);
      rsum[j] += __shfl_xor(rsum[j], off);
      sub[j] += __shfl_xor(sub[j], off);
      tt[j] += __shfl_xor(tt[j], off);
    }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int i = i0 + w + 4 * j;
    if (i >= np) continue;
    double* krow = KF + static_cast<long>(i) * ldk;
    double* yrow = Y + static_cast<long>(i) * ldy;
    if (i < n) {
      // the diagonal, the padding columns, and the right-hand side
      for (long k = n + l; k < ldk; k += 64) krow[k] = 0.0;
      if (l == 0) {
        krow[i] = cnt[j] > 0.0 ? cnt[j] - sub[j] : 1.0;
        yrow[0] = cnt[j] > 0.0 ? (rsum[j] - 1.0) - tt[j] : 0.0;
      }
    } else {
      // padding rows: identity
      for (long k = l; k < ldk; k += 64) krow[k] = k == i ? 1.0 : 0.0;
      if (l == 0) yrow[0] = 0.0;
    }
  }
}

// F_hat from lambda (column 0 of Y); NNR: negative active entries leave the
// next round's mask; every entry of the mask is written (ping-pong buffers).
// One workgroup per 16 rows x one 64-column chunk (grid: chunks x row blocks).
__global__ void __launch_bounds__(256)
lsq_update(const double* __restrict__ F, long ldf, int n, const double* __restrict__ W,
           const uint8_t* __restrict__ mask, const double* __restrict__ Y, long ldy, int nnr,
           uint8_t* __restrict__ mask_next, double* __restrict__ Fo, long ldo, int* __restrict__ negatives) {
  __shared__ double pf[LSQ_KC][LSQ_RB + 1];
  __shared__ uint8_t pm[LSQ_KC][LSQ_RB + 1];
  __shared__ double yk[LSQ_KC];
  const int k0 = blockIdx.x * LSQ_KC, i0 = blockIdx.y * LSQ_RB;
  const int t = threadIdx.x, l = t & 63, w = t >> 6;
  const long ldm = n + 1;
  lsq_stage_partner(F, ldf, mask, ldm, n, i0, k0, pf, pm);
  if (t < LSQ_KC) yk[t] = k0 + t < n ? Y[static_cast<long>(k0 + t) * ldy] : 0.0;
  __syncthreads();
  const int k = k0 + l;
  int neg_count = 0;
  if (k <= n) {
    const double wk = k < n ? W[k] : 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int ii = w + 4 * j, i = i0 + ii;
      if (i >= n) continue;
      const int aik = mask[static_cast<long>(i) * ldm + k];
      double v = 0.0;
      if (aik) {
        const double li = Y[static_cast<long>(i) * ldy];
        const double fik = F[static_cast<long>(i) * ldf + k];
        v = fik - li;
        if (k < n && k != i) {
          const int aki = pm[l][ii];
          const double wi = W[i];
          const double d = wi * wi + wk * wk * aki;
          const double fki = aki ? pf[l][ii] : 0.0;
          const double nu = ((wi * fik - wk * fki) - wi * li + (aki ? wk * yk[l] : 0.0)) / d;
          // a partner held at zero makes the pair's row read W_i F_ik = 0: exactly zero
          v = aki ? v - wi * nu : 0.0;
        }
      }
      const int neg = nnr && aik && v < 0.0;
      neg_count += neg;
      mask_next[static_cast<long>(i) * ldm + k] = aik && !neg;
      Fo[static_cast<long>(i) * ldo + k] = v;
    }
  }
  for (int off = 32; off > 0; off >>= 1) neg_count += __shfl_xor(neg_count, off);
  if (l == 0 && neg_count > 0) atomicAdd(negatives, neg_count);
}

// P = F_sq diag(rho) in FP64, zero outside n x n (refinement residuals).
__global__ void __launch_bounds__(256)
form_p64(const double* __restrict__ F, long ldf, int n, const double* __restrict__ rho,
         double* __restrict__ P, long ldp) {
  const int i = blockIdx.x;
  for (long j = threadIdx.x; j < ldp; j += blockDim.x)
    P[static_cast<long>(i) * ldp + j] = (i < n && j < n) ? F[static_cast<long>(i) * ldf + j] * rho[j] : 0.0;
}

template <class T>
__global__ void __launch_bounds__(256) fill_zero(T* __restrict__ p, long count) {
  for (long q = blockIdx.x * static_cast<long>(blockDim.x) + threadIdx.x; q < count;
       q += static_cast<long>(gridDim.x) * blockDim.x)
    p[q] = T(0);
}

// Inverse of one NB x NB diagonal block D = [A11 A12; A21 A22] (halves of HB),
// no pivoting.  The chain of diagonal blocks needs the product with D^-1, not
// D^-1 itself, so only what that product takes is formed on the chain:
//   I1 = A11^-1,  T = I1 A12,  I2 = (A22 - A21 T)^-1,
// kept as [I1 T; A21 I2] in the block's place in dinv; the L blocks are formed
// from it half by half (lblock_rows), and the launch that starts the panel
// inverses makes it D^-1 for all blocks at once (tri_init_block).
// Blocked by 16: the block is 8 x 8 tiles of 16 x 16 in MFMA accumulator
// layout, and wave w's registers hold tile row w.  Step s takes the pivot tile
// P = M(s,s), R(s,j) = P^-1 M(s,j) (R(s,s) = P^-1) and
//   M(i,j) <- M(i,j) - M(i,s) R(s,j),  M(i,s) <- -M(i,s) R(s,s),
// the scalar in-place Gauss-Jordan update with a 16 x 16 pivot: in the upper
// half's steps for the rows below s only (the rows above take their updates,
// in the same order, while the lower half is inverted), in the lower half's
// for its own rows.  The 16 scalar steps of a pivot tile are a serial chain
// (about 4k cycles) that bounds the kernel; a wave of its own forms pivot tile
// s + 1 from the tiles of step s (two products) and inverts it while the
// others update theirs.  Its FP64 vector operations would wait behind the
// 64-cycle MFMAs of waves on the same SIMD, so it has a SIMD to itself: waves
// 0, 4, 8 of a workgroup share one, and the eight rows are on the other three.
// The steps are unrolled: with tile columns picked at run time the rows took
// 5k to 7k cycles a step instead of 2k to 4k, and bound it.  128 x 128 FP64
// 21.4 us alone (35 us as one full inverse on four SIMDs), FP32 13.0 us.
// Inside a pivot tile the pivot row is broadcast over the lane groups and the
// pivot column along each group by lane permutations of the vector pipe, with
// no LDS round trip on the chain.
// Diagonal dominance of K makes every pivot order stable, so no pivoting is
// needed; the scalar pivots are the same Schur-complement diagonals as in
// unblocked elimination and are checked against the singularity threshold.
constexpr int HB = NB / 2;
constexpr int GJ_THREADS = 64 * 11;

// 1/x: the hardware reciprocal refined to full precision; with e = 1 - x r
// the relative error of r, r (1 + e + e^2) leaves e^3
__device__ __forceinline__ double recip_nr(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}
__device__ __forceinline__ float recip_nr(float x) {
  float r = __builtin_amdgcn_rcpf(x);
  return r * (2.0f - x * r);
}

// 32-bit lane permutations behind the pivot chain: the value of lane Q of each
// group of 16 lanes, and the 16 lanes of group G in every group
template <int Q>
__device__ __forceinline__ unsigned bcast_col32(unsigned x) {
  return __builtin_amdgcn_update_dpp(x, x, 0x150 + Q, 0xf, 0xf, true);  // row_newbcast:Q
}
template <int G>
__device__ __forceinline__ unsigned bcast_group32(unsigned x) {
  const auto h = __builtin_amdgcn_permlane32_swap(x, x, false, false);  // [0]: lanes 0-31 twice, [1]: 32-63 twice
  const unsigned y = h[G >> 1];
  const auto r = __builtin_amdgcn_permlane16_swap(y, y, false, false);  // [0]: even groups twice, [1]: odd ones
  return r[G & 1];
}
template <int Q>
__device__ __forceinline__ double bcast_col(double x) {
  const unsigned long long v = __double_as_longlong(x);
  const unsigned long long lo = bcast_col32<Q>(static_cast<unsigned>(v)), hi = bcast_col32<Q>(static_cast<unsigned>(v >> 32));
  return __longlong_as_double(static_cast<long long>((hi << 32) | lo));
}
template <int Q>
__device__ __forceinline__ float bcast_col(float x) { return __uint_as_float(bcast_col32<Q>(__float_as_uint(x))); }
template <int G>
__device__ __forceinline__ double bcast_group(double x) {
  const unsigned long long v = __double_as_longlong(x);
  const unsigned long long lo = bcast_group32<G>(static_cast<unsigned>(v)), hi = bcast_group32<G>(static_cast<unsigned>(v >> 32));
  return __longlong_as_double(static_cast<long long>((hi << 32) | lo));
}
template <int G>
__device__ __forceinline__ float bcast_group(float x) { return __uint_as_float(bcast_group32<G>(__float_as_uint(x))); }

// w - (column Q of v, broadcast along each group of 16 lanes) * rj
template <int Q>
__device__ __forceinline__ void sub_col_times(double (&w)[4], const double (&v)[4], double rj) {
  // one instruction per element: the broadcast is the multiply-add's own lane
  // permutation (the waits cover the lane permutations before and after it)
  __asm__("s_nop 1\n\t"
          "v_fmac_f64_dpp %0, -%4, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f64_dpp %1, -%5, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f64_dpp %2, -%6, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f64_dpp %3, -%7, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
          "s_nop 1"
          : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3])
          : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(rj), "n"(Q));
}
template <int Q>
__device__ __forceinline__ void sub_col_times(float (&w)[4], const float (&v)[4], float rj) {
#pragma unroll
  for (int r = 0; r < 4; ++r) w[r] = fma(-bcast_col<Q>(v[r]), rj, w[r]);
}

// In-place Gauss-Jordan steps Q..15 of a 16 x 16 tile held by one wave in
// accumulator layout (v[r] = P(orow(l, r), l % 16)); every lane must be active.
// row is row Q in every lane group, piv = P(Q, Q) and d its reciprocal.  The
// chain through the 16 reciprocals binds the tile: step Q forms the next
// pivot and starts its reciprocal from three broadcast entries before the
// tile itself is updated, and carries the next row along instead of
// broadcasting it again.
template <class T, int Q>
__device__ __forceinline__ void pivot_steps(T (&v)[4], T row, T piv, T d, int l, T& pivots) {
  // row q sits in lane group grp(q), register reg(q)
  constexpr auto grp = [](int q) { return sizeof(T) == 8 ? (q & 3) : (q >> 2); };
  constexpr auto reg = [](int q) { return sizeof(T) == 8 ? (q >> 2) : (q & 3); };
  const int li = l & 15, lg = l >> 4;
  T rown = T(0), c = T(0), pn = T(0), dn = T(0);
  if constexpr (Q < 15) {
    rown = bcast_group<grp(Q + 1)>(v[reg(Q + 1)]);  // P(Q + 1, li) before this step
    c = bcast_col<Q>(rown);
    pn = fma(-c, bcast_col<Q + 1>(row) * d, bcast_col<Q + 1>(rown));
    dn = recip_nr(pn);
  }
  pivots = l == Q ? piv : pivots;
  const bool own = li == Q;
  const T rj = own ? d : row * d;  // the new pivot row
  T w[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) w[r] = own ? T(0) : v[r];
  sub_col_times<Q>(w, v, rj);
#pragma unroll
  for (int r = 0; r < 4; ++r) v[r] = w[r];
  v[reg(Q)] = lg == grp(Q) ? rj : w[reg(Q)];
  if constexpr (Q < 15) pivot_steps<T, Q + 1>(v, fma(-c, rj, own ? T(0) : rown), pn, dn, l, pivots);
}

// In-place inverse of such a tile; pivots receives pivot q in lane q.
template <class T>
__device__ __forceinline__ void pivot_inverse(T (&v)[4], int l, T& pivots) {
  const T row = bcast_group<0>(v[0]), piv = bcast_col<0>(row);
  pivot_steps<T, 0>(v, row, piv, recip_nr(piv), l, pivots);
}

constexpr int GJ_LD = NB + 16;  // four rows of 16 FP64 operands in two passes over the banks
template <class T>
struct GjShared {
  static constexpr int BT = 16;
  T sC[NB][BT + 2];      // tile column s before the step
  T sRo[BT][GJ_LD];      // tile row s before the step
  T sR[2][BT][GJ_LD];    // tile row s after it, of two steps
  T sU[2][BT][GJ_LD];    // the upper rows' own pass: the row it takes
  T sP[BT][BT + 1];      // inverse of the pivot tile
  T sD[BT][BT + 1];      // diagonal tile s + 1 before the step
};

// The pivot wave: inverts pivot tile s, and forms tile s + 1 from the tiles of step s.
// AGENT: A was stored by other workgroups of the launch.
template <bool AGENT, class T>
__device__ __forceinline__ T gj_load(const T* p) {
  if constexpr (AGENT) return agent_load(p);
  else return *p;
}
template <class T, bool AGENT>
__device__ __forceinline__ void gj_pivots(const T* __restrict__ A, long lda, Scalars* sc, GjShared<T>& sh) {
  typedef typename Mfma<T>::v4 v4;
  constexpr int BT = 16, NT = NB / BT;
  const int l = threadIdx.x & 63, li = l & 15;
  __builtin_amdgcn_s_setprio(3);  // its dependent operations go first
  const double tiny = sizeof(T) == 8 ? 1e-11 : 1e-5;
  int singular = 0;
  T v[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) v[r] = gj_load<AGENT>(A + static_cast<long>(Mfma<T>::orow(l, r)) * lda + li);
#pragma unroll 1
  for (int s = 0;; ++s) {
    T pivots = T(1);
    pivot_inverse(v, l, pivots);
#pragma unroll
    for (int r = 0; r < 4; ++r) sh.sP[Mfma<T>::orow(l, r)][li] = v[r];
    __syncthreads();  // the step begins
    if (s + 1 < NT) {
      // the next pivot tile: M(s+1, s+1) - M(s+1, s) P^-1 M(s, s+1)
      v4 t = v4{0, 0, 0, 0}, d;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        t = Mfma<T>::mma(sh.sP[li][Mfma<T>::orow(l, kk)], sh.sRo[Mfma<T>::orow(l, kk)][(s + 1) * BT + li], t);
#pragma unroll
      for (int r = 0; r < 4; ++r) d[r] = sh.sD[Mfma<T>::orow(l, r)][li];
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        d = Mfma<T>::mma(-sh.sC[(s + 1) * BT + li][Mfma<T>::orow(l, kk)], t[kk], d);
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = d[r];
    }
    const double ap = fabs(static_cast<double>(pivots));
    singular |= !(ap > tiny && ap <= 1.7976931348623157e308);  // too small, infinite or NaN
    __syncthreads();  // the new tile row s is complete; the old row and column have been read
    if (s + 1 == NT) break;
  }
  if (singular) raise_status(&sc->status, RAD_ESINGULAR);
}

// Tile row w, of the upper or the lower half, through the eight steps.
template <class T, bool UPPER, bool AGENT>
__device__ __forceinline__ void gj_row(const T* __restrict__ A, long lda, T* __restrict__ out, int w,
                                       GjShared<T>& sh) {
  typedef typename Mfma<T>::v4 v4;
  constexpr int BT = 16, NT = NB / BT, NH = NT / 2;
  const int l = threadIdx.x & 63, li = l & 15, lg = l >> 4;
  v4 m[NT];
#pragma unroll
  for (int bj = 0; bj < NT; ++bj)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      m[bj][r] = gj_load<AGENT>(A + static_cast<long>(w * BT + Mfma<T>::orow(l, r)) * lda + bj * BT + li);
  auto put = [&](T* d, int ld, const v4& x) {
#pragma unroll
    for (int r = 0; r < 4; ++r) d[Mfma<T>::orow(l, r) * ld + li] = x[r];
  };
  auto put_row = [&](T(*d)[GJ_LD], int b0) {
#pragma unroll
    for (int bj = b0; bj < NT; ++bj) put(&d[0][bj * BT], GJ_LD, m[bj]);
  };
  auto get_row = [&](const T(*d)[GJ_LD], int b0) {
#pragma unroll
    for (int bj = b0; bj < NT; ++bj)
#pragma unroll
      for (int r = 0; r < 4; ++r) m[bj][r] = d[Mfma<T>::orow(l, r)][bj * BT + li];
  };
  auto store = [&](int b0, int b1) {
#pragma unroll
    for (int bj = b0; bj < b1; ++bj) put(out + static_cast<long>(w) * BT * NB + bj * BT, NB, m[bj]);
  };
  // tile columns [b0, b1) += a (this row's part of a tile column, negated) times a tile row
  auto rank16 = [&](const T(&a)[4], const T(*row)[GJ_LD], int b0, int b1) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int bj = b0; bj < b1; ++bj) m[bj] = Mfma<T>::mma(a[kk], row[4 * kk + lg][bj * BT + li], m[bj]);
  };
  auto column = [&](T(&a)[4]) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) a[kk] = -sh.sC[w * BT + li][4 * kk + lg];
  };
  // tile w of the new tile row s: R(s, j) = P^-1 Ro(s, j), R(s, s) = P^-1
  auto new_row = [&](int s) {
    T* d = &sh.sR[s & 1][0][w * BT];
    if (w == s) {
#pragma unroll
      for (int r = 0; r < 4; ++r) d[Mfma<T>::orow(l, r) * GJ_LD + li] = sh.sP[Mfma<T>::orow(l, r)][li];
    } else {
      v4 x = v4{0, 0, 0, 0};
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) x = Mfma<T>::mma(sh.sP[li][4 * kk + lg], sh.sRo[4 * kk + lg][w * BT + li], x);
      put(d, GJ_LD, x);
    }
  };
  put(&sh.sC[w * BT][0], BT + 2, m[0]);
  if constexpr (UPPER) {
    if (w == 0) put_row(sh.sRo, 0);
    if (w == 1) put(&sh.sD[0][0], BT + 1, m[1]);
#pragma unroll
    for (int s = 0; s < NH; ++s) {
      __syncthreads();
      T av[4];
      column(av);
      new_row(s);
      __syncthreads();
      if (w == s) get_row(sh.sR[s & 1], 0);
      if (w > s) {
        m[s] = v4{0, 0, 0, 0};
        rank16(av, sh.sR[s & 1], 0, NT);
      }
      if (s + 1 < NH) {
        put(&sh.sC[w * BT][0], BT + 2, m[s + 1]);
        if (w == s + 1) put_row(sh.sRo, 0);
        if (s + 2 < NH && w == s + 2) put(&sh.sD[0][0], BT + 1, m[s + 2 < NT ? s + 2 : 0]);
      }
    }
    // what the rows lack: rows 1, 2, 3 taken from those above them
#pragma unroll
    for (int p = 1; p < NH; ++p) {
      put(&sh.sC[w * BT][0], BT + 2, m[p]);
      if (w == p) put_row(sh.sU[p & 1], 0);
      __syncthreads();
      T av[4];
      column(av);
      __syncthreads();
      if (w < p) {
        m[p] = v4{0, 0, 0, 0};
        rank16(av, sh.sU[p & 1], 0, NT);
      }
    }
    store(0, NT);
    __syncthreads();
    __syncthreads();
  } else {
    store(0, NH);  // A21 stays as it is
    T av[4], avp[4];
#pragma unroll
    for (int s = 0; s < NT; ++s) {
      __syncthreads();
      column(av);
      new_row(s);
      __syncthreads();
      if (s < NH) {
        if (s + 1 < NH) rank16(av, sh.sR[s & 1], s + 1, NH);
        if (s == 1 || s == 2) rank16(avp, sh.sR[(s - 1) & 1], NH, NT);
        if (s >= 2) rank16(av, sh.sR[s & 1], NH, NT);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) avp[kk] = av[kk];
      } else if (w == s) {
        get_row(sh.sR[s & 1], NH);
      } else {
        m[s] = v4{0, 0, 0, 0};
        rank16(av, sh.sR[s & 1], NH, NT);
      }
      if (s + 1 < NT) {
        put(&sh.sC[w * BT][0], BT + 2, m[s + 1 < NT ? s + 1 : 0]);
        if (s + 1 >= NH && w == s + 1) put_row(sh.sRo, NH);
        if (s + 2 >= NH && s + 2 < NT && w == s + 2) put(&sh.sD[0][0], BT + 1, m[s + 2 < NT ? s + 2 : 0]);
      }
    }
    store(NH, NT);
  }
}

template <class T, bool AGENT = false>
__device__ __forceinline__ void gj_body(const T* __restrict__ A, long lda, T* __restrict__ out, Scalars* sc,
                                        GjShared<T>& sh) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (wave == 0) {
    gj_pivots<T, AGENT>(A, lda, sc, sh);
  } else if ((wave & 3) == 0) {  // on the pivot wave's SIMD: no work
    for (int s = 0; s < 2 * (NB / 16); ++s) __syncthreads();
  } else {
    // tile rows of waves 1, 2, 3, 5, 6, 7, 9, 10, so that the three SIMDs share the updates
    const int w = (0x64753210 >> (4 * (wave - 1 - wave / 4))) & 15;
    if (w < NB / 32)
      gj_row<T, true, AGENT>(A, lda, out, w, sh);
    else
      gj_row<T, false, AGENT>(A, lda, out, w, sh);
  }
}
template <class T>
__global__ void __launch_bounds__(GJ_THREADS)
gj_inverse(const T* __restrict__ A, long lda, T* __restrict__ out, Scalars* sc) {
  __shared__ GjShared<T> sh;
  gj_body<T>(A, lda, out, sc, sh);
}

// The update of the panel's remaining columns by one block and the half inverses
// of the next diagonal block, in one launch: C -= X U with X (M x NB) and U (NB x
// N) at K = NB, C's first NB x NB corner the next block.  The corner's sixteen
// 32 x 32 tiles come first; the workgroup that stores the last of them inverts
// the corner (nobody waits), while the others form the rest in 64 x 128 tiles.
// Each gives the bits of gemm_tile.  Workgroups have the inversion's eleven
// waves and LDS, one per CU, and eight waves with 32 x 32 of C each; a tile takes K
// in two stages, the second in flight under the first's products.  28 us for up
// to one round of tiles (M x N = 1920 x 896 and less: 19 us of update, then 21 of
// inversion as launches of their own), 30 us at M = 2816.
template <class T>
struct UpdateStage {
  static constexpr int KS = NB / 2;
  T a[64][KS + 2];
  T b[KS][NB + 4];
};
template <class T>
union UpdateShared {
  GjShared<T> gj;
  Tile32<T, false> corner;
  UpdateStage<T> tile;
};

template <class T>
__device__ __forceinline__ void update_tile(const T* __restrict__ X, const T* __restrict__ U, T* __restrict__ C,
                                            long ld, UpdateStage<T>& sh) {
  typedef typename Mfma<T>::v4 v4;
  typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
  constexpr int PV = 16 / sizeof(T), KS = UpdateStage<T>::KS, KC = GemmCfg<T>::KC;
  constexpr int NA = 64 * KS / PV / 512, NBV = KS * NB / PV / 512;
  const int t = threadIdx.x, l = t & 63, li = l & 15, lg = l >> 4, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const bool work = w < 8;  // the other waves only keep step
  const int wr = (w & 1) * 32, wc = (w >> 1) * 32;
  vec ra[NA], rb[NBV];
  auto load = [&](int k0) {
#pragma unroll
    for (int q = 0; q < NA; ++q) {
      const int p = t + 512 * q;
      ra[q] = *reinterpret_cast<const vec*>(X + static_cast<long>(p / (KS / PV)) * ld + k0 + (p % (KS / PV)) * PV);
    }
#pragma unroll
    for (int q = 0; q < NBV; ++q) {
      const int p = t + 512 * q;
      rb[q] = *reinterpret_cast<const vec*>(U + static_cast<long>(k0 + p / (NB / PV)) * ld + (p % (NB / PV)) * PV);
    }
  };
  auto store = [&]() {
#pragma unroll
    for (int q = 0; q < NA; ++q) {
      const int p = t + 512 * q;
      *reinterpret_cast<vec*>(&sh.a[p / (KS / PV)][(p % (KS / PV)) * PV]) = ra[q];
    }
#pragma unroll
    for (int q = 0; q < NBV; ++q) {
      const int p = t + 512 * q;
      *reinterpret_cast<vec*>(&sh.b[p / (NB / PV)][(p % (NB / PV)) * PV]) = rb[q];
    }
  };
  T cv[2][2][4];
  v4 acc[2][2];
  if (work) {
    load(0);
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 2; ++y) {
        acc[x][y] = v4{0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < 4; ++r)
          cv[x][y][r] = C[static_cast<long>(wr + 16 * x + Mfma<T>::orow(l, r)) * ld + wc + 16 * y + li];
      }
  }
#pragma unroll
  for (int k0 = 0; k0 < NB; k0 += KS) {
    if (k0 > 0) __syncthreads();  // the first stage has been read
    if (work) store();
    __syncthreads();
    if (!work) continue;
    if (k0 + KS < NB) load(k0 + KS);
#pragma unroll
    for (int c = 0; c < KS / KC; ++c)
#pragma unroll
      for (int s = 0; s < KC / 4; ++s) {
        const int k = c * KC + lg * (KC / 4) + s;
        T fa[2], fb[2];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          fa[x] = sh.a[wr + 16 * x + li][k];
          fb[x] = sh.b[k][wc + 16 * x + li];
        }
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int y = 0; y < 2; ++y) acc[x][y] = Mfma<T>::mma(fa[x], fb[y], acc[x][y]);
      }
  }
  if (!work) return;
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        C[static_cast<long>(wr + 16 * x + Mfma<T>::orow(l, r)) * ld + wc + 16 * y + li] =
            fma(T(1), cv[x][y][r], T(-1) * acc[x][y][r]);
}

// u: the update (update_args, one segment, M and N multiples of NB); out: the
// next block's place in dinv; sc->arrivals counts the corner's tiles
template <class T>
__global__ void __launch_bounds__(GJ_THREADS)
update_invert(GemmArgs<T> u, T* __restrict__ out, Scalars* sc) {
  __shared__ UpdateShared<T> sh;
  __shared__ int last;
  constexpr int CORNER = (NB / 32) * (NB / 32);
  const int b = blockIdx.x;
  if (b >= CORNER) {
    const int nty = u.M / 64, i = b - CORNER;
    // column by column; the first without the corner's two row tiles
    const int bx = i < nty - 2 ? 0 : 1 + (i - (nty - 2)) / nty;
    const int by = i < nty - 2 ? i + 2 : (i - (nty - 2)) % nty;
    update_tile<T>(u.A + static_cast<long>(by) * 64 * u.lda, u.B[0] + bx * NB,
                   u.C[0] + static_cast<long>(by) * 64 * u.ldc[0] + bx * NB, u.lda, sh.tile);
    return;
  }
  if (threadIdx.x < 256)
    gemm_tile32<T, false, true>(u, b % (NB / 32), b / (NB / 32), sh.corner);
  else
    __syncthreads();  // the tile's one stage
  agent_settle();  // this wave's part of C is stored
  __syncthreads();
  if (threadIdx.x == 0) last = (atomicAdd(&sc->arrivals, 1) + 1) % CORNER == 0;
  __syncthreads();
  if (last) gj_body<T, true>(u.C[0], u.ldc[0], out, sc, sh.gj);
}
template <class T>
inline unsigned update_invert_blocks(const GemmArgs<T>& u) {
  return static_cast<unsigned>((NB / 32) * (NB / 32) + (u.M / 64) * (u.N[0] / NB) - 2);
}

// many diagonal blocks (of different problems) in one launch
template <class T>
struct GjJob {
  const T* A;
  long lda;
  T* out;
  Scalars* sc;
};

template <class T>
__global__ void __launch_bounds__(GJ_THREADS) gj_batched(const GjJob<T>* __restrict__ jobs) {
  __shared__ GjShared<T> sh;
  const GjJob<T> jb = jobs[blockIdx.x];
  gj_body<T>(jb.A, jb.lda, jb.out, jb.sc, sh);
}

// ----------------------------------------------------- panel inverses ---
// W_p = U_pp^-1 and V_p = L_pp^-1 for every 1024-wide panel p by recursive
// doubling over its 128-wide diagonal blocks:
//   [A B; 0 C]^-1 = [A^-1, -A^-1 B C^-1; 0, C^-1],
//   [I 0; E I]^-1 = [I, 0; -E, I] generalised to [X 0; E Y]^-1 = [X^-1, 0; -Y^-1 E X^-1, Y^-1],
// starting from W's diagonal blocks D_k^-1 and V's identity blocks.  Level b
// joins pairs of b-wide inverses; each join is two MFMA products, run for all
// panels and pairs in one launch per stage.
template <class T>
struct TriJob {
  const T* kf;
  long ldk;
  const T* dinv;
  int np;
  T* W;
  T* V;
  long ldw;
  T* tmp;      // tri_tmp_elems scratch
  long ldt;
};

// Workgroups that start the panel inverses of a model of np padded rows.
constexpr int TRI_STRIPS = HB / 16;
__host__ __device__ inline int tri_init_blocks(int np) { return np / NB * TRI_STRIPS; }

// The diagonal blocks of W_p and V_p: D_k^-1 and I.  The blocks on their other
// side are never read (the products with them take op(A) and B as triangular by
// blocks) and stay unwritten.
// D^-1 = [B11 B12; B21 B22] comes from [I1 T; A21 I2] (see gj_row) by
//   B21 = -I2 (A21 I1),  B11 = I1 - T B21,  B12 = -T I2,  B22 = I2;
// column strips of 16 are independent of each other, so a strip of each half
// makes one workgroup (wave w forms rows 16 w .. of each quarter).
template <class T>
__device__ __forceinline__ void tri_init_block(const TriJob<T>& j, int b) {
  typedef typename Mfma<T>::v4 v4;
  constexpr int BT = 16, KK = HB / 4;
  __shared__ T x[HB][BT + 2];
  const int k = b / TRI_STRIPS, c0 = b % TRI_STRIPS * BT;  // block, first column in each half
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
  const int li = l & 15, lg = l >> 4, row = w * BT;
  const T* D = j.dinv + static_cast<long>(k) * NB * NB;
  const int rl = k * NB % NB2;
  const long diag = (static_cast<long>(k * NB / NB2) * NB2 + rl) * j.ldw + rl;
  T* W = j.W + diag;
  // this wave's rows of T, A21 and I2, and the strips of I1 and I2
  T ft[KK], fa[KK], fi[KK], s1[KK], s2[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    fa[kk] = D[(HB + row + li) * NB + 4 * kk + lg];
    s1[kk] = D[(4 * kk + lg) * NB + c0 + li];
    fi[kk] = D[(HB + row + li) * NB + HB + 4 * kk + lg];
    ft[kk] = D[(row + li) * NB + HB + 4 * kk + lg];
    s2[kk] = D[(HB + 4 * kk + lg) * NB + HB + c0 + li];
  }
  v4 i1, i2;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    i1[r] = D[(row + Mfma<T>::orow(l, r)) * NB + c0 + li];
    i2[r] = D[(HB + row + Mfma<T>::orow(l, r)) * NB + HB + c0 + li];
  }
  auto put = [&](int i0, int j0, const v4& v) {
#pragma unroll
    for (int r = 0; r < 4; ++r) W[static_cast<long>(i0 + row + Mfma<T>::orow(l, r)) * j.ldw + j0 + c0 + li] = v[r];
  };
  auto keep = [&](const v4& v) {
#pragma unroll
    for (int r = 0; r < 4; ++r) x[row + Mfma<T>::orow(l, r)][li] = v[r];
  };
  const v4 zero = v4{0, 0, 0, 0};
  v4 u = zero, b12 = zero, b21 = zero;
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) u = Mfma<T>::mma(fa[kk], s1[kk], u);
  keep(u);
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) b12 = Mfma<T>::mma(-ft[kk], s2[kk], b12);
  put(0, HB, b12);
  put(HB, HB, i2);
  __syncthreads();
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) b21 = Mfma<T>::mma(-fi[kk], x[4 * kk + lg][li], b21);
  put(HB, 0, b21);
  __syncthreads();
  keep(b21);
  __syncthreads();
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) i1 = Mfma<T>::mma(-ft[kk], x[4 * kk + lg][li], i1);
  put(0, 0, i1);
  for (int e = threadIdx.x; e < NB * NB / TRI_STRIPS; e += 256) {
    const int i = NB / TRI_STRIPS * (b % TRI_STRIPS) + e / NB, c = e % NB;
    j.V[diag + static_cast<long>(i) * j.ldw + c] = i == c ? T(1) : T(0);
  }
}

template <class T>
__global__ void __launch_bounds__(256, 2) tri_init(TriJob<T> j) {
  tri_init_block<T>(j, blockIdx.x);
}

// Operands of one join at level b: panel p, pair q, matrix mat (0 W, 1 V),
// stage 0 (T = U12 W_bot, T = L21 V_top) or 1 (W12 = -W_top T,
// V21 = -V_bot T).  False when the pair has no bottom half.  Shared by the
// single-model kernel and the batch planner, so both compute identically.
template <class T>
__host__ __device__ inline bool tri_level_args(const TriJob<T>& j, int b, int stage, int p, int q, int mat,
                                               GemmArgs<T>& g) {
  const int nq = NB2 / (2 * b);
  const int c0 = p * NB2;
  const int L = j.np - c0 < NB2 ? j.np - c0 : NB2;
  const int o = 2 * b * q;
  if (o + b >= L) return false;
  const int bb = L - o - b < b ? L - o - b : b;
  T* Wp = j.W + static_cast<long>(p) * NB2 * j.ldw;
  T* Vp = j.V + static_cast<long>(p) * NB2 * j.ldw;
  T* tq = j.tmp + (static_cast<long>(p * nq + q) * 2 + mat) * b * j.ldt;
  const long ldw = j.ldw, ldk = j.ldk;
  g = GemmArgs<T>{};
  g.nseg = 1;
  g.beta = T(0);
  if (mat == 0) {
    if (stage == 0) {
      g.A = j.kf + static_cast<long>(c0 + o) * ldk + (c0 + o + b);
      g.lda = ldk; g.M = b; g.K = bb; g.alpha = T(1);
      g.B[0] = Wp + static_cast<long>(o + b) * ldw + (o + b); g.ldb[0] = ldw;
      g.C[0] = tq; g.ldc[0] = j.ldt; g.N[0] = bb;
      g.btri = 1;
    } else {
      g.A = Wp + static_cast<long>(o) * ldw + o;
      g.lda = ldw; g.M = b; g.K = b; g.alpha = T(-1);
      g.tri = 1;
      g.B[0] = tq; g.ldb[0] = j.ldt;
      g.C[0] = Wp + static_cast<long>(o) * ldw + (o + b); g.ldc[0] = ldw; g.N[0] = bb;
    }
  } else {
    if (stage == 0) {
      g.A = j.kf + static_cast<long>(c0 + o + b) * ldk + (c0 + o);
      g.lda = ldk; g.M = bb; g.K = b; g.alpha = T(1);
      g.B[0] = Vp + static_cast<long>(o) * ldw + o; g.ldb[0] = ldw;
      g.C[0] = tq; g.ldc[0] = j.ldt; g.N[0] = b;
      g.btri = 2;
    } else {
      g.A = Vp + static_cast<long>(o + b) * ldw + (o + b);
      g.lda = ldw; g.M = bb; g.K = bb; g.alpha = T(-1);
      g.tri = 2;
      g.B[0] = tq; g.ldb[0] = j.ldt;
      g.C[0] = Vp + static_cast<long>(o + b) * ldw + o; g.ldc[0] = ldw; g.N[0] = b;
    }
  }
  g.ntile[0] = (g.N[0] + GEMM_TILE - 1) / GEMM_TILE;
  g.ntile[1] = 0;
  return true;
}

// Grid: panels x pairs x 2 matrices x (b/TS)^2 tiles of TS x TS (the joins
// are short latency-bound products, so small tiles spread them over the CUs).
template <class T, int TS>
__global__ void __launch_bounds__(256, TS == 64 ? 4 : 2) tri_level(TriJob<T> j, int b, int stage) {
  const int tpg = (b / TS) * (b / TS);
  const int nq = NB2 / (2 * b);
  int blk = blockIdx.x;
  const int tile = blk % tpg;
  blk /= tpg;
  const int mat = blk % 2;
  blk /= 2;
  GemmArgs<T> g;
  if (!tri_level_args<T>(j, b, stage, blk / nq, blk % nq, mat, g)) return;
  const int ntx = (g.N[0] + TS - 1) / TS, nty = (g.M + TS - 1) / TS;
  if (tile >= ntx * nty) return;
  if constexpr (TS == 64) {
    gemm_tile<T, false, 64>(g, tile % ntx, tile / ntx);
  } else {
    __shared__ Tile32<T, false> sh;
    gemm_tile32<T, false>(g, tile % ntx, tile / ntx, sh);
  }
}

inline unsigned tri_level_blocks(int P2, int b, int ts) {
  return static_cast<unsigned>(P2) * (NB2 / (2 * b)) * 2 * (b / ts) * (b / ts);
}

// L block X = P D^-1 of one diagonal block, in place: 16 RB rows of P (NB
// columns) from [I1 T; A21 I2] (see gj_row):
//   Xb = (Pb - Pa T) I2,   Xa = (Pa - Xb A21) I1.
// A workgroup owns whole rows, so it may overwrite them once they are staged:
// no scratch copy of X and no launch to copy it back.  Wave w forms columns
// 16 w .. 16 w + 15 of each half; its operands of D (the same for every
// workgroup, so they come from L2) are loaded into registers whole, in flight
// together with the staging of P.
template <class T, int RB>
struct LblockShared {
  T p[16 * RB][NB + 2];
  T x[16 * RB][HB + 2];
};
template <class T, int RB>
__device__ __forceinline__ void lblock_rows(T* __restrict__ a0, long lda, const T* __restrict__ D,
                                            LblockShared<T, RB>& sh) {
  typedef typename Mfma<T>::v4 v4;
  typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
  constexpr int PV = 16 / sizeof(T), R = 16 * RB, KK = HB / 4;
  const int t = threadIdx.x, l = t & 63, li = l & 15, lg = l >> 4, wc = (t >> 6) * 16;
  constexpr int NV = R * NB / PV / 256;
  vec ra[NV];
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    const int p = t + 256 * q;
    ra[q] = *reinterpret_cast<const vec*>(a0 + static_cast<long>(p / (NB / PV)) * lda + (p % (NB / PV)) * PV);
  }
  T f[4][KK];  // columns wc + li of T, I2, A21, I1
#pragma unroll
  for (int h = 0; h < 4; ++h)
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const int i0 = (h == 1 || h == 2) ? HB : 0, j0 = h < 2 ? HB : 0;
      f[h][kk] = D[(i0 + 4 * kk + lg) * NB + j0 + wc + li];
    }
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    const int p = t + 256 * q;
    *reinterpret_cast<vec*>(&sh.p[p / (NB / PV)][(p % (NB / PV)) * PV]) = ra[q];
  }
  __syncthreads();  // every row is staged: its place in A may be overwritten
  v4 x[RB];
#pragma unroll
  for (int y = 0; y < RB; ++y) {  // Pb - Pa T
#pragma unroll
    for (int r = 0; r < 4; ++r) x[y][r] = sh.p[16 * y + Mfma<T>::orow(l, r)][HB + wc + li];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) x[y] = Mfma<T>::mma(-sh.p[16 * y + li][4 * kk + lg], f[0][kk], x[y]);
  }
#pragma unroll
  for (int y = 0; y < RB; ++y)  // own columns of Pb, which no other wave reads before the barrier
#pragma unroll
    for (int r = 0; r < 4; ++r) sh.p[16 * y + Mfma<T>::orow(l, r)][HB + wc + li] = x[y][r];
  __syncthreads();
#pragma unroll
  for (int y = 0; y < RB; ++y) {  // Xb
    x[y] = v4{0, 0, 0, 0};
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) x[y] = Mfma<T>::mma(sh.p[16 * y + li][HB + 4 * kk + lg], f[1][kk], x[y]);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      sh.x[16 * y + Mfma<T>::orow(l, r)][wc + li] = x[y][r];
      a0[static_cast<long>(16 * y + Mfma<T>::orow(l, r)) * lda + HB + wc + li] = x[y][r];
    }
  }
  __syncthreads();
#pragma unroll
  for (int y = 0; y < RB; ++y) {  // Pa - Xb A21
#pragma unroll
    for (int r = 0; r < 4; ++r) x[y][r] = sh.p[16 * y + Mfma<T>::orow(l, r)][wc + li];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) x[y] = Mfma<T>::mma(-sh.x[16 * y + li][4 * kk + lg], f[2][kk], x[y]);
#pragma unroll
    for (int r = 0; r < 4; ++r) sh.p[16 * y + Mfma<T>::orow(l, r)][wc + li] = x[y][r];
  }
  __syncthreads();
#pragma unroll
  for (int y = 0; y < RB; ++y) {  // Xa
    x[y] = v4{0, 0, 0, 0};
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) x[y] = Mfma<T>::mma(sh.p[16 * y + li][4 * kk + lg], f[3][kk], x[y]);
#pragma unroll
    for (int r = 0; r < 4; ++r)
      a0[static_cast<long>(16 * y + Mfma<T>::orow(l, r)) * lda + wc + li] = x[y][r];
  }
}
template <class T, int RB>
__global__ void __launch_bounds__(256, 2) lblock_inplace(T* __restrict__ A, long lda, const T* __restrict__ D) {
  __shared__ LblockShared<T, RB> sh;
  lblock_rows<T, RB>(A + static_cast<long>(blockIdx.x) * (16 * RB) * lda, lda, D, sh);
}

// rows: a multiple of NB.  Past 4096 rows (one workgroup per CU at 16 rows)
// 32 rows per workgroup halve the reads of D.
constexpr long LBLOCK_ROWS16 = 4096;
template <class T>
inline hipError_t lblock_run(T* A, long lda, const T* D, int rows, hipStream_t s) {
  ProfScope prof(s, gemm_prof_kind<T>(false), 2.0 * rows * NB * NB, sizeof(T) * (2.0 * rows + NB) * NB);
  if (rows > LBLOCK_ROWS16)
    hipLaunchKernelGGL((lblock_inplace<T, 2>), dim3(static_cast<unsigned>(rows / 32)), dim3(256), 0, s, A, lda, D);
  else
    hipLaunchKernelGGL((lblock_inplace<T, 1>), dim3(static_cast<unsigned>(rows / 16)), dim3(256), 0, s, A, lda, D);
  return hipGetLastError();
}

// dst rows [0, rows) <- src, columns < cols (same precision)
template <class T>
__global__ void __launch_bounds__(256)
copy_rows(const T* __restrict__ src, long lds, T* __restrict__ dst, long ldd, int cols) {
  const long i = blockIdx.x;
  // eight loads per thread in flight (addresses clamped into the row)
  for (int j0 = threadIdx.x; j0 < cols; j0 += 8 * blockDim.x) {
    T v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = src[i * lds + min(j0 + u * static_cast<int>(blockDim.x), cols - 1)];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int j = j0 + u * static_cast<int>(blockDim.x);
      if (j < cols) dst[i * ldd + j] = v[u];
    }
  }
}

// dst (D, rows < n, cols <= n) <- src (S)
template <class S, class D>
__global__ void __launch_bounds__(256)
copy_block(const S* __restrict__ src, long lds, int n, D* __restrict__ dst, long ldd) {
  const int i = blockIdx.x;
  for (int j0 = threadIdx.x; j0 <= n; j0 += 8 * blockDim.x) {  // eight loads per thread in flight
    S v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = src[static_cast<long>(i) * lds + min(j0 + u * static_cast<int>(blockDim.x), n)];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int j = j0 + u * static_cast<int>(blockDim.x);
      if (j <= n) dst[static_cast<long>(i) * ldd + j] = static_cast<D>(v[u]);
    }
  }
}
// max of v over a 256-thread block, merged into *target with one atomic per
// block (every thread of the block must call it)
__device__ inline void block_max(double v, double* target) {
  __shared__ double red[4];
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) atomic_max_nonneg(target, fmax(fmax(red[0], red[1]), fmax(red[2], red[3])));
}

// R = E - X  (rows < n, cols <= n), E from F and eps on the fly
__global__ void __launch_bounds__(256)
residual_init(const double* __restrict__ F, long ldf, int n, const double* __restrict__ eps,
              const double* __restrict__ X, long ldx, double* __restrict__ R, long ldr) {
  const int i = blockIdx.x;
  const double* f = F + static_cast<long>(i) * ldf;
  for (int j = threadIdx.x; j <= n; j += blockDim.x) {
    double e = (j < n) ? f[j] * eps[j] : f[n];
    R[static_cast<long>(i) * ldr + j] = e - X[static_cast<long>(i) * ldx + j];
  }
}

// R = G - L  (rows < n, cols <= n)
__global__ void __launch_bounds__(256)
adj_residual_init(const double* __restrict__ G, long ldg, int n, const double* __restrict__ L, long ldl,
                  double* __restrict__ R, long ldr) {
  const int i = blockIdx.x;
  for (int j = threadIdx.x; j <= n; j += blockDim.x)
    R[static_cast<long>(i) * ldr + j] = G[static_cast<long>(i) * ldg + j] - L[static_cast<long>(i) * ldl + j];
}

// Y32 <- R (rows < n, cols <= n), records max |R|
__global__ void __launch_bounds__(256)
residual_to_rhs(const double* __restrict__ R, long ldr, int n, float* __restrict__ Y, long ldy,
                Scalars* sc) {
  const int i = blockIdx.x;
  double m = 0.0;
  int bad = 0;
  for (int j = threadIdx.x; j <= n; j += blockDim.x) {
    double v = R[static_cast<long>(i) * ldr + j];
    bad |= !(fabs(v) <= 1.0e300);
    m = fmax(m, fabs(v));
    Y[static_cast<long>(i) * ldy + j] = static_cast<float>(v);
  }
  if (bad) raise_status(&sc->status, RAD_ENONFINITE);
  block_max(m, &sc->max_r);
}

// X += Y32 (rows < n, cols <= n), records max |delta|
__global__ void __launch_bounds__(256)
apply_correction(const float* __restrict__ Y, long ldy, int n, double* __restrict__ X, long ldx,
                 Scalars* sc) {
  const int i = blockIdx.x;
  double m = 0.0;
  for (int j = threadIdx.x; j <= n; j += blockDim.x) {
    double d = static_cast<double>(Y[static_cast<long>(i) * ldy + j]);
    m = fmax(m, fabs(d));
    X[static_cast<long>(i) * ldx + j] += d;
  }
  block_max(m, &sc->max_d);
}

// Y (T, np rows x ldy, zero outside n x (n+1)) <- G (fp64); a non-finite
// entry of G raises RAD_ENONFINITE
template <class T>
__global__ void __launch_bounds__(256)
load_rhs(const double* __restrict__ G, long ldg, int n, T* __restrict__ Y, long ldy, Scalars* sc) {
  const int i = blockIdx.x;
  T* y = Y + static_cast<long>(i) * ldy;
  int bad = 0;
  // eight loads per thread in flight: addresses clamped into G, entries
  // outside its n x (n + 1) range replaced by zero afterwards
  const long gi = static_cast<long>(min(i, n - 1)) * ldg;
  for (long j0 = threadIdx.x; j0 < ldy; j0 += 8 * blockDim.x) {
    double g[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) g[u] = G[gi + min(j0 + u * static_cast<long>(blockDim.x), static_cast<long>(n))];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const long j = j0 + u * static_cast<long>(blockDim.x);
      if (j >= ldy) break;
      const bool in = j <= n && i < n;
      const double v = __builtin_unpredictable(in) ? g[u] : 0.0;
      bad |= in && !(fabs(v) <= 1.0e300);
      y[j] = static_cast<T>(v);
    }
  }
  if (bad) raise_status(&sc->status, RAD_ENONFINITE);
}


// REF closure residual: one wave per row sums the n+1 entries; the block's
// maximum of |s_i - 1| goes to blk[blockIdx.x] (no same-address atomics).
__global__ void __launch_bounds__(256)
ref_closure(const double* __restrict__ B, long ldb, int n, double* __restrict__ blk) {
  __shared__ double red[4];
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + w;
  double s = 0.0;
  if (row < n) {
    const double* __restrict__ b = B + static_cast<long>(row) * ldb;
    // eight loads per lane in flight (addresses clamped into the row); the sum
    // still runs over the columns in increasing order
    for (int j0 = l; j0 <= n; j0 += 8 * 64) {
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = b[min(j0 + 64 * u, n)];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (j0 + 64 * u <= n) s += v[u];
    }
  }
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if (l == 0) red[w] = (row < n) ? fabs(s - 1.0) : 0.0;
  __syncthreads();
  if (threadIdx.x == 0) blk[blockIdx.x] = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
}

// REF reciprocity residual max |eps_i A_i B_ij - eps_j A_j B_ji| (eq. 4.4):
// one workgroup per 64 x 64 tile pair (I, J), I <= J; the partner tile goes
// through LDS so both are read as rows; the pair's maximum goes to blk[pair].
__global__ void __launch_bounds__(256)
ref_reciprocity(const double* __restrict__ B, long ldb, int n, int t, const double* __restrict__ eps,
                const double* __restrict__ area, double* __restrict__ blk) {
  __shared__ double sT[64][65];
  __shared__ double wI[64], wJ[64];
  __shared__ double red[4];
  int I, J;
  pair_from_index(blockIdx.x, t, I, J);
  const int tid = threadIdx.x, c = tid & 63, rg = tid >> 6;
  if (tid < 64) {
    const int i = I * 64 + tid;
    wI[tid] = i < n ? eps[i] * area[i] : 0.0;
  } else if (tid < 128) {
    const int j = J * 64 + tid - 64;
    wJ[tid - 64] = j < n ? eps[j] * area[j] : 0.0;
  }
  double v[16];
#pragma unroll
  for (int m = 0; m < 16; ++m) {  // partner tile (J, I)
    const int i = J * 64 + rg + 4 * m, j = I * 64 + c;
    v[m] = (i < n && j < n) ? B[static_cast<long>(i) * ldb + j] : 0.0;
  }
  double u[16];
#pragma unroll
  for (int m = 0; m < 16; ++m) {  // own tile (I, J)
    const int i = I * 64 + rg + 4 * m, j = J * 64 + c;
    u[m] = (i < n && j < n) ? B[static_cast<long>(i) * ldb + j] : 0.0;
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < 16; ++m) sT[rg + 4 * m][c] = wJ[rg + 4 * m] * v[m];
  __syncthreads();
  double mx = 0.0;
#pragma unroll
  for (int m = 0; m < 16; ++m) {
    const int r = rg + 4 * m;
    mx = fmax(mx, fabs(wI[r] * u[m] - sT[c][r]));
  }
  for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off));
  if (c == 0) red[rg] = mx;
  __syncthreads();
  if (tid == 0) blk[blockIdx.x] = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
}

// out[0] = max of the closure block maxima, out[1] = of the reciprocity ones
__global__ void __launch_bounds__(256)
ref_final(const double* __restrict__ bc, int nc, const double* __restrict__ br, long nr, double* __restrict__ out) {
  __shared__ double red[2][4];
  double a = 0.0, b = 0.0;
  for (int q = threadIdx.x; q < nc; q += 256) a = fmax(a, bc[q]);
  for (long q = threadIdx.x; q < nr; q += 256) b = fmax(b, br[q]);
  for (int off = 32; off > 0; off >>= 1) {
    a = fmax(a, __shfl_xor(a, off));
    b = fmax(b, __shfl_xor(b, off));
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    red[0][w] = a;
    red[1][w] = b;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    out[0] = fmax(fmax(red[0][0], red[0][1]), fmax(red[0][2], red[0][3]));
    out[1] = fmax(fmax(red[1][0], red[1][1]), fmax(red[1][2], red[1][3]));
  }
}

// grad_eps[k] = sum_i Lambda_ik F_ik: partial sums over row chunks of 128,
// then a fixed-order sum of the partials (reproducible).
constexpr int GE_ROWS = 128;
__global__ void __launch_bounds__(256)
adj_grad_eps_partial(const double* __restrict__ L, long ldl, const double* __restrict__ F, long ldf,
                     int n, double* __restrict__ part) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  const int c = blockIdx.y;
  if (k >= n) return;
  const int i0 = c * GE_ROWS, i1 = min(n, i0 + GE_ROWS);
  double s = 0.0;
  constexpr int U = 8;  // rows in flight; the sum stays in row order
  for (int a = i0; a < i1; a += U) {
    double x[U], y[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long i = min(a + u, i1 - 1);
      x[u] = L[i * ldl + k];
      y[u] = F[i * ldf + k];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (a + u < i1) s += x[u] * y[u];
  }
  part[static_cast<long>(c) * n + k] = s;
}

__global__ void __launch_bounds__(256)
adj_grad_eps_final(const double* __restrict__ part, int n, int chunks, double* __restrict__ ge) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  double s = 0.0;
  for (int c = 0; c < chunks; ++c) s += part[static_cast<long>(c) * n + k];
  ge[k] = s;
}

// grad_rho[k] = (1/rho_k) sum_j B_kj (Lambda_kj - G_kj), for small rho_k in the
// direct form sum_j B_kj sum_i F_ik Lambda_ij; one workgroup per row
__global__ void __launch_bounds__(256)
adj_grad_rho(const double* __restrict__ L, long ldl, const double* __restrict__ F, long ldf,
             const double* __restrict__ G, long ldg, const double* __restrict__ B, long ldb,
             const double* __restrict__ rho, int n, double* __restrict__ gr) {
  const int k = blockIdx.x;
  __shared__ double red[4];
  const double r = rho[k];
  const double* bk = B + static_cast<long>(k) * ldb;
  double acc = 0.0;
  if (r >= 1e-3) {
    const double *lk = L + static_cast<long>(k) * ldl, *gk = G + static_cast<long>(k) * ldg;
    constexpr int U = 4;
    for (int j0 = threadIdx.x; j0 <= n; j0 += 256 * U) {
      double x[U], y[U], z[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = min(j0 + 256 * u, n);
        x[u] = bk[j];
        y[u] = lk[j];
        z[u] = gk[j];
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (j0 + 256 * u <= n) acc += x[u] * (y[u] - z[u]);
    }
  } else {
    for (int j = threadIdx.x; j <= n; j += 256) {
      double t = 0.0;
      for (int i = 0; i < n; ++i) t += F[static_cast<long>(i) * ldf + k] * L[static_cast<long>(i) * ldl + j];
      acc += bk[j] * t;
    }
  }
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    const double s = red[0] + red[1] + red[2] + red[3];
    gr[k] = r >= 1e-3 ? s / r : s;
  }
}

}  // namespace
}  // namespace rad
