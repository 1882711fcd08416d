// The U side of the partial Fourier form (complex64, r <= 8): the U update of a GDmin
// iteration over many workgroups and the spectral start in one launch.  The same plan as
// the real forms (update.h, subspace.h), with conjugate transposes:
//
//  k_frows : a workgroup per 64 rows: the rows of grad_U f = sum_k h_k b_k^H, U_prev = U, and
//            the block's part of the FP64 Gram X^H X of X = U - eta grad;
//  k_fapply: a row per thread: every workgroup adds the parts in order and factors the
//            Gram, then U = X R^{-1}; one more workgroup does the bookkeeping;
//  k_fsub  : start block, subspace iteration and stop rule in one launch (meet.h).
//
// None is bound by bytes: 64-row blocks are latency of q loads per wave, the rest is the
// serial factorisation.  Measured (launch to launch): k_frows 10 us at n = 9216, q = 64, r = 6
// and 28 us at n = 400, q = 400, r = 4, where blocks of 256 rows by one thread per row took 25 and
// 74 us; k_fapply 10 and 8 us, where two Gram passes in six launches took 37 and 22 us and the
// first iteration 1.05 ms more for eta by one thread's Jacobi sweeps.  The start of 100 steps at
// n = 400: 0.4 ms, in eight launches a step 2.8 ms.
#pragma once
#include "launch.h"
#include "meet.h"
#include "uside.h"

namespace altg {

namespace {

constexpr int kFRowsWaves = 16;
constexpr int kFApplyRows = 256;
constexpr int kFSubThreads = 256, kFSubWaves = kFSubThreads / 64;
constexpr int kFSubBlocksMax = 96;

__device__ __forceinline__ double2 c_fma(double2 a, double2 b, double2 c) {   // a b + c
  return make_double2(fma(a.x, b.x, fma(-a.y, b.y, c.x)), fma(a.x, b.y, fma(a.y, b.x, c.y)));
}
__device__ __forceinline__ double2 c_fma_conj(double2 a, double2 b, double2 c) {   // a conj(b) + c
  return make_double2(fma(a.x, b.x, fma(a.y, b.y, c.x)), fma(a.y, b.x, fma(-a.x, b.y, c.y)));
}

// Entry (i, j) of a Hermitian matrix stored as its upper triangle, row by row.
__device__ __forceinline__ double2 herm_entry(const double2* t, int i, int j, int r) {
  const double2 v = t[tri_index(i, j, r)];
  return i <= j ? v : make_double2(v.x, -v.y);
}

// In-place lower Cholesky factor W = L L^H (real positive diagonal) of the Hermitian
// positive definite r x r matrix W (LDS, row-major, r <= 8) by one wave, right-looking:
// a lane keeps one entry; a step exchanges the current column through LDS.  1 / L_jj in
// rdiag, the smallest and largest pivot in lo and hi.  False if a pivot is not positive.
__device__ inline bool wave_cholesky_span_c(double2* W, double* rdiag, int r, double& lo, double& hi) {
  const int lane = threadIdx.x & 63;
  lo = hi = 0.0;
  const int ri = lane < r * r ? lane / r : 0;
  int ci = lane < r * r ? lane - (lane / r) * r : r;   // r: no entry
  if (ci > ri) ci = r;
  wave_lds_fence();
  double2 w = ci < r ? W[lane] : make_double2(0.0, 0.0);
  for (int j = 0; j < r; ++j) {
    if (ci == j) W[ri * r + j] = w;
    wave_lds_fence();
    const double piv = W[j * r + j].x;
    if (!(piv > 0.0) || !isfinite(piv)) return false;
    lo = j == 0 || piv < lo ? piv : lo;
    hi = j == 0 || piv > hi ? piv : hi;
    const double inv = fast_rcp(piv);
    if (ci > j && ci < r) {   // w -= W[ri][j] conj(W[ci][j]) / piv
      const double2 a = W[ri * r + j], b = W[ci * r + j];
      w = c_fma_conj(make_double2(-a.x * inv, -a.y * inv), b, w);
    }
  }
  if (lane < r) rdiag[lane] = fast_rsqrt(W[lane * r + lane].x);
  wave_lds_fence();
  if (ci < r) {
    const double s = rdiag[ci];
    const double2 v = W[ri * r + ci];
    W[ri * r + ci] = make_double2(v.x * s, ci == ri ? 0.0 : v.y * s);
  }
  wave_lds_fence();
  return true;
}

// Largest eigenvalue of the Hermitian positive semidefinite r x r matrix M (LDS,
// overwritten; T: scratch) by one wave, by squarings as wave_lambda_max.
__device__ inline double wave_lambda_max_c(double2* M, double2* T, int r) {
  const int lane = threadIdx.x & 63, rr = r * r;
  wave_lds_fence();
  double tr = 0.0;
  for (int i = 0; i < r; ++i) tr += M[i * r + i].x;
  if (!(tr > 0.0) || !isfinite(tr)) return 0.0;
  const double first = tr;
  double acc = 0.0, p = 0.5, scale = 1.0 / tr;
  for (int k = 0; k < 56; ++k) {
    if (lane < rr) {
      const int i = lane / r, j = lane - i * r;
      double2 s = make_double2(0.0, 0.0);
      for (int l = 0; l < r; ++l) {
        const double2 a = M[i * r + l], b = M[l * r + j];
        s = c_fma(make_double2(a.x * scale, a.y * scale), make_double2(b.x * scale, b.y * scale), s);
      }
      T[lane] = s;
    }
    wave_lds_fence();
    double t = 0.0;
    for (int i = 0; i < r; ++i) t += T[i * r + i].x;
    if (!(t > 0.0) || !isfinite(t)) return 0.0;
    acc = fma(p, log(t), acc);
    if (t >= 1.0 - 1e-15) break;
    p *= 0.5;
    scale = 1.0 / t;
    double2* x = M;
    M = T;
    T = x;
  }
  return first * exp(acc);
}

// x <- x R^{-1} for one row, R = L^H: x[c] = (x[c] - sum_{p < c} x[p] conj(L[c][p])) / L[c][c].
__device__ __forceinline__ void solve_row_c(double2 (&x)[kFRMax], const double2* L, const double* rdiag, int r) {
#pragma unroll
  for (int c = 0; c < kFRMax; ++c) {
    if (c < r) {
      double2 t = x[c];
#pragma unroll
      for (int p = 0; p < kFRMax; ++p)
        if (p < c) t = c_fma_conj(make_double2(-x[p].x, -x[p].y), L[c * r + p], t);
      x[c] = make_double2(t.x * rdiag[c], t.y * rdiag[c]);
    }
  }
}

// Part of X^H Y over the 64 rows in LDS (row-major, r wide): the upper triangle (a <= b) row
// by row with sym, all r^2 entries without; by a workgroup of WV waves.
template <int WV>
__device__ __forceinline__ void rows_gram64_c(const double2* X, const double2* Y, int r, bool sym, double2* dst) {
  const int lane = threadIdx.x & 63, wave = wave_id();
  const int E = sym ? r * (r + 1) / 2 : r * r;
  for (int e = wave; e < E; e += WV) {
    int a = 0, b = 0;
    if (sym) tri_entry(e, r, a, b);
    else { a = e / r; b = e - a * r; }
    const double2 x = X[lane * r + a], y = Y[lane * r + b];   // conj(x) y
    const double sr = wave_sum_dpp(fma(x.x, y.x, x.y * y.y));
    const double si = wave_sum_dpp(fma(x.x, y.y, -x.y * y.x));
    if (lane == 0) dst[e] = make_double2(sr, si);
  }
}

// Rows 64 jb .. + 63 of sum_k h_k conj(b_k)^T over the columns k0 <= k < k1, by a workgroup
// of WV waves: wave w takes k = k0 + w, then every WV-th, a row per lane; the waves'
// sums are added in order (above 8 waves, w and w + 8 first).  Thread i < 64 r gets row
// i / r, column i % r through put(i, value).
template <int R, int WV, class Put>
__device__ __forceinline__ void frows_grad(const float2* H, const float2* B, int n, int r, int jb, int k0, int k1,
                                           float2 (*red)[64][kFRMax + 1], Put put) {
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
  const int j = jb * 64 + lane, jc = j < n ? j : n - 1;
  float2 acc[R];
#pragma unroll
  for (int c = 0; c < R; ++c) acc[c] = make_float2(0.f, 0.f);
  constexpr int KU = 8;   // loads in flight per lane; the k order of the sum does not depend on it
  for (int kb = k0 + wave; kb < k1; kb += WV * KU) {
    float2 h[KU];
#pragma unroll
    for (int u = 0; u < KU; ++u) {
      const int k = kb + u * WV;
      h[u] = H[(long long)(k < k1 ? k : k0) * n + jc];
    }
#pragma unroll
    for (int u = 0; u < KU; ++u) {
      const int k = kb + u * WV;
      if (k < k1) {
#pragma unroll
        for (int c = 0; c < R; ++c)
          if (c < r) {
            const float2 b = B[(long long)k * r + c];
            acc[c].x = fmaf(h[u].x, b.x, fmaf(h[u].y, b.y, acc[c].x));
            acc[c].y = fmaf(h[u].y, b.x, fmaf(-h[u].x, b.y, acc[c].y));
          }
      }
    }
  }
  constexpr int WS = WV > 8 ? 8 : WV;
  if (wave >= WV - WS)
#pragma unroll
    for (int c = 0; c < R; ++c) red[wave - (WV - WS)][lane][c] = acc[c];
  __syncthreads();
  if constexpr (WV > 8) {
    if (wave < WS)
#pragma unroll
      for (int c = 0; c < R; ++c) {
        const float2 o = red[wave][lane][c];
        red[wave][lane][c] = make_float2(o.x + acc[c].x, o.y + acc[c].y);
      }
    __syncthreads();
  }
  for (int i = tid; i < 64 * r; i += 64 * WV) {
    const int rw = i / r, c = i - rw * r;
    float2 g = red[0][rw][c];
#pragma unroll
    for (int w = 1; w < WS; ++w) {
      g.x += red[w][rw][c].x;
      g.y += red[w][rw][c].y;
    }
    put(i, g);
  }
}

template <int WV, class Put>
__device__ __forceinline__ void frows_grad_r(const float2* H, const float2* B, int n, int r, int jb, int k0, int k1,
                                             float2 (*red)[64][kFRMax + 1], Put put) {
  if (r <= 4) frows_grad<4, WV>(H, B, n, r, jb, k0, k1, red, put);
  else frows_grad<8, WV>(H, B, n, r, jb, k0, k1, red, put);
}

// Sum of `cnt` doubles (offset off of each unit's part, ps apart) over all units into dst
// (LDS); entry e over a contiguous range of units per group of threads, then the groups in order.
template <int TH>
__device__ __forceinline__ void sum_parts_c(const double* part, int ps, int off, int cnt, int units, double* tmp,
                                            double* dst) {
  const int tid = threadIdx.x, grp = sum_groups(TH, cnt, units);
  __syncthreads();
  for (int e = tid; e < cnt * grp; e += TH) {
    const int g = e / cnt, en = e - g * cnt;
    const int b0 = units * g / grp, b1 = units * (g + 1) / grp;
    tmp[e] = sum_strided(part + (long long)b0 * ps + off + en, ps, b1 - b0);
  }
  __syncthreads();
  for (int e = tid; e < cnt; e += TH) {
    double s = tmp[e];
    for (int g = 1; g < grp; ++g) s += tmp[g * cnt + e];
    dst[e] = s;
  }
  __syncthreads();
}

union FRowsShared {
  float2 red[8][64][kFRMax + 1];
  struct {
    double2 X[64 * kFRMax], Y[64 * kFRMax];
  } rows;
};

}  // namespace

enum { FUPD_STEP = 1, FUPD_FIRST = 2 };

__global__ __launch_bounds__(64 * kFRowsWaves) void k_frows(FUpdArgs a) {
  __shared__ FRowsShared S;
  const int tid = threadIdx.x, jb = blockIdx.x;
  const int n = a.n, r = a.r, E = r * (r + 1) / 2;
  const bool have = a.ctl->eta_set != 0;
  if (jb == 0 && tid == 0) *a.upd = have ? FUPD_STEP : FUPD_FIRST;
  const double eta = have ? a.ctl->eta : 0.0;
  const long long base = (long long)jb * 64 * r, nr = (long long)n * r;
  float2 g = make_float2(0.f, 0.f);   // thread i < 64 r: row i / r, column i % r
  frows_grad_r<kFRowsWaves>(a.H, a.B, n, r, jb, 0, a.q, S.red, [&](int, float2 v) { g = v; });
  __syncthreads();
  if (tid < 64 * r) {
    double2 x = make_double2(0.0, 0.0), y = x;
    const long long i = base + tid;
    if (i < nr) {
      a.G[i] = g;
      const float2 u = a.U[i];
      a.Uprev[i] = u;
      x = have ? make_double2(fma(-eta, (double)g.x, (double)u.x), fma(-eta, (double)g.y, (double)u.y))
               : make_double2(u.x, u.y);
      y = make_double2(g.x, g.y);
    }
    S.rows.X[tid] = x;
    S.rows.Y[tid] = y;
  }
  __syncthreads();
  // eta known: the Gram of X; at t = 1: U^H U, G^H G and U^H G
  double2* dst = reinterpret_cast<double2*>(a.part) + (long long)jb * (2 * E + r * r);
  rows_gram64_c<kFRowsWaves>(S.rows.X, S.rows.X, r, true, dst);
  if (!have) {
    rows_gram64_c<kFRowsWaves>(S.rows.Y, S.rows.Y, r, true, dst + E);
    rows_gram64_c<kFRowsWaves>(S.rows.X, S.rows.Y, r, false, dst + 2 * E);
  }
}

__global__ __launch_bounds__(kFApplyRows) void k_fapply(FUpdArgs a) {
  constexpr int kPE = kFRMax * (kFRMax + 1) + kFRMax * kFRMax;   // complex values of a part
  __shared__ double tmp[2 * kPE];
  __shared__ double2 W[kPE], A[2 * kFRMax * kFRMax];
  __shared__ __attribute__((aligned(16))) float2 rows[kFApplyRows][kFRMax + 1];   // second pass: rounded rows
  __shared__ double rdiag[kFRMax], eta_s;
  __shared__ int mode_s;
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_id(), jb = blockIdx.x;
  const int n = a.n, r = a.r, rr = r * r, E = r * (r + 1) / 2, PE = 2 * E + rr, units = (n + 63) / 64;
  const bool first = *a.upd == FUPD_FIRST;
  const int j = jb * kFApplyRows + tid;
  const long long o = (long long)j * r;
  float2 ru[kFRMax], rg[kFRMax];   // this thread's row, loaded ahead of the factorisation
#pragma unroll
  for (int c = 0; c < kFRMax; ++c) {
    ru[c] = c < r && j < n ? a.Uprev[o + c] : make_float2(0.f, 0.f);
    rg[c] = c < r && j < n ? a.G[o + c] : make_float2(0.f, 0.f);
  }
  sum_parts_c<kFApplyRows>(a.part, 2 * PE, 0, 2 * (first ? PE : E), units, tmp, reinterpret_cast<double*>(W));
  if (wave == 0) {
    double eta = first ? 0.0 : a.ctl->eta;
    if (first) {
      if (lane < rr) A[lane] = herm_entry(W + E, lane / r, lane % r, r);
      const double lam = wave_lambda_max_c(A, A + kFRMax * kFRMax, r);
      eta = lam > 0.0 ? a.eta_c / sqrt(lam) : 0.0;
      wave_lds_fence();
    }
    if (lane < rr) {
      const int i = lane / r, jj = lane % r;
      double2 v = herm_entry(W, i, jj, r);
      if (first) {   // U^H U - eta (U^H G + G^H U) + eta^2 G^H G
        const double2 ug = W[2 * E + i * r + jj], gu = W[2 * E + jj * r + i], gg = herm_entry(W + E, i, jj, r);
        v.x = v.x - eta * (ug.x + gu.x) + eta * eta * gg.x;
        v.y = v.y - eta * (ug.y - gu.y) + eta * eta * gg.y;
      }
      A[lane] = v;
    }
    double lo, hi;
    const bool pd = wave_cholesky_span_c(A, rdiag, r, lo, hi);
    if (lane == 0) {
      eta_s = eta;
      mode_s = !pd ? 0 : (lo >= kPivotSpan * hi ? 1 : 2);
    }
  }
  __syncthreads();
  const double eta = eta_s;
  bool ok = mode_s != 0;
  double2 x[kFRMax];
  auto row_x = [&](const float2 (&u)[kFRMax], const float2 (&g)[kFRMax]) {
#pragma unroll
    for (int c = 0; c < kFRMax; ++c)
      x[c] = make_double2(fma(-eta, (double)g[c].x, (double)u[c].x), fma(-eta, (double)g[c].y, (double)u[c].y));
    solve_row_c(x, A, rdiag, r);
  };
  const bool has_rows = jb * kFApplyRows < n;   // the last workgroup has none
  if (mode_s == 2 && has_rows) {   // an ill-conditioned X: once more on the rounded rows, each solved once
    const int grps = kFApplyRows / E, en = tid % E, gr = tid / E;   // a thread: an entry over every grps-th row
    int ra, rb;
    tri_entry(en, r, ra, rb);
    double sr = 0.0, si = 0.0;
    for (int i0 = 0; i0 < n; i0 += kFApplyRows) {
      const int i = i0 + tid;
      float2 u[kFRMax], g[kFRMax];   // rows at or beyond n are zero
#pragma unroll
      for (int c = 0; c < kFRMax; ++c) {
        u[c] = c < r && i < n ? a.Uprev[(long long)i * r + c] : make_float2(0.f, 0.f);
        g[c] = c < r && i < n ? a.G[(long long)i * r + c] : make_float2(0.f, 0.f);
      }
      row_x(u, g);
#pragma unroll
      for (int c = 0; c < kFRMax; ++c)
        if (c < r) rows[tid][c] = make_float2((float)x[c].x, (float)x[c].y);
      __syncthreads();
      if (gr < grps) {
#pragma unroll 8
        for (int k = gr; k < kFApplyRows; k += grps) {
          const float2 xa = rows[k][ra], xb = rows[k][rb];
          sr = fma((double)xa.x, (double)xb.x, fma((double)xa.y, (double)xb.y, sr));
          si = fma((double)xa.x, (double)xb.y, fma(-(double)xa.y, (double)xb.x, si));
        }
      }
      __syncthreads();
    }
    double2* sum = reinterpret_cast<double2*>(&rows[0][0]);   // 4 KiB of 18
    sum[tid] = make_double2(sr, si);
    __syncthreads();
    if (tid < E) {
      for (int g = 1; g < grps; ++g) {
        sr += sum[g * E + tid].x;
        si += sum[g * E + tid].y;
      }
      W[tid] = make_double2(sr, si);
    }
    __syncthreads();
  }
  if (ok && j < n) row_x(ru, rg);
  if (mode_s == 2 && has_rows) {
    __syncthreads();   // the first factor has been used
    if (wave == 0) {
      if (lane < rr) A[lane] = herm_entry(W, lane / r, lane % r, r);
      double lo, hi;
      const bool pd = wave_cholesky_span_c(A, rdiag, r, lo, hi);
      if (lane == 0) mode_s = pd ? 1 : 0;
    }
    __syncthreads();
    ok = mode_s != 0;
    if (ok && j < n) {
#pragma unroll
      for (int c = 0; c < kFRMax; ++c) x[c] = make_double2((double)(float)x[c].x, (double)(float)x[c].y);
      solve_row_c(x, A, rdiag, r);
    }
  }
  if (ok && j < n)
#pragma unroll
    for (int c = 0; c < kFRMax; ++c)
      if (c < r) a.U[o + c] = make_float2((float)x[c].x, (float)x[c].y);
  if (has_rows) {
    if (!ok && jb == 0 && tid == 0) atomicOr(&a.ctl->err, 2);
    return;
  }
  // the last workgroup (no rows): eta, the residual of the iteration and the counters
  double s = 0.0;
  int fl = 0;
  for (int k = tid; k < a.q; k += kFApplyRows) {
    s += a.colrr[k];
    fl |= a.colflags[k];
  }
  if (fl) atomicOr(&a.ctl->err, fl);
  s = wave_sum_dpp(s);
  __syncthreads();
  if (lane == 0) tmp[wave] = s;
  __syncthreads();
  if (tid == 0) {
    if (first) {
      a.ctl->eta = eta;
      a.ctl->eta_set = 1;
    }
    UpdArgs b;   // no hi-only phase and no freeze in this form
    b.ctl = a.ctl;
    b.rlog = a.rlog;
    b.rlog_len = a.rlog_len;
    b.hi_max = 0;
    b.stall = 0.0;
    b.tol = 0.0;
    b.gate_done = 0;
    record_iteration(b, (tmp[0] + tmp[1]) + (tmp[2] + tmp[3]));
  }
}

// ---------------------------------------------------------------- spectral start

namespace {

struct FSubShared {
  union {
    float2 red[kFSubWaves][64][kFRMax + 1];
    struct {
      double2 X[64 * kFRMax], Y[64 * kFRMax];
    } rows;
    double sum[kFSubThreads];
    double2 wsum[kFSubWaves][kFRMax];
  };
  double2 tri[kFRMax * (kFRMax + 1) / 2];
  double2 M[kFRMax * kFRMax];               // the factor, or U_old^H U_new
  double rdiag[kFRMax];
  double val[2];
  int flag;
  int2 roll;
};

}  // namespace

// As k_subspace of the real forms; part of a 64-row unit (doubles): Gram of Z | U_old^H U_new |
// Gram of U_new | change.
__global__ __launch_bounds__(kFSubThreads) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_fsub(FSubArgs a) {
  __shared__ FSubShared S;
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
  const int n = a.n, q = a.q, r = a.r, rr = r * r, E = r * (r + 1) / 2, KS = a.KS;
  const int units = (n + 63) / 64, ps = 2 * (2 * E + rr) + 1;
  const long long nr = (long long)n * r;
  Meeting meet(a.ctl);
  if (!meet.join(a.grace, &S.roll)) return;
  const int me = meet.id, nblk = meet.count;

  auto orth = [&](float2* z, int splits, float2* dst, const float2* old) -> bool {
    for (int ru = me; ru < units; ru += nblk) {
      __syncthreads();
      const long long base = (long long)ru * 64 * r;
      for (int i = tid; i < 64 * r; i += kFSubThreads) {
        float2 x = make_float2(0.f, 0.f);
        if (base + i < nr) {
          x = z[base + i];
          for (int s = 1; s < splits; ++s) {
            const float2 t = z[s * nr + base + i];
            x.x += t.x;
            x.y += t.y;
          }
          if (splits > 1) z[base + i] = x;
        }
        S.rows.X[i] = make_double2(x.x, x.y);
      }
      __syncthreads();
      rows_gram64_c<kFSubWaves>(S.rows.X, S.rows.X, r, true, reinterpret_cast<double2*>(a.part + (long long)ru * (ps + 1)));
    }
    meet();
    for (int pass = 0; pass < 2; ++pass) {
      sum_parts_c<kFSubThreads>(a.part, ps + 1, pass == 0 ? 0 : 2 * (E + rr), 2 * E, units, S.sum,
                                reinterpret_cast<double*>(S.tri));
      if (wave == 0) {
        if (lane < rr) S.M[lane] = herm_entry(S.tri, lane / r, lane % r, r);
        double lo, hi;
        const bool pd = wave_cholesky_span_c(S.M, S.rdiag, r, lo, hi);
        if (lane == 0) S.flag = !pd ? 0 : (lo >= kPivotSpan * hi ? 1 : 2);
      }
      __syncthreads();
      const int mode = S.flag;
      if (mode == 0) return false;
      const bool again = pass == 0 && mode == 2;   // ill-conditioned: once more on the rounded rows
      const float2* src = pass == 0 ? z : dst;
      for (int ru = me; ru < units; ru += nblk) {
        const int j = ru * 64 + tid;
        const long long o = (long long)j * r;
        __syncthreads();
        if (tid < 64) {
          double2 x[kFRMax];
#pragma unroll
          for (int c = 0; c < kFRMax; ++c) {
            const float2 v = c < r && j < n ? src[o + c] : make_float2(0.f, 0.f);
            x[c] = make_double2(v.x, v.y);
          }
          solve_row_c(x, S.M, S.rdiag, r);
#pragma unroll
          for (int c = 0; c < kFRMax; ++c)
            if (c < r) {
              const float2 v = make_float2((float)x[c].x, (float)x[c].y);
              if (j < n) dst[o + c] = v;
              S.rows.X[tid * r + c] = make_double2(v.x, v.y);
            }
        }
        if (old)
          for (int i = tid; i < 64 * r; i += kFSubThreads) {
            const long long oi = (long long)ru * 64 * r + i;
            const float2 v = oi < nr ? old[oi] : make_float2(0.f, 0.f);
            S.rows.Y[i] = make_double2(v.x, v.y);
          }
        __syncthreads();
        double2* pt = reinterpret_cast<double2*>(a.part + (long long)ru * (ps + 1));
        if (again) rows_gram64_c<kFSubWaves>(S.rows.X, S.rows.X, r, true, pt + E + rr);
        else if (old) rows_gram64_c<kFSubWaves>(S.rows.Y, S.rows.X, r, false, pt + E);
        __syncthreads();
      }
      meet();
      if (!again) break;
    }
    return true;
  };

  double prev = 0.0;
  auto decide = [&]() -> bool {   // the change of the last step and the stop rule
    sum_parts_c<kFSubThreads>(a.part, ps + 1, ps - 1, 1, units, S.sum, S.val);
    const double sd = sqrt(S.val[0]);
    const bool conv = sd <= a.tol || (sd <= 1e-3 && prev > 0.0 && sd >= 0.99 * prev);
    if (me == 0 && tid == 0) {
      a.ctl->power_sd = sd;
      a.ctl->power_it += 1;
      if (conv) a.ctl->conv = 1;
    }
    prev = sd;
    return conv;
  };

  float2* cur = a.U;
  float2* nxt = a.V;
  bool ok = orth(a.start, 1, cur, nullptr);
  bool pending = false;
  const int WK = n > 2048 ? kFSubWaves : 1;        // waves that share a column
  for (int p = 0; ok && p < a.iters; ++p) {
    // T[k][c] = sum_j h_k[j] conj(U[j][c]) in FP64
    for (int k0 = me * (kFSubWaves / WK); k0 < q; k0 += nblk * (kFSubWaves / WK)) {
      const int k = k0 + (WK == 1 ? wave : 0), kc = k < q ? k : q - 1;
      const float2* row = a.L0t + (long long)kc * n;
      double2 acc[kFRMax];
#pragma unroll
      for (int c = 0; c < kFRMax; ++c) acc[c] = make_double2(0.0, 0.0);
      const int step = 64 * WK;
#pragma unroll 4
      for (int j = lane + (WK == 1 ? 0 : 64 * wave); j < n; j += step) {
        const float2 h = row[j];
        const double2 hd = make_double2(h.x, h.y);
#pragma unroll
        for (int c = 0; c < kFRMax; ++c)
          if (c < r) {
            const float2 u = cur[(long long)j * r + c];
            acc[c] = c_fma_conj(hd, make_double2(u.x, u.y), acc[c]);
          }
      }
      __syncthreads();
#pragma unroll
      for (int c = 0; c < kFRMax; ++c)
        if (c < r) {
          const double tr = wave_sum_dpp(acc[c].x), ti = wave_sum_dpp(acc[c].y);
          if (lane == 0) S.wsum[wave][c] = make_double2(tr, ti);
        }
      __syncthreads();
      if (WK == 1) {
        if (lane < r && k < q) a.T[(long long)k * r + lane] = make_float2((float)S.wsum[wave][lane].x, (float)S.wsum[wave][lane].y);
      } else if (tid < r && k < q) {
        double2 t = S.wsum[0][tid];
        for (int w = 1; w < kFSubWaves; ++w) {
          t.x += S.wsum[w][tid].x;
          t.y += S.wsum[w][tid].y;
        }
        a.T[(long long)k * r + tid] = make_float2((float)t.x, (float)t.y);
      }
    }
    meet();
    if (pending) {
      pending = false;
      if (decide()) break;
    }
    // Z[j][c] = sum_k h_k[j] conj(T[k][c]) by 64-row units and column splits
    for (int w = me; w < units * KS; w += nblk) {
      const int ru = KS == 1 ? w : w / KS, ks = w - ru * KS;
      const int k0 = (int)((long long)q * ks / KS), k1 = (int)((long long)q * (ks + 1) / KS);
      const long long base = (long long)ru * 64 * r;
      __syncthreads();
      frows_grad_r<kFSubWaves>(a.L0t, a.T, n, r, ru, k0, k1, S.red, [&](int i, float2 g) {
        if (base + i < nr) a.gpart[ks * nr + base + i] = g;
      });
    }
    if (KS > 1) meet();
    __syncthreads();
    ok = orth(a.gpart, KS, nxt, cur);
    if (!ok) break;
    // the change ||U_new - U_old W||_F of this workgroup's rows, W = U_old^H U_new
    sum_parts_c<kFSubThreads>(a.part, ps + 1, 2 * E, 2 * rr, units, S.sum, reinterpret_cast<double*>(S.M));
    for (int ru = me; ru < units; ru += nblk) {
      if (wave == 0) {
        const int j = ru * 64 + lane;
        const long long o = (long long)j * r;
        double acc = 0.0;
        if (j < n) {
          float2 u[kFRMax], v[kFRMax];
#pragma unroll
          for (int e = 0; e < kFRMax; ++e) {
            u[e] = e < r ? cur[o + e] : make_float2(0.f, 0.f);
            v[e] = e < r ? nxt[o + e] : make_float2(0.f, 0.f);
          }
#pragma unroll
          for (int c = 0; c < kFRMax; ++c)
            if (c < r) {
              double2 d = make_double2(v[c].x, v[c].y);
#pragma unroll
              for (int e = 0; e < kFRMax; ++e)
                if (e < r) d = c_fma(make_double2(-(double)u[e].x, -(double)u[e].y), S.M[e * r + c], d);
              acc += d.x * d.x + d.y * d.y;
            }
        }
        acc = wave_sum_dpp(acc);
        if (lane == 0) a.part[(long long)ru * (ps + 1) + ps - 1] = acc;
      }
    }
    __syncthreads();
    pending = true;
    float2* x = cur;
    cur = nxt;
    nxt = x;
  }
  if (pending) {   // the step limit: record the last change
    meet();
    decide();
  }
  if (!ok && me == 0 && tid == 0) atomicOr(&a.ctl->err, 2);
  if (cur != a.U)           // this workgroup's rows, read by no other one any more
    for (int ru = me; ru < units; ru += nblk) {
      const long long base = (long long)ru * 64 * r;
      for (int i = tid; i < 64 * r; i += kFSubThreads)
        if (base + i < nr) a.U[base + i] = cur[base + i];
    }
}

// ---------------------------------------------------------------- launchers

size_t fupd_part_doubles(int n, int r) { return (size_t)((n + 63) / 64) * (size_t)(2 * (r * (r + 1) + r * r) + 2); }

// Column splits of the subspace iteration's L_0 T: a 64-row unit per workgroup, at least 32 columns each.
int fsub_splits(int n, int q) {
  int ks = kFSubBlocksMax / ((n + 63) / 64);
  if (ks > q / 32) ks = q / 32;
  return ks < 1 ? 1 : (ks > 16 ? 16 : ks);
}

hipError_t launch_frows(const FUpdArgs& a, hipStream_t st) {
  (void)hipGetLastError();
  hipLaunchKernelGGL(k_frows, dim3((a.n + 63) / 64), dim3(64 * kFRowsWaves), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_fapply(const FUpdArgs& a, hipStream_t st) {
  (void)hipGetLastError();
  hipLaunchKernelGGL(k_fapply, dim3((a.n + kFApplyRows - 1) / kFApplyRows + 1), dim3(kFApplyRows), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_fsub(const FSubArgs& a_in, hipStream_t st) {
  FSubArgs a = a_in;
  a.grace = roll_grace();
  const int per = a.n > 2048 ? 1 : kFSubWaves;     // columns of a workgroup's round
  const int cols = (a.q + per - 1) / per, rows = (a.n + 63) / 64 * a.KS;
  const int b = cols > rows ? cols : rows;
  (void)hipGetLastError();
  hipLaunchKernelGGL(k_fsub, dim3(b < kFSubBlocksMax ? b : kFSubBlocksMax), dim3(kFSubThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace altg
