// The U update of a GDmin iteration (Alg. 1) over many workgroups, for the real forms:
// grad_U f = sum_k h_k b_k^T, eta at t = 1, U+ = QR(U - eta grad_U f) with a positive
// diagonal R, the residual and the iteration's bookkeeping.  Two launches (three when
// the columns are split for the gradient, see upd_splits in api.hip):
//
//  k_ugrad : a workgroup per 64 rows and column split: its part of grad;
//  k_urows : a workgroup per 64 rows: the rows of grad, U_prev = U, and the block's part
//            of the FP64 Gram matrix of X = U - eta grad;
//  k_uapply: a row per thread: every workgroup adds the parts in order and factors the
//            Gram (the same bits in each), then U = X R^{-1}; one more workgroup does
//            the bookkeeping.
//
// What bounds it is latency: 4 MB of h_k at n = q = 1000, then a chain of small FP64
// steps.  One 1024-thread workgroup for all of it after a gradient launch took 9 + 41
// us there (12 us in all at n = q = 100, 18 + 1028 us at n = 16384, q = 100); workgroups
// that hand over to the last one to arrive cost about 10 us per hand-over in cache
// write-backs, more than a launch; these launches take 9 + 5 + 12 us there (12 and 28).
// At t = 1, eta's eigenvalue took 0.4 ms by a cyclic Jacobi in one thread and takes
// 20 us (wave_lambda_max).
//
// The factor comes from the FP64 Gram of the unrounded X, so one CholeskyQR pass gives
// Q to FP32 rounding whenever cond(X)^2 2^-53 is far below it: a second pass is taken
// only when the pivots span more than kPivotSpan (each workgroup then forms the Gram of
// all the rounded rows itself, 256 rows at a time through LDS: op_qr_step 0.43 ms at
// n = 16384, r = 16 and 38 us at n = 1000, r = 10, where one pass takes 43 and 21 us).
#pragma once
#include "launch.h"
#include "uside.h"

namespace altg {

constexpr int kURowsThreads = kGradWaves * 64;
constexpr int kUApplyRows = 256;            // rows (threads) of a k_uapply workgroup
enum { UPD_FROZEN = 0, UPD_STEP = 1, UPD_FIRST = 2 };

constexpr int kUGradWaves = 4;              // waves of a column split's workgroup

union URowsShared {
  float red[kGradWaves / 2][64][kRMax + 1];
  struct {
    double X[64 * kRMax], Y[64 * kRMax];
  } rows;
};

// One column split of the gradient: rows of block jb over the columns of split ks.
template <int WV>
__device__ __forceinline__ void ugrad_body(const UpdArgs& a, int jb, int ks, float (*red)[64][kRMax + 1]) {
  if (a.gate_done && a.ctl->done) return;
  const int k0 = (int)((long long)a.q * ks / a.KS), k1 = (int)((long long)a.q * (ks + 1) / a.KS);
  const long long nr = (long long)a.n * a.r, base = (long long)jb * 64 * a.r;
  urows_grad_r<WV>(a.H, a.B, a.n, a.r, jb, k0, k1, red, [&](int i, float g) {
    if (base + i < nr) a.gpart[ks * nr + base + i] = g;
  });
}

template <int WV>
__global__ __launch_bounds__(64 * WV) void k_ugrad(UpdArgs a) {
  __shared__ float red[WV > 8 ? 8 : WV][64][kRMax + 1];
  ugrad_body<WV>(a, blockIdx.x, blockIdx.y, red);
}

// Several problems in one launch: block b is (problem, row block, split) = map[b].
__global__ __launch_bounds__(64 * kUGradWaves) void k_ugrad_grp(const UpdArgs* tab, const int4* map) {
  __shared__ float red[kUGradWaves][64][kRMax + 1];
  const int4 mp = map[blockIdx.x];
  const UpdArgs a = tab[mp.x];
  ugrad_body<kUGradWaves>(a, mp.y, mp.z, red);
}

__device__ __forceinline__ void urows_body(const UpdArgs& a, int jb, URowsShared& S) {
  const int tid = threadIdx.x;
  const int n = a.n, r = a.r, E = r * (r + 1) / 2;
  const bool have = a.ctl ? a.ctl->eta_set != 0 : *a.eta_io > 0.0;
  if (jb == 0 && tid == 0) *a.upd = a.gate_done && a.ctl->done ? UPD_FROZEN : (have ? UPD_STEP : UPD_FIRST);
  if (a.gate_done && a.ctl->done) return;
  const double eta = have ? (a.ctl ? a.ctl->eta : *a.eta_io) : 0.0;
  const long long base = (long long)jb * 64 * r, nr = (long long)n * r;
  // thread i < 64 r: row i / r, column i % r (64 r <= kURowsThreads)
  float g = 0.f;
  if (a.H && a.KS == 1) {
    urows_grad_r<kGradWaves>(a.H, a.B, n, r, jb, 0, a.q, S.red, [&](int, float v) { g = v; });
    __syncthreads();   // S is free
  }
  if (!a.part) {   // no room for the parts (the entry point, grad given): k_uapply forms the Grams from the rows
    if (tid < 64 * r && base + tid < nr) a.Uprev[base + tid] = a.U[base + tid];
    return;
  }
  if (tid < 64 * r) {
    double x = 0.0, y = 0.0;
    const long long i = base + tid;
    if (i < nr) {
      if (a.H && a.KS == 1) {
        a.gpart[i] = g;
      } else {          // given, or the column splits in order
        float part[16];
#pragma unroll
        for (int s = 0; s < 16; ++s) part[s] = s < a.KS ? a.gpart[s * nr + i] : 0.f;
        g = part[0];
#pragma unroll
        for (int s = 1; s < 16; ++s) g += part[s];
        if (a.KS > 1) a.gpart[i] = g;
      }
      const float u = a.U[i];
      a.Uprev[i] = u;
      x = have ? fma(-eta, (double)g, (double)u) : (double)u;
      y = (double)g;
    }
    S.rows.X[tid] = x;
    S.rows.Y[tid] = y;
  }
  __syncthreads();
  // eta known: the Gram of X; at t = 1: U^T U, G^T G and U^T G
  double* dst = a.part + (long long)jb * (2 * E + r * r);
  rows_gram64<kGradWaves>(S.rows.X, S.rows.X, r, true, dst);
  if (!have) {
    rows_gram64<kGradWaves>(S.rows.Y, S.rows.Y, r, true, dst + E);
    rows_gram64<kGradWaves>(S.rows.X, S.rows.Y, r, false, dst + 2 * E);
  }
}

__global__ __launch_bounds__(kURowsThreads) void k_urows(UpdArgs a) {
  __shared__ URowsShared S;
  urows_body(a, blockIdx.x, S);
}

// Several problems in one launch: block b is row block map[b].y of problem map[b].x.
__global__ __launch_bounds__(kURowsThreads) void k_urows_grp(const UpdArgs* tab, const int2* map) {
  __shared__ URowsShared S;
  const int2 mp = map[blockIdx.x];
  const UpdArgs a = tab[mp.x];
  urows_body(a, mp.y, S);
}

constexpr int kUPartMax = 2 * (kRMax * (kRMax + 1) / 2) + kRMax * kRMax;   // values of a block's part

struct UApplyShared {
  double sum[kUPartMax > kUApplyRows ? kUPartMax : kUApplyRows];
  double W[kUPartMax];
  double A[2 * kRMax * kRMax];              // the matrix to factor (L afterwards), scratch
  __attribute__((aligned(16))) float rows[kUApplyRows][kRMax + 1];   // second pass: rounded rows
  double rdiag[kRMax];
  double eta;
  int mode;                                 // 0: the Gram is not positive definite, 1 or 2 passes
};

// S.W = the upper triangle of X^T X over all n rows of X, row i as row(i, y) puts it into y, rounded to
// FP32 (rows at or beyond n count as zero, whatever y holds): 256 rows at a time through LDS, by
// FP64 matrix products of four rows each.  Lane l holds column l % 16 of row l / 16 for both operands, and
// column l % 16 of rows l / 16 + 4 v of the result.
template <class Row>
__device__ __forceinline__ void uapply_gram(int n, int r, UApplyShared& S, Row row) {
  typedef double f64x4 __attribute__((ext_vector_type(4)));
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  for (int i0 = 0; i0 < n; i0 += kUApplyRows) {
    double y[kRMax];
    row(i0 + tid, y);
#pragma unroll
    for (int c = 0; c < kRMax; ++c) S.rows[tid][c] = c < r && i0 + tid < n ? (float)y[c] : 0.f;
    __syncthreads();
    float v[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) v[s] = S.rows[64 * wave + 4 * s + (lane >> 4)][lane & 15];
#pragma unroll
    for (int s = 0; s < 16; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64((double)v[s], (double)v[s], acc, 0, 0, 0);
    __syncthreads();
  }
  double* sum = reinterpret_cast<double*>(&S.rows[0][0]);   // 4 x 256 of the waves
#pragma unroll
  for (int v = 0; v < 4; ++v) sum[wave * 256 + ((lane >> 4) + 4 * v) * 16 + (lane & 15)] = acc[v];
  __syncthreads();
  if (tid < r * (r + 1) / 2) {
    int ra, rb;
    tri_entry(tid, r, ra, rb);
    const int e = ra * 16 + rb;
    S.W[tid] = (sum[e] + sum[256 + e]) + (sum[512 + e] + sum[768 + e]);
  }
  __syncthreads();
}

// Workgroup jb < kUApplyRows-row blocks of n updates its rows; the one after them does the
// bookkeeping.
template <bool PARTS>
__device__ __forceinline__ void uapply_body(const UpdArgs& a, int jb, UApplyShared& S) {
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
  const int n = a.n, r = a.r, rr = r * r, E = r * (r + 1) / 2, PE = 2 * E + rr, nb = (n + 63) / 64;
  const int upd = *a.upd;
  if (upd == UPD_FROZEN) return;
  // this thread's row, loaded ahead of the factorisation
  const int j = jb * kUApplyRows + tid;
  const long long o = (long long)j * r;
  float ru[kRMax], rg[kRMax];
#pragma unroll
  for (int c = 0; c < kRMax; ++c) {
    ru[c] = c < r && j < n ? a.Uprev[o + c] : 0.f;
    rg[c] = c < r && j < n ? a.gpart[o + c] : 0.f;
  }
  const bool first = upd == UPD_FIRST;
  double* M = S.A;
  if constexpr (PARTS) {
    // the Gram parts: entry e over a contiguous range of blocks per group of threads,
    // then the groups in order
    const int used = first ? PE : E;
    const int grp = sum_groups(kUApplyRows, used, nb);
    for (int e = tid; e < used * grp; e += kUApplyRows) {
      const int g = e / used, en = e - g * used;
      const int b0 = nb * g / grp, b1 = nb * (g + 1) / grp;
      S.sum[e] = sum_strided(a.part + (long long)b0 * PE + en, PE, b1 - b0);
    }
    __syncthreads();
    for (int e = tid; e < used; e += kUApplyRows) {
      double s = S.sum[e];
      for (int g = 1; g < grp; ++g) s += S.sum[g * used + e];
      S.W[e] = s;
    }
    __syncthreads();
  } else if (first) {   // G^T G for eta
    uapply_gram(n, r, S, [&](int i, double (&y)[kRMax]) {
#pragma unroll
      for (int c = 0; c < kRMax; ++c) y[c] = c < r && i < n ? (double)a.gpart[(long long)i * r + c] : 0.0;
    });
  }
  auto row = [&](int i, double eta, double (&y)[kRMax]) {   // row i of X
#pragma unroll
    for (int c = 0; c < kRMax; ++c)
      y[c] = c < r && i < n ? fma(-eta, (double)a.gpart[(long long)i * r + c], (double)a.Uprev[(long long)i * r + c]) : 0.0;
  };
  auto step_size = [&](int off) -> double {   // at t = 1, from G^T G at S.W + off, by wave 0
    for (int e = lane; e < rr; e += 64) M[e] = S.W[off + tri_index(e / r, e % r, r)];
    const double lam = wave_lambda_max(M, S.A + kRMax * kRMax, r);
    wave_lds_fence();
    return lam > 0.0 ? a.eta_c / sqrt(lam) : 0.0;
  };
  if constexpr (!PARTS) {   // the Gram of the rounded X: always two passes
    if (wave == 0) {
      const double eta = first ? step_size(0) : (a.ctl ? a.ctl->eta : *a.eta_io);
      if (lane == 0) S.eta = eta;
    }
    __syncthreads();
    uapply_gram(n, r, S, [&](int i, double (&y)[kRMax]) { row(i, S.eta, y); });
  }
  if (wave == 0) {
    if (PARTS && first) {
      const double eta = step_size(E);
      // X^T X = U^T U - eta (U^T G + G^T U) + eta^2 G^T G
      for (int e = lane; e < rr; e += 64) {
        const int i = e / r, jj = e % r, t = tri_index(i, jj, r);
        M[e] = S.W[t] - eta * (S.W[2 * E + i * r + jj] + S.W[2 * E + jj * r + i]) + eta * eta * S.W[E + t];
      }
      if (lane == 0) S.eta = eta;
    } else {
      for (int e = lane; e < rr; e += 64) M[e] = S.W[tri_index(e / r, e % r, r)];
      if (PARTS && lane == 0) S.eta = a.ctl ? a.ctl->eta : *a.eta_io;
    }
    double lo, hi;
    const bool pd = wave_cholesky_span(M, S.rdiag, r, lo, hi);
    if (lane == 0) S.mode = !pd ? 0 : (PARTS && lo >= kPivotSpan * hi ? 1 : 2);
  }
  __syncthreads();
  const double eta = S.eta;
  const bool rows = jb * kUApplyRows < n;   // the last workgroup has none
  bool ok = S.mode != 0;
  double x[kRMax];
  if (ok && j < n) {
#pragma unroll
    for (int c = 0; c < kRMax; ++c)
      if (c < r) x[c] = fma(-eta, (double)rg[c], (double)ru[c]);
    solve_row(x, M, S.rdiag, r);
  }
  if (S.mode == 2 && rows) {   // an ill-conditioned X: once more on the rounded rows, each solved once
    uapply_gram(n, r, S, [&](int i, double (&y)[kRMax]) {
      if (i != j) {
        row(i, eta, y);
        solve_row(y, M, S.rdiag, r);
      } else {   // this workgroup's rows are in x
#pragma unroll
        for (int c = 0; c < kRMax; ++c) y[c] = x[c];
      }
    });
    if (wave == 0) {
      for (int e = lane; e < rr; e += 64) M[e] = S.W[tri_index(e / r, e % r, r)];
      double lo, hi;
      const bool pd = wave_cholesky_span(M, S.rdiag, r, lo, hi);
      if (lane == 0) S.mode = pd ? 1 : 0;
    }
    __syncthreads();
    ok = S.mode != 0;
    if (ok && j < n) {
#pragma unroll
      for (int c = 0; c < kRMax; ++c)
        if (c < r) x[c] = (double)(float)x[c];
      solve_row(x, M, S.rdiag, r);
    }
  }
  if (ok && j < n)
#pragma unroll
    for (int c = 0; c < kRMax; ++c)
      if (c < r) a.U[o + c] = (float)x[c];
  if (rows) {
    if (!ok && jb == 0 && tid == 0 && a.ctl) atomicOr(&a.ctl->err, 2);
    return;
  }
  // the last workgroup (no rows): eta, then the residual of the iteration and the
  // counters, recorded whether or not the factorisation failed
  if (!a.ctl) {
    if (first && tid == 0) *a.eta_io = eta;
    return;
  }
  double s = 0.0;
  int fl = 0;
  int k = tid;
  for (; k + 7 * kUApplyRows < a.q; k += 8 * kUApplyRows) {   // in order, the loads eight at a time
    double v[8];
    int f[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      v[u] = a.colrr[k + u * kUApplyRows];
      f[u] = a.colflags[k + u * kUApplyRows];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      s += v[u];
      fl |= f[u];
    }
  }
  for (; k < a.q; k += kUApplyRows) {
    s += a.colrr[k];
    fl |= a.colflags[k];
  }
  if (fl) atomicOr(&a.ctl->err, fl);
  s = wave_sum_dpp(s);
  __syncthreads();   // S.sum is free
  if (lane == 0) S.sum[wave] = s;
  __syncthreads();
  if (tid == 0) {
    if (first) {
      a.ctl->eta = eta;
      a.ctl->eta_set = 1;
    }
    record_iteration(a, (S.sum[0] + S.sum[1]) + (S.sum[2] + S.sum[3]));
  }
}

template <bool PARTS>
__global__ __launch_bounds__(kUApplyRows) void k_uapply(UpdArgs a) {
  __shared__ UApplyShared S;
  uapply_body<PARTS>(a, blockIdx.x, S);
}

__global__ __launch_bounds__(kUApplyRows) void k_uapply_grp(const UpdArgs* tab, const int2* map) {
  __shared__ UApplyShared S;
  const int2 mp = map[blockIdx.x];
  const UpdArgs a = tab[mp.x];
  uapply_body<true>(a, mp.y, S);
}

// ---------------------------------------------------------------- launchers

size_t upd_part_doubles(int n, int r) { return (size_t)((n + 63) / 64) * (size_t)(r * (r + 1) + r * r); }
int uapply_blocks(int n) { return (n + kUApplyRows - 1) / kUApplyRows + 1; }

hipError_t launch_ugrad(const UpdArgs& a, hipStream_t st) {
  (void)hipGetLastError();   // clear a stale error of an earlier, unrelated call
  const dim3 grid((a.n + 63) / 64, a.KS);
  // A GDmin iteration takes 4 waves whatever the launch, so that its sums do not depend on it.  The entry point has few
  // splits (the scratch); where they leave CUs idle, 16 waves: n = 100, q = 20,000, r = 4 53 against 104 us,
  // n = q = 2000, r = 8 (128 workgroups) 14.3 against 20, n = q = 1000, r = 10 14 against 15.4.
  if (!a.ctl && grid.x * grid.y <= 128)
    hipLaunchKernelGGL(k_ugrad<kGradWaves>, grid, dim3(64 * kGradWaves), 0, st, a);
  else
    hipLaunchKernelGGL(k_ugrad<kUGradWaves>, grid, dim3(64 * kUGradWaves), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_ugrad_grp(const UpdArgs* tab, const int4* map, int blocks, hipStream_t st) {
  (void)hipGetLastError();   // clear a stale error of an earlier, unrelated call
  hipLaunchKernelGGL(k_ugrad_grp, dim3(blocks), dim3(64 * kUGradWaves), 0, st, tab, map);
  return hipGetLastError();
}

hipError_t launch_urows(const UpdArgs& a, hipStream_t st) {
  (void)hipGetLastError();   // clear a stale error of an earlier, unrelated call
  hipLaunchKernelGGL(k_urows, dim3((a.n + 63) / 64), dim3(kURowsThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_uapply(const UpdArgs& a, hipStream_t st) {
  (void)hipGetLastError();   // clear a stale error of an earlier, unrelated call
  hipLaunchKernelGGL(a.part ? k_uapply<true> : k_uapply<false>, dim3(uapply_blocks(a.n)), dim3(kUApplyRows), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_urows_grp(const UpdArgs* tab, const int2* map, int blocks, hipStream_t st) {
  (void)hipGetLastError();   // clear a stale error of an earlier, unrelated call
  hipLaunchKernelGGL(k_urows_grp, dim3(blocks), dim3(kURowsThreads), 0, st, tab, map);
  return hipGetLastError();
}

hipError_t launch_uapply_grp(const UpdArgs* tab, const int2* map, int blocks, hipStream_t st) {
  (void)hipGetLastError();   // clear a stale error of an earlier, unrelated call
  hipLaunchKernelGGL(k_uapply_grp, dim3(blocks), dim3(kUApplyRows), 0, st, tab, map);
  return hipGetLastError();
}

}  // namespace altg
