// Device helpers of the U side of the real forms (the gradient reduction, small FP64
// matrices held by one wave in LDS).
#pragma once
#include "common.h"
#include "launch.h"

namespace altg {

// Upper-triangle storage of a symmetric r x r matrix, row by row: entry e is (a, b), a <= b.
__device__ __forceinline__ void tri_entry(int e, int r, int& a, int& b) {
  int base = 0;
  a = 0;
  while (e >= base + (r - a)) {
    base += r - a;
    ++a;
  }
  b = a + (e - base);
}
__device__ __forceinline__ int tri_index(int i, int j, int r) {
  const int a = i < j ? i : j, b = i < j ? j : i;
  return a * r - a * (a - 1) / 2 + (b - a);
}

// sum over b = 0 .. count - 1 of p[b * stride], in that order; the loads go out 8 at a time.
__device__ __forceinline__ double sum_strided(const double* p, long long stride, int count) {
  double s = 0.0;
  int b = 0;
  for (; b + 8 <= count; b += 8) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = p[(long long)(b + u) * stride];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += v[u];
  }
  for (; b < count; ++b) s += p[(long long)b * stride];
  return s;
}

// Groups of threads that share the sum of `cnt` entries over `count` parts: few enough
// that adding the groups afterwards, one thread per entry, is short.
__device__ __forceinline__ int sum_groups(int threads, int cnt, int count) {
  int g = threads / cnt;
  if (g > 8) g = 8;
  if (g > count) g = count;
  return g > 0 ? g : 1;
}

// 1 / sqrt(x) for positive normal x: the hardware estimate and two Newton steps.
__device__ __forceinline__ double fast_rsqrt(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = fma(y, fma(-0.5 * x * y, y, 0.5), y);
  return fma(y, fma(-0.5 * x * y, y, 0.5), y);
}

// In-place lower Cholesky factor of the SPD r x r matrix W (row-major LDS) by one
// wave, right-looking; 1 / L_jj in rdiag, the smallest and largest pivot L_jj^2 in
// lo and hi.  Returns false (wave-uniform) if a pivot is not positive.  A lane keeps
// up to 4 entries of the lower triangle in registers; a step exchanges the current
// column through LDS and takes one reciprocal, and the square roots come at the end,
// all at once.
__device__ inline bool wave_cholesky_span(double* W, double* rdiag, int r, double& lo, double& hi) {
  const int lane = threadIdx.x & 63;
  lo = hi = 0.0;
  int ri[4], ci[4];
  double w[4];
  wave_lds_fence();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int e = lane + 64 * q;
    ri[q] = e < r * r ? e / r : 0;
    ci[q] = e < r * r ? e - (e / r) * r : r;   // r: no entry
    if (ci[q] > ri[q]) ci[q] = r;
    w[q] = ci[q] < r ? W[e] : 0.0;
  }
  for (int j = 0; j < r; ++j) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (ci[q] == j) W[ri[q] * r + j] = w[q];
    wave_lds_fence();
    const double piv = W[j * r + j];
    if (!(piv > 0.0) || !isfinite(piv)) return false;
    lo = j == 0 || piv < lo ? piv : lo;
    hi = j == 0 || piv > hi ? piv : hi;
    const double inv = fast_rcp(piv);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (ci[q] > j && ci[q] < r) w[q] = fma(-W[ri[q] * r + j] * inv, W[ci[q] * r + j], w[q]);
  }
  if (lane < r) rdiag[lane] = fast_rsqrt(W[lane * r + lane]);
  wave_lds_fence();
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (ci[q] < r) W[ri[q] * r + ci[q]] *= rdiag[ci[q]];
  wave_lds_fence();
  return true;
}

// Largest eigenvalue of the symmetric positive semidefinite r x r matrix M (LDS,
// overwritten; T: r x r scratch) by one wave: with M scaled to trace 1,
// lambda = prod_k tr(M_k^2)^(1 / 2^k), M_{k+1} = M_k^2 / tr(M_k^2).  The remaining
// factor lies between r^(-1 / 2^k) and 1; the loop ends when M_k is of rank one to
// rounding (a dozen squarings unless the leading values agree closely) or 2^-k is
// below rounding.  A wave squares a 10 x 10 matrix in about 0.3 us: 0.41 ms for a
// cyclic Jacobi by one thread -> 6 us.  0 for a zero or non-finite matrix.
__device__ inline double wave_lambda_max(double* M, double* T, int r) {
  const int lane = threadIdx.x & 63, rr = r * r;
  wave_lds_fence();
  double tr = 0.0;
  for (int i = 0; i < r; ++i) tr += M[i * r + i];
  if (!(tr > 0.0) || !isfinite(tr)) return 0.0;
  const double first = tr;
  double acc = 0.0, p = 0.5, scale = 1.0 / tr;
  for (int k = 0; k < 56; ++k) {
    for (int e = lane; e < rr; e += 64) {
      const int i = e / r, j = e - i * r;
      double s = 0.0;
      for (int l = 0; l < r; ++l) s = fma(M[i * r + l] * scale, M[l * r + j] * scale, s);
      T[e] = s;
    }
    wave_lds_fence();
    double t = 0.0;
    for (int i = 0; i < r; ++i) t += T[i * r + i];
    if (!(t > 0.0) || !isfinite(t)) return 0.0;
    acc = fma(p, log(t), acc);
    if (t >= 1.0 - 1e-15) break;
    p *= 0.5;
    scale = 1.0 / t;
    double* x = M;
    M = T;
    T = x;
  }
  return first * exp(acc);
}

// smallest / largest pivot for which one CholeskyQR pass is enough
constexpr double kPivotSpan = 1e-6;
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));

// Value of lane I of each 16-lane row, in every lane of the row.
template <int I>
__device__ __forceinline__ float row_bcast(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + I, 0xF, 0xF, false));
}

// acc[e][c] += h[e] * B[k][c], c < R, where lane c of each 16-lane row holds B[k][c].
template <int R, int C = 0>
__device__ __forceinline__ void rank1(float (&acc)[4][R], const float4& h, float b) {
  if constexpr (C < R) {
    const float bc = row_bcast<C>(b);
    acc[0][C] = fmaf(h.x, bc, acc[0][C]);
    acc[1][C] = fmaf(h.y, bc, acc[1][C]);
    acc[2][C] = fmaf(h.z, bc, acc[2][C]);
    acc[3][C] = fmaf(h.w, bc, acc[3][C]);
    rank1<R, C + 1>(acc, h, b);
  }
}

// Rows 64 jb .. + 63 of sum_k h_k b_k^T over the columns k0 <= k < k1, by a workgroup of
// WV waves: thread i < 64 r gets row i / r, column i % r through put(i, value) (rows at
// or beyond n are zero).  Quarter p = lane / 16 of wave w takes k = k0 + 4 w + p, then
// every 4 WV-th, its lanes 4 rows each (16-byte loads, four 256-byte pieces of h_k per
// wave); the quarters, then (above 8 waves) the waves w and w + 8, then the waves are
// added in that order.  R: r rounded up to a multiple of 4.
template <int R, int WV, class Put>
__device__ __forceinline__ void urows_grad(const float* H, const float* B, int n, int r, int jb, int k0, int k1,
                                           float (*red)[64][kRMax + 1], Put put) {
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
  const int l = lane & 15, p = lane >> 4, j = jb * 64 + 4 * l;
  const bool full = (jb + 1) * 64 <= n;
  float acc[4][R];
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int c = 0; c < R; ++c) acc[e][c] = 0.f;
  constexpr int KU = 4;   // loads in flight per wave; the order of the k terms does not depend on it
  for (int kb = k0 + 4 * wave; kb < k1; kb += 4 * WV * KU) {
    float4 h[KU];
    float bv[KU];
#pragma unroll
    for (int u = 0; u < KU; ++u) {
      const int k = kb + p + u * 4 * WV;
      const bool in = k < k1;
      const float* row = H + (long long)(in ? k : k0) * n;
      bv[u] = in && l < r ? B[(long long)k * r + l] : 0.f;
      if (full) {
        const f32x4_u v = *reinterpret_cast<const f32x4_u*>(row + j);
        h[u] = make_float4(v.x, v.y, v.z, v.w);
      } else {
        h[u] = make_float4(j < n ? row[j] : 0.f, j + 1 < n ? row[j + 1] : 0.f, j + 2 < n ? row[j + 2] : 0.f,
                           j + 3 < n ? row[j + 3] : 0.f);
      }
      if (!in) h[u] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int u = 0; u < KU; ++u) rank1<R>(acc, h[u], bv[u]);
  }
  // quarters: afterwards lane (p, l) holds row 4 l + p
  float v[R];
#pragma unroll
  for (int c = 0; c < R; ++c) {
    float t[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float x = acc[e][c] + __shfl_xor(acc[e][c], 16);
      t[e] = x + __shfl_xor(x, 32);
    }
    v[c] = p == 0 ? t[0] : (p == 1 ? t[1] : (p == 2 ? t[2] : t[3]));
  }
  constexpr int WS = WV > 8 ? 8 : WV;   // sums left after the first step
  const int row = 4 * l + p;
  if (wave >= WV - WS)
#pragma unroll
    for (int c = 0; c < R; ++c) red[wave - (WV - WS)][row][c] = v[c];
  __syncthreads();
  if constexpr (WV > 8) {
    if (wave < WS)
#pragma unroll
      for (int c = 0; c < R; ++c) red[wave][row][c] += v[c];
    __syncthreads();
  }
  for (int i = tid; i < 64 * r; i += 64 * WV) {
    const int rw = i / r, c = i - rw * r;
    float g = red[0][rw][c];
#pragma unroll
    for (int w = 1; w < WS; ++w) g += red[w][rw][c];
    put(i, g);
  }
}

template <int WV, class Put>
__device__ __forceinline__ void urows_grad_r(const float* H, const float* B, int n, int r, int jb, int k0, int k1,
                                             float (*red)[64][kRMax + 1], Put put) {
  if (r <= 4) urows_grad<4, WV>(H, B, n, r, jb, k0, k1, red, put);
  else if (r <= 8) urows_grad<8, WV>(H, B, n, r, jb, k0, k1, red, put);
  else if (r <= 12) urows_grad<12, WV>(H, B, n, r, jb, k0, k1, red, put);
  else urows_grad<16, WV>(H, B, n, r, jb, k0, k1, red, put);
}

// Part of X^T Y over the 64 rows in LDS (row-major, r wide): the upper triangle (a <= b)
// row by row with sym, all r^2 entries without; by a workgroup of WV waves.
template <int WV>
__device__ __forceinline__ void rows_gram64(const double* X, const double* Y, int r, bool sym, double* dst) {
  const int lane = threadIdx.x & 63, wave = wave_id();
  const int E = sym ? r * (r + 1) / 2 : r * r;
  for (int e = wave; e < E; e += WV) {
    int a = 0, b = 0;
    if (sym) tri_entry(e, r, a, b);
    else { a = e / r; b = e - a * r; }
    const double s = wave_sum_dpp(X[lane * r + a] * Y[lane * r + b]);
    if (lane == 0) dst[e] = s;
  }
}

// x <- x R^{-1} for one row, R^T = L (row-major r x r in LDS), by forward substitution.
__device__ __forceinline__ void solve_row(double (&x)[kRMax], const double* L, const double* rdiag, int r) {
#pragma unroll
  for (int c = 0; c < kRMax; ++c) {
    if (c < r) {
      double t = x[c];
#pragma unroll
      for (int p = 0; p < kRMax; ++p)
        if (p < c) t = fma(-x[p], L[c * r + p], t);
      x[c] = t * rdiag[c];
    }
  }
}

// End of a GDmin iteration (one thread): the residual from the summed ||r_k||^2, the log,
// the counters, the hi-only phase of a BF16X2 solve and the freeze of batched stepping.
__device__ inline void record_iteration(const UpdArgs& a, double rr) {
  Ctl* c = a.ctl;
  const double resid = c->ynorm2 > 0.0 ? sqrt(rr / c->ynorm2) : sqrt(rr);
  const int t = c->t;
  if (a.rlog && t < a.rlog_len) a.rlog[t] = resid;
  c->resid = resid;
  c->t = t + 1;
  // BF16X2 hi-only phase: switch to hi + lo when the residual stalls or the budget is spent
  if (c->phase == 0 && (t + 1 >= a.hi_max || (t > 0 && resid >= a.stall * c->prev_resid))) {
    c->phase = 1;
    c->refine_t = t + 1;
  }
  c->prev_resid = resid;
  if (a.gate_done && a.tol > 0.0 && resid <= a.tol) c->done = 1;
}

}  // namespace altg
