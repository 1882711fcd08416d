// Device helpers of the U side of the real forms (the gradient reduction, small FP64
// matrices held by one wave in LDS).
#pragma once
#include "common.h"
#include "launch.h"

namespace altg {

// One workgroup of 16 waves per block of 64 rows j; wave w sums the columns
// k = w, w + 16, ... of its split; the 16 wave partials are added in a fixed
// pairwise order.  Row k of B is fetched by lanes 0..r-1 with one vector load
// and broadcast with readlane, so that loads of later columns stay in flight.
__device__ __forceinline__ void grad_body(const float* __restrict__ H, const float* __restrict__ B, int n, int q, int r,
                                          int KS, float* __restrict__ gpart, int jblock, int ks,
                                          float (*red)[64][kRMax + 1]) {
  const int lane = threadIdx.x & 63, ph = wave_id();
  const int j = jblock * 64 + lane;
  const int jc = j < n ? j : n - 1;
  const int k0 = (int)((long long)q * ks / KS), k1 = (int)((long long)q * (ks + 1) / KS);
  float acc[kRMax];
#pragma unroll
  for (int c = 0; c < kRMax; ++c) acc[c] = 0.f;
  constexpr int KU = 16;   // loads in flight per wave; the order of the k terms does not depend on it
  for (int kb = k0 + ph; kb < k1; kb += kGradWaves * KU) {
    float h[KU], bv[KU];
#pragma unroll
    for (int u = 0; u < KU; ++u) {
      const int k = kb + u * kGradWaves;
      const int kc = k < k1 ? k : k0;
      h[u] = H[(long long)kc * n + jc];
      bv[u] = B[(long long)kc * r + (lane < r ? lane : 0)];
    }
#pragma unroll
    for (int u = 0; u < KU; ++u) {
      const bool ok = kb + u * kGradWaves < k1;
      const float hu = ok ? h[u] : 0.f;
#pragma unroll
      for (int c = 0; c < kRMax; ++c)
        if (c < r) acc[c] = fmaf(hu, __int_as_float(__builtin_amdgcn_readlane(__float_as_int(bv[u]), c)), acc[c]);
    }
  }
  // pairwise tree over the waves in a fixed order: (w, w + h) for h = 8, 4, 2, 1
  for (int hh = kGradWaves / 2; hh >= 1; hh >>= 1) {
    if (ph >= hh && ph < 2 * hh)
#pragma unroll
      for (int c = 0; c < kRMax; ++c) red[ph - hh][lane][c] = acc[c];
    __syncthreads();
    if (ph < hh)
#pragma unroll
      for (int c = 0; c < kRMax; ++c) acc[c] += red[ph][lane][c];
    __syncthreads();
  }
  if (ph == 0 && j < n)
    for (int c = 0; c < r; ++c) gpart[((long long)ks * n + j) * r + c] = acc[c];
}

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

// Orders one wave's LDS accesses: they complete in program order, so only the
// compiler has to keep them there.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// 1 / x and 1 / sqrt(x) for positive normal x: the hardware estimate and two Newton steps.
__device__ __forceinline__ double fast_rcp(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(y, fma(-x, y, 1.0), y);
  return fma(y, fma(-x, y, 1.0), y);
}
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
