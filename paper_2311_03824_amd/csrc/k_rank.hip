// Automatic rank of Sec. 2.6 on the GPU (gfx950).
//
// The rank r is the smallest k whose k leading singular values of L_0 hold a
// fraction `energy` (65 % in the paper) of the energy sum_i sigma_i^2 of the
// first K = max(1, floor(min(n, q, m) / 10)).  The K values come from a block
// subspace iteration on L_0 (n x q, given as L_0^T, q x n row-major) with
// b = K + p columns (p <= 8 extra columns speed up the trailing values), each
// step Z = L_0 (L_0^T U) followed by CholeskyQR2 (FP64 Gram, Cholesky and
// R^{-1}), then a Rayleigh-Ritz step: the eigenvalues of M = T^T T, T = L_0^T U,
// are the squared Ritz values, found by a parallel cyclic Jacobi (round-robin
// pairs, all b/2 rotations of a round at once).
//
// Kernels: k_rank_mm (C = A B or A^T B, FP32 tiles staged in LDS), k_rank_gram
// (W = X^T X in FP64), k_rank_chol (one workgroup: W = R^T R, R^{-1}),
// k_rank_jacobi (one workgroup: eigenvalues, their order, the rank).  Every
// reduction runs in a fixed order, so results do not depend on timing.
#include "common.h"
#include "launch.h"

namespace altg {

namespace {

constexpr int kTile = 32;       // output tile of k_rank_mm (kTile x kTile)
constexpr int kKc = 64;         // contraction chunk staged in LDS
constexpr int kGT = 16;         // tile of k_rank_gram (kGT x kGT entries, one per thread)
constexpr int kGRows = 64;      // rows per LDS stage of k_rank_gram

// C (M x N, row-major, ldc) = A' B with A' = A (M x K, row-major lda) or, with
// TRANS, A' = A^T where A is K x M row-major (lda); B is K x N row-major (ldb).
// Four groups of 256 threads take a quarter of every 64-term chunk each, a thread 4 outputs
// of its column in FP32; the next chunk is loaded meanwhile and the groups' sums are added in
// order.  At these sizes a launch has a few workgroups and is bound by the latency of
// its loads and LDS reads (n = 300, q = 200, b = 20: 13 -> 6 us).
template <bool TRANS>
__global__ __launch_bounds__(1024) void k_rank_mm(const float* __restrict__ A, long long lda,
                                                  const float* __restrict__ B, long long ldb, float* __restrict__ C,
                                                  long long ldc, int M, int N, int K) {
  __shared__ __attribute__((aligned(16))) float sa[kKc][kTile + 4];   // sa[kk][i] = A'(i0 + i, k0 + kk)
  __shared__ float sb[kKc][kTile + 1];                                // sb[kk][c] = B(k0 + kk, c0 + c)
  constexpr int kPer = kKc * kTile / 1024, kQ = kKc / 4;
  const int tid = threadIdx.x, grp = tid >> 8, t8 = tid & 255;
  const int i0 = blockIdx.y * kTile, c0 = blockIdx.x * kTile;
  const int tc = t8 & (kTile - 1), ti = (t8 >> 5) * 4;   // this thread: column tc, rows ti .. ti + 3
  float acc[4] = {0.f, 0.f, 0.f, 0.f};
  float va[kPer], vb[kPer];
  auto load = [&](int k0) {
#pragma unroll
    for (int t = 0; t < kPer; ++t) {
      const int e = tid + 1024 * t;
      // A' tile: consecutive threads read consecutive addresses (along k for A, along i for A^T)
      const int ii = TRANS ? e % kTile : e / kKc, kx = TRANS ? e / kTile : e % kKc;
      const int gi = i0 + ii, gk = k0 + kx;
      va[t] = gi < M && gk < K ? (TRANS ? A[(long long)gk * lda + gi] : A[(long long)gi * lda + gk]) : 0.f;
      const int bk = k0 + e / kTile, bc = c0 + e % kTile;
      vb[t] = bk < K && bc < N ? B[(long long)bk * ldb + bc] : 0.f;
    }
  };
  load(0);
  for (int k0 = 0; k0 < K; k0 += kKc) {
#pragma unroll
    for (int t = 0; t < kPer; ++t) {
      const int e = tid + 1024 * t;
      const int ii = TRANS ? e % kTile : e / kKc, kx = TRANS ? e / kTile : e % kKc;
      sa[kx][ii] = va[t];
      sb[e / kTile][e % kTile] = vb[t];
    }
    __syncthreads();
    if (k0 + kKc < K) load(k0 + kKc);
#pragma unroll
    for (int kk = 0; kk < kQ; ++kk) {   // terms beyond K are zero
      const float b = sb[grp * kQ + kk][tc];
      const float4 x = *reinterpret_cast<const float4*>(&sa[grp * kQ + kk][ti]);
      acc[0] = fmaf(x.x, b, acc[0]);
      acc[1] = fmaf(x.y, b, acc[1]);
      acc[2] = fmaf(x.z, b, acc[2]);
      acc[3] = fmaf(x.w, b, acc[3]);
    }
    __syncthreads();
  }
  float4* part = reinterpret_cast<float4*>(&sa[0][0]);   // 2 x 256 entries fit (9 KiB): the groups in two steps
  if (grp >= 2) part[(grp - 2) * 256 + t8] = make_float4(acc[0], acc[1], acc[2], acc[3]);
  __syncthreads();
  if (grp < 2) {
    const float4 o = part[grp * 256 + t8];   // groups 0 + 2 and 1 + 3
    acc[0] += o.x; acc[1] += o.y; acc[2] += o.z; acc[3] += o.w;
  }
  __syncthreads();
  if (grp == 1) part[t8] = make_float4(acc[0], acc[1], acc[2], acc[3]);
  __syncthreads();
  if (grp > 0) return;
  const float4 o = part[t8];
  const float r[4] = {acc[0] + o.x, acc[1] + o.y, acc[2] + o.z, acc[3] + o.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int gi = i0 + ti + e, gc = c0 + tc;
    if (gi < M && gc < N) C[(long long)gi * ldc + gc] = r[e];
  }
}

// W (b x b, FP64) = X^T X for X (rows x b, row-major): one entry per thread of each of
// four groups, which take a quarter of every 64-row stage; the next stage is loaded meanwhile;
// the groups' sums are added in order (n = 300, b = 20: 5 us against 15 with one group and no
// load ahead).
__global__ __launch_bounds__(4 * kGT * kGT) void k_rank_gram(const float* __restrict__ X, int rows, int b,
                                                             double* __restrict__ W) {
  __shared__ float sx[kGRows][2 * kGT + 1];
  __shared__ double part[3][kGT * kGT];
  constexpr int kTh = 4 * kGT * kGT, kPer = kGRows * 2 * kGT / kTh, kQ = kGRows / 4;
  const int tid = threadIdx.x, grp = tid / (kGT * kGT), ent = tid % (kGT * kGT), ta = ent / kGT, tb = ent % kGT;
  const int a0 = blockIdx.y * kGT, b0 = blockIdx.x * kGT;
  float v[kPer];
  auto load = [&](int j0) {
#pragma unroll
    for (int t = 0; t < kPer; ++t) {
      const int e = tid + kTh * t, jj = e / (2 * kGT), cc = e % (2 * kGT);
      const int c = cc < kGT ? a0 + cc : b0 + cc - kGT;
      v[t] = j0 + jj < rows && c < b ? X[(long long)(j0 + jj) * b + c] : 0.f;
    }
  };
  double s = 0.0;
  load(0);
  for (int j0 = 0; j0 < rows; j0 += kGRows) {
#pragma unroll
    for (int t = 0; t < kPer; ++t) {
      const int e = tid + kTh * t;
      sx[e / (2 * kGT)][e % (2 * kGT)] = v[t];
    }
    __syncthreads();
    if (j0 + kGRows < rows) load(j0 + kGRows);
#pragma unroll
    for (int jj = 0; jj < kQ; ++jj)   // rows beyond the last are zero
      s = fma((double)sx[grp * kQ + jj][ta], (double)sx[grp * kQ + jj][kGT + tb], s);
    __syncthreads();
  }
  if (grp > 0) part[grp - 1][ent] = s;
  __syncthreads();
  const int ga = a0 + ta, gb = b0 + tb;
  if (grp == 0 && ga < b && gb < b) W[(long long)ga * b + gb] = ((s + part[0][ent]) + part[1][ent]) + part[2][ent];
}

// One workgroup: W = R^T R (R upper triangular, positive diagonal) in LDS, then
// Xf = R^{-1} (rounded to FP32, for the next product).  A pivot at or below 1e-13
// times the largest diagonal of W (a numerically rank-deficient block) is replaced
// by 1 with a zero row, so the factor stays finite; flag bit 0 records it.
// Elimination without scaling on [W | I], row i minus W[k][i] / pivot times row k, so that a
// step takes one barrier and one reciprocal: W = L D L^T, the right half becomes L^{-1} and is
// held in the lower triangle that the factor leaves free, and R^{-1} = L^{-T} D^{-1/2}.  At b = 20
// 15 us against 29 with three barriers and divisions a step and a serial back
// substitution per column through global memory.
__global__ __launch_bounds__(256) void k_rank_chol(const double* __restrict__ W, int b, float* __restrict__ Xf,
                                                   int* __restrict__ flag) {
  extern __shared__ double sw[];   // b x b: rows of W on and above the diagonal, L^{-1} below it
  __shared__ double rd[kRankBlockMax];   // D, then D^{-1/2}
  const int tid = threadIdx.x, lane = tid & 63, ty = tid >> 4, tx = tid & 15;
  double dmax = 0.0;
  for (int e = lane; e < b; e += 64) dmax = fmax(dmax, W[(long long)e * b + e]);
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) dmax = fmax(dmax, __shfl_xor(dmax, o));
  for (int e = tid; e < b * b; e += 256) {
    const int i = e / b, j = e - i * b;
    sw[e] = j >= i ? W[e] : 0.0;
  }
  __syncthreads();
  const double floor_d = 1e-13 * dmax;
  bool deficient = false;
  for (int k = 0; k < b; ++k) {
    const double d = sw[k * b + k];
    const bool ok = d > floor_d && isfinite(d);
    deficient |= !ok;
    const double inv = ok ? fast_rcp(d) : 0.0;
    if (tid == 0) rd[k] = ok ? d : 1.0;
    for (int i = k + 1 + ty; i < b && ok; i += 16) {
      const double f = -sw[k * b + i] * inv;
      for (int j = tx; j < b; j += 16) {
        if (j >= i) sw[i * b + j] = fma(f, sw[k * b + j], sw[i * b + j]);
        else if (j <= k) sw[i * b + j] = fma(f, j == k ? 1.0 : sw[k * b + j], sw[i * b + j]);
      }
    }
    __syncthreads();
  }
  if (tid == 0 && deficient) atomicOr(flag, 1);
  if (tid < b) rd[tid] = 1.0 / sqrt(rd[tid]);
  __syncthreads();
  for (int e = tid; e < b * b; e += 256) {
    const int i = e / b, c = e - i * b;
    Xf[e] = c < i ? 0.f : (float)((c == i ? 1.0 : sw[c * b + i]) * rd[c]);
  }
}

// One workgroup: eigenvalues of the symmetric b x b matrix M (FP64) by cyclic
// Jacobi with round-robin pairs (b - 1 rounds of b / 2 disjoint rotations per
// sweep, odd b padded with an idle index), until the off-diagonal mass is at
// most 1e-28 of the diagonal mass or 40 sweeps.  Then the eigenvalues in
// descending order, sv[i] = sqrt(max(lambda_i, 0)) for i < K, and the rank:
// the smallest k with sum_{i<k} lambda_i >= energy * sum_{i<K} lambda_i
// (sums in index order, FP64).
__global__ __launch_bounds__(256) void k_rank_jacobi(const double* __restrict__ Mg, int b, int K, double energy,
                                                     double* __restrict__ sv, int* __restrict__ r_out) {
  extern __shared__ double sm[];              // b x b, then the rotations (c, s) of a round
  double* cs = sm + b * b;                    // 2 * (b / 2 + 1)
  __shared__ double red[2][4];
  __shared__ int stop;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int e = tid; e < b * b; e += 256) sm[e] = Mg[e];
  const int bp = b + (b & 1), np = bp / 2;    // players (with an idle one when b is odd), pairs per round
  __syncthreads();
  for (int sweep = 0; sweep < 40; ++sweep) {
    // convergence test: off-diagonal and diagonal mass
    double off = 0.0, dg = 0.0;
    for (int e = tid; e < b * b; e += 256) {
      const int i = e / b, j = e % b;
      const double v = sm[e] * sm[e];
      if (i == j) dg += v;
      else off += v;
    }
    off = wave_sum(off);
    dg = wave_sum(dg);
    if (lane == 0) {
      red[0][wave] = off;
      red[1][wave] = dg;
    }
    __syncthreads();
    if (tid == 0) {
      const double o = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
      const double d = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
      stop = (o <= 1e-28 * d || o == 0.0) ? 1 : 0;
    }
    __syncthreads();
    if (stop) break;
    for (int rd = 0; rd < bp - 1; ++rd) {
      // pair i of this round: positions i and bp - 1 - i of the circle (position 0 fixed)
      auto player = [&](int pos) { return pos == 0 ? 0 : (pos - 1 + rd) % (bp - 1) + 1; };
      for (int i = tid; i < np; i += 256) {
        int p = player(i), q = player(bp - 1 - i);
        if (p > q) {
          const int t = p;
          p = q;
          q = t;
        }
        double c = 1.0, s = 0.0;
        if (q < b) {
          const double apq = sm[p * b + q];
          if (apq != 0.0) {
            const double theta = (sm[q * b + q] - sm[p * b + p]) / (2.0 * apq);
            const double t = (theta >= 0.0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(theta * theta + 1.0));
            c = 1.0 / sqrt(t * t + 1.0);
            s = t * c;
          }
        }
        cs[2 * i] = c;
        cs[2 * i + 1] = s;
      }
      __syncthreads();
      // rows p, q of every pair
      for (int e = tid; e < np * b; e += 256) {
        const int i = e / b, k = e % b;
        int p = player(i), q = player(bp - 1 - i);
        if (p > q) {
          const int t = p;
          p = q;
          q = t;
        }
        if (q >= b) continue;
        const double c = cs[2 * i], s = cs[2 * i + 1];
        const double xp = sm[p * b + k], xq = sm[q * b + k];
        sm[p * b + k] = c * xp - s * xq;
        sm[q * b + k] = s * xp + c * xq;
      }
      __syncthreads();
      // columns p, q of every pair
      for (int e = tid; e < np * b; e += 256) {
        const int i = e / b, k = e % b;
        int p = player(i), q = player(bp - 1 - i);
        if (p > q) {
          const int t = p;
          p = q;
          q = t;
        }
        if (q >= b) continue;
        const double c = cs[2 * i], s = cs[2 * i + 1];
        const double xp = sm[k * b + p], xq = sm[k * b + q];
        sm[k * b + p] = c * xp - s * xq;
        sm[k * b + q] = s * xp + c * xq;
      }
      __syncthreads();
    }
  }
  if (tid == 0) {
    // eigenvalues (the diagonal) in descending order, by selection
    double* lam = cs;   // reuse: b values
    for (int i = 0; i < b; ++i) lam[i] = sm[i * b + i];
    for (int i = 0; i < b; ++i) {
      int best = i;
      for (int j = i + 1; j < b; ++j)
        if (lam[j] > lam[best]) best = j;
      const double t = lam[i];
      lam[i] = lam[best];
      lam[best] = t;
    }
    const int kk = K < b ? K : b;
    double tot = 0.0;
    for (int i = 0; i < kk; ++i) tot += fmax(lam[i], 0.0);
    double cum = 0.0;
    int r = kk;
    for (int i = 0; i < kk; ++i) {
      cum += fmax(lam[i], 0.0);
      if (cum >= energy * tot) {
        r = i + 1;
        break;
      }
    }
    for (int i = 0; i < kk; ++i) sv[i] = sqrt(fmax(lam[i], 0.0));
    *r_out = r;
  }
}

// The real embedding of a complex L_0 = X + iY (n x q), given as L0t (q x n
// complex, L0t[k][j] = L_0[j][k]): E = [[X, -Y], [Y, X]] (2n x 2q), written as its
// transpose Et (2q x 2n, row-major).  The singular values of E are those of L_0,
// each twice.
__global__ void k_rank_embed(const float2* __restrict__ L0t, int q, int n, float* __restrict__ Et) {
  const long long n2 = 2LL * n;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < (long long)q * n;
       e += (long long)gridDim.x * blockDim.x) {
    const long long k = e / n, j = e % n;
    const float2 v = L0t[e];
    Et[k * n2 + j] = v.x;
    Et[k * n2 + n + j] = v.y;
    Et[(q + k) * n2 + j] = -v.y;
    Et[(q + k) * n2 + n + j] = v.x;
  }
}

// U (n x r, row-major) = the first r columns of Ub (n x b, row-major).
__global__ void k_rank_slice(const float* __restrict__ Ub, int n, int b, int r, float* __restrict__ U) {
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < (long long)n * r;
       e += (long long)gridDim.x * blockDim.x) {
    const long long j = e / r;
    const int c = (int)(e % r);
    U[e] = Ub[j * b + c];
  }
}

}  // namespace

size_t rank_lds_bytes(int b) { return (size_t)b * b * sizeof(double) + 2 * (size_t)(b / 2 + 2) * sizeof(double); }

hipError_t launch_rank_mm(bool trans, const float* A, long long lda, const float* B, long long ldb, float* C,
                          long long ldc, int M, int N, int K, hipStream_t st) {
  (void)hipGetLastError();
  const dim3 grid((N + kTile - 1) / kTile, (M + kTile - 1) / kTile);
  if (trans) hipLaunchKernelGGL(k_rank_mm<true>, grid, dim3(1024), 0, st, A, lda, B, ldb, C, ldc, M, N, K);
  else hipLaunchKernelGGL(k_rank_mm<false>, grid, dim3(1024), 0, st, A, lda, B, ldb, C, ldc, M, N, K);
  return hipGetLastError();
}

hipError_t launch_rank_gram(const float* X, int rows, int b, double* W, hipStream_t st) {
  (void)hipGetLastError();
  const dim3 grid((b + kGT - 1) / kGT, (b + kGT - 1) / kGT);
  hipLaunchKernelGGL(k_rank_gram, grid, dim3(4 * kGT * kGT), 0, st, X, rows, b, W);
  return hipGetLastError();
}

hipError_t launch_rank_chol(const double* W, int b, float* Xf, int* flag, hipStream_t st) {
  (void)hipGetLastError();
  hipLaunchKernelGGL(k_rank_chol, dim3(1), dim3(256), (size_t)b * b * sizeof(double), st, W, b, Xf, flag);
  return hipGetLastError();
}

hipError_t launch_rank_jacobi(const double* M, int b, int K, double energy, double* sv, int* r_out,
                              hipStream_t st) {
  (void)hipGetLastError();
  hipLaunchKernelGGL(k_rank_jacobi, dim3(1), dim3(256), rank_lds_bytes(b), st, M, b, K, energy, sv, r_out);
  return hipGetLastError();
}

hipError_t launch_rank_embed(const float* L0t, int q, int n, float* Et, hipStream_t st) {
  (void)hipGetLastError();
  long long g = ((long long)q * n + 255) / 256;
  if (g > 4096) g = 4096;
  if (g < 1) g = 1;
  hipLaunchKernelGGL(k_rank_embed, dim3((unsigned)g), dim3(256), 0, st, reinterpret_cast<const float2*>(L0t), q, n, Et);
  return hipGetLastError();
}

hipError_t launch_rank_slice(const float* Ub, int n, int b, int r, float* U, hipStream_t st) {
  (void)hipGetLastError();
  long long g = ((long long)n * r + 255) / 256;
  if (g > 4096) g = 4096;
  if (g < 1) g = 1;
  hipLaunchKernelGGL(k_rank_slice, dim3((unsigned)g), dim3(256), 0, st, Ub, n, b, r, U);
  return hipGetLastError();
}

}  // namespace altg
