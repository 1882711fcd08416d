// The spectral start of Alg. 1 for the real forms in one launch: orthonormalise the start
// block, then subspace iteration Z = L_0 (L_0^T U), U = Q of Z (CholeskyQR, positive
// diagonal), until ||U_new - U_old (U_old^T U_new)||_F meets the stop rule.
//
// A step is a chain of small dependent pieces (4 MB of L_0 twice at n = q = 1000, then
// r x r algebra), and how many steps run is decided by the data.  As launches, each of up
// to 100 steps took three (55 us a step at n = q = 1000, r = 10, most of it the one
// workgroup that orthonormalised), and the ones after the stop still cost their launches
// (1.7 us each, at the host's 4.6 us): 1400 us for 6 steps.  Here sub_blocks() workgroups
// stay and meet at a counter between the pieces (2.6 us for 32 workgroups, 3.3
// for 64), and the loop ends when the rule fires: 40 us for the start block and 56 us a
// step there; 24 and 17 at n = q = 100, r = 2; 50 and 125 at n = 100, q = 50,000, r = 5;
// 24 and 24 at n = 400, q = 700, r = 1, where three launches a step took 23.
//
// The workgroups need not all be resident (meet.h).  Rows are dealt to workgroups in units and
// every sum runs in a fixed order, so results depend neither on timing nor on how many
// workgroups take part.
#pragma once
#include <algorithm>
#include <cstdlib>

#include "launch.h"
#include "meet.h"
#include "uside.h"

namespace altg {

namespace {

constexpr int kSubThreads = 256, kSubWaves = kSubThreads / 64;
constexpr int kSubBlocksMax = 256;

struct SubShared {
  union {
    float red[kSubWaves][64][kRMax + 1];
    struct {
      double X[64 * kRMax], Y[64 * kRMax];
    } rows;
    double sum[kSubThreads];
  };
  double M[kRMax * kRMax];                  // the factor, or U_old^T U_new
  double rdiag[kRMax];
  double val[2];
  int flag;
  int2 roll;
};

// Part layout of a 64-row unit (doubles): Gram of Z | U_old^T U_new | Gram of U_new | change
__device__ __forceinline__ int part_stride(int r) { return r * (r + 1) + r * r + 1; }

// Sum of `cnt` entries (offset off) over the parts of all units, into dst (LDS); entry e
// over a contiguous range of units per group of threads, then the groups in order.
__device__ __forceinline__ void sum_parts(const SubArgs& a, int off, int cnt, SubShared& S, double* dst, int units) {
  const int tid = threadIdx.x, ps = part_stride(a.r);
  const int grp = sum_groups(kSubThreads, cnt, units);
  __syncthreads();
  for (int e = tid; e < cnt * grp; e += kSubThreads) {
    const int g = e / cnt, en = e - g * cnt;
    const int b0 = units * g / grp, b1 = units * (g + 1) / grp;
    S.sum[e] = sum_strided(a.part + (long long)b0 * ps + off + en, ps, b1 - b0);
  }
  __syncthreads();
  for (int e = tid; e < cnt; e += kSubThreads) {
    double s = S.sum[e];
    for (int g = 1; g < grp; ++g) s += S.sum[g * cnt + e];
    dst[e] = s;
  }
  __syncthreads();
}

// dst (LDS) = X^T Y over all n rows, as rows_gram64 lays it out; for launches without parts.
__device__ __forceinline__ void gram_all(const float* X, const float* Y, int n, int r, bool sym, SubShared& S, double* dst) {
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_id(), E = sym ? r * (r + 1) / 2 : r * r;
  const long long nr = (long long)n * r;
  for (int j0 = 0; j0 < n; j0 += 64) {
    __syncthreads();
    for (int i = tid; i < 64 * r; i += kSubThreads) {
      const long long o = (long long)j0 * r + i;
      S.rows.X[i] = o < nr ? (double)X[o] : 0.0;
      S.rows.Y[i] = o < nr ? (double)Y[o] : 0.0;
    }
    __syncthreads();
    for (int e = wave; e < E; e += kSubWaves) {
      int p = 0, c = 0;
      if (sym) tri_entry(e, r, p, c);
      else { p = e / r; c = e - p * r; }
      const double s = wave_sum_dpp(S.rows.X[lane * r + p] * S.rows.Y[lane * r + c]);
      if (lane == 0) dst[e] = j0 == 0 ? s : dst[e] + s;
    }
  }
  __syncthreads();
}

}  // namespace

// PARTS: Gram parts of the row units in a.part, each computed once; without (a scratch that has no room for
// them), every workgroup forms what it needs over all rows.
template <bool PARTS>
__global__ __launch_bounds__(kSubThreads) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_subspace(SubArgs a) {
  __shared__ SubShared S;
  __shared__ double tri[kRMax * (kRMax + 1) / 2];
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
  const int n = a.n, q = a.q, r = a.r, rr = r * r, E = r * (r + 1) / 2, KS = a.KS;
  const int units = (n + 63) / 64, ps = part_stride(r);
  const long long nr = (long long)n * r;
  Meeting meet(a.ctl);
  if (!meet.join(a.grace, &S.roll)) return;
  const int me = meet.id, nblk = meet.count;
  const int CG = max(1, min(4, (q + 16 * nblk - 1) / (16 * nblk)));   // 16-column blocks a workgroup takes at once

  // dst = Q of the thin QR of z (rows of z already in place: summed over `splits` splits,
  // which end in split 0); with old, also the parts of old^T dst.  False if z is rank
  // deficient.  Ends with every workgroup's rows of dst and parts visible.
  auto orth = [&](float* z, int splits, float* dst, const float* old) -> bool {
    for (int ru = me; ru < units; ru += nblk) {
      __syncthreads();
      const long long base = (long long)ru * 64 * r;
      for (int i = tid; i < 64 * r; i += kSubThreads) {
        float x = 0.f;
        if (base + i < nr) {
          x = z[base + i];
          if (splits <= 4) {
            for (int s = 1; s < splits; ++s) x += z[s * nr + base + i];
          } else {   // in FP64: U against FP64 at n = 100, q = 9000 0.64e-7, with FP32 sums 1.06e-7, with 4 splits 0.75e-7
            double d = (double)x;
            int s = 1;
            for (; s + 8 <= splits; s += 8) {   // in order, the loads eight at a time
              float v[8];
#pragma unroll
              for (int u = 0; u < 8; ++u) v[u] = z[(s + u) * nr + base + i];
#pragma unroll
              for (int u = 0; u < 8; ++u) d += (double)v[u];
            }
            for (; s < splits; ++s) d += (double)z[s * nr + base + i];
            x = (float)d;
          }
          if (splits > 1) z[base + i] = x;
        }
        S.rows.X[i] = (double)x;
      }
      __syncthreads();
      if constexpr (PARTS) rows_gram64<kSubWaves>(S.rows.X, S.rows.X, r, true, a.part + (long long)ru * ps);
    }
    meet();
    for (int pass = 0; pass < 2; ++pass) {
      const float* src = pass == 0 ? z : dst;
      if constexpr (PARTS) sum_parts(a, pass == 0 ? 0 : E + rr, E, S, tri, units);
      else gram_all(src, src, n, r, true, S, tri);
      if (!PARTS) meet();   // dst may be z: every workgroup has read it
      if (wave == 0) {
        for (int e = lane; e < rr; e += 64) S.M[e] = tri[tri_index(e / r, e % r, r)];
        double lo, hi;
        const bool pd = wave_cholesky_span(S.M, S.rdiag, r, lo, hi);
        if (lane == 0) S.flag = !pd ? 0 : (lo >= kPivotSpan * hi ? 1 : 2);
      }
      __syncthreads();
      const int mode = S.flag;
      if (mode == 0) return false;
      const bool again = pass == 0 && mode == 2;   // ill-conditioned: once more on the rounded rows
      for (int ru = me; ru < units; ru += nblk) {
        const int j = ru * 64 + tid;
        const long long o = (long long)j * r;
        if (tid < 64) {
          double x[kRMax];
#pragma unroll
          for (int c = 0; c < kRMax; ++c)
            if (c < r) x[c] = j < n ? (double)src[o + c] : 0.0;
          solve_row(x, S.M, S.rdiag, r);
#pragma unroll
          for (int c = 0; c < kRMax; ++c)
            if (c < r) {
              const float v = (float)x[c];
              if (j < n) dst[o + c] = v;
              S.rows.X[tid * r + c] = (double)v;
            }
        }
        if (old)
          for (int i = tid; i < 64 * r; i += kSubThreads)
            S.rows.Y[i] = (long long)ru * 64 * r + i < nr ? (double)old[(long long)ru * 64 * r + i] : 0.0;
        __syncthreads();
        if constexpr (PARTS) {
          double* pt = a.part + (long long)ru * ps;
          if (again) rows_gram64<kSubWaves>(S.rows.X, S.rows.X, r, true, pt + E + rr);
          else if (old) rows_gram64<kSubWaves>(S.rows.Y, S.rows.X, r, false, pt + E);
          __syncthreads();
        }
      }
      meet();
      if (!again) break;
    }
    return true;
  };

  // the change of the last step, from the units' parts in order, and the stop rule
  double prev = 0.0;
  auto decide = [&]() -> bool {
    if constexpr (PARTS) sum_parts(a, ps - 1, 1, S, S.val, units);
    const double sd = sqrt(S.val[0]);
    // converged at tol, or once the change has stopped shrinking below 1e-3 (by less
    // than 1 % in a step): the FP32 iterate's rounding floor.  A change that still
    // shrinks by a steady factor above 0.9 is a slow iteration, not the floor.
    const bool conv = sd <= a.tol || (sd <= 1e-3 && prev > 0.0 && sd >= 0.99 * prev);
    if (me == 0 && tid == 0) {
      a.ctl->power_sd = sd;
      a.ctl->power_it += 1;
      if (conv) a.ctl->conv = 1;
    }
    prev = sd;
    return conv;
  };

  float* cur = a.U;
  float* nxt = a.V;
  bool ok = orth(a.start, 1, cur, nullptr);
  bool pending = false;
  for (int p = 0; ok && p < a.iters; ++p) {
    // T = L_0^T U on the matrix cores, 16 columns k by r at a time, the rows j split over the
    // workgroup's waves 16 at a time: lane (i, p) holds 4 rows of column i, and the four
    // products of a group take row 4 p + e of it, e = 0..3, for both operands.  Up to four such blocks of
    // columns go through LDS together, where each workgroup has that many.
    for (int kb = me * 16 * CG; kb < q; kb += nblk * 16 * CG) {
      typedef float f32x4 __attribute__((ext_vector_type(4)));
      const int i = lane & 15, p4 = 4 * (lane >> 4);
      __syncthreads();
      for (int cg = 0; cg < CG && kb + 16 * cg < q; ++cg) {
        const int k = kb + 16 * cg + i;
        const float* row = a.L0t + (long long)(k < q ? k : q - 1) * n;
        constexpr int SU = 4;   // 16-row groups in flight per wave
        // the FP32 sums end with the loads in flight (16 products each) and are added in FP64: sums of n / 32
        // products in FP32 round worse than the sums over lanes that they replaced (U against FP64 at
        // n = q = 1000, mean of 40 draws: 1.13e-7, over lanes 0.96e-7, these 0.91e-7; ten steps 597 and 600 us,
        // at n = 20,000, q = 50: 1393 and 1462).  All products in FP64: 671 and 2950 us.
        double tot[4] = {0.0, 0.0, 0.0, 0.0};
        for (int s0 = wave * 16; s0 < n; s0 += kSubWaves * 16 * SU) {
          float x[SU][4], u[SU][4];
#pragma unroll
          for (int g = 0; g < SU; ++g) {
            const int j = s0 + g * kSubWaves * 16 + p4;
            if (j + 4 <= n) {
              const f32x4_u v = *reinterpret_cast<const f32x4_u*>(row + j);
              x[g][0] = v.x; x[g][1] = v.y; x[g][2] = v.z; x[g][3] = v.w;
            } else {
#pragma unroll
              for (int e = 0; e < 4; ++e) x[g][e] = j + e < n ? row[j + e] : 0.f;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) u[g][e] = i < r && j + e < n ? cur[(long long)(j + e) * r + i] : 0.f;
          }
          f32x4 acc[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[e] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int g = 0; g < SU; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[g][e], u[g][e], acc[e], 0, 0, 0);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            tot[e] += ((double)acc[0][e] + (double)acc[1][e]) + ((double)acc[2][e] + (double)acc[3][e]);
        }
        // lane (i, p) holds column i of rows 4 p .. 4 p + 3 of the 16 x 16 result
#pragma unroll
        for (int e = 0; e < 4; ++e) S.red[wave][16 * cg + p4 + e][i] = (float)tot[e];
      }
      __syncthreads();
      for (int t = tid; t < 16 * CG * r; t += kSubThreads) {
        const int kk = t / r, c = t - kk * r;
        if (kb + kk < q) {
          double v = S.red[0][kk][c];
#pragma unroll
          for (int w = 1; w < kSubWaves; ++w) v += (double)S.red[w][kk][c];
          a.T[(long long)(kb + kk) * r + c] = (float)v;
        }
      }
    }
    meet();
    if (pending) {
      pending = false;
      if (decide()) break;
    }
    // Z = L_0 T by 64-row units and column splits
    for (int w = me; w < units * KS; w += nblk) {
      const int ru = KS == 1 ? w : w / KS, ks = w - ru * KS;
      const int k0 = (int)((long long)q * ks / KS), k1 = (int)((long long)q * (ks + 1) / KS);
      const long long base = (long long)ru * 64 * r;
      __syncthreads();
      urows_grad_r<kSubWaves>(a.L0t, a.T, n, r, ru, k0, k1, S.red, [&](int i, float g) {
        if (base + i < nr) a.gpart[ks * nr + base + i] = g;
      });
    }
    if (KS > 1) meet();
    __syncthreads();
    ok = orth(a.gpart, KS, nxt, cur);
    if (!ok) break;
    // the change ||U_new - U_old W||_F of this workgroup's rows, W = U_old^T U_new,
    // summed directly from the residual entries; decided after the next meeting
    if constexpr (PARTS) sum_parts(a, E, rr, S, S.M, units);
    else gram_all(cur, nxt, n, r, false, S, S.M);
    double all = 0.0;   // without parts: the units of all workgroups, in order
    for (int ru = PARTS ? me : 0; ru < units; ru += PARTS ? nblk : 1) {
      if (wave == 0) {
        const int j = ru * 64 + lane;
        const long long o = (long long)j * r;
        double acc = 0.0;
        if (j < n) {
          float u[kRMax], v[kRMax];
#pragma unroll
          for (int e = 0; e < kRMax; ++e) {
            u[e] = e < r ? cur[o + e] : 0.f;
            v[e] = e < r ? nxt[o + e] : 0.f;
          }
#pragma unroll
          for (int c = 0; c < kRMax; ++c)
            if (c < r) {
              double d = (double)v[c];
#pragma unroll
              for (int e = 0; e < kRMax; ++e)
                if (e < r) d = fma(-(double)u[e], S.M[e * r + c], d);
              acc = fma(d, d, acc);
            }
        }
        acc = wave_sum_dpp(acc);
        if constexpr (PARTS) {
          if (lane == 0) a.part[(long long)ru * ps + ps - 1] = acc;
        } else {
          all += acc;
        }
      }
    }
    if (!PARTS && tid == 0) S.val[0] = all;
    __syncthreads();
    pending = true;
    float* x = cur;
    cur = nxt;
    nxt = x;
  }
  if (pending) {   // the step limit: record the last change (after a failed step, the one before)
    meet();
    decide();
  }
  if (!ok && me == 0 && tid == 0) atomicOr(&a.ctl->err, 2);
  if (cur != a.U)           // this workgroup's rows, read by no other one any more
    for (int ru = me; ru < units; ru += nblk) {
      const long long base = (long long)ru * 64 * r;
      for (int i = tid; i < 64 * r; i += kSubThreads)
        if (base + i < nr) a.U[base + i] = cur[base + i];
    }
}

// ---------------------------------------------------------------- launcher

size_t sub_part_doubles(int n, int r) { return (size_t)((n + 63) / 64) * (size_t)(r * (r + 1) + r * r + 1); }

// Workgroups: as many as have 16 columns for L_0^T U or rows of their own, at most
// kSubBlocksMax.
static int sub_blocks(int n, int q) {
  const int cols = (q + 15) / 16, rows = (n + 63) / 64;
  const int b = cols > rows ? cols : rows;
  return b < kSubBlocksMax ? b : kSubBlocksMax;
}

// Column splits of Z: a 64-row unit per workgroup with at least 32 columns each; at most 2 below 512
// columns and 4 below 2048, where a split more saves less than its plane costs to add (n = q = 100:
// 3 splits 1 % slower than 2 over a solve), 32 above (n = 100, q = 50,000: 0.13 ms a step, 0.48 with 4).
int sub_splits(int n, int q) {
  int ks = sub_blocks(n, q) / ((n + 63) / 64);
  const int cap = q < 512 ? 2 : (q < 2048 ? 4 : 32);
  if (ks > q / 32) ks = q / 32;
  if (ks > cap) ks = cap;
  return ks < 1 ? 1 : ks;
}

// ALTGDMIN_START_GRACE_US forces the wait for late workgroups (tests: 0 closes the roll at once).
int roll_grace() {
  if (const char* f = std::getenv("ALTGDMIN_START_GRACE_US")) {
    const int us = std::atoi(f);
    if (us >= 0 && us <= 1000000) return 100 * us;
  }
  return kRollGrace;
}

hipError_t launch_subspace(const SubArgs& a_in, int max_splits, hipStream_t st) {
  SubArgs a = a_in;
  a.grace = roll_grace();
  a.KS = std::min(sub_splits(a.n, a.q), max_splits);
  (void)hipGetLastError();   // clear a stale error of an earlier, unrelated call
  hipLaunchKernelGGL(a.part ? k_subspace<true> : k_subspace<false>, dim3(sub_blocks(a.n, a.q)), dim3(kSubThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace altg
