// The U side of AltGDmin-LR+S for gfx950: the U update of a GDmin iteration (update.h) and
// the spectral start (subspace.h), and the small kernels beside them: sums over the
// columns, the control block, fills and copies, start blocks and restored supports.
#include "launch.h"
#include "subspace.h"
#include "update.h"

namespace altg {

// ||Y||_F^2 from the per-column values, fixed order.
__global__ __launch_bounds__(kQRThreads) void k_sum_ctl(const double* colrr, int q, Ctl* ctl) {
  __shared__ double sh[kQRThreads];
  const int tid = threadIdx.x;
  double s = 0.0;
  for (int k = tid; k < q; k += kQRThreads) s += colrr[k];
  sh[tid] = s;
  __syncthreads();
  for (int st = kQRThreads / 2; st > 0; st >>= 1) {
    if (tid < st) sh[tid] += sh[tid + st];
    __syncthreads();
  }
  if (tid == 0) ctl->ynorm2 = sh[0];
}

__global__ void k_set_phase(Ctl* ctl, int phase) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    ctl->phase = phase;
    ctl->refine_t = phase ? 0 : -1;
  }
}

__global__ void k_reset_ctl(Ctl* ctl, int full) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    ctl->eta = 0.0;
    ctl->eta_set = 0;
    ctl->t = 0;
    ctl->resid = 0.0;
    ctl->prev_resid = 0.0;
    ctl->done = 0;
    ctl->bar = 0;
    ctl->roll = 0;
    ctl->members = 0;
    if (full) {
      ctl->power_sd = 0.0;
      ctl->ynorm2 = 0.0;
      ctl->conv = 0;
      ctl->power_it = 0;
      ctl->err = 0;
    }
  }
}

__global__ void k_fill_int(int* p, int v, long long count) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < count; i += (long long)gridDim.x * blockDim.x) p[i] = v;
}

// U[j][c] = 1 if j % r == c else 0: an orthogonal start block with disjoint supports.
__global__ void k_fill_basis(float* U, int n, int r) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < (long long)n * r; i += (long long)gridDim.x * blockDim.x) {
    const int j = (int)(i / r), c = (int)(i % r);
    U[i] = (j % r == c) ? 1.f : 0.f;
  }
}

__global__ void k_copy_f(float* dst, const float* src, long long count) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < count; i += (long long)gridDim.x * blockDim.x) dst[i] = src[i];
}

__global__ void k_copy_i(int* dst, const int* src, long long count) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < count; i += (long long)gridDim.x * blockDim.x) dst[i] = src[i];
}

// A support loaded into a solver (altgdmin_set_state) must hold rho distinct
// in-range indices in ascending order in every column; a column that does not
// gets the no-start support 0 .. rho - 1 with zero values and error bit 2.
// One 64-thread workgroup per column; vpe = floats per value (2 for complex).
__global__ void k_check_support(int* idx, float* val, int vpe, int q, int rho, int n, int* flags) {
  const int k = blockIdx.x, lane = threadIdx.x;
  if (k >= q) return;
  int* ik = idx + (long long)k * rho;
  float* vk = val + (long long)k * rho * vpe;
  int bad = 0;
  for (int t = lane; t < rho; t += 64) {
    const int j = ik[t];
    bad |= (j < 0 || j >= n || (t > 0 && j <= ik[t - 1])) ? 1 : 0;
  }
  if (__ballot(bad != 0) == 0ull) return;
  for (int t = lane; t < rho; t += 64) {
    ik[t] = t;
    for (int c = 0; c < vpe; ++c) vk[(long long)t * vpe + c] = 0.f;
  }
  if (lane == 0) flags[k] |= 4;
}

__global__ void k_put_words(long long* dst, StateWords w) {
  if (threadIdx.x < kStateWords && blockIdx.x == 0) dst[threadIdx.x] = w.v[threadIdx.x];
}

__global__ void k_sum_partials(const float* gpart, int KS, long long nr, float* out) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < nr; i += (long long)gridDim.x * blockDim.x) {
    float s = gpart[i];
    for (int ks = 1; ks < KS; ++ks) s += gpart[(long long)ks * nr + i];
    out[i] = s;
  }
}

// ---------------------------------------------------------------- launchers

static inline int grid_for(long long count, int block) {
  long long g = (count + block - 1) / block;
  if (g < 1) g = 1;
  if (g > 4096) g = 4096;
  return (int)g;
}

hipError_t launch_sum_ctl(const double* colrr, int q, Ctl* ctl, hipStream_t st) {
  (void)hipGetLastError();   // clear a stale error of an earlier, unrelated call
  hipLaunchKernelGGL(k_sum_ctl, dim3(1), dim3(kQRThreads), 0, st, colrr, q, ctl);
  return hipGetLastError();
}

hipError_t launch_reset_ctl(Ctl* ctl, int full, hipStream_t st) {
  (void)hipGetLastError();   // clear a stale error of an earlier, unrelated call
  hipLaunchKernelGGL(k_reset_ctl, dim3(1), dim3(64), 0, st, ctl, full);
  return hipGetLastError();
}

hipError_t launch_set_phase(Ctl* ctl, int phase, hipStream_t st) {
  (void)hipGetLastError();   // clear a stale error of an earlier, unrelated call
  hipLaunchKernelGGL(k_set_phase, dim3(1), dim3(64), 0, st, ctl, phase);
  return hipGetLastError();
}

hipError_t launch_fill_int(int* p, int v, long long count, hipStream_t st) {
  (void)hipGetLastError();   // clear a stale error of an earlier, unrelated call
  hipLaunchKernelGGL(k_fill_int, dim3(grid_for(count, 256)), dim3(256), 0, st, p, v, count);
  return hipGetLastError();
}

hipError_t launch_fill_basis(float* U, int n, int r, hipStream_t st) {
  (void)hipGetLastError();   // clear a stale error of an earlier, unrelated call
  hipLaunchKernelGGL(k_fill_basis, dim3(grid_for((long long)n * r, 256)), dim3(256), 0, st, U, n, r);
  return hipGetLastError();
}

hipError_t launch_copy_f(float* dst, const float* src, long long count, hipStream_t st) {
  (void)hipGetLastError();   // clear a stale error of an earlier, unrelated call
  hipLaunchKernelGGL(k_copy_f, dim3(grid_for(count, 256)), dim3(256), 0, st, dst, src, count);
  return hipGetLastError();
}

hipError_t launch_sum_partials(const float* gpart, int KS, long long nr, float* out, hipStream_t st) {
  (void)hipGetLastError();   // clear a stale error of an earlier, unrelated call
  hipLaunchKernelGGL(k_sum_partials, dim3(grid_for(nr, 256)), dim3(256), 0, st, gpart, KS, nr, out);
  return hipGetLastError();
}

hipError_t launch_check_support(int* idx, float* val, int vpe, int q, int rho, int n, int* flags, hipStream_t st) {
  (void)hipGetLastError();   // clear a stale error of an earlier, unrelated call
  if (q < 1 || rho < 1) return hipSuccess;
  hipLaunchKernelGGL(k_check_support, dim3(q), dim3(64), 0, st, idx, val, vpe, q, rho, n, flags);
  return hipGetLastError();
}

hipError_t launch_put_words(long long* dst, const StateWords& w, hipStream_t st) {
  (void)hipGetLastError();   // clear a stale error of an earlier, unrelated call
  hipLaunchKernelGGL(k_put_words, dim3(1), dim3(64), 0, st, dst, w);
  return hipGetLastError();
}

hipError_t launch_copy_i(int* dst, const int* src, long long count, hipStream_t st) {
  (void)hipGetLastError();   // clear a stale error of an earlier, unrelated call
  hipLaunchKernelGGL(k_copy_i, dim3(grid_for(count, 256)), dim3(256), 0, st, dst, src, count);
  return hipGetLastError();
}

}  // namespace altg
