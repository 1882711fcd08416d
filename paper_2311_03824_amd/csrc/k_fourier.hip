// Partial Fourier form of the measurement operators (gfx950).
//
// A_k keeps the rows mask_k of the unitary 2D DFT of 96 x 96 complex frames
// (x_k flattened row-major; frequency index u = u1 * 96 + u2), so
// A_k x = (F x)[mask_k] and A_k^H v = F^H (v scattered to mask_k).  All data are
// complex64 (float2 = re, im); every transpose of the real path is a conjugate
// transpose and HardThreshold ranks by modulus.  Per GDmin iteration of Alg. 1:
//
//   k_fu   : F U (the DFT of each column of U): a row pass and a column pass,
//            one 96-point line per 32 lanes;
//   k_fcol : per column k (one 1024-thread workgroup): P_k = (F U)[mask_k],
//            G_k = P_k^H P_k and its inverse in FP64, the projected IHT of
//            Alg. 2 (tau iterations, three 2D FFTs each), b_k by least squares
//            (eq. (bk_LS)), r_k and h_k = A_k^H r_k;
//   k_frows, k_fapply (fourier_u.h): grad_U f = sum_k h_k b_k^H, eta at t = 1, U - eta
//            grad orthonormalised with a real positive diagonal, the residual.
// The initialisation uses k_fcol with M = A_k (IHT from 0, then the columns of
// L_0 = [A_k^H (y_k - A_k s_k)]) and k_fsub (the start block and the subspace iteration).
//
// 2D FFT.  A frame lives in LDS as 96 rows of 97 complex values (one pad column
// keeps the column pass free of bank conflicts).  Each 96-point transform is
// done by a group of 32 lanes: lane l holds elements l, l + 32, l + 64; a
// radix-3 butterfly with twiddles W96^(l k2) is followed by a 32-point radix-2
// decimation-in-frequency transform across the lanes (ds_swizzle exchanges), so
// lane l ends with outputs 3 bitrev5(l) + k2.  Rows first, then columns; the
// unitary scale 1/96 is applied in the column pass.
//
// Other frame sizes (n1 x n2 with n = n1 n2 <= 4096 and lines of at most 1024
// points; e.g. the 20 x 20 frames or the 1 x 400 rows of a 1D DFT) take the
// generic instantiation (GEN) of the column kernel: frames are stored unpadded
// and each 2D DFT is a row pass and a column pass of direct line DFTs, every
// output a sum over its line in index order with twiddles W_N^((u j) mod N) from
// a table in LDS (n1 + n2 entries); up to four outputs per thread are held in
// registers across a barrier, so the passes run in place.  k_fu_gen is the same
// transform of the columns of U.
#include "common.h"
#include "fourier_u.h"
#include "launch.h"

namespace altg {

namespace {

__device__ __forceinline__ float2 c_add(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 c_sub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 c_mul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 c_scale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }

// |v|^2 as the ranking key: two products and one sum, each rounded to FP32.
__device__ __forceinline__ float c_abs2_key(float2 v) {
#pragma clang fp contract(off)
  const float a = v.x * v.x;
  const float b = v.y * v.y;
  return a + b;
}

__device__ __forceinline__ int fpos(int j) { return j + j / kFN; }   // element j -> padded grid slot

template <int H>
__device__ __forceinline__ float2 swz_xor(float2 v) {
  // ds_swizzle bit mode inside groups of 32 lanes: partner = lane ^ H
  constexpr int pat = (H << 10) | 0x1f;
  return make_float2(__int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v.x), pat)),
                     __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v.y), pat)));
}

template <bool INV>
__device__ __forceinline__ float2 twid(const float2* tw, int e) {   // W96^e (conjugated for the inverse)
  const float2 w = tw[e];
  return INV ? make_float2(w.x, -w.y) : w;
}

template <bool INV, int H>
__device__ __forceinline__ void dif_stage(float2 (&v)[3], int l, const float2* tw) {
  const bool up = (l & H) != 0;
  const float2 w = twid<INV>(tw, 3 * ((l & (H - 1)) * (16 / H)));   // W32^((l mod H) 16 / H)
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float2 t = swz_xor<H>(v[a]);
    v[a] = up ? c_mul(c_sub(t, v[a]), w) : c_add(v[a], t);
  }
}

// 96-point DFT by the 32 lanes of a group: in v[a] = x[l + 32 a], out v[a] = X[3 bitrev5(l) + a].
template <bool INV>
__device__ __forceinline__ void fft96(float2 (&v)[3], int l, const float2* tw) {
  const float2 w1 = twid<INV>(tw, 32), w2 = twid<INV>(tw, 64);   // W3, W3^2
  const float2 x0 = v[0], x1 = v[1], x2 = v[2];
  v[0] = c_add(c_add(x0, x1), x2);
  v[1] = c_mul(c_add(c_add(x0, c_mul(x1, w1)), c_mul(x2, w2)), twid<INV>(tw, l));
  v[2] = c_mul(c_add(c_add(x0, c_mul(x1, w2)), c_mul(x2, w1)), twid<INV>(tw, 2 * l));
  dif_stage<INV, 16>(v, l, tw);
  dif_stage<INV, 8>(v, l, tw);
  dif_stage<INV, 4>(v, l, tw);
  dif_stage<INV, 2>(v, l, tw);
  dif_stage<INV, 1>(v, l, tw);
}

// Unitary 2D DFT (INV: its inverse) of the frame in `grid`, in place.  All 1024
// threads call it; it ends with a barrier.
template <bool INV>
__device__ __attribute__((noinline)) void fft2_grid(float2* grid, const float2* tw) {
  const int g = threadIdx.x >> 5, l = threadIdx.x & 31;
  const int k1 = (int)(__builtin_bitreverse32((unsigned)l) >> 27);
  for (int rr = 0; rr < 3; ++rr) {
    float2* row = grid + (g + 32 * rr) * kFP;
    float2 v[3] = {row[l], row[l + 32], row[l + 64]};
    fft96<INV>(v, l, tw);
    row[3 * k1] = v[0];
    row[3 * k1 + 1] = v[1];
    row[3 * k1 + 2] = v[2];
  }
  __syncthreads();
  const float s = 1.0f / kFN;
  for (int cc = 0; cc < 3; ++cc) {
    float2* col = grid + g + 32 * cc;
    float2 v[3] = {col[l * kFP], col[(l + 32) * kFP], col[(l + 64) * kFP]};
    fft96<INV>(v, l, tw);
    col[(3 * k1) * kFP] = c_scale(v[0], s);
    col[(3 * k1 + 1) * kFP] = c_scale(v[1], s);
    col[(3 * k1 + 2) * kFP] = c_scale(v[2], s);
  }
  __syncthreads();
}

__device__ __forceinline__ void zero_grid(float2* grid, int count = kFGrid) {
  for (int t = threadIdx.x; t < count; t += kFThreads) grid[t] = make_float2(0.f, 0.f);
}

// Unitary 2D DFT (INV: inverse) of an unpadded n1 x n2 frame in `grid`, in place,
// by direct line sums: first X[j1][u2] = sum_j2 x[j1][j2] W_n2^(u2 j2), then
// X[u1][u2] = scale sum_j1 X[j1][u2] W_n1^(u1 j1), each sum in index order.  tw
// holds W_n1^t (t < n1) then W_n2^t (t < n2).  All threads of the workgroup call
// it (blockDim.x = kFThreads, n1 n2 <= kFGenPer kFThreads); it ends with a barrier.
template <bool INV>
__device__ __attribute__((noinline)) void dft2_gen(float2* grid, const float2* tw, int n1, int n2, float scale) {
  const int n = n1 * n2;
  const float2* tw1 = tw;
  const float2* tw2 = tw + n1;
  float2 acc[kFGenPer];
#pragma unroll
  for (int e = 0; e < kFGenPer; ++e) {
    const int t = threadIdx.x + e * kFThreads;
    float2 sum = make_float2(0.f, 0.f);
    if (t < n) {
      const int j1 = t / n2, u2 = t - j1 * n2;
      const float2* row = grid + j1 * n2;
      int w = 0;   // (u2 j2) mod n2
      for (int j2 = 0; j2 < n2; ++j2) {
        const float2 x = row[j2], tt = twid<INV>(tw2, w);
        sum.x = fmaf(x.x, tt.x, fmaf(-x.y, tt.y, sum.x));
        sum.y = fmaf(x.x, tt.y, fmaf(x.y, tt.x, sum.y));
        w += u2;
        if (w >= n2) w -= n2;
      }
    }
    acc[e] = sum;
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < kFGenPer; ++e) {
    const int t = threadIdx.x + e * kFThreads;
    if (t < n) grid[t] = acc[e];
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < kFGenPer; ++e) {
    const int t = threadIdx.x + e * kFThreads;
    float2 sum = make_float2(0.f, 0.f);
    if (t < n) {
      const int u1 = t / n2, u2 = t - u1 * n2;
      int w = 0;   // (u1 j1) mod n1
      for (int j1 = 0; j1 < n1; ++j1) {
        const float2 x = grid[j1 * n2 + u2], tt = twid<INV>(tw1, w);
        sum.x = fmaf(x.x, tt.x, fmaf(-x.y, tt.y, sum.x));
        sum.y = fmaf(x.x, tt.y, fmaf(x.y, tt.x, sum.y));
        w += u1;
        if (w >= n1) w -= n1;
      }
    }
    acc[e] = c_scale(sum, scale);
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < kFGenPer; ++e) {
    const int t = threadIdx.x + e * kFThreads;
    if (t < n) grid[t] = acc[e];
  }
  __syncthreads();
}

// Sum over the workgroup of NV doubles per thread, in a fixed order (DPP inside
// each wave, then the 16 wave totals in wave order).  out[0..NV) in LDS; ends
// with a barrier.  red holds kFWaves * NV doubles.
template <int NV>
__device__ void fblock_sum(double (&v)[NV], double* red, double* out) {
  const int lane = threadIdx.x & 63, wave = wave_id();
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] = wave_sum_dpp(v[i]);
  if (lane == 0)
#pragma unroll
    for (int i = 0; i < NV; ++i) red[wave * NV + i] = v[i];
  __syncthreads();
  if (threadIdx.x < NV) {
    double s = 0.0;
    for (int w = 0; w < kFWaves; ++w) s += red[w * NV + threadIdx.x];
    out[threadIdx.x] = s;
  }
  __syncthreads();
}

// Whether HardThreshold keeps the support marked in the bitmap `mark`: it does
// when every key on it is larger than every key off it (with a tie or a NaN key
// the full select decides).  slot holds 3 kFWaves words of LDS; a barrier on
// entry to the reduction and on exit.
template <class Val>
__device__ bool fsupport_kept(Val val, int n, const unsigned* mark, unsigned* slot) {
  const int lane = threadIdx.x & 63, wave = wave_id();
  unsigned kmin = 0xffffffffu, kmax = 0u;
  bool bad = false;
  for (int j = threadIdx.x; j < n; j += kFThreads) {
    const unsigned key = __float_as_uint(c_abs2_key(val(j)));
    bad |= key > 0x7f800000u;
    if ((mark[j >> 5] >> (j & 31)) & 1u)
      kmin = min(kmin, key);
    else
      kmax = max(kmax, key);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    kmin = min(kmin, __shfl_xor(kmin, o));
    kmax = max(kmax, __shfl_xor(kmax, o));
  }
  const bool wbad = __ballot(bad) != 0ull;
  if (lane == 0) {
    slot[3 * wave] = kmin;
    slot[3 * wave + 1] = kmax;
    slot[3 * wave + 2] = wbad ? 1u : 0u;
  }
  __syncthreads();
  unsigned mn = 0xffffffffu, mx = 0u, b = 0u;
#pragma unroll
  for (int w = 0; w < kFWaves; ++w) {
    mn = min(mn, slot[3 * w]);
    mx = max(mx, slot[3 * w + 1]);
    b |= slot[3 * w + 2];
  }
  __syncthreads();
  return b == 0u && mn > mx;
}

// Whether any thread of the workgroup has f != 0 (every thread calls it; a
// barrier on entry and on exit).  slot holds kFWaves ints of LDS.
__device__ bool fblock_any(int f, int* slot) {
  const int lane = threadIdx.x & 63, wave = wave_id();
  const bool any = __ballot(f != 0) != 0ull;
  if (lane == 0) slot[wave] = any ? 1 : 0;
  __syncthreads();
  int r = 0;
#pragma unroll
  for (int w = 0; w < kFWaves; ++w) r |= slot[w];
  __syncthreads();
  return r != 0;
}

// Exclusive prefix sum of one int per thread over the workgroup in thread order;
// *total gets the sum.  tmp holds kFWaves + 1 ints.
__device__ int fblock_exscan(int v, int* tmp, int* total) {
  const int lane = threadIdx.x & 63, wave = wave_id();
  int incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(incl, o);
    if (lane >= o) incl += t;
  }
  if (lane == 63) tmp[wave] = incl;
  __syncthreads();
  int base = 0, all = 0;
  for (int w = 0; w < kFWaves; ++w) {
    const int t = tmp[w];
    base += w < wave ? t : 0;
    all += t;
  }
  *total = all;
  __syncthreads();
  return base + incl - v;
}

// HardThreshold support of n complex values: the rho largest keys |v|^2 (FP32,
// as c_abs2_key), lower index first on ties, written ascending to idx[0..rho).
// Thread t owns the contiguous elements [t c, t c + c), c = ceil(n / 1024).
// Byte-wise radix selection with a 256-bin LDS histogram.  Returns the number of
// NaN keys seen.  hist holds 256 + 8 ints, tmp kFWaves + 1 ints.
template <class Val>
__device__ int fselect(Val val, int n, int rho, int* idx, int* hist, int* tmp) {
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
  const int per = (n + kFThreads - 1) / kFThreads;
  const int j0 = tid * per;
  const int j1 = min(n, j0 + per);
  int* ctl = hist + 256;
  unsigned prefix = 0u, pmask = 0u;
  int remaining = rho;
  int nanc = 0;
  for (int d = 3; d >= 0; --d) {
    const int shift = 8 * d;
    for (int b = tid; b < 256; b += kFThreads) hist[b] = 0;
    if (d == 3 && tid == 0) ctl[2] = 0;
    __syncthreads();
    for (int j = j0; j < j1; ++j) {
      const unsigned key = __float_as_uint(c_abs2_key(val(j)));
      if (d == 3) nanc += key > 0x7f800000u ? 1 : 0;
      if ((key & pmask) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1);
    }
    if (d == 3 && nanc) atomicAdd(&ctl[2], nanc);
    __syncthreads();
    if (wave == 0) {
      const int h0 = hist[4 * lane], h1 = hist[4 * lane + 1], h2 = hist[4 * lane + 2], h3 = hist[4 * lane + 3];
      const int lsum = h0 + h1 + h2 + h3;
      int incl = lsum;   // inclusive suffix sum over lanes >= lane
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_down(incl, o);
        if (lane + o < 64) incl += t;
      }
      int acc = incl - lsum;
      const int hb[4] = {h3, h2, h1, h0};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (acc < remaining && remaining <= acc + hb[q]) {
          ctl[0] = 4 * lane + 3 - q;
          ctl[1] = remaining - acc;
        }
        acc += hb[q];
      }
    }
    __syncthreads();
    remaining = ctl[1];
    prefix |= (unsigned)ctl[0] << shift;
    pmask |= 255u << shift;
    __syncthreads();
  }
  const unsigned T = prefix;
  int ngt = 0, neq = 0;
  for (int j = j0; j < j1; ++j) {
    const unsigned key = __float_as_uint(c_abs2_key(val(j)));
    ngt += key > T ? 1 : 0;
    neq += key == T ? 1 : 0;
  }
  int tot;
  const int eq_base = fblock_exscan(neq, tmp, &tot);
  const int take_eq = max(0, min(neq, remaining - eq_base));
  const int nsel = ngt + take_eq;
  const int pos0 = fblock_exscan(nsel, tmp, &tot);
  int pos = pos0, eqs = 0;
  for (int j = j0; j < j1; ++j) {
    const unsigned key = __float_as_uint(c_abs2_key(val(j)));
    bool sel = key > T;
    if (key == T) {
      sel = eqs < take_eq;
      ++eqs;
    }
    if (sel && pos < rho) idx[pos++] = j;
  }
  const int nan_total = ctl[2];
  __syncthreads();
  return nan_total;
}

// G^{-1} of a Hermitian positive definite r x r matrix (complex FP64, row-major
// double2 = re, im), by the workgroup: Cholesky G = L L^H (real positive
// diagonal) column by column, thread j + 1 + t computing L[j + 1 + t][j]; then
// thread c solves L y = e_c and L^H x = y for column c.  Returns false (identity
// in Ginv) if a pivot is not positive.
__device__ bool fblock_chol_inverse(const double2* G, double2* L, double2* Ginv, double2* Y, int r) {
  const int tid = threadIdx.x;
  for (int j = 0; j < r; ++j) {
    double s = G[j * r + j].x;
    for (int p = 0; p < j; ++p) s -= L[j * r + p].x * L[j * r + p].x + L[j * r + p].y * L[j * r + p].y;
    if (!(s > 0.0)) {
      for (int i = tid; i < r * r; i += kFThreads) Ginv[i] = make_double2((i % (r + 1) == 0) ? 1.0 : 0.0, 0.0);
      __syncthreads();
      return false;
    }
    const double d = sqrt(s);
    const int i = j + 1 + tid;
    if (i < r) {
      double tr = G[i * r + j].x, ti = G[i * r + j].y;
      for (int p = 0; p < j; ++p) {   // t -= L[i][p] conj(L[j][p])
        const double2 a = L[i * r + p], b = L[j * r + p];
        tr -= a.x * b.x + a.y * b.y;
        ti -= a.y * b.x - a.x * b.y;
      }
      L[i * r + j] = make_double2(tr / d, ti / d);
    }
    if (tid == 0) L[j * r + j] = make_double2(d, 0.0);
    if (tid < j) L[tid * r + j] = make_double2(0.0, 0.0);
    __syncthreads();
  }
  if (tid < r) {
    const int c = tid;
    for (int i = c; i < r; ++i) {
      double tr = (i == c) ? 1.0 : 0.0, ti = 0.0;
      for (int p = c; p < i; ++p) {   // t -= L[i][p] y[p]
        const double2 a = L[i * r + p], y = Y[p * r + c];
        tr -= a.x * y.x - a.y * y.y;
        ti -= a.x * y.y + a.y * y.x;
      }
      const double dd = L[i * r + i].x;
      Y[i * r + c] = make_double2(tr / dd, ti / dd);
    }
    for (int i = r - 1; i >= 0; --i) {
      double tr = i >= c ? Y[i * r + c].x : 0.0, ti = i >= c ? Y[i * r + c].y : 0.0;
      for (int p = i + 1; p < r; ++p) {   // t -= conj(L[p][i]) x[p]
        const double2 a = L[p * r + i], x = Ginv[p * r + c];
        tr -= a.x * x.x + a.y * x.y;
        ti -= a.x * x.y - a.y * x.x;
      }
      const double dd = L[i * r + i].x;
      Ginv[i * r + c] = make_double2(tr / dd, ti / dd);
    }
  }
  __syncthreads();
  return true;
}

}  // namespace

// ---------------------------------------------------------------- k_fcol

// LDS layout of the column kernel (bytes)
struct FColLayout {
  size_t gridA, gridB, tw, red, gi, dsum, gx, sidx, sval, gT, hist, tmp, total;
  // grid: complex elements of each of the two frame grids; ntw: twiddles
  __host__ __device__ FColLayout(int rho, int r, int grid = kFGrid, int ntw = kFN) {
    size_t o = 0;
    gridA = o; o = align16(o + 8 * (size_t)grid);
    gridB = o; o = align16(o + 8 * (size_t)grid);
    tw = o;    o = align16(o + 8 * (size_t)ntw);
    red = o;   o = align16(o + 8 * (size_t)kFWaves * (2 * kFRMax + 2));
    gi = o;    o = align16(o + 16 * (size_t)r * r);
    dsum = o;  o = align16(o + 8 * (size_t)(2 * kFRMax + 2));
    gx = o;    o = align16(o + 16 * (size_t)kFRMax);
    sidx = o;  o = align16(o + 4 * (size_t)rho);
    sval = o;  o = align16(o + 8 * (size_t)rho);
    gT = o;    o = align16(o + 8 * (size_t)rho);
    hist = o;  o = align16(o + 4 * (size_t)(256 + 8));
    tmp = o;   o = align16(o + 4 * (size_t)(kFWaves + 1));
    total = o;
  }
};

// Grid elements of a generic frame: the frame (n), or the rows of P_k staged for
// the Gram (m rows of kFRMax + 1 complex values over both grids), whichever is more.
__host__ __device__ inline int fgen_grid(int n, int m) {
  int need = (m * (kFRMax + 1) + 1) / 2;
  // grid B also holds the Cholesky work arrays: 2 kFRMax^2 double2 = 4 kFRMax^2 complex slots
  if (need < 4 * kFRMax * kFRMax) need = 4 * kFRMax * kFRMax;
  return ((n > need ? n : need) + 3) / 4 * 4;
}

size_t fcol_lds_bytes(int rho, int r, int n, int m, int n1, int n2) {
  if (n1 == kFN && n2 == kFN) return FColLayout(rho, r).total;
  return FColLayout(rho, r, fgen_grid(n, m), n1 + n2).total;
}

template <int R, bool GEN>
__global__ __launch_bounds__(kFThreads) void k_fcol(FColArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int tid = threadIdx.x, k = blockIdx.x;
  const int n = a.n, m = a.m, r = a.r, rho = a.rho;
  const bool gd = a.mode == FCOL_GD;
  const int gsize = GEN ? n : kFGrid;              // grid slots a transform touches
  const int ntw = GEN ? a.n1 + a.n2 : kFN;
  const FColLayout lay = GEN ? FColLayout(rho, r, fgen_grid(n, m), ntw) : FColLayout(rho, r);
  const float gscale = GEN ? (float)(1.0 / sqrt((double)n)) : 0.f;
  // element j -> grid slot (the 96 x 96 grid has a pad column)
  auto pos = [&](int j) { return GEN ? j : fpos(j); };
  auto dft2 = [&](float2* g, const float2* t, bool inv) {
    if constexpr (GEN) {
      if (inv) dft2_gen<true>(g, t, a.n1, a.n2, gscale);
      else dft2_gen<false>(g, t, a.n1, a.n2, gscale);
    } else {
      if (inv) fft2_grid<true>(g, t);
      else fft2_grid<false>(g, t);
    }
  };
  float2* gA = reinterpret_cast<float2*>(smem + lay.gridA);
  float2* gB = reinterpret_cast<float2*>(smem + lay.gridB);
  float2* tw = reinterpret_cast<float2*>(smem + lay.tw);
  double* red = reinterpret_cast<double*>(smem + lay.red);
  double2* Gi = reinterpret_cast<double2*>(smem + lay.gi);
  double* dsum = reinterpret_cast<double*>(smem + lay.dsum);
  double2* gx = reinterpret_cast<double2*>(smem + lay.gx);
  int* sidx = reinterpret_cast<int*>(smem + lay.sidx);
  float2* sval = reinterpret_cast<float2*>(smem + lay.sval);
  float2* gT = reinterpret_cast<float2*>(smem + lay.gT);
  int* hist = reinterpret_cast<int*>(smem + lay.hist);
  int* tmp = reinterpret_cast<int*>(smem + lay.tmp);

  for (int t = tid; t < ntw; t += kFThreads) tw[t] = a.tw[t];
  // the measurement rows i = tid, tid + 1024 of this thread, in registers
  int mi[2];
  bool ok[2];
  float2 yv[2];
  int flags = 0;
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int i = tid + kFThreads * e;
    const int raw = i < m ? a.mask[(long long)k * m + i] : 0;
    const bool inr = raw >= 0 && raw < n;
    if (i < m && !inr) flags |= 4;   // a frequency index out of range: the row is left out
    ok[e] = i < m && inr;
    mi[e] = ok[e] ? raw : 0;
    yv[e] = ok[e] ? a.Y[(long long)k * a.ldy + i] : make_float2(0.f, 0.f);
  }
  // rows i of P_k = rows mask_k[i] of F U, read once into registers (the GD
  // steps use them about a dozen times; each re-read from L2 was a round trip
  // on the critical path).  At R = 6, 8 this costs a few spilled registers.
  float2 Pc[2][R];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const float2* src = a.FU + (long long)mi[e] * r;
#pragma unroll
    for (int c = 0; c < R; ++c) Pc[e][c] = (gd && ok[e] && c < r) ? src[c] : make_float2(0.f, 0.f);
  }
  auto Prow = [&](int e, float2 (&p)[R]) {
#pragma unroll
    for (int c = 0; c < R; ++c) p[c] = Pc[e][c];
  };
  int nz = 0;
  for (int e = tid; e < rho; e += kFThreads) {
    int j = e;   // s = 0 on the support 0 .. rho - 1 when there is no start (kept if tau = 0)
    float2 v = make_float2(0.f, 0.f);
    if (gd) {
      j = a.Sidx[(long long)k * rho + e];
      v = a.Sval[(long long)k * rho + e];
      if (j < 0 || j >= n) {   // invalid state: flag it and keep every access in bounds
        flags |= 4;
        j = 0;
        v = make_float2(0.f, 0.f);
      }
    }
    sidx[e] = j;
    sval[e] = v;
    nz |= v.x != 0.f || v.y != 0.f;
  }
  // a start whose values are all zero (an initialisation with tau0 = 0) is s = 0
  // with no support yet: T then comes from HardThreshold(g), as for no start
  const bool start = fblock_any(nz, tmp);

  // G_k = P_k^H P_k (FP64) and its inverse.  The rows of P_k are staged in the
  // two grids (free at this point); wave w sums the entries w, w + 16, ... of
  // the upper triangle with its lanes over the rows (fixed DPP order).
  if (gd) {
    constexpr int PS = R + 1;   // LDS row stride of P_k (complex values)
    float2* Pl = gA;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int i = tid + kFThreads * e;
      if (i < m) {
        float2 p[R];
        Prow(e, p);
#pragma unroll
        for (int c = 0; c < R; ++c) Pl[i * PS + c] = p[c];
      }
    }
    __syncthreads();
    double2* Gl = reinterpret_cast<double2*>(red);   // r x r
    {
      const int lane = tid & 63, wave = wave_id();
      const int E = r * (r + 1) / 2;
      for (int e = wave; e < E; e += kFWaves) {
        int ra = 0, base = 0;
        while (e >= base + (r - ra)) {
          base += r - ra;
          ++ra;
        }
        const int rb = ra + (e - base);
        double sr = 0.0, si = 0.0;
        for (int i = lane; i < m; i += 64) {   // conj(P[i][ra]) P[i][rb]
          const float2 pa = Pl[i * PS + ra], pb = Pl[i * PS + rb];
          sr = fma((double)pa.x, (double)pb.x, fma((double)pa.y, (double)pb.y, sr));
          si = fma((double)pa.x, (double)pb.y, fma(-(double)pa.y, (double)pb.x, si));
        }
        sr = wave_sum_dpp(sr);
        si = wave_sum_dpp(si);
        if (lane == 0) {
          Gl[ra * r + rb] = make_double2(sr, si);
          Gl[rb * r + ra] = make_double2(sr, -si);
        }
      }
    }
    __syncthreads();
    double2* Ll = reinterpret_cast<double2*>(gB);   // the staged rows are no longer needed
    double2* Yl = Ll + kFRMax * kFRMax;
    if (!fblock_chol_inverse(Gl, Ll, Gi, Yl, r)) flags |= 2;
  }

  // gx = G_k^{-1} x for the complex x in dsum[0 .. 2r), entry ra by thread ra
  // (one 36-term FP64 chain per workgroup rather than per thread); one barrier.
  auto ginv_apply = [&]() {
    if (tid < r) {
      double dr = 0.0, di = 0.0;
      for (int cb = 0; cb < r; ++cb) {
        const double2 g = Gi[tid * r + cb];
        const double xr = dsum[2 * cb], xi = dsum[2 * cb + 1];
        dr += g.x * xr - g.y * xi;
        di += g.x * xi + g.y * xr;
      }
      gx[tid] = make_double2(dr, di);
    }
    __syncthreads();
  };

  // v <- v - P_k G_k^{-1} P_k^H v for the two rows of this thread
  auto project = [&](float2 (&v)[2]) {
    double c[2 * R];
#pragma unroll
    for (int cc = 0; cc < 2 * R; ++cc) c[cc] = 0.0;
#pragma unroll
    for (int e = 0; e < 2; ++e) {   // conj(P[i][cc]) v[i]
      float2 p[R];
      Prow(e, p);
#pragma unroll
      for (int cc = 0; cc < R; ++cc) {
        c[2 * cc] += (double)p[cc].x * v[e].x + (double)p[cc].y * v[e].y;
        c[2 * cc + 1] += (double)p[cc].x * v[e].y - (double)p[cc].y * v[e].x;
      }
    }
    fblock_sum<2 * R>(c, red, dsum);
    ginv_apply();
    float2 d[R];
#pragma unroll
    for (int ra = 0; ra < R; ++ra) d[ra] = ra < r ? make_float2((float)gx[ra].x, (float)gx[ra].y) : make_float2(0.f, 0.f);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      float2 p[R];
      Prow(e, p);
      float2 s = v[e];
#pragma unroll
      for (int ra = 0; ra < R; ++ra) s = c_sub(s, c_mul(p[ra], d[ra]));
      v[e] = ok[e] ? s : make_float2(0.f, 0.f);
    }
  };

  auto sum_sq = [&](float2 (&v)[2]) -> double {
    double s[1] = {0.0};
#pragma unroll
    for (int e = 0; e < 2; ++e) s[0] += (double)v[e].x * v[e].x + (double)v[e].y * v[e].y;
    fblock_sum<1>(s, red, dsum);
    return dsum[0];
  };

  // A_k s (the sparse s in sidx/sval) into grid B, gathered at this thread's rows
  auto apply_sparse = [&](const int* id, const float2* vl, int cnt, float2 (&out)[2]) {
    zero_grid(gB, gsize);
    __syncthreads();
    for (int e = tid; e < cnt; e += kFThreads) gB[pos(id[e])] = vl[e];
    __syncthreads();
    dft2(gB, tw, false);
#pragma unroll
    for (int e = 0; e < 2; ++e) out[e] = ok[e] ? gB[pos(mi[e])] : make_float2(0.f, 0.f);
    __syncthreads();
  };
  // A_k^H v into grid A
  auto apply_adj = [&](float2 (&v)[2]) {
    zero_grid(gA, gsize);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 2; ++e)
      if (ok[e]) gA[pos(mi[e])] = v[e];
    __syncthreads();
    dft2(gA, tw, true);
  };

  // A_k s at this thread's rows.  When a HardThreshold step keeps the support
  // T, the new s is s - mu g_T, so A_k s moves by -mu A_k g_T = -mu w, which is
  // already at hand: the next transform of s is skipped (equal up to rounding
  // order).  mark is a bitmap of T over n, kept in grid B between transforms.
  float2 as[2] = {make_float2(0.f, 0.f), make_float2(0.f, 0.f)};
  bool have = start, known = !start;   // without a start s = 0, so A_k s = 0
  unsigned* mark = reinterpret_cast<unsigned*>(gB);
  const int words = (n + 31) >> 5;
  const int tau = rho > 0 ? a.tau : 0;
  for (int it = 0; it < tau; ++it) {
    // u = M s - z: A s - y (projected in the GD iterations)
    float2 u[2];
    if (!known) apply_sparse(sidx, sval, rho, as);
#pragma unroll
    for (int e = 0; e < 2; ++e) u[e] = ok[e] ? c_sub(as[e], yv[e]) : make_float2(0.f, 0.f);
    if (gd) project(u);
    // g = M^H u = A^H u (u lies in the range of the projector)
    apply_adj(u);
    // T: the current support, or that of HardThreshold(g) when s = 0
    if (!have) {
      flags |= fselect([&](int j) { return gA[pos(j)]; }, n, rho, sidx, hist, tmp) ? 1 : 0;
      for (int e = tid; e < rho; e += kFThreads) sval[e] = make_float2(0.f, 0.f);
      __syncthreads();
    }
    double gg_part = 0.0;
    for (int e = tid; e < rho; e += kFThreads) {
      const float2 g = gA[pos(sidx[e])];
      gT[e] = g;
      gg_part += (double)g.x * g.x + (double)g.y * g.y;
    }
    // w = M g_T: only ||w||^2 is needed.  With the projector, ||Pi w||^2 =
    // ||w||^2 - Re(c^H G^{-1} c) with c = P_k^H w, one reduction together with
    // ||g_T||^2.
    float2 w[2];
    apply_sparse(sidx, gT, rho, w);
    double gg, ww;
    {
      double v[2 * R + 2];
#pragma unroll
      for (int cc = 0; cc < 2 * R + 2; ++cc) v[cc] = 0.0;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        v[2 * R] += (double)w[e].x * w[e].x + (double)w[e].y * w[e].y;
        if (gd) {
          float2 p[R];
          Prow(e, p);
#pragma unroll
          for (int cc = 0; cc < R; ++cc) {
            v[2 * cc] += (double)p[cc].x * w[e].x + (double)p[cc].y * w[e].y;
            v[2 * cc + 1] += (double)p[cc].x * w[e].y - (double)p[cc].y * w[e].x;
          }
        }
      }
      v[2 * R + 1] = gg_part;
      fblock_sum<2 * R + 2>(v, red, dsum);
      gg = dsum[2 * R + 1];
      ww = dsum[2 * R];
      if (gd) {
        ginv_apply();
        double q = 0.0;   // Re(c^H G^{-1} c)
        for (int ra = 0; ra < r; ++ra) q += dsum[2 * ra] * gx[ra].x + dsum[2 * ra + 1] * gx[ra].y;
        ww = fmax(ww - q, 0.0);
      }
    }
    const bool okmu = ww > 0.0 && isfinite(ww) && isfinite(gg);
    const float mu = okmu ? (float)(gg / ww) : 0.f;
    // v = s - mu g in grid A, then HardThreshold
    for (int t = tid; t < gsize; t += kFThreads) gA[t] = c_scale(gA[t], -mu);
    for (int t = tid; t < words; t += kFThreads) mark[t] = 0u;
    __syncthreads();
    for (int e = tid; e < rho; e += kFThreads) {
      const int j = sidx[e];
      gA[pos(j)] = c_add(gA[pos(j)], sval[e]);
      atomicOr(&mark[j >> 5], 1u << (j & 31));
    }
    __syncthreads();
    // most steps keep T: then sidx (ascending) is already the selection
    if (!fsupport_kept([&](int j) { return gA[pos(j)]; }, n, mark, reinterpret_cast<unsigned*>(red)))
      flags |= fselect([&](int j) { return gA[pos(j)]; }, n, rho, sidx, hist, tmp) ? 1 : 0;
    int moved = 0;
    for (int e = tid; e < rho; e += kFThreads) {
      const int j = sidx[e];
      sval[e] = gA[pos(j)];
      moved |= ((mark[j >> 5] >> (j & 31)) & 1u) ^ 1u;
    }
    known = !fblock_any(moved, tmp);
    if (known && mu != 0.f)
#pragma unroll
      for (int e = 0; e < 2; ++e) as[e] = c_sub(as[e], c_scale(w[e], mu));
    have = true;
  }

  // A_k s_k and e_k = y_k - A_k s_k
  float2 ev[2];
  if (rho > 0 && !known) apply_sparse(sidx, sval, rho, as);
#pragma unroll
  for (int e = 0; e < 2; ++e) ev[e] = ok[e] ? c_sub(yv[e], as[e]) : make_float2(0.f, 0.f);

  float2* Hk = a.H + (long long)k * n;
  if (gd) {
    // b_k = G_k^{-1} P_k^H e_k; r_k = P_k b_k - e_k; h_k = A_k^H r_k
    double c[2 * R + 1];
#pragma unroll
    for (int cc = 0; cc < 2 * R + 1; ++cc) c[cc] = 0.0;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      float2 p[R];
      Prow(e, p);
#pragma unroll
      for (int cc = 0; cc < R; ++cc) {
        c[2 * cc] += (double)p[cc].x * ev[e].x + (double)p[cc].y * ev[e].y;
        c[2 * cc + 1] += (double)p[cc].x * ev[e].y - (double)p[cc].y * ev[e].x;
      }
      c[2 * R] += (double)ev[e].x * ev[e].x + (double)ev[e].y * ev[e].y;
    }
    fblock_sum<2 * R + 1>(c, red, dsum);
    ginv_apply();
    float2 b[R];
#pragma unroll
    for (int ra = 0; ra < R; ++ra) b[ra] = ra < r ? make_float2((float)gx[ra].x, (float)gx[ra].y) : make_float2(0.f, 0.f);
    if (tid < r) {
      float2 bo = b[0];
#pragma unroll
      for (int ra = 0; ra < R; ++ra)
        if (ra == tid) bo = b[ra];
      a.Bt[(long long)k * r + tid] = bo;
    }
    // ||r_k||^2 = ||e_k||^2 - Re(c^H b_k), since G_k b_k = c = P_k^H e_k
    double cb_re = 0.0;
    for (int ra = 0; ra < r; ++ra) cb_re += dsum[2 * ra] * gx[ra].x + dsum[2 * ra + 1] * gx[ra].y;
    const double d_rr = dsum[2 * R] - cb_re;
    const double rr = d_rr < 0.0 ? 0.0 : d_rr;   // rounding below zero clamped; a NaN stays NaN
    if (tid == 0) a.colrr[k] = rr;
    __syncthreads();   // dsum is read above by every thread
    float2 rv[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      float2 p[R];
      Prow(e, p);
      float2 s = make_float2(-ev[e].x, -ev[e].y);
#pragma unroll
      for (int ra = 0; ra < R; ++ra) s = c_add(s, c_mul(p[ra], b[ra]));
      rv[e] = ok[e] ? s : make_float2(0.f, 0.f);
    }
    apply_adj(rv);
  } else {
    // initialisation: ||y_k||^2 and the column A_k^H (y_k - A_k s_k) of L_0
    const double yy = sum_sq(yv);
    if (tid == 0) a.colrr[k] = yy;
    apply_adj(ev);
  }
  for (int j = tid; j < n; j += kFThreads) Hk[j] = gA[pos(j)];
  for (int e = tid; e < rho; e += kFThreads) {
    a.Sidx[(long long)k * rho + e] = sidx[e];
    a.Sval[(long long)k * rho + e] = sval[e];
  }
  if (flags) atomicOr(&a.flags[k], flags);
}

// ---------------------------------------------------------------- U side

// F U, the unitary 2D DFT of each of U's r columns (n x r, row-major; frame
// element (j1, j2) at row j1 * 96 + j2), in two launches that each give one
// 96-point line to a group of 32 lanes: PASS 0 transforms the rows (j1, c) of U
// into FU, PASS 1 the columns (u2, c) of FU in place, with the 1/96 scale (the
// same transform and scaling as fft2_grid).  A group reads its whole line before
// it writes (the lane exchanges need every lane's loads), and no two groups share
// an element, so the column pass can run in place.  kFN r is even, so a wave's
// two groups exit together.
template <int PASS>
__global__ __launch_bounds__(64) void k_fu(const float2* U, int r, const float2* tw, float2* FU) {
  const int gid = blockIdx.x * 2 + (threadIdx.x >> 5), l = threadIdx.x & 31;
  if (gid >= kFN * r) return;
  const int line = gid / r, c = gid - line * r;
  const int k1 = (int)(__builtin_bitreverse32((unsigned)l) >> 27);
  const long long stride = PASS == 0 ? (long long)r : (long long)kFN * r;
  const long long base = PASS == 0 ? (long long)line * kFN * r + c : (long long)line * r + c;
  const float2* src = (PASS == 0 ? U : FU) + base;
  float2 v[3] = {src[l * stride], src[(l + 32) * stride], src[(l + 64) * stride]};
  fft96<false>(v, l, tw);
  float2* dst = FU + base;
  const float s = 1.0f / kFN;
#pragma unroll
  for (int a = 0; a < 3; ++a) dst[(3 * k1 + a) * stride] = PASS == 0 ? v[a] : c_scale(v[a], s);
}

// F U for a generic frame: one workgroup per column c of U; the column is staged
// in LDS, transformed by dft2_gen and written back (the same transform and scale
// as the column kernel's).
__global__ __launch_bounds__(kFThreads) void k_fu_gen(const float2* U, int n, int r, int n1, int n2,
                                                      const float2* tw, float2* FU) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  float2* grid = reinterpret_cast<float2*>(smem);
  float2* twl = grid + n;
  const int c = blockIdx.x;
  for (int t = threadIdx.x; t < n1 + n2; t += kFThreads) twl[t] = tw[t];
  for (int j = threadIdx.x; j < n; j += kFThreads) grid[j] = U[(long long)j * r + c];
  __syncthreads();
  dft2_gen<false>(grid, twl, n1, n2, (float)(1.0 / sqrt((double)n)));
  for (int j = threadIdx.x; j < n; j += kFThreads) FU[(long long)j * r + c] = grid[j];
}

__global__ void k_ftwiddle(float2* tw) {
  const int t = threadIdx.x;
  if (t < kFN) {
    double s, c;
    sincospi(-2.0 * t / kFN, &s, &c);
    tw[t] = make_float2((float)c, (float)s);
  }
}

// Twiddles of a generic frame: W_n1^t (t < n1), then W_n2^t (t < n2), W_N = exp(-2 pi i / N).
__global__ void k_ftwiddle_gen(float2* tw, int n1, int n2) {
  for (int t = threadIdx.x + blockIdx.x * blockDim.x; t < n1 + n2; t += blockDim.x * gridDim.x) {
    const int N = t < n1 ? n1 : n2, e = t < n1 ? t : t - n1;
    double s, c;
    sincospi(-2.0 * e / N, &s, &c);
    tw[t] = make_float2((float)c, (float)s);
  }
}

__global__ void k_fbasis(float2* U, int n, int r) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < (long long)n * r;
       i += (long long)gridDim.x * blockDim.x) {
    const int j = (int)(i / r), c = (int)(i % r);
    U[i] = make_float2((j % r == c) ? 1.f : 0.f, 0.f);
  }
}

// ---------------------------------------------------------------- launchers

#define FR_SWITCH(R_, CALL)  \
  switch (R_) {              \
    case 2: CALL(2); break;  \
    case 4: CALL(4); break;  \
    case 6: CALL(6); break;  \
    default: CALL(8); break; \
  }

static int fr_bucket(int r) { return r <= 2 ? 2 : (r <= 4 ? 4 : (r <= 6 ? 6 : 8)); }

template <int RR, bool GEN>
static hipError_t launch_fcol_inst(const FColArgs& a, size_t lds, hipStream_t st) {
  static bool attr_set = false;   // the LDS limit is raised once, before any graph capture
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void*)k_fcol<RR, GEN>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)kFLdsMax);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipLaunchKernelGGL((k_fcol<RR, GEN>), dim3(a.q), dim3(kFThreads), lds, st, a);
  return hipSuccess;
}

hipError_t launch_fcol(const FColArgs& a, hipStream_t st) {
  const bool gen = !(a.n1 == kFN && a.n2 == kFN);
  const size_t lds = fcol_lds_bytes(a.rho, a.r, a.n, a.m, a.n1, a.n2);
  if (lds > kFLdsMax) return hipErrorInvalidValue;
  (void)hipGetLastError();
  hipError_t e;
#define FCOL_CALL(RR) e = gen ? launch_fcol_inst<RR, true>(a, lds, st) : launch_fcol_inst<RR, false>(a, lds, st)
  FR_SWITCH(fr_bucket(a.r), FCOL_CALL)
#undef FCOL_CALL
  if (e != hipSuccess) return e;
  return hipGetLastError();
}

hipError_t launch_fu_gen(const float2* U, int n, int r, int n1, int n2, const float2* tw, float2* FU,
                         hipStream_t st) {
  (void)hipGetLastError();
  const size_t lds = 8 * (size_t)(n + n1 + n2);
  hipLaunchKernelGGL(k_fu_gen, dim3(r), dim3(kFThreads), lds, st, U, n, r, n1, n2, tw, FU);
  return hipGetLastError();
}

hipError_t launch_ftwiddle_gen(float2* tw, int n1, int n2, hipStream_t st) {
  (void)hipGetLastError();
  hipLaunchKernelGGL(k_ftwiddle_gen, dim3((n1 + n2 + 255) / 256), dim3(256), 0, st, tw, n1, n2);
  return hipGetLastError();
}

hipError_t launch_fu(const float2* U, int r, const float2* tw, float2* FU, hipStream_t st) {
  (void)hipGetLastError();
  const int blocks = kFN * r / 2;   // two 32-lane groups per 64-thread workgroup
  hipLaunchKernelGGL(k_fu<0>, dim3(blocks), dim3(64), 0, st, U, r, tw, FU);
  hipLaunchKernelGGL(k_fu<1>, dim3(blocks), dim3(64), 0, st, U, r, tw, FU);
  return hipGetLastError();
}

hipError_t launch_ftwiddle(float2* tw, hipStream_t st) {
  (void)hipGetLastError();
  hipLaunchKernelGGL(k_ftwiddle, dim3(1), dim3(128), 0, st, tw);
  return hipGetLastError();
}

hipError_t launch_fbasis(float2* U, int n, int r, hipStream_t st) {
  (void)hipGetLastError();
  hipLaunchKernelGGL(k_fbasis, dim3(64), dim3(256), 0, st, U, n, r);
  return hipGetLastError();
}

}  // namespace altg
