// Overlaps of Eq. (QUV) (App. D) from frequency-domain inputs: the step that
// prepares Q, U and V for the likelihood.  On a two-sided grid of N samples
// in FFT order (f_i = i df for i < (N+1)/2, (i - N) df otherwise), with the
// weight w_ki = 2 df / S_k(|f_i|) on |f_i| > f_low and 0 elsewhere,
//   Q_k,m(t_n) = sum_i w_ki conj(h_m(f_i)) d_k(f_i) e^{2 pi i f_i t_n}, t_n = n / (N df),
// is an unnormalized inverse DFT of the weighted product (a pruned two-step
// transform of the wanted rows, or for the largest problems one batched complex
// FFT of length N over every detector and mode), and
//   U_k,mm' = sum_i w_ki conj(h_m(f_i)) h_m'(f_i),
//   V_k,mm' = sum_i w_ki h_m(-f_i) h_m'(f_i)
// are weighted Gram sums over the grid, by chunks of it reduced in a fixed order.
#include <hipfft/hipfft.h>

#include "common.h"
#include "internal.h"

#include <algorithm>

namespace rift {

__device__ __forceinline__ double quv_w(int64_t i, int64_t N, double df, double f_low, double S) {
  const double f = (double)(i < (N + 1) / 2 ? i : i - N) * df;
  return fabs(f) > f_low ? 2.0 * df / S : 0.0;
}

// X[k][m][i] = w_ki conj(h_m(f_i)) d_k(f_i)
__global__ void __launch_bounds__(256) quv_weight_kernel(int M, int64_t N, double df, double f_low,
                                                         const double2 *data, const double *psd,
                                                         const double2 *modes, double2 *X) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= N) return;
  const int km = blockIdx.y, k = km / M, m = km % M;
  const double w = quv_w(i, N, df, f_low, psd[(size_t)k * N + i]);
  double2 x = {0.0, 0.0};
  if (w != 0.0) {
    const double2 h = modes[(size_t)m * N + i], d = data[(size_t)k * N + i];
    x.x = w * (h.x * d.x + h.y * d.y);
    x.y = w * (h.x * d.y - h.y * d.x);
  }
  X[(size_t)km * N + i] = x;
}

// Q[k][r][m] = X[k][m][(row0 + r) mod N] (after the transform)
__global__ void __launch_bounds__(256) quv_gather_kernel(int M, int64_t N, int64_t row0, int64_t n_rows,
                                                         const double2 *X, double2 *Q) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n_rows) return;
  const int km = blockIdx.y, k = km / M, m = km % M;
  const int64_t n = ((row0 + r) % N + N) % N;
  Q[((size_t)k * n_rows + r) * M + m] = X[(size_t)km * N + n];
}

// ---- Q by a pruned two-step transform -----------------------------------------
// Only n_rows of the N outputs of each series are wanted (about 1000 of 32768),
// and they need no plan: with N = A B, i = B a + b and c = n mod A,
//   Q[n] = sum_b e^{2 pi i b n / N} S[c][b],   S[c][b] = sum_a x[B a + b] e^{2 pi i a c / A},
// which costs N A + n_rows B products per series; the host takes the divisor A
// that makes this least (near sqrt(n_rows), at most kMaxA).  Bound by FP64
// vector work: 0.13e9 complex products for 63 series, N = 32768, 999 rows (59
// and 97 us), where the FFT library's plan alone takes 14 ms to make and
// destroy; the whole call 16.4 -> 0.97 ms, most of it the copies.
constexpr int kMaxA = 64;
constexpr int kBT = 64;  // b per workgroup of the first step
// Both steps add in runs of eight terms, the second its N / A / 8 runs with
// Kahan's compensation: the error of one long sum grows with its length, the
// FFT's with log N.  Largest error over the largest |Q| of a steep spectrum at N
// = 4096, 32749 (prime: one step of N terms) and 2^18: by the FFT library
// 3.5e-16, 1.7e-15 and 1.5e-15; as long sums 2.4e-15, 1.1e-14 and 5.3e-14; in
// runs 2.4e-16, 4.9e-16 and 9.8e-16 (the call 2 % slower at the size above).
constexpr int kSub = 8;

// S[series][c][b]; x = w conj(h) d is formed here.  A workgroup takes 64 b of
// one series; each of its four wavefronts a quarter of the c, eight at a time.
__global__ void __launch_bounds__(256) quv_step1_kernel(int M, int64_t N, int A, double df, double f_low,
                                                        const double2 *data, const double *psd,
                                                        const double2 *modes, double2 *S) {
  __shared__ double2 x[kMaxA][kBT];
  __shared__ double2 tw[kMaxA];
  const int64_t B = N / A;
  const int km = blockIdx.y, k = km / M, m = km % M;
  const int64_t b0 = (int64_t)blockIdx.x * kBT;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t b = b0 + lane;
  if ((int)threadIdx.x < A) sincospi(2.0 * threadIdx.x / A, &tw[threadIdx.x].y, &tw[threadIdx.x].x);
  for (int a = wave; a < A; a += 4) {
    double2 v = {0.0, 0.0};
    if (b < B) {
      const int64_t i = B * a + b;
      const double w = quv_w(i, N, df, f_low, psd[(size_t)k * N + i]);
      if (w != 0.0) {
        const double2 h = modes[(size_t)m * N + i], d = data[(size_t)k * N + i];
        v.x = w * (h.x * d.x + h.y * d.y);
        v.y = w * (h.x * d.y - h.y * d.x);
      }
    }
    x[a][lane] = v;
  }
  __syncthreads();
  for (int c0 = 8 * wave; c0 < A; c0 += 32) {
    double2 acc[8];
    int ph[8];
#pragma unroll
    for (int q = 0; q < 8; q++) {
      acc[q] = double2{0.0, 0.0};
      ph[q] = 0;
    }
    for (int a0 = 0; a0 < A; a0 += kSub) {
      double2 sub[8];
#pragma unroll
      for (int q = 0; q < 8; q++) sub[q] = double2{0.0, 0.0};
      for (int a = a0; a < min(A, a0 + kSub); a++) {
        const double2 v = x[a][lane];
#pragma unroll
        for (int q = 0; q < 8; q++) {
          const double2 t = tw[ph[q]];
          sub[q].x = fma(v.x, t.x, fma(-v.y, t.y, sub[q].x));
          sub[q].y = fma(v.x, t.y, fma(v.y, t.x, sub[q].y));
          ph[q] += c0 + q;  // a (c0 + q) mod A, below 2 kMaxA before
          while (ph[q] >= A) ph[q] -= A;
        }
      }
#pragma unroll
      for (int q = 0; q < 8; q++) {
        acc[q].x += sub[q].x;
        acc[q].y += sub[q].y;
      }
    }
    if (b < B) {
#pragma unroll
      for (int q = 0; q < 8; q++)
        if (c0 + q < A) S[((size_t)km * A + c0 + q) * B + b] = acc[q];
    }
  }
}

// Q[k][r][m] over the rows of one residue c: a workgroup takes 8 of them (r =
// r0 + A t) and every mode of detector k, 32 b at a time through LDS.
__global__ void __launch_bounds__(256) quv_step2_kernel(int M, int64_t N, int A, int64_t row0, int64_t n_rows,
                                                        const double2 *S, double2 *Q) {
  __shared__ double2 sx[32][33], w[8][32];
  const int64_t B = N / A;
  const int c = blockIdx.y, k = blockIdx.z;
  // smallest r >= 0 with (row0 + r) mod A = c
  const int64_t r0 = ((c - row0) % A + A) % A;
  const int row = threadIdx.x >> 5, m = threadIdx.x & 31;
  const int64_t r = r0 + (int64_t)A * (8 * (int64_t)blockIdx.x + row);
  if (r0 + (int64_t)A * 8 * blockIdx.x >= n_rows) return;  // the whole workgroup
  const int64_t n = ((row0 + r) % N + N) % N;
  double qr = 0.0, qi = 0.0, er = 0.0, ei = 0.0;  // the sums and what their roundings have added
  auto add = [](double &sum, double &err, double v) {
    const double y = v - err, t = sum + y;
    err = (t - sum) - y;
    sum = t;
  };
  for (int64_t b0 = 0; b0 < B; b0 += 32) {
    __syncthreads();
    for (int e = threadIdx.x; e < 32 * M; e += 256) {
      const int mm = e >> 5, j = e & 31;
      sx[j][mm] = b0 + j < B ? S[((size_t)(k * M + mm) * A + c) * B + b0 + j] : double2{0.0, 0.0};
    }
    {
      const int64_t ph = ((b0 + m) * n) % N;  // (m: this thread's b in the tile)
      sincospi(2.0 * (double)ph / (double)N, &w[row][m].y, &w[row][m].x);
    }
    __syncthreads();
    if (m < M)
      for (int j0 = 0; j0 < 32; j0 += kSub) {
        double sr = 0.0, si = 0.0;
#pragma unroll
        for (int j = 0; j < kSub; j++) {
          const double2 v = sx[j0 + j][m], t = w[row][j0 + j];
          sr = fma(v.x, t.x, fma(-v.y, t.y, sr));
          si = fma(v.x, t.y, fma(v.y, t.x, si));
        }
        add(qr, er, sr);
        add(qi, ei, si);
      }
  }
  if (m < M && r < n_rows) Q[((size_t)k * n_rows + r) * M + m] = double2{qr, qi};
}

// ---- U and V ----------------------------------------------------------------------
// Partial Gram sums of detector k over a chunk of the grid: the weighted mode
// values of 16 grid points at a time go through LDS, and every thread keeps
// up to four (m, m') entries of both.  Each input is read once per chunk and
// detector (one workgroup per entry read the modes M times from L2: 151 us at
// K = 3, M = 21, N = 32768, now 87); bound by LDS reads, 48 bytes per entry and
// point.
constexpr int kGT = 16;       // grid points per tile
constexpr int kGChunk = 512;  // grid points per workgroup
__global__ void __launch_bounds__(256) quv_gram_kernel(int M, int64_t N, double df, double f_low, const double *psd,
                                                       const double2 *modes, double2 *part) {
  __shared__ double2 h[kMaxModes][kGT + 1], wh[kMaxModes][kGT + 1], hn[kMaxModes][kGT + 1];
  const int k = blockIdx.y;
  const int64_t i0 = (int64_t)blockIdx.x * kGChunk, i1 = min(N, i0 + kGChunk);
  double2 u[4], v[4];
#pragma unroll
  for (int q = 0; q < 4; q++) u[q] = v[q] = double2{0.0, 0.0};
  for (int64_t i = i0; i < i1; i += kGT) {
    __syncthreads();
    for (int e = threadIdx.x; e < M * kGT; e += 256) {
      const int m = e / kGT, j = e % kGT;
      double2 a = {0.0, 0.0}, an = {0.0, 0.0};
      double w = 0.0;
      if (i + j < i1) w = quv_w(i + j, N, df, f_low, psd[(size_t)k * N + i + j]);
      if (w != 0.0) {
        a = modes[(size_t)m * N + i + j];
        an = modes[(size_t)m * N + (N - i - j) % N];
      }
      h[m][j] = a;
      wh[m][j] = double2{w * a.x, w * a.y};
      hn[m][j] = an;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int e = threadIdx.x + 256 * q;
      if (e < M * M) {
        const int m = e / M, mp = e % M;
        // (the tile's sum, then the chunk's: one long sum rounds more)
        double2 su = {0.0, 0.0}, sv = {0.0, 0.0};
#pragma unroll 4
        for (int j = 0; j < kGT; j++) {
          const double2 a = h[m][j], an = hn[m][j], b = wh[mp][j];
          su.x = fma(a.x, b.x, fma(a.y, b.y, su.x));
          su.y = fma(a.x, b.y, fma(-a.y, b.x, su.y));
          sv.x = fma(an.x, b.x, fma(-an.y, b.y, sv.x));
          sv.y = fma(an.x, b.y, fma(an.y, b.x, sv.y));
        }
        u[q].x += su.x;
        u[q].y += su.y;
        v[q].x += sv.x;
        v[q].y += sv.y;
      }
    }
  }
  double2 *out = part + ((size_t)blockIdx.x * gridDim.y + k) * 2 * M * M;
#pragma unroll
  for (int q = 0; q < 4; q++) {
    const int e = threadIdx.x + 256 * q;
    if (e < M * M) {
      out[e] = u[q];
      out[M * M + e] = v[q];
    }
  }
}

// U and V from the chunks' sums, in chunk order (a wavefront per entry: lane
// by lane a strided part, then a fixed tree)
__global__ void __launch_bounds__(64) quv_gram_sum_kernel(int KMM, int MM, int n_chunks, const double2 *part,
                                                          double2 *U, double2 *V) {
  const int e = blockIdx.x, k = e / MM, mm = e % MM, lane = threadIdx.x;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  for (int c = lane; c < n_chunks; c += 64) {
    const double2 *p = part + ((size_t)c * (KMM / MM) + k) * 2 * MM;
    s[0] += p[mm].x;
    s[1] += p[mm].y;
    s[2] += p[MM + mm].x;
    s[3] += p[MM + mm].y;
  }
  for (int o = 32; o > 0; o >>= 1)
    for (int q = 0; q < 4; q++)
      s[q] += __hiloint2double(__shfl_xor(__double2hiint(s[q]), o), __shfl_xor(__double2loint(s[q]), o));
  if (lane == 0) {
    U[e] = double2{s[0], s[1]};
    V[e] = double2{s[2], s[3]};
  }
}

// bad[0]: some data or mode value is not finite; bad[1]: the first in-band PSD
// value (index k N + i, ordered by i then k) that is not finite and positive
__global__ void __launch_bounds__(256) quv_check_kernel(int K, int64_t N, int64_t n_data, int64_t n_modes, double df,
                                                        double f_low, const double *data, const double *psd,
                                                        const double *modes, unsigned long long *bad) {
  const int64_t stride = (int64_t)gridDim.x * 256, t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  bool nf = false;
  for (int64_t i = t; i < n_data; i += stride) nf |= !isfinite(data[i]);
  for (int64_t i = t; i < n_modes; i += stride) nf |= !isfinite(modes[i]);
  if (nf) atomicOr(&bad[0], 1ull);
  for (int64_t i = t; i < N; i += stride) {
    const double f = (double)(i < (N + 1) / 2 ? i : i - N) * df;
    if (fabs(f) <= f_low) continue;
    for (int k = 0; k < K; k++) {
      const double S = psd[(size_t)k * N + i];
      if (!(S > 0.0) || !isfinite(S)) {
        atomicMin(&bad[1], (unsigned long long)(i * K + k));
        break;
      }
    }
  }
}

hipError_t quv_check(int K, int M, int64_t N, double df, double f_low, const double *data, const double *psd,
                     const double *modes, unsigned long long *bad, hipStream_t st) {
  hipError_t e = fill_u32((uint32_t *)bad, 2, 0u, st);
  if (e == hipSuccess) e = fill_u32((uint32_t *)(bad + 1), 2, 0xffffffffu, st);
  if (e != hipSuccess) return e;
  const int64_t nd = 2 * (int64_t)K * N, nm = 2 * (int64_t)M * N;
  const unsigned grid = (unsigned)std::min<int64_t>(1024, (nm + 255) / 256);
  hipLaunchKernelGGL(quv_check_kernel, dim3(grid), dim3(256), 0, st, K, N, nd, nm, df, f_low, data, psd, modes, bad);
  return hipGetLastError();
}

// The divisor A <= kMaxA of N that makes N A + n_rows N / A least; 0 where the
// products of all series would then take longer than the FFT library's plan
// and transform (1e11 products are about 20 ms; the plan 14).
static int quv_split(int K, int M, int64_t N, int64_t n_rows) {
  int best = 0;
  double cost = 0.0;
  for (int A = 1; A <= kMaxA; A++) {
    if (N % A) continue;
    const double c = (double)N * A + (double)n_rows * (double)(N / A);
    if (best == 0 || c < cost) {
      best = A;
      cost = c;
    }
  }
  // (the second step's phases b n are products below N^2, in 64 bits)
  return cost * K * M <= 5.0e10 && (double)N * (double)N < 9.0e18 ? best : 0;
}

int64_t quv_part_chunks(int64_t N) { return (N + kGChunk - 1) / kGChunk; }

hipError_t quv_device(int K, int M, int64_t N, double df, double f_low, const double *data, const double *psd,
                      const double *modes, int64_t row0, int64_t n_rows, double *X, double *part, double *Q, double *U,
                      double *V, hipStream_t st) {
  const int A = quv_split(K, M, N, n_rows);
  if (n_rows > 0 && A > 0) {
    const int64_t B = N / A;
    hipLaunchKernelGGL(quv_step1_kernel, dim3((unsigned)((B + kBT - 1) / kBT), (unsigned)(K * M)), dim3(256), 0, st, M,
                       N, A, df, f_low, (const double2 *)data, psd, (const double2 *)modes, (double2 *)X);
    const int64_t per = (n_rows + A - 1) / A;  // rows of a residue, at most
    hipLaunchKernelGGL(quv_step2_kernel, dim3((unsigned)((per + 7) / 8), (unsigned)A, (unsigned)K), dim3(256), 0, st,
                       M, N, A, row0, n_rows, (const double2 *)X, (double2 *)Q);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  } else if (n_rows > 0) {
    const dim3 gw((unsigned)((N + 255) / 256), (unsigned)(K * M));
    hipLaunchKernelGGL(quv_weight_kernel, gw, dim3(256), 0, st, M, N, df, f_low, (const double2 *)data, psd,
                       (const double2 *)modes, (double2 *)X);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipfftHandle plan;
    int n = (int)N;
    if (hipfftPlanMany(&plan, 1, &n, nullptr, 1, n, nullptr, 1, n, HIPFFT_Z2Z, K * M) != HIPFFT_SUCCESS)
      return hipErrorUnknown;
    hipfftResult r = hipfftSetStream(plan, st);
    if (r == HIPFFT_SUCCESS)
      r = hipfftExecZ2Z(plan, (hipfftDoubleComplex *)X, (hipfftDoubleComplex *)X, HIPFFT_BACKWARD);
    (void)hipfftDestroy(plan);
    if (r != HIPFFT_SUCCESS) return hipErrorUnknown;
    const dim3 gg((unsigned)((n_rows + 255) / 256), (unsigned)(K * M));
    hipLaunchKernelGGL(quv_gather_kernel, gg, dim3(256), 0, st, M, N, row0, n_rows, (const double2 *)X,
                       (double2 *)Q);
  }
  const int64_t nc = quv_part_chunks(N);
  hipLaunchKernelGGL(quv_gram_kernel, dim3((unsigned)nc, (unsigned)K), dim3(256), 0, st, M, N, df, f_low, psd,
                     (const double2 *)modes, (double2 *)part);
  hipLaunchKernelGGL(quv_gram_sum_kernel, dim3((unsigned)(K * M * M)), dim3(64), 0, st, K * M * M, M * M, (int)nc,
                     (const double2 *)part, (double2 *)U, (double2 *)V);
  return hipGetLastError();
}

}  // namespace rift
