// FP64 evaluation of ln L_t and its gradient on the FP64 matrix cores, for
// FP64 handles, from the same sorted tiles as the FP32 path (k_mfma.hip).
//
// A wavefront takes a tile of 16 samples of one delay bin, whose stencils
// start 0..bin_w-1 rows above the bin's lower edge, so per detector the
// contraction z_k[r](s) = Re sum_m conj(a_km) Q_k[r][m] over 16 rows is T
// instructions v_mfma_f64_16x16x4f64 (T = ceil(M / 2)), with Q read straight
// from the handle's row layout: the workgroup's four tiles mostly share their
// bin, so three of four reads hit in L1, and one instruction of 64 cycles
// needs no more than 512 bytes.  The rows of the block before stay in
// registers; with them in a 32-row buffer in LDS each lane reads the 7 rows
// its 4 window samples need at its sample's own offset.
//
// Forward: a max-shifted log-sum-exp with a lazily moved reference.  Adjoint:
// one sweep, the softmax weights p_j formed against a reference shared by a
// sample's four lanes (streaming softmax, moved only when a block exceeds it
// by 64), H_k from the derivative interpolation, the transposed interpolation
// c_k[r] and G_k = Q_k^T c_k as a second matrix product over the same rows;
// the chain rule follows in k_bwd.hip.  A term below e^-60 of the reference
// is taken as zero (the sums it would enter are at least 1, n_t of them are
// below 1e-19 of that), so a block far from the peak costs no exponentials
// and, in the adjoint, no second product.
//
// The vector form (k_plain.hip) reads Q once per 4 to 16 samples and holds a
// whole window in LDS: 2e5 samples at K = 3, M = 21, n_t = 820 took 10.2 ms
// there; FP64 peak of the matrix instruction as measured is 65.7 TFLOP/s.
#include "common.h"
#include "internal.h"
#include "mfma_tile.h"

#include <algorithm>
#include <type_traits>

namespace rift {

typedef double d2 __attribute__((ext_vector_type(2)));
typedef double d4 __attribute__((ext_vector_type(4)));

constexpr double kTiny = -60.0;  // nats below the reference where a term is zero

__device__ __forceinline__ double shfl_xor_d(double v, int o) {
  return __hiloint2double(__shfl_xor(__double2hiint(v), o), __shfl_xor(__double2loint(v), o));
}

template <int T, int K, bool BWD>
__global__ void __launch_bounds__(256) eval64_kernel(MfmaArgsT<double> a, int item_lo, int item_hi, int cls) {
  constexpr int U = T / 2, OD = T & 1;      // pairs of instructions; an odd one
  constexpr int MT = (4 * T + 15) / 16;     // 16-element tiles of G
  constexpr int ZB = 32 * 16;               // doubles of a window buffer: rows of the last two blocks
  __shared__ double zbuf_all[kWaves * ZB];
  __shared__ double pbuf_all[BWD ? kWaves * ZB : 1];
  __shared__ uint32_t unit_sh;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int s = lane & 15, g = lane >> 4;
  double *const zbuf = zbuf_all + wave * ZB;  // [row][sample]
  double *const pbuf = pbuf_all + (BWD ? wave * ZB : 0);
  const uint32_t t_lo = a.item_tiles[item_lo], t_hi = a.item_tiles[item_hi];

  for (;;) {
    __syncthreads();  // every wavefront has read the last unit
    if (threadIdx.x == 0) unit_sh = atomicAdd(&a.ctl[1 + cls], 1u);
    __syncthreads();
    const uint32_t n = __builtin_amdgcn_readfirstlane(unit_sh);
    if (n >= (t_hi - t_lo + 3u) / 4u) break;  // the same for the whole workgroup
    const uint32_t t = t_lo + 4u * n + wave;
    if (t >= t_hi) continue;
    uint32_t key = __builtin_amdgcn_readfirstlane(a.tile_key[t]);
    if (key == kNoBin) continue;  // the tiles that round a point up to groups of 4
    const int it = __builtin_amdgcn_readfirstlane(a.tile_item[t]);
    const PointDev &p = a.pts[a.items.point[it]];
    const int NT = __builtin_amdgcn_readfirstlane(p.n_t), P = __builtin_amdgcn_readfirstlane(p.pad);
    const int Lpad = __builtin_amdgcn_readfirstlane(p.Lpad), E = 2 * __builtin_amdgcn_readfirstlane(p.M);
    const RIFT_GLOBAL double *const Q = gp(uniform_ptr((const double *)p.Q));
    int lo_k[K];
    const RIFT_GLOBAL double *qk[K];
#pragma unroll
    for (int k = 0; k < K; k++) {
      const int q = (int)(key % (uint32_t)p.nq);
      key /= (uint32_t)p.nq;
      lo_k[k] = __builtin_amdgcn_readfirstlane(q * p.bin_w - P);
      qk[k] = Q + (size_t)(k * Lpad + P + lo_k[k]) * E;
    }
    const RIFT_GLOBAL CoefTileT<double> *ct = gp(a.ctile + t);
    const int flag = ct->flag[s];
    bool valid = flag == 1;
    const int64_t top = a.item_cop[it] + (int64_t)(t - a.item_tiles[it]) * K * (4 * T) * kTS;
    const RIFT_GLOBAL double *yop = gp(a.cop + top + s);
    // element of instruction tt in lane group g: 8 u + 2 g + i (tt = 2 u + i),
    // two neighbours per lane and pair, then 8 U + g; the sample operands take
    // the same ones (zero past 2 M), so rows may be read past their end
    double Bop[K][T];
    {
      double yr[T], yi[T];
#pragma unroll
      for (int tt = 0; tt < T; tt++) {
        const int e = tt < 2 * U ? 8 * (tt >> 1) + 2 * g : (8 * U + g) & ~1;
        yr[tt] = yop[kTS * e];
        yi[tt] = yop[kTS * (e + 1)];
      }
#pragma unroll
      for (int k = 0; k < K; k++) {
        const double xr = ct->xf[k][0][s], xi = ct->xf[k][1][s];
#pragma unroll
        for (int tt = 0; tt < T; tt++) {
          const bool im = tt < 2 * U ? (tt & 1) != 0 : (g & 1) != 0;
          Bop[k][tt] = im ? fma(xr, yi[tt], xi * yr[tt]) : fma(xr, yr[tt], -xi * yi[tt]);
        }
      }
    }
    double w[K][4], wd[BWD ? K : 1][4];
    int zr[K];  // this lane's first row of a window read, in doubles
    int sh[K];
#pragma unroll
    for (int k = 0; k < K; k++) {
      const double mu = ct->mu[k][s];
      cr_weights<double>(mu, w[k]);
      if constexpr (BWD) cr_dweights<double>(mu, wd[k]);
      sh[k] = valid ? ct->n[k][s] - lo_k[k] : 0;
      if (sh[k] < 0 || sh[k] > kBinW - 1) {
        valid = false;
        sh[k] = 0;
      }
    }
#pragma unroll
    for (int k = 0; k < K; k++) zr[k] = 16 * (4 * g + sh[k]) + s;
    const int JB = (NT + 15) >> 4, rem = NT - 16 * (JB - 1);

    d4 acc[K];  // the last block's rows (4 i + g in register i)
    auto put = [&](const d4 &z, int row) {
#pragma unroll
      for (int i = 0; i < 4; i++) zbuf[16 * (row + 4 * i + g) + s] = z[i];
    };
    const int arow = s * E + 2 * g, atail = s * E + 8 * U + g;
    auto product = [&](int k, int b) {
      const RIFT_GLOBAL double *q = qk[k] + (size_t)(16 * b) * E;
      d2 A[U > 0 ? U : 1];
      double At = 0.0;
#pragma unroll
      for (int u = 0; u < U; u++) A[u] = *(const RIFT_GLOBAL d2 *)(q + 8 * u + arow);
      if constexpr (OD) At = q[atail];
      d4 c = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int u = 0; u < U; u++) {
        c = __builtin_amdgcn_mfma_f64_16x16x4f64(A[u][0], Bop[k][2 * u], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f64_16x16x4f64(A[u][1], Bop[k][2 * u + 1], c, 0, 0, 0);
      }
      if constexpr (OD) c = __builtin_amdgcn_mfma_f64_16x16x4f64(At, Bop[k][T - 1], c, 0, 0, 0);
      return c;
    };

    // the reference (m_ref: per lane in the forward, per sample in the
    // adjoint) and the sums kept against it
    double m_ref = 0.0, s_run = 0.0;
    double hsum[K], pp[4] = {0.0, 0.0, 0.0, 0.0};  // adjoint: H_k, the last window block's p
    d4 gacc[BWD ? K : 1][MT];
    bool any_prev = false;
    if constexpr (BWD) {
#pragma unroll
      for (int k = 0; k < K; k++) {
        hsum[k] = 0.0;
#pragma unroll
        for (int mt = 0; mt < MT; mt++) gacc[k][mt] = d4{0.0, 0.0, 0.0, 0.0};
      }
    }
    // G_k += Q_k^T c_k over row block rb; pbuf holds p of window blocks rb - 1
    // and rb.  Instruction q takes rows 4 g + q, element 16 mt + s.
    auto gproduct = [&](int rb) {
#pragma unroll
      for (int k = 0; k < K; k++) {
        const double *pr = pbuf + 16 * (13 + 4 * g - sh[k]) + s;  // p of row 16 rb + 4 g, tap 3
        double pv[7], c[4];
#pragma unroll
        for (int o = 0; o < 7; o++) pv[o] = pr[16 * o];
#pragma unroll
        for (int q = 0; q < 4; q++)
          c[q] = w[k][0] * pv[q + 3] + w[k][1] * pv[q + 2] + w[k][2] * pv[q + 1] + w[k][3] * pv[q];
        const RIFT_GLOBAL double *qr = qk[k] + (size_t)(16 * rb + 4 * g) * E + s;
#pragma unroll
        for (int q = 0; q < 4; q++)
#pragma unroll
          for (int mt = 0; mt < MT; mt++)
            gacc[BWD ? k : 0][mt] =
                __builtin_amdgcn_mfma_f64_16x16x4f64(qr[(size_t)q * E + 16 * mt], c[q], gacc[BWD ? k : 0][mt], 0, 0, 0);
      }
    };
#pragma unroll
    for (int k = 0; k < K; k++) acc[k] = product(k, 0);
    for (int b = 1; b <= JB; b++) {
      // block b's rows, then window samples 16 (b - 1) + 4 g + i
      double ell[4], zd[BWD ? K : 1][4];
#pragma unroll
      for (int i = 0; i < 4; i++) ell[i] = -m_ref;
#pragma unroll
      for (int k = 0; k < K; k++) {
        put(acc[k], 0);
        acc[k] = product(k, b);
        put(acc[k], 16);
        wave_sync();
        double z[7];
#pragma unroll
        for (int o = 0; o < 7; o++) z[o] = zbuf[zr[k] + 16 * o];
        wave_sync();
#pragma unroll
        for (int i = 0; i < 4; i++) {
          ell[i] = fma(w[k][0], z[i], ell[i]);
          ell[i] = fma(w[k][1], z[i + 1], ell[i]);
          ell[i] = fma(w[k][2], z[i + 2], ell[i]);
          ell[i] = fma(w[k][3], z[i + 3], ell[i]);
          if constexpr (BWD)
            zd[k][i] = wd[k][0] * z[i] + wd[k][1] * z[i + 1] + wd[k][2] * z[i + 2] + wd[k][3] * z[i + 3];
        }
      }
      if (b == JB) {
#pragma unroll
        for (int i = 0; i < 4; i++) ell[i] = 4 * g + i < rem ? ell[i] : -INFINITY;
      }
      double cmax = fmax(fmax(ell[0], ell[1]), fmax(ell[2], ell[3]));
      if constexpr (BWD) {
        cmax = fmax(cmax, shfl_xor_d(cmax, 16));
        cmax = fmax(cmax, shfl_xor_d(cmax, 32));
      }
      if ((b == 1 || cmax > 64.0) && cmax > -INFINITY) {
        const double f = b == 1 ? 0.0 : exp(-cmax);
        s_run *= f;
        if constexpr (BWD) {
#pragma unroll
          for (int i = 0; i < 4; i++) pp[i] *= f;
#pragma unroll
          for (int k = 0; k < K; k++) {
            hsum[k] *= f;
#pragma unroll
            for (int mt = 0; mt < MT; mt++) gacc[k][mt] *= f;
          }
        }
        m_ref += cmax;
#pragma unroll
        for (int i = 0; i < 4; i++) ell[i] -= cmax;
      }
      // (of the values, not of their maximum, which leaves a NaN out: a NaN
      // window value, of an overflowing sample, must reach the sums)
      const bool any = __any(!(ell[0] <= kTiny && ell[1] <= kTiny && ell[2] <= kTiny && ell[3] <= kTiny));
      double pj[4] = {0.0, 0.0, 0.0, 0.0};
      if (any) {
#pragma unroll
        for (int i = 0; i < 4; i++) pj[i] = ell[i] <= kTiny ? 0.0 : exp(ell[i]);
        s_run += (pj[0] + pj[1]) + (pj[2] + pj[3]);
        if constexpr (BWD) {
#pragma unroll
          for (int k = 0; k < K; k++)
#pragma unroll
            for (int i = 0; i < 4; i++) hsum[k] = fma(pj[i], zd[k][i], hsum[k]);
        }
      }
      if constexpr (BWD) {
        if (any || any_prev) {
#pragma unroll
          for (int i = 0; i < 4; i++) {
            pbuf[16 * (4 * g + i) + s] = pp[i];
            pbuf[16 * (16 + 4 * g + i) + s] = pj[i];
          }
          wave_sync();
          gproduct(b - 1);
          wave_sync();
        }
#pragma unroll
        for (int i = 0; i < 4; i++) pp[i] = pj[i];
        any_prev = any;
      }
    }
    if constexpr (BWD) {
      if (any_prev) {  // the last row block: window block JB does not exist
#pragma unroll
        for (int i = 0; i < 4; i++) {
          pbuf[16 * (4 * g + i) + s] = pp[i];
          pbuf[16 * (16 + 4 * g + i) + s] = 0.0;
        }
        wave_sync();
        gproduct(JB);
        wave_sync();
      }
    }
    // combine a sample's four lanes (in the forward each with its own reference)
    double mr = BWD || s_run > 0.0 ? m_ref : -INFINITY, mo = mr;
    if constexpr (!BWD) {
      mo = fmax(mo, shfl_xor_d(mo, 16));
      mo = fmax(mo, shfl_xor_d(mo, 32));
      s_run *= exp(mr - mo);
    }
    s_run += shfl_xor_d(s_run, 16);
    s_run += shfl_xor_d(s_run, 32);
    double lt = (mo - ct->B[s]) + log(s_run) - log((double)NT);
    if (!valid || !isfinite(lt)) {
      lt = NAN;
      valid = false;
    }
    const int col = ct->col[s];
    if constexpr (BWD) {
      const double inv = 1.0 / s_run;
      if (flag != 0) {
        RIFT_GLOBAL double *ho = gpw(a.hop + (size_t)t * (kMaxDet * kTS));
#pragma unroll
        for (int k = 0; k < K; k++) {
          double h = hsum[k];
          h += shfl_xor_d(h, 16);
          h += shfl_xor_d(h, 32);
          if (g == 0) ho[k * kTS + s] = valid ? h * inv : NAN;
        }
        RIFT_GLOBAL double *go = gpw(a.gop + top);
#pragma unroll
        for (int k = 0; k < K; k++)
#pragma unroll
          for (int mt = 0; mt < MT; mt++)
#pragma unroll
            for (int i = 0; i < 4; i++) {
              const int e = 16 * mt + 4 * i + g;
              if (e < 4 * T) go[((size_t)k * 4 * T + e) * kTS + s] = gacc[k][mt][i] * inv;
            }
      }
    }
    if (flag != 0 && g == 0) {
      if (a.lnL) gpw(a.lnL)[col] = lt;
      if (a.lnw) gpw(a.lnw)[col] = lt + (a.ln_ratio ? gp(a.ln_ratio)[col] : 0.0);
    }
  }
}

template <int T, int K, bool BWD>
static void launch64_tkb(const MfmaArgsT<double> &a, int lo, int hi, int cls, hipStream_t st) {
  static int per_cu = 0;
  if (per_cu == 0) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, eval64_kernel<T, K, BWD>, 256, 0) != hipSuccess || nb < 1)
      nb = 1;
    per_cu = nb;
  }
  const int grid = std::max(1, std::min(a.grid / 4 * per_cu, (a.max_tiles + 3) / 4));
  hipLaunchKernelGGL((eval64_kernel<T, K, BWD>), dim3(grid), dim3(256), 0, st, a, lo, hi, cls);
}

template <int T>
static void launch64(const MfmaArgsT<double> &a, int K, int lo, int hi, int cls, hipStream_t st) {
  const bool bwd = a.grad != nullptr;
  if (K == 1) bwd ? launch64_tkb<T, 1, true>(a, lo, hi, cls, st) : launch64_tkb<T, 1, false>(a, lo, hi, cls, st);
  else if (K == 2) bwd ? launch64_tkb<T, 2, true>(a, lo, hi, cls, st) : launch64_tkb<T, 2, false>(a, lo, hi, cls, st);
  else bwd ? launch64_tkb<T, 3, true>(a, lo, hi, cls, st) : launch64_tkb<T, 3, false>(a, lo, hi, cls, st);
}

hipError_t mfma64_run(const MfmaArgsT<double> &a, const int *class_T, const int *class_K, const int *class_item0,
                      int n_classes, const int *mclass_M, const int *mclass_item0, const int64_t *mclass_tiles,
                      int n_mclasses, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  if (a.total <= 0) return hipSuccess;
  hipError_t e = mfma_prepare<double>(a, mclass_M, mclass_item0, mclass_tiles, n_mclasses, st);
  if (e != hipSuccess) return e;
  if (ev0) (void)hipEventRecord(ev0, st);
  for (int c = 0; c < n_classes; c++) {
    const int lo = class_item0[c], hi = class_item0[c + 1], K = class_K[c];
    switch (class_T[c]) {
#define RIFT_T_CASE(TT) \
  case TT: launch64<TT>(a, K, lo, hi, c, st); break;
      RIFT_T_CASE(1) RIFT_T_CASE(2) RIFT_T_CASE(3) RIFT_T_CASE(4) RIFT_T_CASE(5) RIFT_T_CASE(6) RIFT_T_CASE(7)
      RIFT_T_CASE(8) RIFT_T_CASE(9) RIFT_T_CASE(10) RIFT_T_CASE(11) RIFT_T_CASE(12) RIFT_T_CASE(13)
      RIFT_T_CASE(14) RIFT_T_CASE(15) RIFT_T_CASE(16)
#undef RIFT_T_CASE
      default: return hipErrorInvalidValue;
    }
  }
  e = hipGetLastError();
  if (ev1) (void)hipEventRecord(ev1, st);
  if (e != hipSuccess || !a.grad) return e;
  return chain_launch<double>(a, mclass_M, mclass_item0, mclass_tiles, n_mclasses, st);
}

}  // namespace rift
