// FP64 refinement of the FP32 matrix-core adjoint on the window samples that
// hold a sample's softmax mass.
//
// d ln L_t / d theta = sum_j p_j d ell_j / d theta is an average under the
// window softmax p_j (App. D Eq. (def:lnL:Decomposed) differentiated).  For a
// sample whose likelihood is loud, the data term and the quadratic term B
// are both large and nearly cancel in each gradient component, and the FP32
// rounding of the contraction, carried into p_j, G_k and H_k, is then a
// visible fraction of the component.  The mass of such a sample lies in a
// few window samples: the main peak, or, for a loud template at a wrong sky
// position, the top few spikes of the noise.  The FP32 sweep keeps, per
// sample, the three 16-sample window blocks with the largest maxima and the
// largest maximum of all other blocks; when that one is more than
// kRefineNats below the sample's maximum, the blocks within kRefineNats of
// the maximum hold all but n_t e^-kRefineNats of the mass, and this kernel
// redoes the sample over them in FP64 (coefficients, B, the contraction of
// the rows the blocks need, ell_j, p_j, H_k, c_k, G_k and the chain rule),
// writing its gradient and ln L_t.  Other samples keep the FP32 result:
// their ell_j come within kRefineNats of the maximum in more than three
// blocks, so the terms of their sums are comparatively small and so is the
// rounding.
//
// A workgroup takes up to 16 samples of one delay bin, a wavefront per detector
// (all detectors in one wavefront need some 300 registers).  The sweep lists
// the samples to refine of each of its work units (up to 64 slots of a bin), so
// that these tiles are full however few of a sorted tile's samples need it,
// and none is started in vain.  The samples of a tile share their
// delay bin, so the blocks that one of them needs start at the same rows for
// all, and they mostly need the same ones: the workgroup walks the union of
// their blocks (a sample takes part in its own only, so that its result does
// not depend on its neighbours), the contraction and G_k = Q_k^T c_k on the FP64 matrix cores as in the FP64
// path (k_eval64.hip), with Q from the FP32 matrix-core layout (FP32 values,
// exact in FP64); ell_j is summed over the detectors through LDS.  U and V
// enter as one real matrix per detector,
//     W = [Ur + Vr, -Ui - Vi; Ui - Vi, Ur - Vr]   (rows, columns re / im),
// for which B = 1/4 a^T W a and d ln L / d a = G - 1/2 W a: one more matrix
// product per tile.  The chain rule is then three complex sums over the modes
// per detector, sum conj(Y) v, sum conj(dY / d iota) v and sum conj(i m Y) v
// with v = G - 1/2 W a, each lane over the elements it holds.
//
// A wavefront per sample (lanes over rows, modes and window samples, vector
// FP64, the sums over the wavefront) took 574 us for 1e5 samples at K = 3,
// M = 21, n_t = 820, half of them near the source, and 231 us for prior draws,
// by 1540 vector instructions and 87 loads a sample.
// The sorted tiles themselves took 261 and 294 us: of prior draws four samples a
// tile, and a workgroup for every tile (some 10 ns each).  This form takes 202
// and 176 us.
#include "common.h"
#include "internal.h"
#include "mfma_tile.h"

#include <algorithm>

namespace rift {

typedef float f2 __attribute__((ext_vector_type(2)));
typedef double d2 __attribute__((ext_vector_type(2)));
typedef double d4 __attribute__((ext_vector_type(4)));

constexpr double kTiny = -60.0;  // nats below the reference where a term is zero

__device__ __forceinline__ double shfl_xor_d(double v, int o) {
  return __hiloint2double(__shfl_xor(__double2hiint(v), o), __shfl_xor(__double2loint(v), o));
}

template <int T>
__global__ void __launch_bounds__(64 * kMaxDet) __attribute__((amdgpu_waves_per_eu(3))) refine_kernel(MfmaArgs a, int item_lo, int cls) {
  constexpr int U = T / 2, OD = T & 1;   // pairs of instructions; an odd one
  constexpr int E = 4 * T;               // elements per row
  constexpr int MT = (E + 15) / 16;      // 16-element tiles of G
  constexpr int ZB = 32 * kTS;
  // per wavefront in turn: the rows of the last two blocks [row][sample], its
  // detector's terms of the window samples, p of the last two blocks, its sums
  __shared__ double buf_all[kMaxDet * ZB];
  __shared__ double yt[2 * T][4][kTS];   // Y_m, dY_m / d iota (zero past M)
  __shared__ double em_sh[2 * T];        // m
  __shared__ double tg[5][2][kTS];       // sin, cos of alpha - gmst, delta, psi, iota / 2, phi
  const int lane = threadIdx.x & 63, s = lane & 15, g = lane >> 4;
  const int k = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), K = blockDim.x >> 6;
  double *const buf = buf_all + k * ZB;
  // (one tile per workgroup: in a loop over tiles the compiler keeps the
  // constants of the FP64 functions in some 100 registers)
  if (blockIdx.x >= *cp(a.ctl + kCtlUnits2 + cls)) return;
  const RIFT_CONST RefineTile &rt = *cp(a.rtile + *cp(a.item_tiles + item_lo) + blockIdx.x);
  const bool on = s < rt.n;
  const uint32_t slot = (uint32_t)gp(a.rslot)[rt.first + (on ? s : 0)];
  const SampleRec rec = a.rec[slot];
  RIFT_GLOBAL int *const jr = gpw(a.jrng) + 2 * (size_t)slot;
  const int b01 = jr[0], b2n = jr[1], nb = b2n >> 16;
  uint32_t key = rt.key;
  const int pt = rt.point;
  const RIFT_CONST PointDev &p = *cp(a.pts + pt);
  const int NT = p.n_t, P = p.pad, M = p.M;
  const int JB = (NT + 15) >> 4, rem = NT - 16 * (JB - 1);
  for (int i = 0; i < k; i++) key /= (uint32_t)p.nq;
  const int lo = __builtin_amdgcn_readfirstlane((int)(key % (uint32_t)p.nq) * p.bin_w - P);
  const RIFT_GLOBAL float *const qk = gp(p.Qm) + (size_t)(k * p.Lpad + P + lo) * E;
  double th[7];
#pragma unroll
  for (int d = 0; d < 7; d++) th[d] = (double)rec.th[d];
  // an angle per lane group: the first four by the first wavefront, phi by the last
  for (int i = k == 0 ? 0 : 4; i < (k == K - 1 ? 5 : 4); i += 4) {
    const int d = i + g;
    const double arg = d == 0   ? th[RIFT_ALPHA] - p.gmst
                       : d == 1 ? th[RIFT_DELTA]
                       : d == 2 ? th[RIFT_PSI]
                       : d == 3 ? 0.5 * th[RIFT_IOTA]
                                : th[RIFT_PHI];
    double sv, cv;
    sincos(arg, &sv, &cv);
    if (d < 5) {
      tg[d][0][s] = sv;
      tg[d][1][s] = cv;
    }
  }
  __syncthreads();
  auto trig = [&] {
    SkyTrig tr;
    tr.sh = tg[0][0][s];
    tr.ch = tg[0][1][s];
    tr.sd = tg[1][0][s];
    tr.cd = tg[1][1][s];
    tr.sp = tg[2][0][s];
    tr.cp = tg[2][1][s];
    return tr;
  };

  // ---- harmonics: 4 K lanes per sample, one mode each --------------------------
  {
    const double si = tg[3][0][s], ci = tg[3][1][s], s1 = tg[4][0][s], c1 = tg[4][1][s];
    const double u = ci * ci, hs = si * ci, hc = 0.5 * (ci * ci - si * si);
#pragma unroll 1
    for (int m = 4 * k + g; m < 2 * T; m += 4 * K) {
      // Y = s^par P(u) e^{i m phi}, s = sin(iota) / 2, u = cos^2(iota / 2)
      // (the whole row of coefficients, zero past the degree, in one go)
      const int mc = min(m, M - 1), par = p.hpar[mc], em = p.em[mc];
      double h[kMaxHDeg + 1], P1 = 0.0, dP = 0.0, cr, cim;
#pragma unroll
      for (int j = 0; j <= kMaxHDeg; j++) h[j] = p.hpoly[mc][j];
#pragma unroll
      for (int j = kMaxHDeg; j >= 0; j--) {
        dP = fma(dP, u, P1);
        P1 = fma(P1, u, h[j]);
      }
      double y = par ? hs * P1 : P1, dy = par ? hc * P1 - hs * hs * dP : -hs * dP;
      if (m >= M) y = dy = 0.0;
      phase_m(em, c1, s1, cr, cim);
      yt[m][0][s] = y * cr;
      yt[m][1][s] = y * cim;
      yt[m][2][s] = dy * cr;
      yt[m][3][s] = dy * cim;
      if (s == 0) em_sh[m] = (double)em;
    }
  }
  double D[9], rc[3];
#pragma unroll
  for (int i = 0; i < 9; i++) D[i] = p.D[k][i];
#pragma unroll
  for (int i = 0; i < 3; i++) rc[i] = p.rc[k][i];
  double xr, xi;
  {
    double Fp, Fc;
    antenna(D, trig(), Fp, Fc);
    const double x = on ? p.d_ref / th[RIFT_DIST] : 0.0;
    xr = x * Fp;
    xi = x * Fc;
  }
  const int n = on ? (int)gp(a.rec)[slot].n[k] : lo;
  double w[4], wd[4];
  {
    const double mu = on ? (th[RIFT_TAU] + delay(rc, trig())) * p.f_s - (double)n : 0.0;
    cr_weights<double>(mu, w);
    cr_dweights<double>(mu, wd);
  }
  const int sh = min(max(n - lo, 0), kBinW - 1);  // a tile's samples are of its bin
  __syncthreads();  // the harmonics

  // sum over the elements of a row operand times a_km = x F_k Y_m:
  // instructions 2 u + i take element 8 u + 2 g + i, the odd last one 8 U + g
  auto contract = [&](auto even, auto odd_last) {
    d4 c = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int u = 0; u < U; u++) {
      const double yr = yt[4 * u + g][0][s], yi = yt[4 * u + g][1][s];
      double qr, qi;
      even(u, qr, qi);
      c = __builtin_amdgcn_mfma_f64_16x16x4f64(qr, fma(xr, yr, -xi * yi), c, 0, 0, 0);
      c = __builtin_amdgcn_mfma_f64_16x16x4f64(qi, fma(xr, yi, xi * yr), c, 0, 0, 0);
    }
    if constexpr (OD) {
      const double yr = yt[4 * U + (g >> 1)][0][s], yi = yt[4 * U + (g >> 1)][1][s];
      c = __builtin_amdgcn_mfma_f64_16x16x4f64(odd_last(), (g & 1) ? fma(xr, yi, xi * yr) : fma(xr, yr, -xi * yi), c,
                                               0, 0, 0);
    }
    return c;
  };
  const int arow = s * E + 2 * g, atail = s * E + 8 * U + g;
  f2 A[U > 0 ? U : 1];
  float At = 0.f;
  auto rows = [&](int b) {  // row block b's operands
    const RIFT_GLOBAL float *q = qk + (size_t)(16 * b) * E;
#pragma unroll
    for (int u = 0; u < U; u++) A[u] = *(const RIFT_GLOBAL f2 *)(q + 8 * u + arow);
    if constexpr (OD) At = q[atail];
  };
  auto product = [&] {
    return contract(
        [&](int u, double &qr, double &qi) {
          qr = (double)A[u][0];
          qi = (double)A[u][1];
        },
        [&] { return (double)At; });
  };
  auto put = [&](const d4 &z, int row) {  // register i of lane group g: row 4 i + g
#pragma unroll
    for (int i = 0; i < 4; i++) buf[16 * (row + 4 * i + g) + s] = z[i];
  };

  // ---- the blocks that any of the samples needs, in ascending order -----------
  d4 acc = {0.0, 0.0, 0.0, 0.0}, gacc[MT];
#pragma unroll
  for (int mt = 0; mt < MT; mt++) gacc[mt] = d4{0.0, 0.0, 0.0, 0.0};
  double m_ref = 0.0, s_run = 0.0, hsum = 0.0, pp[4] = {0.0, 0.0, 0.0, 0.0};
  // G_k += Q_k^T c_k over row block rb, with p of window blocks rb - 1 (pa)
  // and rb (pb).  Instruction q takes rows 4 g + q, element 16 mt + s (past
  // the last element: the next row's, of results that are not used).
  float qv[4][MT];
  auto grows = [&](int rb) {
    const RIFT_GLOBAL float *qr = qk + (size_t)(16 * rb + 4 * g) * E + s;
#pragma unroll
    for (int q = 0; q < 4; q++)
#pragma unroll
      for (int mt = 0; mt < MT; mt++) qv[q][mt] = qr[q * E + 16 * mt];
  };
  auto gproduct = [&](const double (&pa)[4], const double (&pb)[4]) {
#pragma unroll
    for (int i = 0; i < 4; i++) {
      buf[16 * (4 * g + i) + s] = pa[i];
      buf[16 * (16 + 4 * g + i) + s] = pb[i];
    }
    wave_sync();
    const double *pr = buf + 16 * (13 + 4 * g - sh) + s;  // p of row 16 rb + 4 g, tap 3
    double pv[7], c[4];
#pragma unroll
    for (int o = 0; o < 7; o++) pv[o] = pr[16 * o];
#pragma unroll
    for (int q = 0; q < 4; q++) c[q] = w[0] * pv[q + 3] + w[1] * pv[q + 2] + w[2] * pv[q + 1] + w[3] * pv[q];
    // (a narrow peak often has no weight in one of the two row blocks; a NaN counts)
    if (__any(c[0] != 0.0 || c[1] != 0.0 || c[2] != 0.0 || c[3] != 0.0)) {
#pragma unroll
      for (int q = 0; q < 4; q++)
#pragma unroll
        for (int mt = 0; mt < MT; mt++)
          gacc[mt] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)qv[q][mt], c[q], gacc[mt], 0, 0, 0);
    }
    wave_sync();
  };
  const double none[4] = {0.0, 0.0, 0.0, 0.0};
  // (a sample takes part in its own blocks only: what it gets does not depend
  // on the samples that share its tile)
  constexpr int kNone = 0x7fffffff;
  const int c0 = on ? b01 & 0xffff : kNone, c1 = on && nb > 1 ? (int)((uint32_t)b01 >> 16) : kNone,
            c2 = on && nb > 2 ? b2n & 0xffff : kNone;
  int last = -2;
  for (;;) {
    const int own = min(min(c0 > last ? c0 : kNone, c1 > last ? c1 : kNone), c2 > last ? c2 : kNone);
    const int c = __builtin_amdgcn_readfirstlane(wave_min(own));
    if (c >= JB) break;  // no further one
    if (c != last + 1) {
      rows(c);
      if (last >= 0) {
        grows(last + 1);
        gproduct(pp, none);
      }
#pragma unroll
      for (int i = 0; i < 4; i++) pp[i] = 0.0;
      acc = product();
    }
    rows(c + 1);
    put(acc, 0);
    acc = product();
    put(acc, 16);
    grows(c);
    wave_sync();
    double z[7], ell[4], zd[4];
#pragma unroll
    for (int o = 0; o < 7; o++) z[o] = buf[16 * (4 * g + sh + o) + s];
    wave_sync();
#pragma unroll
    for (int i = 0; i < 4; i++) {
      buf[64 * i + lane] = w[0] * z[i] + w[1] * z[i + 1] + w[2] * z[i + 2] + w[3] * z[i + 3];
      zd[i] = wd[0] * z[i] + wd[1] * z[i + 1] + wd[2] * z[i + 2] + wd[3] * z[i + 3];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; i++) ell[i] = -m_ref;
#pragma unroll
    for (int kk = 0; kk < kMaxDet; kk++)
      if (kk < K)
#pragma unroll
        for (int i = 0; i < 4; i++) ell[i] += buf_all[kk * ZB + 64 * i + lane];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; i++)
      if (own != c || (c == JB - 1 && 4 * g + i >= rem)) ell[i] = -INFINITY;
    // the reference of a sample: its first block's maximum, moved when a block
    // exceeds it by 64
    const bool first = c == min(min(c0, c1), c2);
    double cmax = fmax(fmax(ell[0], ell[1]), fmax(ell[2], ell[3]));
    cmax = fmax(cmax, shfl_xor_d(cmax, 16));
    cmax = fmax(cmax, shfl_xor_d(cmax, 32));
    if ((first || cmax > 64.0) && cmax > -INFINITY) {
      const double f = first ? 0.0 : exp(-cmax);
      s_run *= f;
      hsum *= f;
#pragma unroll
      for (int i = 0; i < 4; i++) pp[i] *= f;
#pragma unroll
      for (int mt = 0; mt < MT; mt++) gacc[mt] *= f;
      m_ref += cmax;
#pragma unroll
      for (int i = 0; i < 4; i++) ell[i] -= cmax;
    }
    double pj[4];
#pragma unroll
    for (int i = 0; i < 4; i++) pj[i] = ell[i] <= kTiny ? 0.0 : exp(ell[i]);  // (a NaN reaches the sums)
    s_run += (pj[0] + pj[1]) + (pj[2] + pj[3]);
#pragma unroll
    for (int i = 0; i < 4; i++) hsum = fma(pj[i], zd[i], hsum);
    gproduct(pp, pj);
#pragma unroll
    for (int i = 0; i < 4; i++) pp[i] = pj[i];
    last = c;
  }
  if (last >= 0) {
    grows(last + 1);
    gproduct(pp, none);
  }
  s_run += shfl_xor_d(s_run, 16);
  s_run += shfl_xor_d(s_run, 32);
  const double inv = 1.0 / s_run;

  // ---- v = G - 1/2 W a, the sums of the chain rule -----------------------------
  double s0r = 0.0, s0i = 0.0, s1r = 0.0, s1i = 0.0, s2r = 0.0, s2i = 0.0, sbr = 0.0, sbi = 0.0;
#pragma unroll
  for (int mt = 0; mt < MT; mt++) {
    // W a of elements 16 mt + ...: this lane's row of W is 16 mt + s, its
    // columns the two of the instructions' modes (a is zero past M, and
    // results past 2 M are not used: indices are clamped)
    const bool odd = (s & 1) != 0;
    const size_t urow = ((size_t)k * M + min(8 * mt + (s >> 1), M - 1)) * M;
    wave_sync();  // (the harmonics read again for each tile of rows, not kept)
    __builtin_amdgcn_sched_barrier(0);
    d2 W[U + OD];
    auto mode = [&](int u) { return min(u < U ? 4 * u + g : 4 * U + (g >> 1), M - 1); };
#pragma unroll
    for (int u = 0; u < U + OD; u++) {
      const d2 v = *(const RIFT_GLOBAL d2 *)(gp(p.U) + 2 * (urow + mode(u)));
      W[u] = odd ? d2{v[1], v[0]} : d2{v[0], -v[1]};
    }
    if (p.V) {
#pragma unroll
      for (int u = 0; u < U + OD; u++) {
        const d2 v = *(const RIFT_GLOBAL d2 *)(gp(p.V) + 2 * (urow + mode(u)));
        W[u] -= odd ? d2{v[1], v[0]} : d2{-v[0], v[1]};
      }
    }
    const d4 wa = contract(
        [&](int u, double &wre, double &wim) {
          wre = W[u][0];
          wim = W[u][1];
        },
        [&] { return (g & 1) ? W[U + OD - 1][1] : W[U + OD - 1][0]; });
    wave_sync();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 4; i++) {
      if (16 * mt + 4 * i >= E) continue;
      const int m = 8 * mt + 2 * i + (g >> 1);  // element 16 mt + 4 i + g
      const double v = gacc[mt][i] * inv - 0.5 * wa[i];
      // v (even g) or i v (odd g) times conj(Y): (p, q) = (Yr, -Yi) or (Yi, Yr)
      const double yr = yt[m][0][s], yi = yt[m][1][s], dr = yt[m][2][s], di = yt[m][3][s];
      const double yp = (g & 1) ? yi : yr, yq = (g & 1) ? yr : -yi;
      const double dp = (g & 1) ? di : dr, dq = (g & 1) ? dr : -di;
      const double em = em_sh[m];
      s0r = fma(yp, v, s0r);
      s0i = fma(yq, v, s0i);
      s1r = fma(dp, v, s1r);
      s1i = fma(dq, v, s1i);
      s2r = fma(em * yq, v, s2r);  // conj(i m Y) = -i m conj(Y)
      s2i = fma(-em * yp, v, s2i);
      sbr = fma(yp, wa[i], sbr);
      sbi = fma(yq, wa[i], sbi);
    }
  }
  // this detector's parts: Re(conj(x F) S), F = Fp + i Fc; B in out[7]
  // (the distance and the angles read again, not kept through the blocks)
  wave_sync();
  const double dist = (double)gp(a.rec)[slot].th[RIFT_DIST], x = p.d_ref / dist;
  const SkyTrig tr = trig();
  double out[8], Fp, Fc, dFa[2], dFd[2];
  antenna(D, tr, Fp, Fc, dFa, dFd);
  auto re = [&](double fr, double fi, double sr, double s_i) { return x * (fr * sr + fi * s_i); };
  // arrival times: f_s H_k d(dt_k) / d(alpha, delta) and f_s H_k for tau
  const double H = hsum * inv * p.f_s;
  out[RIFT_ALPHA] = re(dFa[0], dFa[1], s0r, s0i) - H * (rc[0] * (-tr.cd * tr.sh) + rc[1] * (tr.cd * tr.ch));
  out[RIFT_DELTA] =
      re(dFd[0], dFd[1], s0r, s0i) - H * (rc[0] * (-tr.sd * tr.ch) + rc[1] * (-tr.sd * tr.sh) + rc[2] * tr.cd);
  out[RIFT_PSI] = re(2.0 * Fc, -2.0 * Fp, s0r, s0i);  // dF / dpsi = -2 i F
  out[RIFT_IOTA] = re(Fp, Fc, s1r, s1i);
  out[RIFT_PHI] = re(Fp, Fc, s2r, s2i);
  out[RIFT_DIST] = -re(Fp, Fc, s0r, s0i) / dist;
  out[RIFT_TAU] = H;
  out[7] = 0.25 * re(Fp, Fc, sbr, sbi);
#pragma unroll
  for (int d = 0; d < 8; d++) {
    out[d] += shfl_xor_d(out[d], 16);
    out[d] += shfl_xor_d(out[d], 32);
    if (g == 0) buf[16 * d + s] = out[d];
  }
  __syncthreads();
  if (k == 0 && on && g == 0) {
#pragma unroll
    for (int d = 0; d < 8; d++) {
      out[d] = buf_all[16 * d + s];
      if (K > 1) out[d] += buf_all[ZB + 16 * d + s];
      if (K > 2) out[d] += buf_all[2 * ZB + 16 * d + s];
    }
    const double lt = m_ref + log(s_run) - log((double)NT) - out[7];
    if (isfinite(lt)) {
      const int64_t col = rec.col;
      const double gi = a.gin ? (double)gp(a.gin)[col] : 1.0;
#pragma unroll
      for (int d = 0; d < 7; d++) gpw(a.grad)[d * a.stride + col] = (float)(gi * out[d]);
      if (a.lnL) gpw(a.lnL)[col] = (float)lt;
    } else {
      jr[1] = 0;  // left to the chain rule of the FP32 sweep
    }
  }
}

template <int T>
static void launch_refine(const MfmaArgs &a, int K, int lo, int cls, int64_t tiles, hipStream_t st) {
  hipLaunchKernelGGL((refine_kernel<T>), dim3((unsigned)tiles), dim3(64 * K), 0, st, a, lo, cls);
}

hipError_t refine_backward(const MfmaArgs &a, int T, int K, int lo, int cls, int64_t tiles, hipStream_t st) {
  if (a.total <= 0 || tiles <= 0 || !a.jrng) return hipSuccess;
  switch (T) {
#define RIFT_T_CASE(TT) \
  case TT: launch_refine<TT>(a, K, lo, cls, tiles, st); break;
    RIFT_T_CASE(1) RIFT_T_CASE(2) RIFT_T_CASE(3) RIFT_T_CASE(4) RIFT_T_CASE(5) RIFT_T_CASE(6) RIFT_T_CASE(7)
    RIFT_T_CASE(8) RIFT_T_CASE(9) RIFT_T_CASE(10) RIFT_T_CASE(11) RIFT_T_CASE(12) RIFT_T_CASE(13)
    RIFT_T_CASE(14) RIFT_T_CASE(15) RIFT_T_CASE(16)
#undef RIFT_T_CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace rift
