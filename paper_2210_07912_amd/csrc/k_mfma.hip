// FP32 evaluation of ln L_t on the matrix cores (gfx950): the passes before
// the evaluation kernel (k_eval.hip) and the adjoint (k_bwd.hip).
//
// The data term of App. D Eq. (def:lnL:Decomposed), summed over the window,
// needs for every sample s and detector k the real contraction
//     z_k[r](s) = Re sum_m conj(a_{k,m}(s)) Q_k[r][m]
// over the rows r its arrival time selects.  Over a common run of rows for a
// tile of samples this is a dense product
//     Z_k = Qr_k (rows x 2M) * A_k (2M x samples)
// with the real and imaginary parts of Q and a as the inner dimension.  The
// rows a sample needs depend on its own delay, so samples are first sorted
// into bins of equal integer delay (per detector, bins of 14 rows); a tile
// holds 16 samples of one bin, whose windows then start within 13 rows of
// each other and share one run of rows.  Bins are padded to whole tiles (for
// the evaluation kernel, whose wavefronts take two, to whole pairs), so tile t
// is sorted slots [16 t, 16 t + 16).
//
// Kernels, in launch order:
//   bin_kernel    integer delays n_k, bin key, per-sort-block bin counts
//   colscan       per point of many sort blocks: their offsets in each bin
//   scan_kernel   per point: the same for few sort blocks, tiles and work
//                 units before each bin; then before each point; per-class
//                 counters reset
//   scatter       a 40-byte record (theta, column, n_k) at the sorted slot; the
//                 point and bin of every tile, the work units (up to
//                 unit_tiles tiles of one bin each) and the padding slots
//   coef_kernel   one thread per slot, FP64: antenna patterns, harmonics
//                 (polynomial tables), Y_m (rounded to FP32) and x F_k, the
//                 quadratic term B, and the interpolation fraction mu_k
#include "common.h"
#include "dmarg.h"
#include "internal.h"
#include "mfma_tile.h"

#include <algorithm>

namespace rift {

// ---- layouts of Q for the matrix cores, once per point ------------------------
// Qm [K][Lpad][E] (FP32, zero past 2 M) and Qs [K][3 ceil(E / 8)][Lpad][8]
// (three BF16 parts of each value) from the row layout Q [K][Lpad][2 M]; one
// thread per row and group of 8 elements.
__global__ void __launch_bounds__(256) layout_kernel(const float *Q, float *Qm, bf8 *Qs, int K, int Lpad, int M2, int E) {
  const int r = blockIdx.x * 256 + threadIdx.x, j = blockIdx.y, k = blockIdx.z;
  if (r >= Lpad) return;
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; e++) {
    v[e] = 8 * j + e < M2 ? Q[((size_t)k * Lpad + r) * M2 + 8 * j + e] : 0.f;
    if (8 * j + e < E) Qm[((size_t)k * Lpad + r) * E + 8 * j + e] = v[e];
  }
  bf8 q[3];
  split3(v, q[0], q[1], q[2]);
  const int C = 3 * gridDim.y;
#pragma unroll
  for (int i = 0; i < 3; i++) Qs[((size_t)k * C + 3 * j + i) * Lpad + r] = q[i];
}

hipError_t mfma_layouts(const float *Q, float *Qm, void *Qs, int K, int Lpad, int M2, int E, hipStream_t st) {
  hipLaunchKernelGGL(layout_kernel, dim3((Lpad + 255) / 256, (E + 7) / 8, K), dim3(256), 0, st, Q, Qm, (bf8 *)Qs, K,
                     Lpad, M2, E);
  return hipGetLastError();
}

// ---- 1. integer delays, bin keys, per-block bin counts ----------------------
// A sort block is TH U consecutive samples of one point (a.sort_block: 4096,
// or 1024 and 256 for calls too small to fill the device with those).  Counts
// go to an LDS histogram (the point's bins), then to the block's row of the
// global block histogram; no global atomics, so no contention on busy bins.
// Bound by the latency of the FP64 sky trigonometry: 4096 samples in one block
// of 1024 threads took 22 us, in 16 of 256 6 us.
__device__ __forceinline__ int block_item(const ItemsDev &it, int b) {
  int lo = 0, hi = it.n_items;  // blk0[lo] <= b < blk0[hi]
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (it.blk0[mid] <= b) lo = mid; else hi = mid;
  }
  return lo;
}

template <typename R, int TH, int U>
__global__ void __launch_bounds__(TH) bin_kernel(MfmaArgsT<R> a) {
  extern __shared__ uint32_t cnt_l[];
  if (blockIdx.x == 0 && threadIdx.x == 0) a.ctl[kCtlScan] = 0u;  // points scanned (scan_kernel)
  const int it = block_item(a.items, blockIdx.x);
  const int lb = blockIdx.x - a.items.blk0[it];
  const RIFT_CONST PointDev &p = *cp(a.pts + __builtin_amdgcn_readfirstlane(a.items.point[it]));
  const int nb = a.items.bin0[it + 1] - a.items.bin0[it];
  const bool lds = nb <= kLdsBins;
  uint32_t *cnt = lds ? cnt_l : a.bhist + a.items.hoff[it] + (int64_t)lb * nb;
  for (int i = threadIdx.x; i < nb; i += TH) cnt[i] = 0u;
  __syncthreads();
  const int64_t n = a.items.cnt[it];
  const int64_t j0 = (int64_t)lb * (TH * U), j1 = min(n, j0 + TH * U);
  // the sort block's samples, U per thread: all their parameters are loaded
  // before any is used, so the loads of a thread's samples are in flight
  // together
  R th[U][7];
#pragma unroll
  for (int u = 0; u < U; u++) {
    const int64_t j = j0 + threadIdx.x + (int64_t)u * TH;
    const int64_t col = a.items.off[it] + (j < j1 ? j : j0);
#pragma unroll
    for (int d = 0; d < 7; d++) th[u][d] = a.theta[d * a.stride + col];
  }
  const int K = p.K, pad = p.pad, bin_w = p.bin_w, nq = p.nq;
#pragma unroll
  for (int u = 0; u < U; u++) {
    const int64_t j = j0 + threadIdx.x + (int64_t)u * TH;
    if (j >= j1) break;
    const int64_t f = a.items.samp0[it] + j;
    const double io = th[u][RIFT_IOTA], ph = th[u][RIFT_PHI], di = th[u][RIFT_DIST], ta = th[u][RIFT_TAU];
    const SkyTrig tr = sky_trig(th[u][RIFT_ALPHA], th[u][RIFT_DELTA], 0.0, p.gmst);
    // n_k = floor((tau + dt_k) f_s), valid when the 4-tap stencil stays inside
    // the stored rows for every window sample: -pad <= n_k <= pad
    bool ok = isfinite(ta) && isfinite(tr.ch) && isfinite(tr.sd) && isfinite(io) && isfinite(ph) &&
              (a.dmarg || (isfinite(di) && di > 0.0)) && isfinite((double)th[u][RIFT_PSI]);
    int nk[kMaxDet];
#pragma unroll
    for (int k = 0; k < kMaxDet; k++) {
      nk[k] = 0;
      if (k < K) {
        const double rc[3] = {p.rc[k][0], p.rc[k][1], p.rc[k][2]};
        const double sk = (ta + delay(rc, tr)) * p.f_s, fl = floor(sk);
        const bool okk = isfinite(sk) && fl >= -pad && fl <= pad;
        ok = ok && okk;
        nk[k] = okk ? (int)fl : 0;
      }
    }
    uint32_t key = 0, mul = 1;
#pragma unroll
    for (int k = 0; k < kMaxDet; k++) {
      if (!ok) nk[k] = 0;
      if (k < K) {
        key += (ok ? (uint32_t)((nk[k] + pad) / bin_w) : 0u) * mul;
        mul *= nq;
      }
    }
    // the four int16 of the sample, one 8-byte store
    *(uint2 *)(a.nsh + f * 4) = make_uint2((uint32_t)(uint16_t)nk[0] | (uint32_t)(uint16_t)nk[1] << 16,
                                           (uint32_t)(uint16_t)nk[2] | (ok ? 1u << 16 : 0u));
    a.key[f] = key;
    atomicAdd(&cnt[key], 1u);
  }
  __syncthreads();
  if (lds) {
    uint32_t *row = a.bhist + a.items.hoff[it] + (int64_t)lb * nb;
    for (int i = threadIdx.x; i < nb; i += TH) row[i] = cnt_l[i];
  }
}

// ---- 2. scans: block offsets within each bin, tiles before each bin and point --
// Column scan of the [sort block][bin] histogram of one point with more than
// kScanRows sort blocks or kLdsBins bins: a workgroup takes 64 bins; its 16 wavefronts each sum
// a sixteenth of the sort blocks, then rewrite their share as running offsets.
// Reads are coalesced along the bins, and every point's bins are spread over
// many workgroups.  (Fewer: scan_kernel's own threads do it, a launch less; of
// 132651 bins they took 250 us, this 12.)
constexpr int kScanBins = 64;
constexpr int kScanRanges = 16;  // block ranges per column scan: 1024 threads
constexpr int kScanRows = 16;
__host__ __device__ constexpr bool own_colscan(int blocks, int bins) { return blocks > kScanRows || bins > kLdsBins; }

template <typename R>
__global__ void __launch_bounds__(kScanRanges * kScanBins) colscan_kernel(MfmaArgsT<R> a) {
  __shared__ uint32_t part[kScanRanges][kScanBins];
  const int q = threadIdx.x >> 6, bl = threadIdx.x & 63;
  for (int it = blockIdx.y; it < a.items.n_items; it += gridDim.y) {
    const int b0 = a.items.bin0[it], nb = a.items.bin0[it + 1] - b0;
    const int nblk = a.items.blk0[it + 1] - a.items.blk0[it];
    if ((int)blockIdx.x * kScanBins >= nb || !own_colscan(nblk, nb)) continue;  // uniform over the workgroup
    const int lb_per = (nblk + kScanRanges - 1) / kScanRanges;
    const int b = (int)blockIdx.x * kScanBins + bl;
    const int lo = min(nblk, q * lb_per), hi = min(nblk, lo + lb_per);
    uint32_t *h = a.bhist + a.items.hoff[it];
    uint32_t sum = 0;
    if (b < nb)
      for (int lb = lo; lb < hi; lb++) sum += h[(int64_t)lb * nb + b];
    __syncthreads();  // part[] of the previous item fully read
    part[q][bl] = sum;
    __syncthreads();
    uint32_t run = 0;
    for (int i = 0; i < q; i++) run += part[i][bl];
    if (b < nb) {
      for (int lb = lo; lb < hi; lb++) {
        const uint32_t v = h[(int64_t)lb * nb + b];
        h[(int64_t)lb * nb + b] = run;
        run += v;
      }
      if (q == kScanRanges - 1) a.count[b0 + b] = run;
    }
  }
}

// tiles of each bin (bins padded to whole tiles, for the evaluation to whole
// pairs of them, the 32 samples of its wavefronts), work units of each bin
// (groups of up to unit_tiles of its tiles), and their prefixes per point
__device__ __forceinline__ uint32_t bin_tiles(int unit_tiles, uint32_t cnt) {
  const uint32_t w = unit_tiles == 8 ? 2u : 1u;
  return w * ((cnt + w * kTS - 1) / (w * kTS));
}

// exclusive prefix of v over the 1024 threads of a workgroup, and its total
template <typename V>
__device__ __forceinline__ V block_scan(V v, V *wsum, V &total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  V x = v;
  for (int o = 1; o < 64; o <<= 1) {
    const V y = (V)__shfl_up((unsigned long long)x, o);
    if (lane >= o) x += y;
  }
  __syncthreads();  // wsum free
  if (lane == 63) wsum[wave] = x;
  __syncthreads();
  V before = 0;
  total = 0;
#pragma unroll 4  // (whole, the scheduler of this file loads all at once and spills 14 registers)
  for (int i = 0; i < 16; i++) {
    if (i < wave) before += wsum[i];
    total += wsum[i];
  }
  return before + x - v;
}

// One workgroup per point: the column scan of its few sort blocks (more:
// colscan_kernel has done it), then the tiles and units before each bin.  The
// workgroup that finishes last (a device counter) also takes the prefixes over
// the points and resets the per-class counters.
template <typename R>
__global__ void __launch_bounds__(1024) scan_kernel(MfmaArgsT<R> a) {
  __shared__ uint64_t wsum[16];
  __shared__ bool last_sh;
  const int it = blockIdx.x, tid = threadIdx.x;
  const int b0 = a.items.bin0[it], nb = a.items.bin0[it + 1] - b0;
  const int nblk = a.items.blk0[it + 1] - a.items.blk0[it];
  const uint32_t U = (uint32_t)a.unit_tiles;
  if (!own_colscan(nblk, nb)) {
    uint32_t *h = a.bhist + a.items.hoff[it];
    for (int b = tid; b < nb; b += 1024) {
      uint32_t v[kScanRows], run = 0;
#pragma unroll
      for (int lb = 0; lb < kScanRows; lb++) v[lb] = lb < nblk ? h[(int64_t)lb * nb + b] : 0u;
#pragma unroll
      for (int lb = 0; lb < kScanRows; lb++) {
        if (lb < nblk) h[(int64_t)lb * nb + b] = run;
        run += v[lb];
      }
      a.count[b0 + b] = run;
    }
    __syncthreads();
  }
  // a contiguous run of bins per thread; tiles and units as one 64-bit sum
  const int per = (nb + 1023) / 1024, lo = min(nb, tid * per), hi = min(nb, lo + per);
  auto of = [&](uint32_t cnt) {
    const uint32_t tb = bin_tiles(a.unit_tiles, cnt);
    return (uint64_t)tb | (uint64_t)((tb + U - 1) / U) << 32;
  };
  uint64_t sum = 0, all;
  for (int b = lo; b < hi; b++) sum += of(a.count[b0 + b]);
  uint64_t run = block_scan<uint64_t>(sum, wsum, all);
  for (int b = lo; b < hi; b++) {
    a.bin_tile[b0 + b] = (uint32_t)run;
    a.bin_unit[b0 + b] = (uint32_t)(run >> 32);
    run += of(a.count[b0 + b]);
  }
  const uint32_t rt = (uint32_t)all, ru = (uint32_t)(all >> 32);
  if (tid == 0) {
    // whole groups of 4 tiles per point; read by another workgroup
    __hip_atomic_store(&a.item_tiles[it + 1], (rt + 3u) & ~3u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&a.item_units[it + 1], ru, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t done = __hip_atomic_fetch_add(&a.ctl[kCtlScan], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    last_sh = done + 1 == (uint32_t)a.items.n_items;
  }
  __syncthreads();
  if (!last_sh) return;
  const int ni = a.items.n_items;
  uint64_t ct = 0, cc = 0;  // tiles and units; coefficient storage: K 2Mp 16 values per tile of each point
  for (int c0 = 0; c0 < ni; c0 += 1024) {
    const int i = c0 + tid;
    uint64_t t = 0, c = 0, tt, tc;
    if (i < ni) {
      const uint32_t nt = __hip_atomic_load(&a.item_tiles[i + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const uint32_t nu = __hip_atomic_load(&a.item_units[i + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      t = (uint64_t)nt | (uint64_t)nu << 32;
      const PointDev &p = a.pts[a.items.point[i]];
      c = (uint64_t)nt * (uint64_t)(p.K * 2 * p.Mp * kTS);
    }
    const uint64_t xt = ct + block_scan<uint64_t>(t, wsum, tt) + t;
    const uint64_t xc = cc + block_scan<uint64_t>(c, wsum, tc);
    if (i < ni) {
      a.item_tiles[i + 1] = (uint32_t)xt;
      a.item_units[i + 1] = (uint32_t)(xt >> 32);
      a.item_cop[i] = (int64_t)xc;
    }
    ct += tt;
    cc += tc;
  }
  if (tid == 0) {
    a.item_tiles[0] = 0;
    a.item_units[0] = 0;
    a.ctl[0] = (uint32_t)ct;
  }
  if (tid < kMaxClasses) a.ctl[1 + tid] = a.ctl[kCtlUnits2 + tid] = 0;
}

// ---- 3. one record per sample at its (padded) sorted slot; the tiles -----------
// The first n_sort_blocks workgroups scatter their samples' records.  The
// others take one tile per thread: its point and bin, the work unit it opens
// (every unit_tiles-th tile of a bin opens one, for itself and the next ones),
// and the padding slots (flag 0) that the scatter leaves: the rest of a bin's
// last tiles and, past the last bin, the tiles that round the point up to
// groups of 4.  The tile's bin is found by bisection of the point's tile
// prefixes, so a bin that holds most of a call's samples (a proposal
// concentrated on a source) costs no more than the same number of tiles in
// many bins: one thread per bin took 877 us for 1e6 samples with half of them
// in a few bins, one per tile 6 us.
template <typename R>
__device__ __forceinline__ void tile_setup(const MfmaArgsT<R> &a, uint32_t t) {
  if (t >= a.ctl[0]) return;
  int lo = 0, hi = a.items.n_items;  // item_tiles[lo] <= t < item_tiles[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (a.item_tiles[mid] <= t) lo = mid; else hi = mid;
  }
  const int it = lo;
  a.tile_item[t] = it;
  const uint32_t x = t - a.item_tiles[it];  // tile within the point
  const int b0 = a.items.bin0[it];
  lo = b0;  // last bin with bin_tile <= x (an empty bin shares its prefix with the next one)
  hi = a.items.bin0[it + 1];
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (a.bin_tile[mid] <= x) lo = mid; else hi = mid;
  }
  const uint32_t cnt = a.count[lo], c = x - a.bin_tile[lo], tb = bin_tiles(a.unit_tiles, cnt);
  const uint32_t U = (uint32_t)a.unit_tiles;
  a.tile_key[t] = c < tb ? (uint32_t)(lo - b0) : kNoBin;
  if (c < tb && c % U == 0u) {
    WorkUnit w;
    w.tile = t;
    w.ntiles = min(U, tb - c);
    w.key = (uint32_t)(lo - b0);
    a.unit[a.item_units[it] + a.bin_unit[lo] + c / U] = w;
  }
  const uint32_t used = c < tb && cnt > kTS * c ? min((uint32_t)kTS, cnt - kTS * c) : 0u;
  SampleRec z;
  for (int d = 0; d < 7; d++) z.th[d] = 0.f;
  z.col = 0;
  z.n[0] = z.n[1] = z.n[2] = 0;
  z.flag = 0;
  for (uint32_t q = used; q < (uint32_t)kTS; q++) a.rec[(int64_t)kTS * t + q] = z;
}

template <typename R, int TH, int U>
__global__ void __launch_bounds__(TH) scatter_kernel(MfmaArgsT<R> a) {
  extern __shared__ uint32_t cur_l[];
  if ((int)blockIdx.x >= a.n_sort_blocks) {
    tile_setup(a, (blockIdx.x - (uint32_t)a.n_sort_blocks) * TH + threadIdx.x);
    return;
  }
  const int it = block_item(a.items, blockIdx.x);
  const int lb = blockIdx.x - a.items.blk0[it];
  const int b0 = a.items.bin0[it], nb = a.items.bin0[it + 1] - b0;
  const bool lds = nb <= kLdsBins;
  uint32_t *cur = lds ? cur_l : a.bhist + a.items.hoff[it] + (int64_t)lb * nb;
  if (lds) {
    const uint32_t *row = a.bhist + a.items.hoff[it] + (int64_t)lb * nb;
    for (int i = threadIdx.x; i < nb; i += TH) cur_l[i] = row[i];
  }
  __syncthreads();
  const int64_t n = a.items.cnt[it];
  const int64_t j0 = (int64_t)lb * (TH * U), j1 = min(n, j0 + TH * U);
  const uint32_t tbase = a.item_tiles[it];
  // U samples per thread, their loads issued together
  SampleRec rec[U];
  uint32_t key[U];
#pragma unroll
  for (int u = 0; u < U; u++) {
    const int64_t jj = j0 + threadIdx.x + (int64_t)u * TH, j = jj < j1 ? jj : j0;
    const int64_t f = a.items.samp0[it] + j;
    const int64_t col = a.items.off[it] + j;
    key[u] = a.key[f];
#pragma unroll
    for (int d = 0; d < 7; d++) rec[u].th[d] = sizeof(R) == 4 ? (float)a.theta[d * a.stride + col] : 0.f;
    rec[u].col = (int)col;
    const uint2 nw = *(const uint2 *)(a.nsh + f * 4);
    rec[u].n[0] = (int16_t)(nw.x & 0xffffu);
    rec[u].n[1] = (int16_t)(nw.x >> 16);
    rec[u].n[2] = (int16_t)(nw.y & 0xffffu);
    rec[u].flag = (nw.y >> 16) ? 1 : 2;
  }
#pragma unroll
  for (int u = 0; u < U; u++) {
    if (j0 + threadIdx.x + (int64_t)u * TH >= j1) break;
    const uint32_t r = atomicAdd(&cur[key[u]], 1u);
    a.rec[kTS * (tbase + a.bin_tile[b0 + key[u]]) + r] = rec[u];
  }
}

// ---- 4. per-sample coefficients (FP64), tile-major ---------------------------
// Quadratic term with the Hermitian (U) and symmetric (V) packing of the
// host: q_k = Y^dag U_k Y = sum_{m <= m'} Re(conj(Y_m) c_{mm'} Y_m'),
// t_k = Y^T V_k Y = sum_{m <= m'} c'_{mm'} Y_m Y_m', with the off-diagonal
// factor 2 folded into c, c'; B = x^2/4 sum_k [|F_k|^2 q_k + Re(F_k^2 t_k)].
// A block is 4 whole tiles of one point, so the point's constants are read
// through the constant address space (scalar loads) and every branch on them
// is uniform.  The packed tables are zero for detectors past K and F_k = 0
// there, so the pair sums run over all kMaxDet detectors without branches.
// Per tile the pass stores Y_m (2 M_p floats per sample, shared by the
// detectors) and x F_k (in the tile record); the evaluation kernels form the
// B operands a_km = x F_k Y_m themselves.
// Harmonics use the polynomial form of the host tables (Horner in
// u = cos^2(iota/2)).  MC > 0: the mode count is a compile-time constant, Y
// lives in registers and the pair sums unroll (table values as scalar
// operands).  MC = 0 is the general form, with Y staged in LDS and the sums
// in loops; points with a V table always take it (the host gives them
// classes of their own: a second unrolled pass would keep every mode product
// of the first alive).  Padding and invalid slots run the same code on a
// harmless angle set and store zeros.
template <int MC, typename R>
__global__ void __launch_bounds__(64) coef_kernel(MfmaArgsT<R> a, int item_lo, int item_hi) {
  constexpr int YS = MC > 0 ? 1 : 64;
  constexpr int YM = MC > 0 ? 1 : kMaxModes;
  constexpr int YR = MC > 0 ? MC : 1;
  __shared__ double Ys[YS][YM][2];
  const int64_t t_lo = a.item_tiles[item_lo], t_hi = a.item_tiles[item_hi];
  const int64_t t_blk = t_lo + 4 * (int64_t)blockIdx.x;
  if (t_blk >= t_hi) return;  // whole block (items hold whole blocks of 4 tiles)
  const int64_t pos = t_blk * kTS + threadIdx.x;
  const int64_t t = pos / kTS;
  const int s = (int)(pos % kTS);
  const SampleRec rec = a.rec[pos];
  const int it = __builtin_amdgcn_readfirstlane(a.tile_item[t_blk]);
  const int pt = __builtin_amdgcn_readfirstlane(a.items.point[it]);
  const RIFT_CONST PointDev &p = *cp(a.pts + pt);
  const int K = p.K, E = 2 * p.Mp;
  const int M = MC > 0 ? MC : p.M;
  RIFT_GLOBAL R *op = gpw(a.cop + a.item_cop[it] + (int64_t)(t - a.item_tiles[it]) * K * E * kTS + s);
  RIFT_GLOBAL CoefTileT<R> *ct = gpw(a.ctile + t);
  const bool pad = rec.flag == 0;
  const bool valid = rec.flag == 1;
  double th[7];
#pragma unroll
  for (int d = 0; d < 7; d++) {
    const double v = sizeof(R) == 4 ? (double)rec.th[d] : (double)a.theta[d * a.stride + (valid ? rec.col : 0)];
    th[d] = valid ? v : (d == RIFT_DIST ? 1.0 : 0.0);
  }
  const double x = a.dmarg ? 1.0 : p.d_ref / th[RIFT_DIST];  // distance marginalization: the terms at D_ref
  constexpr double kUnit = sizeof(R) == 4 ? kLog2e : 1.0;  // FP32: base-2 units for the window's exp2 / log2
  const double xl = valid ? x * kUnit : 0.0;
  SkyTrig tr = sky_trig(th[RIFT_ALPHA], th[RIFT_DELTA], th[RIFT_PSI], p.gmst);
  double Fr[kMaxDet], Fi[kMaxDet];
#pragma unroll
  for (int k = 0; k < kMaxDet; k++) {
    Fr[k] = Fi[k] = 0.0;
    if (k < K) {
      double D[9], rc[3];
#pragma unroll
      for (int i = 0; i < 9; i++) D[i] = p.D[k][i];
#pragma unroll
      for (int i = 0; i < 3; i++) rc[i] = p.rc[k][i];
      antenna(D, tr, Fr[k], Fi[k]);
      const int n = (int)rec.n[k];
      const double sk = (th[RIFT_TAU] + delay(rc, tr)) * p.f_s;
      ct->mu[k][s] = valid ? (R)(sk - (double)n) : R(0);
      ct->n[k][s] = valid ? n : 1 << 28;
    } else {
      ct->mu[k][s] = R(0);
      ct->n[k][s] = 1 << 28;
    }
    ct->xf[k][0][s] = (R)(xl * Fr[k]);
    ct->xf[k][1][s] = (R)(xl * Fi[k]);
  }
  // harmonics: Y_m = (sin(iota)/2)^par P_m(cos^2(iota/2)) exp(i m phi), with
  // exp(i m phi) by repeated products of exp(i phi)
  double ci, si, c1, s1;
  sincos(0.5 * th[RIFT_IOTA], &si, &ci);
  sincos(th[RIFT_PHI], &s1, &c1);
  const double u = ci * ci, hs = si * ci;
  double Yr[YR], Yi[YR];
  double (*Yl)[2] = Ys[MC > 0 ? 0 : threadIdx.x];
#pragma unroll
  for (int m = 0; m < (MC > 0 ? MC : kMaxModes); m++) {
    if (m >= M) break;
    double yr, yi;
    if constexpr (sizeof(R) == 4) {
      harmonic_ym(p, m, u, hs, c1, s1, yr, yi);
    } else {
      // the Wigner sum itself: the polynomial's cancellation costs a digit
      // (4e-15 of ln L_t at l <= 4 against 4e-16), which only FP64 shows
      double cm, sm;
      phase_m(p.em[m], c1, s1, cm, sm);
      harmonic(p, m, ci, si, cm, sm, yr, yi);
    }
    if constexpr (MC > 0) {
      Yr[m] = yr;
      Yi[m] = yi;
    } else {
      Yl[m][0] = yr;
      Yl[m][1] = yi;
    }
    // elements 2m, 2m + 1 of the tile's harmonic block; the evaluation
    // kernels form a_km = (x F_k) Y_m from it and xf
    op[(2 * m) * kTS] = valid ? (R)yr : R(0);
    op[(2 * m + 1) * kTS] = valid ? (R)yi : R(0);
  }
  for (int e = 2 * M; e < E; e++) op[e * kTS] = R(0);
  double q[kMaxDet] = {0.0, 0.0, 0.0}, vr[kMaxDet] = {0.0, 0.0, 0.0}, vi[kMaxDet] = {0.0, 0.0, 0.0};
  // conj(Y_m) Y_m' against U, Y_m Y_m' against V
  auto upair = [&](const auto *T, int idx, double ymr, double ymi, double ypr, double ypi) {
    const double pr = ymr * ypr + ymi * ypi, pi = ymr * ypi - ymi * ypr;
#pragma unroll
    for (int k = 0; k < kMaxDet; k++) {
      const double ur = T[(idx * kMaxDet + k) * 2], ui = T[(idx * kMaxDet + k) * 2 + 1];
      q[k] = fma(-ui, pi, fma(ur, pr, q[k]));
    }
    // unrolled: one wait per four pairs of table loads
    if ((idx & 3) == 3) __builtin_amdgcn_sched_barrier(0);
  };
  auto vpair = [&](const auto *T, int idx, double ymr, double ymi, double ypr, double ypi) {
    const double sr = ymr * ypr - ymi * ypi, s_i = ymr * ypi + ymi * ypr;
#pragma unroll
    for (int k = 0; k < kMaxDet; k++) {
      const double wr = T[(idx * kMaxDet + k) * 2], wi = T[(idx * kMaxDet + k) * 2 + 1];
      vr[k] = fma(-wi, s_i, fma(wr, sr, vr[k]));
      vi[k] = fma(wi, sr, fma(wr, s_i, vi[k]));
    }
  };
  const RIFT_CONST double *Uq = cp(p.Upk);
  if constexpr (MC > 0) {
#pragma unroll
    for (int m = 0; m < MC; m++)
#pragma unroll
      for (int mp = m; mp < MC; mp++) upair(Uq, m * MC - m * (m - 1) / 2 + (mp - m), Yr[m], Yi[m], Yr[mp], Yi[mp]);
  } else {
    int idx = 0;
    for (int m = 0; m < M; m++)
      for (int mp = m; mp < M; mp++, idx++) upair(Uq, idx, Yl[m][0], Yl[m][1], Yl[mp][0], Yl[mp][1]);
    if (p.Vpk) {
      const RIFT_CONST double *Vq = cp(p.Vpk);
      idx = 0;
      for (int m = 0; m < M; m++)
        for (int mp = m; mp < M; mp++, idx++) vpair(Vq, idx, Yl[m][0], Yl[m][1], Yl[mp][0], Yl[mp][1]);
    }
  }
  double b = 0.0;
#pragma unroll
  for (int k = 0; k < kMaxDet; k++) {
    const double f2 = Fr[k] * Fr[k] + Fi[k] * Fi[k];
    const double F2r = Fr[k] * Fr[k] - Fi[k] * Fi[k], F2i = 2.0 * Fr[k] * Fi[k];
    b += f2 * q[k] + (F2r * vr[k] - F2i * vi[k]);
  }
  ct->B[s] = valid ? (R)(0.25 * x * x * b * kUnit) : R(0);
  ct->col[s] = pad ? -1 : (int)rec.col;
  ct->flag[s] = valid ? 1 : (pad ? 0 : 2);
}

// the sort: sort blocks of TH U samples
template <typename R, int TH, int U>
static void sort_launch(const MfmaArgsT<R> &a, hipStream_t st) {
  const size_t lds = sizeof(uint32_t) * (size_t)std::min(a.max_item_bins, kLdsBins);
  hipLaunchKernelGGL((bin_kernel<R, TH, U>), dim3(a.n_sort_blocks), dim3(TH), lds, st, a);
  if (own_colscan(a.max_item_blocks, a.max_item_bins))
    hipLaunchKernelGGL(colscan_kernel<R>,
                       dim3((unsigned)((a.max_item_bins + kScanBins - 1) / kScanBins), std::min(a.items.n_items, 65535)),
                       dim3(kScanRanges * kScanBins), 0, st, a);
  hipLaunchKernelGGL(scan_kernel<R>, dim3(a.items.n_items), dim3(1024), 0, st, a);
  hipLaunchKernelGGL((scatter_kernel<R, TH, U>), dim3((unsigned)(a.n_sort_blocks + (a.max_tiles + TH - 1) / TH)), dim3(TH),
                     lds, st, a);
}

template <typename R>
hipError_t mfma_prepare(const MfmaArgsT<R> &a, const int *mclass_M, const int *mclass_item0,
                        const int64_t *mclass_tiles, int n_mclasses, hipStream_t st) {
  if (a.sort_block == 256) sort_launch<R, 256, 1>(a, st);
  else if (a.sort_block == 1024) sort_launch<R, 256, 4>(a, st);
  else sort_launch<R, 1024, 4>(a, st);
  for (int c = 0; c < n_mclasses; c++) {
    const int lo = mclass_item0[c], hi = mclass_item0[c + 1];
    const dim3 grid((unsigned)(((int64_t)kTS * mclass_tiles[c] + 63) / 64));
    switch (mclass_M[c]) {  // negative: points with a V table, general form
      case 2: hipLaunchKernelGGL((coef_kernel<2, R>), grid, dim3(64), 0, st, a, lo, hi); break;
      case 5: hipLaunchKernelGGL((coef_kernel<5, R>), grid, dim3(64), 0, st, a, lo, hi); break;
      case 9: hipLaunchKernelGGL((coef_kernel<9, R>), grid, dim3(64), 0, st, a, lo, hi); break;
      case 21: hipLaunchKernelGGL((coef_kernel<21, R>), grid, dim3(64), 0, st, a, lo, hi); break;
      default: hipLaunchKernelGGL((coef_kernel<0, R>), grid, dim3(64), 0, st, a, lo, hi); break;
    }
  }
  return hipGetLastError();
}
template hipError_t mfma_prepare<float>(const MfmaArgsT<float> &, const int *, const int *, const int64_t *, int,
                                        hipStream_t);
template hipError_t mfma_prepare<double>(const MfmaArgsT<double> &, const int *, const int *, const int64_t *, int,
                                         hipStream_t);

}  // namespace rift
