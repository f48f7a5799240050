// Four-step FFT passes of a large level's Toeplitz-plus-Cross matvec (Sec. 3.2,
// eq. (ccs3.4), eq. (split01)): L = L1 * L2 points, three HBM passes.
//   pass 1 (k_col_fwd): vector formation fused in front (smoothing start,
//            restriction, prolongation, refinement update), column FFTs of
//            length L2, four-step twiddle;
//   pass 2 (k_row):     for a row pair (k2, L2-k2): row FFTs, the 2x2 spectral
//            product (bins f and -f sit in the paired rows), inverse row FFTs,
//            inverse twiddle;
//   pass 3 (k_col_inv): inverse column FFTs, Cross terms, residual / Jacobi /
//            output epilogue.
// Two families of kernels, by the level's geometry:
//  - the mid-size levels' (columns of 64..512 points in tiles of 4, rows of
//    128..1024) hold 8 elements to a thread and one tile or row pair to a
//    workgroup of 32..256 threads.  Latency bounds them (a pass moves a few MB
//    at most), so every operand, twiddle and spectrum is fetched at the start,
//    the transforms make one to three LDS exchanges (fft8_sig; none of them
//    with a barrier where a wavefront holds the tile), and the w_o row is
//    finished by a workgroup of its own.  With the transforms in LDS (seven to
//    ten barriers), general spectra loaded after them and block 0 reducing the
//    w_o row, a row pass took 6.2..8.5 us at L = 2^13..2^17 and 9.1 and 11.8 at
//    2^18 and 2^19, a column pass 3.8..6.9 and 6.6..12.2; now 4.3..4.8, 5.2 and
//    7.2, and 2.9..5.4 and 4.5..9.3 (FP32, kernel trace of a solve with
//    N = 2^20), beside the 1.7 us between two dependent kernels;
//  - the largest levels' hold 16: tiles of kCap4 or 2 kCap4 values,
//    so that each row segment of a real vector spans 32 bytes rather than 16
//    (the column passes there are bound by the number of distinct cache lines
//    their loads touch), and rows of 2048 or 4096 points (L >= 2^22, whose
//    columns then come in tiles of 8 or 4).
// Every global load of a pass is issued in compile-time batches into
// registers, with clamped addresses and masked values, before any of them is
// used.  Internal header.
#pragma once

#include <type_traits>

#include "kernel_common.hpp"

namespace amg {

// ---------------------------------------------------------------------------
// Pass 1.  Thread tid owns column j1 = c0 + (tid mod T) at the EPT rows
// i0 + e*di, i0 = tid / T, di = L2 / EPT.  The signal's upper half (rows from
// L2/2 on) is zero but for the setup's circulant columns, so only EPT/2 rows
// are loaded.
// ---------------------------------------------------------------------------
// The two families' tile geometry: columns of 2^LOG2 points, 2^LOGTC to a tile.
template <int LOG2, int LOGTC>
struct ColGeom {
  static constexpr int kLog2 = LOG2, kLogTC = LOGTC;
  static constexpr bool kMid = LOG2 + LOGTC <= 11;  // 8 elements per thread
  static constexpr int EPT = kMid ? 8 : 16;
  static constexpr int NT = (1 << (LOG2 + LOGTC)) / EPT;
  static constexpr bool kWave = NT <= 64;
  static constexpr int kLds = lds_slots(1 << (LOG2 + LOGTC)) * (kMid && !kWave ? 2 : 1);
  static_assert(NT >= 32 && NT <= 2 * kNT4, "workgroup size");
};

// The lane that holds wave_sum63's result in a workgroup of NT threads.
template <int NT>
__device__ __forceinline__ int sum_lane() {
  return NT < 64 ? NT - 1 : 63;
}
// Sum of one value per thread over the workgroup, in two halves so that the
// barrier between them is one the FFT has anyway: wave partials to red, then
// (after a barrier) their sum in index order, by one thread.
template <int NT, typename T>
__device__ __forceinline__ void block_part(T v, T* red) {
  v = wave_sum63(v);
  if ((threadIdx.x & 63) == sum_lane<NT>()) red[threadIdx.x >> 6] = v;
}
template <int NT, typename T>
__device__ __forceinline__ T block_total(const T* red) {
  T s = red[0];
#pragma unroll
  for (int w = 1; w < NT / 64; ++w) s += red[w];
  return s;
}

// Whether a pass reads the Cross vectors at i.  In the large tiles, which
// memory bounds, it does where they may be nonzero; the other lanes read entry
// 0 and multiply by zero - the same sums, and beyond the horizon a line per
// load in place of a quarter of the bytes of a product's column passes (product
// at N = 2^22, general, FP64: 320 -> 285 us; CG solve at N = 2^22, mixed: 8152
// -> 7544).  The mid-size tiles, which latency bounds, read all: the test in
// front of their loads made them 1 - 2 % slower.
template <typename G, typename T>
__device__ __forceinline__ bool cross_at(const LevelDev<T>& lv, int i) {
  return G::kMid || i < (int)lv.ext || i >= lv.n - (int)lv.ext;
}

template <typename T, int MODE, typename G>
__device__ __forceinline__ void col_fwd_body(const LevelDev<T>& lv, const ColIn<T>& in,
                                             cplx<T>* buf, const Twiddles<T>& tw, T* part) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  const Lds<T> lds{reinterpret_cast<cplx<T>*>(smem_raw)};
  constexpr int EPT = G::EPT, NT = G::NT, LOG2 = G::kLog2, logTC = G::kLogTC;
  __shared__ T red[NT / 64 + 1];
  const int n = lv.n;
  const int L = 1 << lv.logL;
  constexpr int tcols = 1 << logTC;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int j1 = tile * tcols + (threadIdx.x & (tcols - 1));
  const int i0 = threadIdx.x >> logTC;
  constexpr int di = (1 << LOG2) / EPT;
  constexpr int KJ = MODE == COL_SETUP ? EPT : EPT / 2;  // rows with data
  // elements per load batch
  constexpr int CH = KJ < 8 ? KJ : 8;
  // the w_o entry (tile 0, thread 0): its operands are fetched first
  constexpr bool kWo = MODE != COL_SETUP && MODE != COL_MV;
  const bool wo_thread = kWo && tile == 0 && threadIdx.x == 0;
  T wo0 = 0, wo1 = 0, wo2 = 0;
  if (wo_thread) {
    if constexpr (MODE == COL_PRE) {
      wo0 = lv.b[n];
    } else if constexpr (MODE == COL_PRE_RESTRICT) {
      wo0 = in.x[2 * n];
      wo1 = in.x[2 * n + 1];
      wo2 = in.x[2 * n + 2];
    } else if constexpr (MODE == COL_PROLONG) {
      wo0 = lv.u[n];
      wo1 = prolong_at(in.x, n, n);
    } else if constexpr (MODE == COL_OUTER_UPDATE) {
      wo0 = (T)in.xo[n];
      wo1 = in.e_is_float ? (T)((const float*)in.e)[n] : (T)((const double*)in.e)[n];
    }
  }
  FftTw8<T> ft;
  RunTw<T, EPT> rt;
  // the damped inverse diagonal of the two blocks, one division per thread
  const T wdv = in.omega / lv.dv, wdw = in.omega / lv.dw;
  T dot = 0;
  cplx<T> a[EPT];  // formed vector at rows i0 + e*di of column j1
#pragma unroll
  for (int e0 = 0; e0 < KJ; e0 += CH) {
    int jj[CH];
    bool ok[CH];
    T r0[CH], r1[CH], r2[CH], r3[CH], r4[CH], r5[CH], qq[CH], zz[CH];
    // (a) loads only
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int j = j1 + ((i0 + (e0 + c) * di) << lv.logL1);
      jj[c] = j;
      if constexpr (MODE == COL_SETUP) {
        ok[c] = true;
        r0[c] = (T)circ_col(in.gx, n, L, j);
        r1[c] = (T)circ_col(in.gy, n, L, j);
      } else {
        // only the last row's last column is past n - 1
        ok[c] = e0 + c < KJ - 1 || j < n;
        const int js = ok[c] ? j : 0, jw = n + 1 + js;
        const bool nz = cross_at<G>(lv, js);
        const int jc = nz ? js : 0;
        qq[c] = lv.q[jc];
        zz[c] = lv.zeta[jc];
        qq[c] = nz ? qq[c] : T(0);
        zz[c] = nz ? zz[c] : T(0);
        if constexpr (MODE == COL_MV) {
          r0[c] = in.x[js];
          r1[c] = in.x[jw];
        } else if constexpr (MODE == COL_PRE) {
          r0[c] = lv.b[js];
          r1[c] = lv.b[jw];
        } else if constexpr (MODE == COL_PRE_RESTRICT) {
          r0[c] = in.x[2 * js];
          r1[c] = in.x[2 * js + 1];
          r2[c] = in.x[2 * js + 2];
          r3[c] = in.x[2 * jw];
          r4[c] = in.x[2 * jw + 1];
          r5[c] = in.x[2 * jw + 2];
        } else if constexpr (MODE == COL_PROLONG) {
          // coarse vector length = n (2 n_c + 1 = n)
          int lo, hi;
          bool ml, mh;
          r0[c] = lv.u[js];
          r1[c] = lv.u[jw];
          prolong_idx(js, n, lo, hi, ml, mh);
          r2[c] = in.x[lo];
          r3[c] = in.x[hi];
          r2[c] = ml ? r2[c] : T(0);
          r3[c] = mh ? r3[c] : T(0);
          prolong_idx(jw, n, lo, hi, ml, mh);
          r4[c] = in.x[lo];
          r5[c] = in.x[hi];
          r4[c] = ml ? r4[c] : T(0);
          r5[c] = mh ? r5[c] : T(0);
        } else {  // COL_OUTER_UPDATE (T = double)
          r0[c] = (T)in.xo[js];
          r1[c] = (T)in.xo[jw];
        }
      }
    }
    if constexpr (MODE == COL_OUTER_UPDATE) {
      if (in.e_is_float) {
        const float* ef = static_cast<const float*>(in.e);
#pragma unroll
        for (int c = 0; c < CH; ++c) {
          const int js = ok[c] ? jj[c] : 0;
          r2[c] = (T)ef[js];
          r3[c] = (T)ef[n + 1 + js];
        }
      } else {
        const double* ed = static_cast<const double*>(in.e);
#pragma unroll
        for (int c = 0; c < CH; ++c) {
          const int js = ok[c] ? jj[c] : 0;
          r2[c] = (T)ed[js];
          r3[c] = (T)ed[n + 1 + js];
        }
      }
    }
    if constexpr (G::kMid) {  // every twiddle of the pass, behind the operands
      if (e0 + CH >= KJ) {
        ft.load(LOG2, i0, FftTab8<T>{tw.tail, kTailLog});
        run_tw_load<T, EPT>(tw, lv.logL, j1 * i0, j1 * di, rt);
      }
    }
    // (b) vector formation, stores, Cross dot product
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int j = jj[c], jw = n + 1 + j;
      T v = r0[c], w = r1[c];
      if constexpr (MODE == COL_PRE || MODE == COL_PRE_RESTRICT) {
        if constexpr (MODE == COL_PRE_RESTRICT) {
          const T bv = T(0.25) * (r0[c] + T(2) * r1[c] + r2[c]);
          const T bw = T(0.25) * (r3[c] + T(2) * r4[c] + r5[c]);
          if (ok[c]) {
            lv.b[j] = bv;
            lv.b[jw] = bw;
          }
          v = bv;
          w = bw;
        }
        if (lv.dinv) {  // variable diagonal (weakly singular levels)
          const int js = ok[c] ? j : 0;
          v = in.omega * v * lv.dinv[js];
          w = in.omega * w * lv.dinv[n + 1 + js];
        } else {
          v = wdv * v;
          w = wdw * w;
        }
        if (ok[c]) {
          lv.u[j] = v;
          lv.u[jw] = w;
        }
      } else if constexpr (MODE == COL_PROLONG) {
        v = r0[c] + T(0.5) * (r2[c] + r3[c]);
        w = r1[c] + T(0.5) * (r4[c] + r5[c]);
        if (ok[c]) {
          lv.u[j] = v;
          lv.u[jw] = w;
        }
      } else if constexpr (MODE == COL_OUTER_UPDATE) {
        v = r0[c] + r2[c];
        w = r1[c] + r3[c];
        if (ok[c]) {
          in.xo[j] = v;
          in.xo[jw] = w;
        }
      }
      if (!ok[c]) v = w = T(0);
      if constexpr (MODE != COL_SETUP) dot += qq[c] * v + zz[c] * w;
      a[e0 + c] = cplx<T>{v, w};
    }
  }
#pragma unroll
  for (int e = KJ; e < EPT; ++e) a[e] = {T(0), T(0)};
  if (wo_thread) {
    if constexpr (MODE == COL_PRE) {
      lv.u[n] = in.omega * wo0 * (lv.dinv ? lv.dinv[n] : T(1) / lv.o);
    } else if constexpr (MODE == COL_PRE_RESTRICT) {
      const T bo = T(0.25) * (wo0 + T(2) * wo1 + wo2);
      lv.b[n] = bo;
      lv.u[n] = in.omega * bo * (lv.dinv ? lv.dinv[n] : T(1) / lv.o);
    } else if constexpr (MODE == COL_PROLONG) {
      lv.u[n] = wo0 + wo1;
    } else if constexpr (MODE == COL_OUTER_UPDATE) {
      in.xo[n] = (double)wo0 + (double)wo1;
    }
  }
  // the w_o row's partial sum; the FFT's first barrier publishes the waves'
  if constexpr (MODE != COL_SETUP) block_part<NT>(dot, red);
  if constexpr (G::kMid) {
    fft8_sig<T, LOG2, logTC, G::kWave, 0>(a, lds, lds_slots(1 << (LOG2 + logTC)),
                                          threadIdx.x & (tcols - 1), i0, ft);
    twiddle_run_mul_pre<T, EPT, false>(rt, a);
  } else {
    // the thread's rows i0 + e*di are the positions j0 + e*L2/16 of its
    // last-pass butterfly (j0 = i0): first and last passes on registers
    const FftGeom g{LOG2, logTC, 0, logTC, kTwLog, true};
    fft_reg16<T, NT, false>(a, lds, g, threadIdx.x & (tcols - 1), i0, tw.base);
    twiddle_run_mul<T, EPT, false>(tw, lv.logL, j1 * i0, j1 * di, a);
  }
#pragma unroll
  for (int e = 0; e < EPT; ++e) stg(buf + j1 + ((i0 + e * di) << lv.logL1), a[e]);
  if constexpr (MODE != COL_SETUP) {
    if (threadIdx.x == 0) part[tile] = block_total<NT>(red);
  }
}

template <typename T, int MODE, typename G>
__global__ __launch_bounds__(G::NT) __attribute__((amdgpu_waves_per_eu(2)))
void k_col_fwd(LevelDev<T> lv, ColIn<T> in, cplx<T>* buf, Twiddles<T> tw, T* part) {
  col_fwd_body<T, MODE, G>(lv, in, buf, tw, part);
}
// The same pass for a batch of instances of one geometry: block (x, y) runs
// tile x of instance y with that instance's arguments (gated by its solve
// state), so each instance's arithmetic is that of its own launch.
template <typename T, int MODE, typename G>
__global__ __launch_bounds__(G::NT) __attribute__((amdgpu_waves_per_eu(2)))
void k_col_fwd_b(const PassArgs<T>* __restrict__ args, Twiddles<T> tw) {
  const PassArgs<T>* a = args + blockIdx.y;
  if (gate_skip(a->st, a->gate)) return;
  const LevelDev<T> lv = a->lv;
  const ColIn<T> in = a->in;
  col_fwd_body<T, MODE, G>(lv, in, a->buf, tw, a->part);
}

// ---------------------------------------------------------------------------
// Pass 2.  Row pair (item, L2-item), or (0, L2/2) for item 0, one to a
// workgroup; one workgroup more finishes the w_o row
// y_o = q.v + o w_o + zeta.w_bar from pass 1's partial sums (block 0 did both
// and held the pass back by its reduction and the dependent load of w_o), with
// a snapshot of the input's w_o (pass 3 may update u[n] in place (Jacobi) while
// its other blocks still need the value the product used).
// ---------------------------------------------------------------------------
template <typename T, int NT>
__device__ __forceinline__ void finish_wo(const LevelDev<T>& lv, const T* part, int npart,
                                          const T* xin, T* red) {
  const T wo = xin[lv.n];
  T v = 0;
  for (int i = threadIdx.x; i < npart; i += NT) v += part[i];
  block_part<NT>(v, red);
  __syncthreads();
  if (threadIdx.x == 0) {
    lv.scal[0] = block_total<NT>(red) + lv.o * wo;
    lv.scal[1] = wo;
  }
}

// Slot of the partner of bin p of row s (f = k2 + L2 k1 pairs with -f): in the
// other row at L1-1-p for item != 0; within row 0 at (L1-p) mod L1 and within
// row L2/2 at L1-1-p for item 0.
__device__ __forceinline__ int row_partner(int item, int s, int p, int L1) {
  if (item != 0) return s == 0 ? L1 + (L1 - 1 - p) : (L1 - 1 - p);
  return s == 0 ? ((L1 - p) & (L1 - 1)) : L1 + (L1 - 1 - p);
}

// Row pair with L1 = 16 NT / 2 (each thread owns one radix-16 butterfly of
// the last pass: row s = tid / (L1/16), j0 = tid mod (L1/16), positions
// p = j0 + e L1/16).  Loads feed the first FFT pass directly; the spectral
// product exchanges the partner bins through LDS once; the last inverse pass
// feeds the twiddle and the stores.  NT = kNT4: rows of 2048 points;
// NT = 2 kNT4: rows of 4096 (the levels with L >= 2^22, whose columns then
// stay short enough for wide tiles of 8 or 4 columns).
template <typename T, bool SPECTRAL, bool SYM, int NT = kNT4>
__device__ __forceinline__ void row_pair_regs(const LevelDev<T>& lv, Lds<T> lds, cplx<T>* buf,
                                              const Twiddles<T>& tw, int item) {
  constexpr int Q = 16 * NT / 2 / 16;  // L1/16 butterflies per row
  // log2 L1: the geometry is a compile-time constant
  constexpr int kLog1 = NT == kNT4 ? 11 : 12;
  static_assert((1 << kLog1) == 16 * Q, "row length of the register row pass");
  constexpr int L1 = 1 << kLog1;
  const int L2 = 1 << lv.logL2;
  const int tid = threadIdx.x;
  const int s = tid / Q, j0 = tid % Q;
  const int k2 = item == 0 ? (s == 0 ? 0 : L2 / 2) : (s == 0 ? item : L2 - item);
  const int row = k2 << kLog1;
  cplx<T> a[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) a[e] = ldg(buf + row + j0 + e * Q);
  // SPD spectra at the thread's positions: FP32 fetches them under the
  // forward FFT; FP64 right after it (holding them across the FFT would spill)
  constexpr bool kEarly = sizeof(T) == 4;
  T g1[16], g2[16];
  auto load_spec = [&]() {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      g1[e] = lv.g1[row + j0 + e * Q];
      g2[e] = lv.g2[row + j0 + e * Q];
    }
  };
  if (kEarly && SPECTRAL && SYM) load_spec();
  const FftGeom g{kLog1, 1, kLog1, 0, kTwLog, false};
  fft_reg16<T, NT, false>(a, lds, g, s, j0, tw.base);
  if (!kEarly && SPECTRAL && SYM) load_spec();
  if constexpr (!SPECTRAL) {
#pragma unroll
    for (int e = 0; e < 16; ++e) stg(buf + row + j0 + e * Q, a[e]);
  } else {
    __syncthreads();  // last-pass LDS reads done before the exchange writes
#pragma unroll
    for (int e = 0; e < 16; ++e) lds[(s << kLog1) + j0 + e * Q] = a[e];
    __syncthreads();
    auto partner = [&](int e) { return lds[row_partner(item, s, j0 + e * Q, L1)]; };
    if constexpr (SYM) {
      // G1 real, G2 = i g2: Y = g1 z + i g2 conj(z')
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const cplx<T> zp = partner(e);
        a[e] = {g1[e] * a[e].x + g2[e] * zp.y, g1[e] * a[e].y + g2[e] * zp.x};
      }
    } else {
      const cplx<T>* G1 = reinterpret_cast<const cplx<T>*>(lv.g1);
      const cplx<T>* G2 = reinterpret_cast<const cplx<T>*>(lv.g2);
#pragma unroll
      for (int e0 = 0; e0 < 16; e0 += 4) {
        cplx<T> h1[4], h2[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          h1[c] = ldg(G1 + row + j0 + (e0 + c) * Q);
          h2[c] = ldg(G2 + row + j0 + (e0 + c) * Q);
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
          a[e0 + c] = cmul(h1[c], a[e0 + c]) + cmul(h2[c], conj(partner(e0 + c)));
      }
    }
    __syncthreads();  // partner reads done before the inverse FFT writes LDS
    fft_reg16<T, NT, true>(a, lds, g, s, j0, tw.base);
    twiddle_run_mul<T, 16, true>(tw, lv.logL, j0 * k2, Q * k2, a);
#pragma unroll
    for (int e = 0; e < 16; ++e) stg(buf + row + j0 + e * Q, a[e]);
  }
}

// The mid-size levels' row pair: 2^LOG1 <= 1024 points to a row, 8 elements to
// a thread, L1/8 threads to a row; the spectra of both kinds are fetched under
// the forward transform.
template <typename T, bool SPECTRAL, bool SYM, int LOG1>
__device__ __forceinline__ void row8_body(const LevelDev<T>& lv, Lds<T> lds, cplx<T>* buf,
                                          const Twiddles<T>& tw, int item) {
  constexpr int Q = 1 << (LOG1 - 3), L1 = 1 << LOG1, NT = 2 * Q, half = lds_slots(2 * L1);
  constexpr bool kWave = NT <= 64;
  constexpr int X = fft8_exchanges(LOG1);
  const int L2 = 1 << lv.logL2;
  const int s = threadIdx.x / Q, j0 = threadIdx.x % Q;
  const int k2 = item == 0 ? (s == 0 ? 0 : L2 / 2) : (s == 0 ? item : L2 - item);
  const int row = k2 << LOG1;
  cplx<T> a[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) a[e] = ldg(buf + row + j0 + e * Q);
  FftTw8<T> ft;
  ft.load(LOG1, j0, FftTab8<T>{tw.tail, kTailLog});
  using S = std::conditional_t<SYM, T, cplx<T>>;
  S g1[8], g2[8];
  RunTw<T, 8> rt;
  if constexpr (SPECTRAL) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      g1[e] = reinterpret_cast<const S*>(lv.g1)[row + j0 + e * Q];
      g2[e] = reinterpret_cast<const S*>(lv.g2)[row + j0 + e * Q];
    }
    run_tw_load<T, 8>(tw, lv.logL, j0 * k2, Q * k2, rt);
  }
  fft8_sig<T, LOG1, 0, kWave, 0>(a, lds, half, s << LOG1, j0, ft);
  if constexpr (SPECTRAL) {
    const Lds<T> ex{lds.p + (!kWave && (X & 1) ? half : 0)};
#pragma unroll
    for (int e = 0; e < 8; ++e) ex.p[lds_slot((s << LOG1) + j0) + e * lds_step(LOG1 - 3)] = a[e];
    fft_sync<kWave>();
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const cplx<T> zp = ex[row_partner(item, s, j0 + e * Q, L1)];
      // conj(Y): the inverse transform is conj(F(conj Y))
      if constexpr (SYM) {  // G1 real, G2 = i g2
        a[e] = {g1[e] * a[e].x + g2[e] * zp.y, -(g1[e] * a[e].y + g2[e] * zp.x)};
      } else {
        a[e] = conj(cmul(g1[e], a[e]) + cmul(g2[e], conj(zp)));
      }
    }
    // One buffer: the first pass writes where other lanes' partner reads are
    // pending, and with radix 2 or 4 its values do not depend on all of them.
    if constexpr (kWave) fft_sync<true>();
    fft8_sig<T, LOG1, 0, kWave, X + 1>(a, lds, half, s << LOG1, j0, ft);
#pragma unroll
    for (int e = 0; e < 8; ++e) a[e] = conj(a[e]);
    twiddle_run_mul_pre<T, 8, true>(rt, a);
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) stg(buf + row + j0 + e * Q, a[e]);
}

// Threads of a row pass: rows of 4096 and 2048 points with 16 elements to a
// thread, shorter ones with 8.
constexpr int row_nt(int logL1) { return logL1 >= 11 ? 1 << (logL1 - 3) : 1 << (logL1 - 2); }
constexpr int row_lds(int logL1) {  // slots; two buffers where the 8-element form has barriers
  return lds_slots(2 << logL1) * (logL1 < 11 && row_nt(logL1) > 64 ? 2 : 1);
}
template <typename T, bool SPECTRAL, bool SYM, int LOG1>
__device__ __forceinline__ void row_body(const LevelDev<T>& lv, cplx<T>* buf, const Twiddles<T>& tw,
                                         const T* part, int npart, const T* xin) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  constexpr int NT = row_nt(LOG1);
  const Lds<T> lds{reinterpret_cast<cplx<T>*>(smem_raw)};
  __shared__ T red[NT / 64 + 1];
  const int item = blockIdx.x;
  if (SPECTRAL && item == 1 << (lv.logL2 - 1)) {  // past the last row pair
    finish_wo<T, NT>(lv, part, npart, xin, red);
    return;
  }
  if constexpr (LOG1 >= 11) row_pair_regs<T, SPECTRAL, SYM, NT>(lv, lds, buf, tw, item);
  else row8_body<T, SPECTRAL, SYM, LOG1>(lv, lds, buf, tw, item);
}

// Rows of 4096 points, FP32 symmetric: at most 128 registers, so that two
// workgroups fit on a CU (70 KB of LDS each).
constexpr int row_waves(int logL1, size_t elem, bool sym) {
  return logL1 == 12 && elem == 4 && sym ? 4 : 2;
}
template <typename T, bool SPECTRAL, bool SYM, int LOG1>
__global__ __launch_bounds__(row_nt(LOG1))
__attribute__((amdgpu_waves_per_eu(row_waves(LOG1, sizeof(T), SYM))))
void k_row(LevelDev<T> lv, cplx<T>* buf, Twiddles<T> tw, const T* part, int npart, const T* xin) {
  row_body<T, SPECTRAL, SYM, LOG1>(lv, buf, tw, part, npart, xin);
}
template <typename T, bool SPECTRAL, bool SYM, int LOG1>
__global__ __launch_bounds__(row_nt(LOG1))
__attribute__((amdgpu_waves_per_eu(row_waves(LOG1, sizeof(T), SYM))))
void k_row_b(const PassArgs<T>* __restrict__ args, Twiddles<T> tw) {
  const PassArgs<T>* a = args + blockIdx.y;
  if (gate_skip(a->st, a->gate)) return;
  const LevelDev<T> lv = a->lv;
  row_body<T, SPECTRAL, SYM, LOG1>(lv, a->buf, tw, a->part, a->npart, a->xin);
}

// ---------------------------------------------------------------------------
// Pass 3.  Same ownership as pass 1; the outputs j < n are the rows
// j2 < L2/2, i.e. e < EPT/2.  The epilogue's operands are fetched before the
// FFT so their latency overlaps it.
// ---------------------------------------------------------------------------
template <typename T, int MODE, typename G>
__device__ __forceinline__ void col_inv_body(const LevelDev<T>& lv, const EpiOut<T>& out,
                                             const cplx<T>* buf, const Twiddles<T>& tw,
                                             double* part) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  const Lds<T> lds{reinterpret_cast<cplx<T>*>(smem_raw)};
  constexpr int EPT = G::EPT, NT = G::NT, LOG2 = G::kLog2, logTC = G::kLogTC;
  constexpr int KH = EPT / 2, tcols = 1 << logTC, di = (1 << LOG2) / EPT;
  __shared__ double red[NT / 64 + 1];
  const int n = lv.n;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int j1 = tile * tcols + (threadIdx.x & (tcols - 1));
  const int i0 = threadIdx.x >> logTC;
  cplx<T> a[EPT];  // rows i0 + e*di of column j1
#pragma unroll
  for (int e = 0; e < EPT; ++e) a[e] = ldg(buf + j1 + ((i0 + e * di) << lv.logL1));
  FftTw8<T> ft;
  if constexpr (G::kMid) ft.load(LOG2, i0, FftTab8<T>{tw.tail, kTailLog});
  const T wo = lv.scal[1];  // the matvec input's w_o (see finish_wo)
  // the w_o row (tile 0, thread 0): its operands are fetched first
  const bool wo_thread = tile == 0 && threadIdx.x == 0;
  T yo = 0, wb = 0, wu = 0;
  double wbo = 0.0;
  if (wo_thread) {
    yo = lv.scal[0];
    if constexpr (MODE == EPI_RESID || MODE == EPI_SMOOTH) wb = lv.b[n];
    if constexpr (MODE == EPI_SMOOTH) wu = lv.u[n];
    if constexpr (MODE == EPI_OUTER) wbo = out.bo[n] - (out.ynear ? out.ynear[n] : 0.0);
  }
  bool ok[KH];
  int jj[KH];
  T pp[KH], xx[KH], b0[KH], b1[KH], u0[KH], u1[KH];
  double o0[KH], o1[KH], q0[KH], q1[KH];
#pragma unroll
  for (int e = 0; e < KH; ++e) {
    const int j = j1 + ((i0 + e * di) << lv.logL1);
    ok[e] = e < KH - 1 || j < n;  // only the last row's last column is past n - 1
    jj[e] = j;
    const int js = ok[e] ? j : 0, jw = n + 1 + js;
    const bool nz = cross_at<G>(lv, js);
    const int jc = nz ? js : 0;
    pp[e] = lv.p[jc];
    xx[e] = lv.xi[jc];
    pp[e] = nz ? pp[e] : T(0);
    xx[e] = nz ? xx[e] : T(0);
    if constexpr (MODE == EPI_RESID || MODE == EPI_SMOOTH) {
      b0[e] = lv.b[js];
      b1[e] = lv.b[jw];
    }
    if constexpr (MODE == EPI_SMOOTH && (sizeof(T) == 4 || EPT < 16)) {
      u0[e] = lv.u[js];
      u1[e] = lv.u[jw];
    }
    if constexpr (MODE == EPI_OUTER) {
      o0[e] = out.bo[js];
      o1[e] = out.bo[jw];
      q0[e] = out.ynear ? out.ynear[js] : 0.0;
      q1[e] = out.ynear ? out.ynear[jw] : 0.0;
    }
  }
  if constexpr (G::kMid) {  // the inverse transform is conj(F(conj Y))
#pragma unroll
    for (int e = 0; e < EPT; ++e) a[e] = conj(a[e]);
    fft8_sig<T, LOG2, logTC, G::kWave, 0>(a, lds, lds_slots(1 << (LOG2 + logTC)),
                                          threadIdx.x & (tcols - 1), i0, ft);
#pragma unroll
    for (int e = 0; e < KH; ++e) a[e] = conj(a[e]);
  } else {
    const FftGeom g{LOG2, logTC, 0, logTC, kTwLog, true};
    fft_reg16<T, NT, true>(a, lds, g, threadIdx.x & (tcols - 1), i0, tw.base);
  }
  if constexpr (MODE == EPI_SMOOTH && sizeof(T) == 8 && EPT == 16) {
    // FP64 full tiles: the iterate is fetched after the FFT (register budget)
#pragma unroll
    for (int e = 0; e < KH; ++e) {
      const int js = ok[e] ? jj[e] : 0;
      u0[e] = lv.u[js];
      u1[e] = lv.u[n + 1 + js];
    }
  }
  const bool band = lv.bc != nullptr;  // weakly singular levels: + B x, variable diagonal
  const T wdv = out.omega / lv.dv, wdw = out.omega / lv.dw;  // Jacobi factors, constant diagonal
  double ss = 0.0;
#pragma unroll
  for (int e = 0; e < KH; ++e) {
    if (!ok[e]) continue;
    const int j = jj[e], jw = n + 1 + j;
    const cplx<T> y = a[e];
    T yv = y.x + pp[e] * wo;
    T yw = y.y + xx[e] * wo;
    if (band) {
      yv += lv.bc[j];
      yw += lv.bc[jw];
    }
    if constexpr (MODE == EPI_MV) {
      out.y[j] = yv;
      out.y[jw] = yw;
    } else if constexpr (MODE == EPI_RESID) {
      lv.r[j] = b0[e] - yv;
      lv.r[jw] = b1[e] - yw;
    } else if constexpr (MODE == EPI_SMOOTH) {
      if (band) {
        lv.u[j] = u0[e] + out.omega * (b0[e] - yv) * lv.dinv[j];
        lv.u[jw] = u1[e] + out.omega * (b1[e] - yw) * lv.dinv[jw];
      } else {
        lv.u[j] = u0[e] + wdv * (b0[e] - yv);
        lv.u[jw] = u1[e] + wdw * (b1[e] - yw);
      }
    } else {  // EPI_OUTER
      const double rv = o0[e] - ((double)yv + q0[e]), rw = o1[e] - ((double)yw + q1[e]);
      out.ro[j] = rv;
      out.ro[jw] = rw;
      if (out.r32) {
        out.r32[j] = (float)rv;
        out.r32[jw] = (float)rw;
      }
      ss += rv * rv + rw * rw;
    }
  }
  if (wo_thread) {
    if (band) yo += lv.bc[n];
    if constexpr (MODE == EPI_MV) {
      out.y[n] = yo;
    } else if constexpr (MODE == EPI_RESID) {
      lv.r[n] = wb - yo;
    } else if constexpr (MODE == EPI_SMOOTH) {
      lv.u[n] = wu + out.omega * (wb - yo) * (band ? lv.dinv[n] : T(1) / lv.o);
    } else {
      const double ro = wbo - (double)yo;
      out.ro[n] = ro;
      if (out.r32) out.r32[n] = (float)ro;
      ss += ro * ro;
    }
  }
  if constexpr (MODE == EPI_OUTER) {
    block_part<NT>(ss, red);
    __syncthreads();
    if (threadIdx.x == 0) part[tile] = block_total<NT>(red);
  }
}

template <typename T, int MODE, typename G>
__global__ __launch_bounds__(G::NT) __attribute__((amdgpu_waves_per_eu(2)))
void k_col_inv(LevelDev<T> lv, EpiOut<T> out, const cplx<T>* buf, Twiddles<T> tw, double* part) {
  col_inv_body<T, MODE, G>(lv, out, buf, tw, part);
}
template <typename T, int MODE, typename G>
__global__ __launch_bounds__(G::NT) __attribute__((amdgpu_waves_per_eu(2)))
void k_col_inv_b(const PassArgs<T>* __restrict__ args, Twiddles<T> tw) {
  const PassArgs<T>* a = args + blockIdx.y;
  if (gate_skip(a->st, a->gate)) return;
  const LevelDev<T> lv = a->lv;
  const EpiOut<T> out = a->out;
  col_inv_body<T, MODE, G>(lv, out, a->buf, tw, a->npart_out);
}

// ---------------------------------------------------------------------------
// Launchers: the level geometry picks the instance; a geometry that no plan
// has is refused (hipErrorInvalidValue).
// ---------------------------------------------------------------------------
template <int V>
using IC = std::integral_constant<int, V>;
// f(ColGeom) for columns of 2^logL2 points in tiles of tcols.
template <typename F>
hipError_t col_pick(int logL1, int logL2, int tcols, F&& f) {
  if (tcols < 1 || (1 << logL1) % tcols) return hipErrorInvalidValue;
  switch (100 * logL2 + tcols) {
    case 604: return f(ColGeom<6, 2>{});
    case 704: return f(ColGeom<7, 2>{});
    case 804: return f(ColGeom<8, 2>{});
    case 904: return f(ColGeom<9, 2>{});
    case 908: return f(ColGeom<9, 3>{});
    case 1008: return f(ColGeom<10, 3>{});
    case 1104: return f(ColGeom<11, 2>{});
    default: return hipErrorInvalidValue;
  }
}
// f(log2 of the row length).
template <typename F>
hipError_t row_pick(int logL1, F&& f) {
  switch (logL1) {
    case 7: return f(IC<7>{});
    case 8: return f(IC<8>{});
    case 9: return f(IC<9>{});
    case 10: return f(IC<10>{});
    case 11: return f(IC<11>{});
    case 12: return f(IC<12>{});
    default: return hipErrorInvalidValue;
  }
}

template <typename T, int MODE>
hipError_t col_fwd_go(int grid, hipStream_t s, const LevelDev<T>& lv, const ColIn<T>& in,
                      cplx<T>* buf, const Twiddles<T>& tw, T* part) {
  return col_pick(lv.logL1, lv.logL2, lv.tcols, [&](auto g) {
    using G = decltype(g);
    return launch_lds(k_col_fwd<T, MODE, G>, grid, G::NT, sizeof(cplx<T>) * G::kLds, s, lv, in,
                      buf, tw, part);
  });
}
template <typename T, int MODE>
hipError_t col_inv_go(int grid, hipStream_t s, const LevelDev<T>& lv, const EpiOut<T>& out,
                      const cplx<T>* buf, const Twiddles<T>& tw, double* part) {
  return col_pick(lv.logL1, lv.logL2, lv.tcols, [&](auto g) {
    using G = decltype(g);
    return launch_lds(k_col_inv<T, MODE, G>, grid, G::NT, sizeof(cplx<T>) * G::kLds, s, lv, out,
                      buf, tw, part);
  });
}
template <typename T, bool SPECTRAL, bool SYM>
hipError_t row_go(int grid, hipStream_t s, const LevelDev<T>& lv, cplx<T>* buf,
                  const Twiddles<T>& tw, const T* part, int npart, const T* xin) {
  return row_pick(lv.logL1, [&](auto g) {
    constexpr int LOG1 = decltype(g)::value;
    return launch_lds(k_row<T, SPECTRAL, SYM, LOG1>, grid, row_nt(LOG1),
                      sizeof(cplx<T>) * row_lds(LOG1), s, lv, buf, tw, part, npart, xin);
  });
}

// Modes built for FP32 (the V-cycle) and FP64 (everything).
template <typename T>
constexpr bool col_mode_built(int mode) {
  return sizeof(T) == 8 || mode == COL_MV || mode == COL_PRE || mode == COL_PRE_RESTRICT ||
         mode == COL_PROLONG;
}
template <typename T>
constexpr bool epi_mode_built(int mode) {
  return sizeof(T) == 8 || mode == EPI_MV || mode == EPI_RESID || mode == EPI_SMOOTH;
}

template <typename T>
hipError_t launch_col_fwd(int mode, const LevelDev<T>& lv, const ColIn<T>& in, cplx<T>* buf,
                          const Twiddles<T>& tw, T* part, hipStream_t s) {
  if (!col_mode_built<T>(mode)) return hipErrorInvalidValue;
  const int grid = col_blocks(lv.logL1, lv.tcols);
  switch (mode) {
    case COL_MV: return col_fwd_go<T, COL_MV>(grid, s, lv, in, buf, tw, part);
    case COL_PRE: return col_fwd_go<T, COL_PRE>(grid, s, lv, in, buf, tw, part);
    case COL_PRE_RESTRICT: return col_fwd_go<T, COL_PRE_RESTRICT>(grid, s, lv, in, buf, tw, part);
    case COL_PROLONG: return col_fwd_go<T, COL_PROLONG>(grid, s, lv, in, buf, tw, part);
    default: break;
  }
  if constexpr (sizeof(T) == 8) {
    switch (mode) {
      case COL_OUTER_UPDATE:
        return col_fwd_go<T, COL_OUTER_UPDATE>(grid, s, lv, in, buf, tw, part);
      case COL_SETUP: return col_fwd_go<T, COL_SETUP>(grid, s, lv, in, buf, tw, part);
      default: break;
    }
  }
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_row(int spectral, const LevelDev<T>& lv, cplx<T>* buf, const Twiddles<T>& tw,
                      const T* part, int npart, const T* xin, hipStream_t s) {
  if (lv.logL2 < 1) return hipErrorInvalidValue;
  const int pairs = (1 << lv.logL2) / 2;
  if (spectral && lv.sym)
    return row_go<T, true, true>(pairs + 1, s, lv, buf, tw, part, npart, xin);
  if (spectral) return row_go<T, true, false>(pairs + 1, s, lv, buf, tw, part, npart, xin);
  if constexpr (sizeof(T) == 8)
    return row_go<T, false, false>(pairs, s, lv, buf, tw, part, npart, xin);
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_col_inv(int mode, const LevelDev<T>& lv, const EpiOut<T>& out,
                          const cplx<T>* buf, const Twiddles<T>& tw, double* part,
                          hipStream_t s) {
  if (!epi_mode_built<T>(mode)) return hipErrorInvalidValue;
  const int grid = col_blocks(lv.logL1, lv.tcols);
  switch (mode) {
    case EPI_MV: return col_inv_go<T, EPI_MV>(grid, s, lv, out, buf, tw, part);
    case EPI_RESID: return col_inv_go<T, EPI_RESID>(grid, s, lv, out, buf, tw, part);
    case EPI_SMOOTH: return col_inv_go<T, EPI_SMOOTH>(grid, s, lv, out, buf, tw, part);
    default: break;
  }
  if constexpr (sizeof(T) == 8) {
    if (mode == EPI_OUTER) return col_inv_go<T, EPI_OUTER>(grid, s, lv, out, buf, tw, part);
  }
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Batched launches: `count` instances of one level geometry (the geometry of
// `geom`; each instance's own arguments in the device table `args`), block
// row y = instance y.  Same kernels bodies, same per-instance arithmetic.
// ---------------------------------------------------------------------------
template <typename T>
hipError_t launch_col_fwd_batch(int mode, const LevelDev<T>& geom, const PassArgs<T>* args,
                                int count, const Twiddles<T>& tw, hipStream_t s) {
  if (count < 1 || count > 65535 || !col_mode_built<T>(mode)) return hipErrorInvalidValue;
  const dim3 grid(col_blocks(geom.logL1, geom.tcols), count);
  auto go = [&](auto M) {
    constexpr int MODE = decltype(M)::value;
    return col_pick(geom.logL1, geom.logL2, geom.tcols, [&](auto g) {
      using G = decltype(g);
      return launch_lds(k_col_fwd_b<T, MODE, G>, grid, G::NT, sizeof(cplx<T>) * G::kLds, s, args,
                        tw);
    });
  };
  switch (mode) {
    case COL_MV: return go(IC<COL_MV>{});
    case COL_PRE: return go(IC<COL_PRE>{});
    case COL_PRE_RESTRICT: return go(IC<COL_PRE_RESTRICT>{});
    case COL_PROLONG: return go(IC<COL_PROLONG>{});
    default: break;
  }
  if constexpr (sizeof(T) == 8) {
    if (mode == COL_OUTER_UPDATE) return go(IC<COL_OUTER_UPDATE>{});
  }
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_row_batch(const LevelDev<T>& geom, const PassArgs<T>* args, int count,
                            const Twiddles<T>& tw, hipStream_t s) {
  if (count < 1 || count > 65535 || geom.logL2 < 1) return hipErrorInvalidValue;
  const dim3 grid((1 << geom.logL2) / 2 + 1, count);
  auto go = [&](auto SY) {
    constexpr bool SYM = decltype(SY)::value != 0;
    return row_pick(geom.logL1, [&](auto g) {
      constexpr int LOG1 = decltype(g)::value;
      return launch_lds(k_row_b<T, true, SYM, LOG1>, grid, row_nt(LOG1),
                        sizeof(cplx<T>) * row_lds(LOG1), s, args, tw);
    });
  };
  return geom.sym ? go(IC<1>{}) : go(IC<0>{});
}

template <typename T>
hipError_t launch_col_inv_batch(int mode, const LevelDev<T>& geom, const PassArgs<T>* args,
                                int count, const Twiddles<T>& tw, hipStream_t s) {
  if (count < 1 || count > 65535 || !epi_mode_built<T>(mode)) return hipErrorInvalidValue;
  const dim3 grid(col_blocks(geom.logL1, geom.tcols), count);
  auto go = [&](auto M) {
    constexpr int MODE = decltype(M)::value;
    return col_pick(geom.logL1, geom.logL2, geom.tcols, [&](auto g) {
      using G = decltype(g);
      return launch_lds(k_col_inv_b<T, MODE, G>, grid, G::NT, sizeof(cplx<T>) * G::kLds, s, args,
                        tw);
    });
  };
  switch (mode) {
    case EPI_MV: return go(IC<EPI_MV>{});
    case EPI_RESID: return go(IC<EPI_RESID>{});
    case EPI_SMOOTH: return go(IC<EPI_SMOOTH>{});
    default: break;
  }
  if constexpr (sizeof(T) == 8) {
    if (mode == EPI_OUTER) return go(IC<EPI_OUTER>{});
  }
  return hipErrorInvalidValue;
}

}  // namespace amg
