// HIP kernels of the block-structured V-cycle (Algorithm 2) with FFT-based
// Toeplitz-plus-Cross matrix-vector products (Sec. 3.2, eq. (ccs3.4),
// eq. (split01)) for gfx950.
//
// Each level's matvec works on the packed complex signal z = v + i w_bar
// (zero-padded to L = 2(n+1)); one complex FFT replaces the two real ones,
// and the 2x2 block product becomes, bin by bin,
//     Y[f] = G1[f] Z[f] + G2[f] conj(Z[-f]),
//     G1 = (A^ + D^ + i(C^ - B^))/2,  G2 = (A^ - D^ + i(C^ + B^))/2,
// with A^..D^ the spectra of the four circulant embeddings.  The inverse FFT
// of Y gives A v + B_bar w_bar in its real part and C_bar v + D_bar w_bar in
// its imaginary part.  Large levels run the FFT as a four-step transform in
// three HBM passes (column FFTs, row FFT + spectral product + inverse row FFT,
// inverse column FFTs) with the vector formation (smoothing, restriction,
// prolongation, refinement update) fused into the first pass and the residual
// / Jacobi epilogue fused into the last.  Small levels run the whole V-cycle
// below them in one workgroup with the FFT and its twiddles in LDS.
#include "kernel_common.hpp"

#include <algorithm>
#include <type_traits>

namespace amg {

// ---------------------------------------------------------------------------
// Tail levels: L <= 2^12, one workgroup of 512 threads, FFT and twiddles in LDS.
// ---------------------------------------------------------------------------
// One compute unit runs a whole cycle here, so latency bounds it: every step
// is a chain of loads, the FFT's LDS exchanges and the epilogue.  Thread
// j0 < L/8 holds the elements j0 + e L/8 of a level in registers from the
// prologue through both FFTs to the epilogue (fft8: five LDS exchanges with
// the partner bins' at L = 512, seven above, against eleven and thirteen when
// every pass went through LDS), and what one step hands to the next (a
// residual to restrict, a correction to prolong) stays in LDS.  Kernel time per
// V-cycle: FP32 from L = 2^12 77 -> 55 us, FP64 from L = 2^11 62 -> 42 us; an
// FP64 product with L = 2^9 6.7 -> 3.7 us, a residual with L = 2^11 11.4 ->
// 8.3 us.
//
// Dynamic LDS starts after a kernel's static LDS; it is declared 16-byte
// aligned so that the complex FP64 accesses (16-byte LDS instructions) stay
// aligned whatever the static variables add up to (an 8-byte offset made the
// FP64 FFT passes 3.5 times slower).
constexpr int kTailZ = 2 * kFft8Half;  // FFT slots: one signal of 2^12 or two of 2^11
constexpr int kTailRed = kNTT / 64 + 2;  // wave partials, w_o
template <typename T>
struct TailLds {
  Lds<T> z;     // kTailZ complex
  cplx<T>* tw;  // kTailTw twiddles e^{-2 pi i m / 2^kTailLog}
  T* x;         // a level vector between steps (2^kTailLog)
  T* red;       // kTailRed
};

template <typename T>
__device__ __forceinline__ TailLds<T> tail_lds(unsigned char* smem) {
  TailLds<T> s;
  s.z.p = reinterpret_cast<cplx<T>*>(smem);
  s.tw = s.z.p + kTailZ;
  s.x = reinterpret_cast<T*>(s.tw + kTailTw);
  s.red = s.x + (1 << kTailLog);
  return s;
}
constexpr size_t tail_lds_bytes(size_t elem) {
  return elem * (2 * (size_t)(kTailZ + kTailTw) + (1 << kTailLog) + kTailRed);
}
// A single product's LDS: the FFT slots and the partials (no table, no vector).
constexpr size_t tail_mv_lds_bytes(size_t elem, int logL) {
  return elem * (2 * (size_t)(logL <= 9 ? lds_slots(512) : kTailZ) + kTailRed);
}

// The level descriptors a tail call visits, copied to LDS once at kernel start
// (one round trip instead of a dependent scalar load at every step), and read
// back as wave-uniform values so that their pointers stay scalar.
template <typename T>
__device__ __forceinline__ void tail_levels_to_lds(const LevelDev<T>* levels, int first, int last,
                                                   LevelDev<T>* lvs) {
  static_assert(sizeof(LevelDev<T>) % 4 == 0, "descriptor copied as 32-bit words");
  constexpr int W = sizeof(LevelDev<T>) / 4;
  const int total = (last - first + 1) * W;
  const unsigned* src = reinterpret_cast<const unsigned*>(levels + first);
  unsigned* dst = reinterpret_cast<unsigned*>(lvs);
  for (int i = threadIdx.x; i < total; i += kNTT) dst[i] = src[i];
}
// (Pointers are rebuilt through the global address space so that accesses
// through them compile to global, not flat, memory instructions.)
template <typename T>
__device__ __forceinline__ T* ptr_uniform(T* p) {
  const unsigned long long v = reinterpret_cast<unsigned long long>(p);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
  using G = __attribute__((address_space(1))) T;
  return (T*)(G*)(((unsigned long long)hi << 32) | lo);
}
template <typename T>
__device__ __forceinline__ T val_uniform(T x) {
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)));
  } else {
    const unsigned long long v = __builtin_bit_cast(unsigned long long, x);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
    return __builtin_bit_cast(T, ((unsigned long long)hi << 32) | lo);
  }
}
template <typename T>
__device__ __forceinline__ LevelDev<T> lv_uniform(const LevelDev<T>& x) {
  LevelDev<T> o;
  o.n = __builtin_amdgcn_readfirstlane(x.n);
  o.logL = __builtin_amdgcn_readfirstlane(x.logL);
  o.logL1 = __builtin_amdgcn_readfirstlane(x.logL1);
  o.logL2 = __builtin_amdgcn_readfirstlane(x.logL2);
  o.tcols = __builtin_amdgcn_readfirstlane(x.tcols);
  o.sym = __builtin_amdgcn_readfirstlane(x.sym);
  o.g1 = ptr_uniform(x.g1);
  o.g2 = ptr_uniform(x.g2);
  o.p = ptr_uniform(x.p);
  o.q = ptr_uniform(x.q);
  o.xi = ptr_uniform(x.xi);
  o.zeta = ptr_uniform(x.zeta);
  o.o = val_uniform(x.o);
  o.dv = val_uniform(x.dv);
  o.dw = val_uniform(x.dw);
  o.b = ptr_uniform(x.b);
  o.u = ptr_uniform(x.u);
  o.r = ptr_uniform(x.r);
  o.scal = ptr_uniform(x.scal);
  o.bsub = ptr_uniform(x.bsub);
  o.bmain = ptr_uniform(x.bmain);
  o.bsup = ptr_uniform(x.bsup);
  o.dinv = ptr_uniform(x.dinv);
  o.bc = ptr_uniform(x.bc);
  return o;
}

// The damped inverse diagonals of a call's levels, formed once in parallel at
// kernel start (a division costs tens of dependent instructions per step).
template <typename T>
struct TailDamp {
  T wv[2], ww[2];  // w / dv, w / dw for the pre- and post-smoothing factor
  T io;            // 1 / o
};
template <typename T>
__device__ __forceinline__ void tail_damp_to_lds(const LevelDev<T>* levels, int first, int last,
                                                 T wpre, T wpost, TailDamp<T>* damp) {
  const int t = kNTT - 1 - (int)threadIdx.x;  // the last wave: the others copy
  if (t >= 0 && t <= last - first) {
    const LevelDev<T>* lv = levels + first + t;
    const T dv = lv->dv, dw = lv->dw;
    damp[t] = {{wpre / dv, wpost / dv}, {wpre / dw, wpost / dw}, T(1) / lv->o};
  }
}

// Spectra at the thread's bins j0 + e L/8.
template <typename T, bool SYM>
struct TailSpec {
  using G = std::conditional_t<SYM, T, cplx<T>>;
  G g1[8], g2[8];
};
template <typename T, bool SYM>
__device__ __forceinline__ void tail_spec_load(const LevelDev<T>& lv, int j0, int q,
                                               TailSpec<T, SYM>& sp) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int f = j0 + (e << q);
    if constexpr (SYM) {
      sp.g1[e] = lv.g1[f];
      sp.g2[e] = lv.g2[f];
    } else {
      sp.g1[e] = ldg(reinterpret_cast<const cplx<T>*>(lv.g1) + f);
      sp.g2[e] = ldg(reinterpret_cast<const cplx<T>*>(lv.g2) + f);
    }
  }
}

// a holds the packed input at the thread's elements; leaves conj(y_v + i y_w)
// (without the Cross terms) there: the inverse transform is conj(F(conj Y)).
// Called by the whole workgroup, or by its first wavefront where that holds
// the signal (LOGL <= 9; 0: L <= 256 at run time).
// mid runs between the transforms, where the caller loads what its epilogue
// needs and finishes the w_o row's partial sum.
template <typename T, bool SYM, int LOGL, typename TW, typename F>
__device__ __forceinline__ void tail_fft_spectral(cplx<T> (&a)[8], Lds<T> z, int logLr, int j0,
                                                  bool act, const TailSpec<T, SYM>& sp,
                                                  const TW& tw, F&& mid) {
  constexpr bool kWave = LOGL <= 9;
  constexpr bool kPing = LOGL == 10 || LOGL == 11;
  const int logL = LOGL ? LOGL : logLr;
  const int L = 1 << logL, q = logL - 3;
  fft8<T, LOGL>(a, z, logLr, j0, act, tw);
  const Lds<T> ex{z.p + (kPing ? kFft8Half : 0)};
  if constexpr (!kPing && !kWave) __syncthreads();
  if (act) {
    const int sj = lds_slot(j0);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if constexpr (LOGL != 0) ex.p[sj + e * lds_step(q)] = a[e];
      else ex[j0 + (e << q)] = a[e];
    }
  }
  mid();
  fft_sync<kWave>();
  if (act) {
    // slot of bin L - j0 - 7 2^q; bin 0 is its own partner
    const int sr = lds_slot(L - j0) - 7 * lds_step(q);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      cplx<T> zp;
      if constexpr (LOGL == 0) zp = ex[(L - j0 - (e << q)) & (L - 1)];
      else if (e == 0) zp = ex.p[j0 == 0 ? 0 : sr + 7 * lds_step(q)];
      else zp = ex.p[sr + (7 - e) * lds_step(q)];
      if constexpr (SYM) {  // G1 real, G2 = i g2
        a[e] = {sp.g1[e] * a[e].x + sp.g2[e] * zp.y, -(sp.g1[e] * a[e].y + sp.g2[e] * zp.x)};
      } else {
        a[e] = conj(cmul(sp.g1[e], a[e]) + cmul(sp.g2[e], conj(zp)));
      }
    }
  }
  if constexpr (!kPing) fft_sync<kWave>();
  fft8<T, LOGL>(a, z, logLr, j0, act, tw);
}

// One matvec step of a tail level: form u (prologue), y = A u, then the
// residual or Jacobi epilogue.  The prologue's source is the LDS vector the
// previous step left (src null) or, for a restriction at the call's first
// level, the fine residual src in memory.  b and u stay in memory between
// a level's steps; the same thread writes and reads them.  The result goes
// to the LDS vector and, for a smoothing step, to u.  wv, ww, io: w / dv,
// w / dw, 1 / o.
template <typename T, bool BAND, bool SYM, int LOGL, typename F>
__device__ __forceinline__ void tail_step(const LevelDev<T>& lv, int pro, int epi, const T* src,
                                          T w, T wv, T ww, T io, const TailLds<T>& s, F&& idle) {
  constexpr bool kWave = LOGL <= 9;
  constexpr int J = 4;  // owned elements j < n (the packed signal's upper half is zero)
  const int logL = LOGL ? LOGL : lv.logL;
  const int L = 1 << logL, n = L / 2 - 1, q = logL - 3;
  const int j0 = opaque((int)threadIdx.x);  // (not hoisted out of the step loop)
  const bool act = j0 < L / 8;
  const bool restr = pro == TP_PRE_RESTRICT, prol = pro == TP_PROLONG;
  // the thread's elements j0 + e L/8, e < 4, all lie in the level but for the
  // last thread's last
  auto in = [&](int e) { return (LOGL != 0 && e < J - 1) || j0 + (e << q) < n; };
  T pj[J], xj[J], qq[J], zz[J], bv[J], bw[J], uv[J], uw[J], dv0[J], dv1[J];
  int js[J];
  T bo = T(0), uo = T(0), dio = io;
  TailSpec<T, SYM> sp;
  const FftTab8<T> tw{s.tw, kTailLog};
  if (act) {
#pragma unroll
    for (int e = 0; e < J; ++e) js[e] = in(e) ? j0 + (e << q) : 0;
    // loads in the order of their use: the iterate, the spectra, the rest
    if (prol || pro == TP_USE_U) {
#pragma unroll
      for (int e = 0; e < J; ++e) {
        uv[e] = lv.u[js[e]];
        uw[e] = lv.u[n + 1 + js[e]];
      }
      if (j0 == 0) uo = lv.u[n];
    }
    auto restrict_from = [&](const T* r) {
#pragma unroll
      for (int e = 0; e < J; ++e) {
        bv[e] = restrict_at(r, js[e]);
        bw[e] = restrict_at(r, n + 1 + js[e]);
      }
      if (j0 == 0) bo = restrict_at(r, n);
    };
    auto b_load = [&] {
#pragma unroll
      for (int e = 0; e < J; ++e) {
        bv[e] = lv.b[js[e]];
        bw[e] = lv.b[n + 1 + js[e]];
      }
      if (j0 == 0) bo = lv.b[n];
    };
    if (restr && src) restrict_from(src);
    if (pro == TP_PRE_B) b_load();
    if constexpr (BAND) {
#pragma unroll
      for (int e = 0; e < J; ++e) {
        dv0[e] = lv.dinv[js[e]];
        dv1[e] = lv.dinv[n + 1 + js[e]];
      }
      if (j0 == 0) dio = lv.dinv[n];
    }
    tail_spec_load<T, SYM>(lv, j0, q, sp);
#pragma unroll
    for (int e = 0; e < J; ++e) {
      qq[e] = lv.q[js[e]];
      zz[e] = lv.zeta[js[e]];
    }
    if (prol || pro == TP_USE_U) b_load();
    if (restr && !src) restrict_from(s.x);
    if (prol) {
#pragma unroll
      for (int e = 0; e < J; ++e) {
        uv[e] += prolong_at(s.x, n, js[e]);
        uw[e] += prolong_at(s.x, n, n + 1 + js[e]);
      }
      if (j0 == 0) uo += prolong_at(s.x, n, n);
    } else if (pro != TP_USE_U) {  // from zero: u = w D^{-1} b
#pragma unroll
      for (int e = 0; e < J; ++e) {
        uv[e] = (BAND ? w * dv0[e] : wv) * bv[e];
        uw[e] = (BAND ? w * dv1[e] : ww) * bw[e];
      }
      uo = w * bo * dio;
    }
#pragma unroll
    for (int e = 0; e < J; ++e) {
      const int j = j0 + (e << q), jw = n + 1 + j;
      if (in(e)) {
        if (restr) {
          lv.b[j] = bv[e];
          lv.b[jw] = bw[e];
        }
        if (epi == TE_RESID && pro != TP_USE_U) {
          lv.u[j] = uv[e];
          lv.u[jw] = uw[e];
        }
      } else {
        uv[e] = uw[e] = T(0);
      }
    }
    if (j0 == 0) {
      if (restr) lv.b[n] = bo;
      if (epi == TE_RESID && pro != TP_USE_U) lv.u[n] = uo;
      s.red[kNTT / 64] = uo;
    }
  }
  if constexpr (BAND) {  // u beside its neighbours, for the band's product
    __syncthreads();     // the prologue's reads of s.x are done
    if (act) {
#pragma unroll
      for (int e = 0; e < J; ++e) {
        const int j = j0 + (e << q);
        if (in(e)) {
          s.x[j] = uv[e];
          s.x[n + 1 + j] = uw[e];
        }
      }
      if (j0 == 0) s.x[n] = uo;
    }
    __syncthreads();
  }
  cplx<T> a[8];
  if (!kWave || j0 < 64) {
#pragma unroll
    for (int e = 0; e < J; ++e) {
      a[e] = {uv[e], uw[e]};
      a[e + J] = {T(0), T(0)};
    }
    tail_fft_spectral<T, SYM, LOGL>(a, s.z, logL, j0, act, sp, tw, [&] {
      T dot = T(0);  // inactive threads add zero
      if (act) {
#pragma unroll
        for (int e = 0; e < J; ++e) {
          dot += qq[e] * uv[e] + zz[e] * uw[e];
          pj[e] = lv.p[js[e]];
          xj[e] = lv.xi[js[e]];
        }
      }
      dot = wave_sum63(dot);
      if ((j0 & 63) == 63) s.red[j0 >> 6] = dot;
    });
  } else {
    idle();
  }
  T nv[J], nw[J], no = T(0);
  // The band's entries, loaded in one batch, and (B u)_i from them, u in s.x.  Each
  // behind a test of its own waited for the one before: a W-cycle of N = 2^13
  // 1.07 -> 1.00 ms, the set-up that forms its bottom 156 -> 130 ms (FP64).
  // Fetched between the transforms they would spill.
  T bm[2 * J + 1], bl[2 * J + 1], bu[2 * J + 1];
  auto band_load = [&](int k, int i) {
    bm[k] = lv.bmain[i];
    bl[k] = lv.bsub[i];
    bu[k] = lv.bsup[i];
  };
  auto bandu = [&](int k, int i) {
    const T y0 = bm[k] * s.x[i], y1 = __builtin_elementwise_fma(bl[k], s.x[i > 0 ? i - 1 : 0], y0);
    const T y2 = i > 0 ? y1 : y0;
    const T y3 = __builtin_elementwise_fma(bu[k], s.x[i < 2 * n ? i + 1 : i], y2);
    return i < 2 * n ? y3 : y2;
  };
  if (act) {
    const T uof = s.red[kNTT / 64];
    if constexpr (BAND) {
#pragma unroll
      for (int e = 0; e < J; ++e) {
        band_load(e, js[e]);
        band_load(J + e, n + 1 + js[e]);
      }
      if (j0 == 0) band_load(2 * J, n);
    }
#pragma unroll
    for (int e = 0; e < J; ++e) {
      T yv = a[e].x + pj[e] * uof, yw = xj[e] * uof - a[e].y;
      if constexpr (BAND) {
        yv += bandu(e, js[e]);
        yw += bandu(J + e, n + 1 + js[e]);
      }
      const T rv = bv[e] - yv, rw = bw[e] - yw;
      nv[e] = epi == TE_RESID ? rv : uv[e] + (BAND ? w * dv0[e] : wv) * rv;
      nw[e] = epi == TE_RESID ? rw : uw[e] + (BAND ? w * dv1[e] : ww) * rw;
    }
    if (j0 == 0) {
      T yo = lv.o * uo;
      for (int k = 0; k < (L / 8 + 63) / 64; ++k) yo += s.red[k];
      if constexpr (BAND) yo += bandu(2 * J, n);
      no = epi == TE_RESID ? bo - yo : uo + w * (bo - yo) * dio;
    }
  }
  if constexpr (BAND) __syncthreads();  // the band's reads of s.x are done
  if (act) {
#pragma unroll
    for (int e = 0; e < J; ++e) {
      const int j = j0 + (e << q), jw = n + 1 + j;
      if (in(e)) {
        s.x[j] = nv[e];
        s.x[jw] = nw[e];
        if (epi == TE_SMOOTH) {
          lv.u[j] = nv[e];
          lv.u[jw] = nw[e];
        }
      }
    }
    if (j0 == 0) {
      s.x[n] = no;
      if (epi == TE_SMOOTH) lv.u[n] = no;
    }
  }
  __syncthreads();  // s.x published; z and red reusable
}

// The step in the level's geometry: the sizes a tail mostly visits with it as
// compile-time constants.  idle: run by the wavefronts that have no part in a
// level of one wavefront.
template <typename T, bool BAND, bool SYM, typename F>
__device__ __forceinline__ void tail_step_any(const LevelDev<T>& lv, int pro, int epi,
                                              const T* src, T w, T wv, T ww, T io,
                                              const TailLds<T>& s, F&& idle) {
  switch (lv.logL) {
    case 12: tail_step<T, BAND, SYM, 12>(lv, pro, epi, src, w, wv, ww, io, s, idle); break;
    case 11: tail_step<T, BAND, SYM, 11>(lv, pro, epi, src, w, wv, ww, io, s, idle); break;
    case 10: tail_step<T, BAND, SYM, 10>(lv, pro, epi, src, w, wv, ww, io, s, idle); break;
    case 9: tail_step<T, BAND, SYM, 9>(lv, pro, epi, src, w, wv, ww, io, s, idle); break;
    default: tail_step<T, BAND, SYM, 0>(lv, pro, epi, src, w, wv, ww, io, s, idle); break;
  }
}

// Coarsest level: u = A_c^{-1} b with the inverse formed at setup from the
// LU factors (partial pivoting), or the matrix of a folded sub-cycle (CoarseLU).
// b (in LDS, FP64) is restricted from the previous step's residual; u goes to
// the LDS vector and to memory.  A thread holds R = 16 / sizeof(M) neighbouring
// rows and one of P parts of the columns, which it sums in ascending order; the
// partial sums are added in part order through LDS.  One compute unit bounds
// it: it loads 57..62 B per clock in 16-byte pieces but only 30 in 8-byte ones
// (m = 255: 1.9 us in FP32, 3.6 us in FP64), so every load is 16 bytes wide and
// four to eight of them are in flight while the previous four are summed.  One
// row to a thread, loaded eight columns at a time and the rest one by one, took
// 5.2 us in FP32 and 8.0 us in FP64; now 3.0 and 4.4.  The FP32 V-cycle
// reads the matrix's FP32 rounding when there is one.
template <typename M>
__device__ __forceinline__ void coarse_rows(const M* a, const double* bk, int ld, int at, int cp,
                                            double (&acc)[16 / sizeof(M)]) {
  constexpr int R = 16 / sizeof(M), kU = 4;  // cp is a multiple of 8
  using V = M __attribute__((ext_vector_type(R)));
  V v0[kU], v1[kU], v2[kU];
  auto load = [&](V (&v)[kU], int c0) {
    if (c0 < cp) {
      const M* ac = a + (int64_t)c0 * ld;
#pragma unroll
      for (int c = 0; c < kU; ++c) v[c] = *reinterpret_cast<const V*>(ac + (int64_t)c * ld + at);
    }
  };
  auto sum = [&](const V (&v)[kU], int c0) {
#pragma unroll
    for (int c = 0; c < kU; ++c) {
      const double b = bk[c0 + c];
#pragma unroll
      for (int r = 0; r < R; ++r) acc[r] += (double)v[c][r] * b;
    }
  };
  load(v0, 0);
  load(v1, kU);
  for (int c0 = 0;;) {
    load(v2, c0 + 2 * kU);
    sum(v0, c0);
    if ((c0 += kU) >= cp) break;
    load(v0, c0 + 2 * kU);
    sum(v1, c0);
    if ((c0 += kU) >= cp) break;
    load(v1, c0 + 2 * kU);
    sum(v2, c0);
    if ((c0 += kU) >= cp) break;
  }
}
template <typename T, typename M>
__device__ __forceinline__ void coarse_apply(const M* a, int m, T* u, T* x, double* bs) {
  constexpr int R = 16 / sizeof(M);
  const int ld = m + 1;  // a power of two, at least 8
  const int P = min(min(8, ld / 8), kNTT * R / ld), cp = ld / P;
  double* part = bs + ld;  // P * ld partial sums
  const int g = threadIdx.x & (ld / R - 1), k = threadIdx.x / (ld / R);
  if (k < P) {
    double acc[R] = {};
    coarse_rows(a, bs + k * cp, ld, k * cp * ld + g * R, cp, acc);
#pragma unroll
    for (int r = 0; r < R; ++r) part[k * ld + g * R + r] = acc[r];
  }
  __syncthreads();
  for (int r = threadIdx.x; r < m; r += kNTT) {
    double acc = part[r];
    for (int c = 1; c < P; ++c) acc += part[c * ld + r];
    x[r] = u[r] = (T)acc;
  }
}
// src: the fine residual in memory (the call's only level); else the LDS
// vector, or the level's b where `own` is set (no finer level).
template <typename T>
__device__ __forceinline__ void coarse_solve(const CoarseLU& lu, const LevelDev<T>& lc,
                                             const T* src, bool own, const TailLds<T>& s) {
  double* bs = reinterpret_cast<double*>(s.z.p);
  for (int i = threadIdx.x; i < lu.m; i += kNTT)
    bs[i] = (double)(own ? lc.b[i] : (src ? restrict_at(src, i) : restrict_at(s.x, i)));
  if (threadIdx.x == 0) bs[lu.m] = 0.0;
  __syncthreads();
  bool done = false;
  if constexpr (sizeof(T) == 4) {
    if (lu.ainv32) {
      coarse_apply(lu.ainv32, lu.m, lc.u, s.x, bs);
      done = true;
    }
  }
  if (!done) coarse_apply(lu.ainv, lu.m, lc.u, s.x, bs);
  __syncthreads();
}

// Pulls the matrix coarse_solve will read into this XCD's L2 (the large levels
// have evicted it since the previous cycle; a folded sub-cycle's matrix is up
// to 2 MB): one word per 128-byte line, by the threads t of nt, in batches of 8
// lines per thread with clamped addresses, folded into one value that is
// stored only if it equals a constant, so that the loads stay live.  The
// wavefronts that the step before the solve leaves idle do it (at kernel
// start it delayed the first step by 1 us).
template <typename T>
__device__ __forceinline__ void coarse_warm(const CoarseLU& lu, int t, int nt, T* sink) {
  const char* p = reinterpret_cast<const char*>(lu.ainv);
  long bytes = (long)lu.m * lu.m * 8;
  if constexpr (sizeof(T) == 4) {
    if (lu.ainv32) {
      p = reinterpret_cast<const char*>(lu.ainv32);
      bytes = (long)lu.m * lu.m * 4;
    }
  }
  constexpr int K = 8;
  const long batch = (long)K * nt * 128;  // bytes covered per batch
  unsigned acc = 0;
  for (long base = 0; base < bytes; base += batch) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      long off = base + ((long)t + (long)k * nt) * 128;
      off = off < bytes ? off : bytes - 4;
      acc ^= *reinterpret_cast<const unsigned*>(p + off);
    }
  }
  if (acc == 0x5bd1e995u) sink[0] = T(0);
}

// What a cycle or step-program kernel sets up before its steps: the level
// descriptors, the damping factors and the twiddle table in LDS.
template <typename T>
__device__ __forceinline__ TailLds<T> tail_begin(unsigned char* smem, const LevelDev<T>* levels,
                                                 int first, int last, T wpre, T wpost,
                                                 const Twiddles<T>& tw, LevelDev<T>* lvs,
                                                 TailDamp<T>* damp) {
  const TailLds<T> s = tail_lds<T>(smem);
  tail_damp_to_lds(levels, first, last, wpre, wpost, damp);
  tail_levels_to_lds(levels, first, last, lvs);
  cplx<T> t[kTailTw / kNTT];
#pragma unroll
  for (int k = 0; k < kTailTw / kNTT; ++k) t[k] = ldg(tw.tail + threadIdx.x + k * kNTT);
#pragma unroll
  for (int k = 0; k < kTailTw / kNTT; ++k) s.tw[threadIdx.x + k * kNTT] = t[k];
  __syncthreads();
  return s;
}

template <typename T, bool BAND, bool SYM>
__device__ __forceinline__ void tail_vcycle_body(const LevelDev<T>* levels, int first, int last,
                                                 const T* rf, int m1, int m2, T wpre, T wpost,
                                                 const CoarseLU& lu, const Twiddles<T>& tw) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  __shared__ LevelDev<T> lvs[kTailMaxLev];
  __shared__ TailDamp<T> damp[kTailMaxLev];
  __shared__ T warm_sink;
  const TailLds<T> s = tail_begin<T>(smem_raw, levels, first, last, wpre, wpost, tw, lvs, damp);
  // One loop over the V-cycle's matvec steps (a single inlined tail_step per
  // geometry): descend (level first..last-1, m1 sweeps each, residual on the
  // last one), the coarsest solve, then ascend (prolongation + m2 post-sweeps).
  bool up = false;
  for (int l = first, sweep = 0;;) {
    if (!up && l == last) {  // coarsest level: b = R r_fine, exact solve by LU
      const bool only = last == first;
      coarse_solve<T>(lu, lv_uniform(lvs[last - first]), only ? rf : nullptr, only && !rf, s);
      up = true;
      sweep = 0;
      if (--l < first) break;
    }
    int pro = TP_USE_U, epi = TE_SMOOTH;
    if (sweep == 0) pro = up ? TP_PROLONG : (l == first && !rf ? TP_PRE_B : TP_PRE_RESTRICT);
    if (!up && sweep == m1 - 1) epi = TE_RESID;
    const TailDamp<T>& d = damp[l - first];
    const bool warm = l == last - 1 && epi == TE_RESID;  // the coarsest solve is next
    tail_step_any<T, BAND, SYM>(
        lv_uniform(lvs[l - first]), pro, epi, l == first ? rf : nullptr, up ? wpost : wpre,
        val_uniform(d.wv[up]), val_uniform(d.ww[up]), val_uniform(d.io), s, [&] {
          if (warm) coarse_warm<T>(lu, (int)threadIdx.x - 64, kNTT - 64, &warm_sink);
        });
    if (++sweep < (up ? m2 : m1)) continue;
    sweep = 0;
    if (!up) ++l;
    else if (--l < first) break;
  }
}

template <typename T, bool BAND, bool SYM>
__global__ __launch_bounds__(kNTT) __attribute__((amdgpu_waves_per_eu(2)))
void k_tail_vcycle(const LevelDev<T>* levels, int first, int last, const T* rf, int m1, int m2,
                   T wpre, T wpost, CoarseLU lu, Twiddles<T> tw) {
  tail_vcycle_body<T, BAND, SYM>(levels, first, last, rf, m1, m2, wpre, wpost, lu, tw);
}
// One block per instance: the small levels of a batch of handles in one launch.
// FP32: at most 128 registers, so that two instances share a CU (71 KB of LDS
// each); an FP64 one has it to itself (138 KB).
template <typename T, bool BAND, bool SYM>
__global__ __launch_bounds__(kNTT) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 && !BAND ? 4 : 2)))
void k_tail_vcycle_b(const TailArgs<T>* __restrict__ args, Twiddles<T> tw) {
  const TailArgs<T>* a = args + blockIdx.x;
  if (gate_skip(a->st, a->gate)) return;
  const CoarseLU lu = a->lu;
  tail_vcycle_body<T, BAND, SYM>(a->levels, a->first, a->last, a->rf, a->m1, a->m2, a->wpre,
                                 a->wpost, lu, tw);
}

// A cycle's small-level part as a program of steps built on the host (the
// W-cycle: the second visit of a level smooths from its current iterate and
// recomputes the residual; see TailOp).  A restriction or prolongation
// follows the step that left its source in LDS, as in the V-cycle.
template <typename T, bool BAND, bool SYM>
__global__ __launch_bounds__(kNTT) __attribute__((amdgpu_waves_per_eu(2)))
void k_tail_program(const LevelDev<T>* levels, int first, int last, const T* rf,
                    const TailOp* ops, int nops, T wpre, T wpost, CoarseLU lu, Twiddles<T> tw) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  __shared__ LevelDev<T> lvs[kTailMaxLev];
  __shared__ TailDamp<T> damp[kTailMaxLev];
  __shared__ T warm_sink;
  const TailLds<T> s = tail_begin<T>(smem_raw, levels, first, last, wpre, wpost, tw, lvs, damp);
  coarse_warm<T>(lu, threadIdx.x, kNTT, &warm_sink);
  for (int k = 0; k < nops; ++k) {
    const TailOp op = ops[k];
    if (op.flags & TAILOP_COARSE) {  // coarsest level: b = R r_fine, exact solve
      const bool only = last == first;
      coarse_solve<T>(lu, lv_uniform(lvs[last - first]), only ? rf : nullptr, only && !rf, s);
      continue;
    }
    const int l = op.level;
    const bool up = (op.flags & TAILOP_UP) != 0;
    const TailDamp<T>& d = damp[l - first];
    tail_step_any<T, BAND, SYM>(
        lv_uniform(lvs[l - first]), op.pro, op.epi, l == first ? rf : nullptr, up ? wpost : wpre,
        val_uniform(d.wv[up]), val_uniform(d.ww[up]), val_uniform(d.io), s, [] {});
  }
}

// Stopping test of the outer iteration (Sec. 5): ||r_i|| / ||r_0|| < tol.
__device__ void finish_state(SolveState* st, double s, double tol, int max_iter, double* hist,
                             int verify) {
  if (st->done) return;
  const double nrm = sqrt(s);
  if (st->iter == 0) {
    st->r0 = nrm;
    st->best = 1.0;
  }
  const double rel = (st->r0 > 0.0) ? nrm / st->r0 : 0.0;
  st->relres = rel;
  hist[st->iter] = rel;
  if (!(rel == rel) || isinf(rel)) {
    st->status = 2;
    st->done = 1;
  } else if (rel < tol) {
    if (verify) {  // a recurrence's residual: b - A x decides (gm_check_state)
      st->cycle_end = 1;
    } else {
      st->status = 0;
      st->done = 1;
    }
  } else if (rel > 1e3 * st->best) {
    st->status = 2;
    st->done = 1;
  } else if (st->iter >= max_iter) {
    st->status = 1;
    st->done = 1;
  }
  if (rel < st->best) st->best = rel;
  if (!st->done && !st->cycle_end) st->iter += 1;
}
__device__ __forceinline__ void gm_check_state(SolveState* st, double v, double tol, int max_iter,
                                               double* hist, int stall) {
  if (st->done) return;
  const double rel = sqrt(v) / st->r0;
  st->relres = rel;
  hist[st->iter] = rel;
  st->cycle_end = 0;
  if (!(rel == rel) || isinf(rel)) {
    st->status = 2;
    st->done = 1;
  } else if (rel < tol) {
    st->status = 0;
    st->done = 1;
  } else if (st->iter >= max_iter || (stall && st->vtrue > 0.0 && rel >= 0.9 * st->vtrue)) {
    st->status = 1;
    st->done = 1;
  } else {
    st->iter += 1;
    // the next recurrence starts from this residual: the growth test of
    // finish_state measures from here (a Krylov method's 2-norm residual is
    // not monotone, and a restart can start above the recurrence's minimum)
    st->best = rel;
    st->cg_first = 1;  // CG restarts from it
  }
  st->vtrue = rel;
}

// One thread of a round's last kernel: the stop test of the residual's squared
// norm s.
__device__ __forceinline__ void stop_state(const StopTest& t, double s) {
  if (t.begin) {  // the solve's first stop test starts its state
    *t.st = SolveState{};
    t.st->cg_first = 1;
  }
  if (t.check) gm_check_state(t.st, s, t.tol, t.max_iter, t.hist, t.verify);
  else finish_state(t.st, s, t.tol, t.max_iter, t.hist, t.verify);
}
// The workgroup (at least a wavefront, past a barrier behind the state's last
// write): the state and the history entry the round wrote (iter, or iter - 1
// where it advanced it) into pinned host memory, by the kernel that made them
// - a kernel for it cost the round 5 us more.
__device__ __forceinline__ void publish_state(const SolveState* st, SolveState* host,
                                              const double* hist) {
  static_assert(sizeof(SolveState) % 4 == 0 && sizeof(SolveState) / 4 <= 64, "state words");
  if (!host) return;
  const int w = threadIdx.x, i = st->iter - w;
  if (w < 2 && i >= 0 && i < kHistHost) hist_host(host)[i] = hist[i];
  if (w < (int)(sizeof(SolveState) / 4))
    reinterpret_cast<unsigned*>(host)[w] = reinterpret_cast<const unsigned*>(st)[w];
  __threadfence_system();
}

// One tail-level matvec: y = A x (EPI_MV) or the outer residual with the
// refinement update fused in front (COL_OUTER_UPDATE + EPI_OUTER).  A single
// product: its twiddles come straight from memory beside the other operands
// (the whole LDS table cost 2 us of the 7 us of a product with L = 512).
template <typename T, int CM, int EM, bool SYM, int LOGL>
__device__ __forceinline__ void tail_matvec_geom(const LevelDev<T>& lv, const ColIn<T>& in,
                                                 const EpiOut<T>& out, const Twiddles<T>& tws,
                                                 double* part, const StopTest& stop) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  __shared__ double redd[kNTT / 64];
  constexpr bool kWave = LOGL <= 9;
  constexpr int J = 4;
  const int logL = LOGL ? LOGL : lv.logL;
  const int L = 1 << logL, n = L / 2 - 1, q = logL - 3;
  const Lds<T> z{reinterpret_cast<cplx<T>*>(smem_raw)};
  T* red = reinterpret_cast<T*>(smem_raw + tail_mv_lds_bytes(sizeof(T), logL)) - kTailRed;
  const int j0 = threadIdx.x;
  const bool act = j0 < L / 8;
  auto in_level = [&](int e) { return (LOGL != 0 && e < J - 1) || j0 + (e << q) < n; };
  const T* x = out.xin;
  TailSpec<T, SYM> sp;
  FftTw8<T> tw;
  T pj[J], xj[J], qq[J], zz[J], xv[J], xw[J];
  double bv[J], bw[J], bo = 0.0;
  T wo = T(0);
  int js[J];
  if (act) {
#pragma unroll
    for (int e = 0; e < J; ++e) {
      js[e] = in_level(e) ? j0 + (e << q) : 0;
      xv[e] = x[js[e]];
      xw[e] = x[n + 1 + js[e]];
    }
    wo = x[n];
    if constexpr (CM == COL_OUTER_UPDATE) {
      auto add = [&](const auto* c) {
#pragma unroll
        for (int e = 0; e < J; ++e) {
          xv[e] += (T)c[js[e]];
          xw[e] += (T)c[n + 1 + js[e]];
        }
        wo += (T)c[n];
      };
      if (in.e_is_float) add(static_cast<const float*>(in.e));
      else add(static_cast<const double*>(in.e));
    }
    tw.load(logL, j0, FftTab8<T>{tws.tail, kTailLog});
    tail_spec_load<T, SYM>(lv, j0, q, sp);
#pragma unroll
    for (int e = 0; e < J; ++e) {
      qq[e] = lv.q[js[e]];
      zz[e] = lv.zeta[js[e]];
      pj[e] = lv.p[js[e]];
      xj[e] = lv.xi[js[e]];
      if constexpr (EM == EPI_OUTER) {
        bv[e] = out.bo[js[e]];
        bw[e] = out.bo[n + 1 + js[e]];
      }
    }
    if (EM == EPI_OUTER && j0 == 0) bo = out.bo[n];
    if (!in_level(J - 1)) xv[J - 1] = xw[J - 1] = T(0);
    if constexpr (LOGL == 0) {
#pragma unroll
      for (int e = 0; e < J - 1; ++e)
        if (!in_level(e)) xv[e] = xw[e] = T(0);
    }
  }
  const bool band = lv.bmain != nullptr;  // weakly singular levels
  if constexpr (CM == COL_OUTER_UPDATE) {
    __syncthreads();  // every thread has read the old w_o
    if (act) {
#pragma unroll
      for (int e = 0; e < J; ++e) {
        if (in_level(e)) {
          in.xo[js[e]] = xv[e];
          in.xo[n + 1 + js[e]] = xw[e];
        }
      }
      if (j0 == 0) in.xo[n] = wo;
    }
    if (band) __syncthreads();  // the band reads its neighbours' new values
  }
  cplx<T> a[8];
  if (!kWave || j0 < 64) {
#pragma unroll
    for (int e = 0; e < J; ++e) {
      a[e] = {xv[e], xw[e]};
      a[e + J] = {T(0), T(0)};
    }
    tail_fft_spectral<T, SYM, LOGL>(a, z, logL, j0, act, sp, tw, [&] {
      T dot = T(0);  // inactive threads add zero
      if (act) {
#pragma unroll
        for (int e = 0; e < J; ++e) dot += qq[e] * xv[e] + zz[e] * xw[e];
      }
      dot = wave_sum63(dot);
      if ((j0 & 63) == 63) red[j0 >> 6] = dot;
    });
  }
  // band product of x (weakly singular levels) at index i of the block-ordered vector
  auto bandx = [&](int i) {
    T y = lv.bmain[i] * x[i];
    if (i > 0) y += lv.bsub[i] * x[i - 1];
    if (i < 2 * n) y += lv.bsup[i] * x[i + 1];
    return y;
  };
  double ss = 0.0;
  auto put = [&](int i, T y, double b) {
    if (band) y += bandx(i);
    if constexpr (EM == EPI_MV) {
      out.y[i] = y;
    } else {
      const double r = b - ((double)y + (out.ynear ? out.ynear[i] : 0.0));
      out.ro[i] = r;
      if (out.r32) out.r32[i] = (float)r;
      ss += r * r;
    }
  };
  if (act) {
#pragma unroll
    for (int e = 0; e < J; ++e) {
      if (in_level(e)) {
        put(js[e], a[e].x + pj[e] * wo, bv[e]);
        put(n + 1 + js[e], xj[e] * wo - a[e].y, bw[e]);
      }
    }
    if (j0 == 0) {
      T yo = lv.o * wo;
      for (int k = 0; k < (L / 8 + 63) / 64; ++k) yo += red[k];
      put(n, yo, bo);
    }
  }
  if constexpr (EM == EPI_OUTER) {
    ss = wave_sum63(ss);
    if ((j0 & 63) == 63) redd[j0 >> 6] = ss;
    __syncthreads();
    if (j0 == 0) {
      double sum = redd[0];
      for (int k = 1; k < kNTT / 64; ++k) sum += redd[k];
      part[0] = sum;
      if (stop.st) stop_state(stop, sum);
    }
    if (stop.st) {
      __syncthreads();  // thread 0's state writes before the copy
      publish_state(stop.st, stop.host, stop.hist);
    }
  }
}
template <typename T, int CM, int EM>
__device__ __forceinline__ void tail_matvec_body(const LevelDev<T>& lv, const ColIn<T>& in,
                                                 const EpiOut<T>& out, const Twiddles<T>& tw,
                                                 double* part, const StopTest& stop) {
  auto go = [&](auto sym) {
    constexpr bool SYM = decltype(sym)::value;
    switch (lv.logL) {
      case 12: tail_matvec_geom<T, CM, EM, SYM, 12>(lv, in, out, tw, part, stop); break;
      case 11: tail_matvec_geom<T, CM, EM, SYM, 11>(lv, in, out, tw, part, stop); break;
      case 10: tail_matvec_geom<T, CM, EM, SYM, 10>(lv, in, out, tw, part, stop); break;
      case 9: tail_matvec_geom<T, CM, EM, SYM, 9>(lv, in, out, tw, part, stop); break;
      default: tail_matvec_geom<T, CM, EM, SYM, 0>(lv, in, out, tw, part, stop); break;
    }
  };
  if (lv.sym) go(std::true_type{});
  else go(std::false_type{});
}

template <typename T, int CM, int EM>
__global__ __launch_bounds__(kNTT) __attribute__((amdgpu_waves_per_eu(2)))
void k_tail_matvec(LevelDev<T> lv, ColIn<T> in, EpiOut<T> out, Twiddles<T> tw, double* part) {
  tail_matvec_body<T, CM, EM>(lv, in, out, tw, part, StopTest{});
}
// The outer residual of a small finest level with the stop test behind it: the
// one workgroup has the whole norm.  As a kernel of its own the test took 4 of
// a round's 60 us at N = 2^10, and its start 1.7 more.
template <int CM>
__global__ __launch_bounds__(kNTT) __attribute__((amdgpu_waves_per_eu(2)))
void k_tail_outer(LevelDev<double> lv, ColIn<double> in, EpiOut<double> out, Twiddles<double> tw,
                  double* part, StopTest stop) {
  tail_matvec_body<double, CM, EPI_OUTER>(lv, in, out, tw, part, stop);
}
template <typename T, int CM, int EM>
__global__ __launch_bounds__(kNTT) __attribute__((amdgpu_waves_per_eu(2)))
void k_tail_matvec_b(const PassArgs<T>* __restrict__ args, Twiddles<T> tw) {
  const PassArgs<T>* a = args + blockIdx.x;
  if (gate_skip(a->st, a->gate)) return;
  const LevelDev<T> lv = a->lv;
  const ColIn<T> in = a->in;
  const EpiOut<T> out = a->out;
  tail_matvec_body<T, CM, EM>(lv, in, out, tw, a->npart_out, StopTest{});
}

// Setup: FFT (natural order) of c_x + i c_y for a tail level.
template <int LOGL>
__device__ __forceinline__ void tail_fft_setup(int logl, const double* gx, const double* gy,
                                               cplx<double>* out, const Twiddles<double>& tws) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  const Lds<double> z{reinterpret_cast<cplx<double>*>(smem_raw)};
  const int logL = LOGL ? LOGL : logl;
  const int L = 1 << logL, n = L / 2 - 1, q = logL - 3;
  const int j0 = threadIdx.x;
  const bool act = j0 < L / 8;
  cplx<double> a[8];
  FftTw8<double> tw;
  if (act) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int j = j0 + (e << q);
      a[e] = {circ_col(gx, n, L, j), circ_col(gy, n, L, j)};
    }
    tw.load(logL, j0, FftTab8<double>{tws.tail, kTailLog});
  }
  if (LOGL > 9 || j0 < 64) fft8<double, LOGL>(a, z, logL, j0, act, tw);
  if (act) {
#pragma unroll
    for (int e = 0; e < 8; ++e) out[j0 + (e << q)] = a[e];
  }
}
// Setup: spectra of the four blocks from two packed transforms
// Z1 = F(c_A + i c_B), Z2 = F(c_C + i c_D); A^ = (Z1 + conj Z1(-f))/2,
// B^ = (Z1 - conj Z1(-f))/(2i), etc.; G1, G2 as above, divided by L.
__device__ __forceinline__ void combine_at(int pos, int logL, int logL1, int logL2,
                                           const cplx<double>* z1, const cplx<double>* z2, int sym,
                                           double* g1, double* g2, float* g1f, float* g2f) {
  const int L = 1 << logL;
  int pp;
  if (logL2 == 0) {
    pp = (L - pos) & (L - 1);
  } else {
    const int L1 = 1 << logL1, L2 = 1 << logL2;
    const int k2 = pos >> logL1, k1 = pos & (L1 - 1);
    const int f = k2 + L2 * k1;
    const int fn = (L - f) & (L - 1);
    pp = (fn & (L2 - 1)) * L1 + (fn >> logL2);
  }
  const cplx<double> a1 = z1[pos], b1 = conj(z1[pp]), a2 = z2[pos], b2 = conj(z2[pp]);
  const cplx<double> Ah = scale(a1 + b1, 0.5), Ch = scale(a2 + b2, 0.5);
  const cplx<double> Bh = scale(rot<double, false>(a1 - b1), 0.5);  // (z - conj)/(2i)
  const cplx<double> Dh = scale(rot<double, false>(a2 - b2), 0.5);
  const double sc = 0.5 / (double)L;
  const cplx<double> G1 = scale((Ah + Dh) + rot<double, true>(Ch - Bh), sc);
  const cplx<double> G2 = scale((Ah - Dh) + rot<double, true>(Ch + Bh), sc);
  if (sym) {
    g1[pos] = G1.x;
    g2[pos] = G2.y;
    if (g1f) {
      g1f[pos] = (float)G1.x;
      g2f[pos] = (float)G2.y;
    }
  } else {
    g1[2 * pos] = G1.x;
    g1[2 * pos + 1] = G1.y;
    g2[2 * pos] = G2.x;
    g2[2 * pos + 1] = G2.y;
    if (g1f) {
      g1f[2 * pos] = (float)G1.x;
      g1f[2 * pos + 1] = (float)G1.y;
      g2f[2 * pos] = (float)G2.x;
      g2f[2 * pos + 1] = (float)G2.y;
    }
  }
}
__global__ void k_combine(int logL, int logL1, int logL2, const cplx<double>* z1,
                          const cplx<double>* z2, int sym, double* g1, double* g2, float* g1f,
                          float* g2f) {
  const int pos = blockIdx.x * blockDim.x + threadIdx.x;
  if (pos < (1 << logL)) combine_at(pos, logL, logL1, logL2, z1, z2, sym, g1, g2, g1f, g2f);
}

// The small levels' spectra, a workgroup per level: both transforms and their
// combination, where three launches per level stood (27 for nine levels,
// 5 us each; here the largest level's workgroup takes 20 us in all).
template <int LOGL>
__device__ __forceinline__ void tail_spectra(const TailSpectra& e, const Twiddles<double>& tw) {
  const int L = 1 << (LOGL ? LOGL : e.logL);
  tail_fft_setup<LOGL>(e.logL, e.a, e.b, e.z, tw);
  __syncthreads();  // the first transform's LDS reads
  tail_fft_setup<LOGL>(e.logL, e.c, e.d, e.z + L, tw);
  __syncthreads();  // both transforms, written by other threads
  for (int pos = threadIdx.x; pos < L; pos += kNTT)
    combine_at(pos, e.logL, e.logL, 0, e.z, e.z + L, e.sym, e.g1, e.g2, e.g1f, e.g2f);
}
__global__ __launch_bounds__(kNTT) __attribute__((amdgpu_waves_per_eu(2)))
void k_tail_spectra(TailSpectraTable t, Twiddles<double> tw) {
  const TailSpectra e = t.lv[blockIdx.x];
  switch (e.logL) {
    case 12: tail_spectra<12>(e, tw); break;
    case 11: tail_spectra<11>(e, tw); break;
    case 10: tail_spectra<10>(e, tw); break;
    case 9: tail_spectra<9>(e, tw); break;
    default: tail_spectra<0>(e, tw); break;
  }
}

__global__ __launch_bounds__(256) void k_finish(StopTest t, const double* part, int npart) {
  __shared__ double red[256 / 64];
  double v = 0.0;
  for (int i = threadIdx.x; i < npart; i += 256) v += part[i];
  const double s = block_sum<double, 256>(v, red);
  if (threadIdx.x == 0) stop_state(t, s);
  __syncthreads();  // thread 0's state writes before the copy
  publish_state(t.st, t.host, t.hist);
}

__global__ __launch_bounds__(256) void k_finish_b(const FinishArgs* __restrict__ args) {
  __shared__ double red[256 / 64];
  const FinishArgs* a = args + blockIdx.x;
  if (gate_skip(a->st, a->gate)) return;
  double v = 0.0;
  for (int i = threadIdx.x; i < a->npart; i += 256) v += a->part[i];
  const double s = block_sum<double, 256>(v, red);
  if (threadIdx.x == 0) finish_state(a->st, s, a->tol, a->max_iter, a->hist, a->verify);
  if (a->host) {
    __syncthreads();  // thread 0's state writes before the copy
    constexpr int W = sizeof(SolveState) / 4;
    if (threadIdx.x < W)
      reinterpret_cast<unsigned*>(a->host)[threadIdx.x] =
          reinterpret_cast<const unsigned*>(a->st)[threadIdx.x];
    __threadfence_system();
  }
}

__global__ void k_copy_d2f(const double* a, float* b, int64_t m) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < m) b[i] = (float)a[i];
}

// ---------------------------------------------------------------------------
// Conjugate gradients preconditioned by the V-cycle (SPD case).  Dot products
// and norms sum fixed contiguous chunks (one per block) and reduce the block
// partials in index order, so every run gives the same bits.  The scalars
// live in the solve state on the device; a finished solve (done) leaves them
// and the vectors untouched.
// ---------------------------------------------------------------------------
template <typename TZ>
__device__ __forceinline__ void vdot_body(const double* a, const TZ* z, const double* c, int64_t m,
                                          int64_t chunk, double* part) {
  __shared__ double red[kVecNT / 64];
  const int64_t i0 = (int64_t)blockIdx.x * chunk;
  const int64_t i1 = i0 + chunk < m ? i0 + chunk : m;
  double s0 = 0.0, s1 = 0.0;
  for (int64_t i = i0 + threadIdx.x; i < i1; i += kVecNT) {
    const double zi = (double)z[i];
    s0 += a[i] * zi;
    if (c) s1 += c[i] * zi;
  }
  s0 = block_sum<double, kVecNT>(s0, red);
  s1 = block_sum<double, kVecNT>(s1, red);
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = s0;
    part[2 * blockIdx.x + 1] = s1;
  }
}
template <typename TZ>
__global__ __launch_bounds__(kVecNT) void k_vdot(const double* a, const TZ* z, const double* c,
                                                 int64_t m, int64_t chunk, double* part) {
  vdot_body<TZ>(a, z, c, m, chunk, part);
}
// Batched: block (x, y) is chunk x of instance y (the instance's own
// partition: vec_blocks(m) chunks of vec_chunk(m)).
template <typename TZ>
__global__ __launch_bounds__(kVecNT) void k_vdot_b(const VdotArgs* __restrict__ args) {
  const VdotArgs* g = args + blockIdx.y;
  if (gate_skip(g->st, g->gate)) return;
  if ((int)blockIdx.x >= vec_blocks(g->m)) return;
  vdot_body<TZ>(g->a, static_cast<const TZ*>(g->z), g->c, g->m, vec_chunk(g->m), g->part);
}

__device__ __forceinline__ void cg_scalar_body(SolveState* st, const double* part, int nb,
                                               int stage) {
  __shared__ double red[kVecNT / 64];
  double v0 = 0.0, v1 = 0.0;
  for (int i = threadIdx.x; i < nb; i += kVecNT) {
    v0 += part[2 * i];
    v1 += part[2 * i + 1];
  }
  v0 = block_sum<double, kVecNT>(v0, red);
  v1 = block_sum<double, kVecNT>(v1, red);
  if (threadIdx.x != 0 || st->done) return;
  bool bad = !(v0 > 0.0) || isinf(v0);  // <r, z> and <p, A p> must be positive (SPD)
  if (stage == CG_INIT) {
    st->rz = v0;
    st->beta = 0.0;
  } else if (stage == CG_ALPHA) {
    st->alpha = st->rz / v0;
  } else {
    // Polak-Ribiere: <z_new, r_new - r_old> / <z_old, r_old>
    st->beta = (v0 - v1) / st->rz;
    st->rz = v0;
  }
  if (bad) {
    st->status = 2;  // AMG_DIVERGED: the operator or the preconditioner is not SPD
    st->done = 1;
  }
}
__global__ __launch_bounds__(kVecNT) void k_cg_scalar(SolveState* st, const double* part, int nb,
                                                      int stage) {
  cg_scalar_body(st, part, nb, stage);
}
__global__ __launch_bounds__(kVecNT) void k_cg_scalar_b(const CgArgs* __restrict__ args,
                                                        int stage) {
  const CgArgs* g = args + blockIdx.x;
  if (gate_skip(g->st, g->gate)) return;
  const int sg = stage == CG_AUTO ? (g->st->cg_first ? CG_INIT : CG_BETA) : stage;
  cg_scalar_body(g->st, g->part, g->nb, sg);
}

__device__ __forceinline__ void cg_update_body(const SolveState* st, double* x, const double* p,
                                               double* r, double* r_old, const double* q,
                                               float* r32, int64_t m, int64_t chunk,
                                               double* npart) {
  __shared__ double red[kVecNT / 64];
  if (st->done) return;  // uniform: every thread of every block returns
  const double alpha = st->alpha;
  const int64_t i0 = (int64_t)blockIdx.x * chunk;
  const int64_t i1 = i0 + chunk < m ? i0 + chunk : m;
  double ss = 0.0;
  for (int64_t i = i0 + threadIdx.x; i < i1; i += kVecNT) {
    x[i] += alpha * p[i];
    const double ro = r[i], rn = ro - alpha * q[i];
    r_old[i] = ro;
    r[i] = rn;
    if (r32) r32[i] = (float)rn;
    ss += rn * rn;
  }
  ss = block_sum<double, kVecNT>(ss, red);
  if (threadIdx.x == 0) npart[blockIdx.x] = ss;
}
__global__ __launch_bounds__(kVecNT) void k_cg_update(const SolveState* st, double* x,
                                                      const double* p, double* r, double* r_old,
                                                      const double* q, float* r32, int64_t m,
                                                      int64_t chunk, double* npart) {
  cg_update_body(st, x, p, r, r_old, q, r32, m, chunk, npart);
}
// Batched; block 0 also clears the instance's cg_first (the direction of
// this step has been formed).
__global__ __launch_bounds__(kVecNT) void k_cg_update_b(const CgArgs* __restrict__ args) {
  const CgArgs* g = args + blockIdx.y;
  if (gate_skip(g->st, g->gate)) return;
  if ((int)blockIdx.x >= vec_blocks(g->m)) return;
  cg_update_body(g->st, g->x, g->p, g->r, g->r_old, g->q, g->r32, g->m, vec_chunk(g->m), g->npart);
  if (blockIdx.x == 0 && threadIdx.x == 0) g->st->cg_first = 0;
}

// ---------------------------------------------------------------------------
// Restarted flexible GMRES (right preconditioner = one V-cycle per step).
// Classical Gram-Schmidt applied twice: each pass is one multi-dot (all
// <v_i, w> of the pass in one launch, fixed-order block partials) and one
// update; the small dense work (Givens rotations, the triangular solve) runs
// in one thread.  Every kernel returns at once when the solve is done.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kVecNT) void k_gm_start(const SolveState* st, const double* r,
                                                     double* v0, double* g, int64_t m,
                                                     double* vin64, float* vin32) {
  if (st->done) return;
  const double beta = st->relres * st->r0;
  const double inv = 1.0 / beta;
  const int64_t i = (int64_t)blockIdx.x * kVecNT + threadIdx.x;
  if (i == 0) g[0] = beta;
  if (i >= m) return;
  const double v = r[i] * inv;
  v0[i] = v;
  if (vin64) vin64[i] = v;
  if (vin32) vin32[i] = (float)v;
}

__global__ __launch_bounds__(kVecNT) void k_gm_dot(const double* V, int cnt, const double* w,
                                                   int64_t m, int64_t chunk, double* part) {
  __shared__ double red[kVecNT / 64];
  const int g0 = blockIdx.y * kGmGroup;
  const int64_t i0 = (int64_t)blockIdx.x * chunk;
  const int64_t i1 = i0 + chunk < m ? i0 + chunk : m;
  double acc[kGmGroup];
#pragma unroll
  for (int k = 0; k < kGmGroup; ++k) acc[k] = 0.0;
  for (int64_t i = i0 + threadIdx.x; i < i1; i += kVecNT) {
    const double wi = w[i];
#pragma unroll
    for (int k = 0; k < kGmGroup; ++k)
      if (g0 + k < cnt) acc[k] += V[(int64_t)(g0 + k) * m + i] * wi;
  }
#pragma unroll
  for (int k = 0; k < kGmGroup; ++k) {
    const double t = block_sum<double, kVecNT>(acc[k], red);
    if (threadIdx.x == 0 && g0 + k < cnt) part[(int64_t)(g0 + k) * gridDim.x + blockIdx.x] = t;
  }
}

__global__ __launch_bounds__(kVecNT) void k_gm_reduce(const SolveState* st, const double* part,
                                                      int nb, int cnt, double* hcur, double* hcol,
                                                      int accumulate) {
  __shared__ double red[kVecNT / 64];
  if (st->done) return;
  for (int k = 0; k < cnt; ++k) {
    double v = 0.0;
    for (int b = threadIdx.x; b < nb; b += kVecNT) v += part[(int64_t)k * nb + b];
    v = block_sum<double, kVecNT>(v, red);
    if (threadIdx.x == 0) {
      hcur[k] = v;
      hcol[k] = accumulate ? hcol[k] + v : v;
    }
  }
}

__global__ __launch_bounds__(kVecNT) void k_gm_axpy(const SolveState* st, double* w,
                                                    const double* V, const double* hcur, int cnt,
                                                    int64_t m, int64_t chunk, double* npart) {
  __shared__ double red[kVecNT / 64];
  __shared__ double hs[kGmMax + 1];
  if (st->done) return;
  for (int k = threadIdx.x; k < cnt; k += kVecNT) hs[k] = hcur[k];
  __syncthreads();
  const int64_t i0 = (int64_t)blockIdx.x * chunk;
  const int64_t i1 = i0 + chunk < m ? i0 + chunk : m;
  double ss = 0.0;
  for (int64_t i = i0 + threadIdx.x; i < i1; i += kVecNT) {
    double v = w[i];
    for (int k = 0; k < cnt; ++k) v -= hs[k] * V[(int64_t)k * m + i];
    w[i] = v;
    ss += v * v;
  }
  if (npart) {
    ss = block_sum<double, kVecNT>(ss, red);
    if (threadIdx.x == 0) npart[blockIdx.x] = ss;
  }
}

__device__ __forceinline__ void gm_givens_state(SolveState* st, double* H, int j, double* cs,
                                                double* sn, double* g, double* hn_out, double v,
                                                double tol, int max_iter, int restart,
                                                double* hist) {
  if (st->done) return;
  const double hn = sqrt(v);
  *hn_out = hn;
  double* Hj = H + (int64_t)j * (kGmMax + 1);
  Hj[j + 1] = hn;
  for (int i = 0; i < j; ++i) {
    const double a = Hj[i], c = Hj[i + 1];
    Hj[i] = cs[i] * a + sn[i] * c;
    Hj[i + 1] = -sn[i] * a + cs[i] * c;
  }
  const double d = hypot(Hj[j], Hj[j + 1]);
  if (!(d > 0.0) || isinf(d)) {  // singular or non-finite Hessenberg column
    st->status = 2;
    st->done = 1;
    return;
  }
  cs[j] = Hj[j] / d;
  sn[j] = Hj[j + 1] / d;
  Hj[j] = d;
  Hj[j + 1] = 0.0;
  g[j + 1] = -sn[j] * g[j];
  g[j] = cs[j] * g[j];
  const double est = fabs(g[j + 1]) / st->r0;
  st->relres = est;
  hist[st->iter] = est;
  if (!(est == est) || isinf(est)) {
    st->status = 2;
    st->done = 1;
    return;
  }
  if (est < tol || j + 1 >= restart || st->iter >= max_iter || hn == 0.0)
    st->cycle_end = 1;
  else
    st->iter += 1;
}
__global__ __launch_bounds__(kVecNT) void k_gm_givens(StopTest t, double* H, int j, double* cs,
                                                      double* sn, double* g, double* hn_out,
                                                      const double* npart, int nb, int restart) {
  __shared__ double red[kVecNT / 64];
  double v = 0.0;
  for (int b = threadIdx.x; b < nb; b += kVecNT) v += npart[b];
  v = block_sum<double, kVecNT>(v, red);
  if (threadIdx.x == 0)
    gm_givens_state(t.st, H, j, cs, sn, g, hn_out, v, t.tol, t.max_iter, restart, t.hist);
  __syncthreads();  // thread 0's state writes before the copy
  publish_state(t.st, t.host, t.hist);
}

__global__ __launch_bounds__(kVecNT) void k_gm_scale(const SolveState* st, double* w,
                                                     const double* hn, int64_t m, double* vin64,
                                                     float* vin32) {
  if (st->done || st->cycle_end) return;
  const int64_t i = (int64_t)blockIdx.x * kVecNT + threadIdx.x;
  if (i >= m) return;
  const double v = w[i] / *hn;
  w[i] = v;
  if (vin64) vin64[i] = v;
  if (vin32) vin32[i] = (float)v;
}

__global__ void k_gm_solve(const SolveState* st, const double* H, const double* g, int k,
                           double* y) {
  if (threadIdx.x != 0 || st->done) return;
  for (int i = k - 1; i >= 0; --i) {
    double v = g[i];
    for (int l = i + 1; l < k; ++l) v -= H[(int64_t)l * (kGmMax + 1) + i] * y[l];
    y[i] = v / H[(int64_t)i * (kGmMax + 1) + i];
  }
}

__global__ __launch_bounds__(kVecNT) void k_gm_xupdate(const SolveState* st, double* x,
                                                       const double* Z, const double* y, int k,
                                                       int64_t m) {
  __shared__ double ys[kGmMax];
  if (st->done) return;
  for (int l = threadIdx.x; l < k; l += kVecNT) ys[l] = y[l];
  __syncthreads();
  const int64_t i = (int64_t)blockIdx.x * kVecNT + threadIdx.x;
  if (i >= m) return;
  double v = x[i];
  for (int l = 0; l < k; ++l) v += ys[l] * Z[(int64_t)l * m + i];
  x[i] = v;
}

__global__ __launch_bounds__(kVecNT) void k_gm_check_b(const FinishArgs* __restrict__ args) {
  __shared__ double red[kVecNT / 64];
  const FinishArgs* a = args + blockIdx.x;
  if (gate_skip(a->st, a->gate)) return;
  double v = 0.0;
  for (int b = threadIdx.x; b < a->npart; b += kVecNT) v += a->part[b];
  v = block_sum<double, kVecNT>(v, red);
  if (threadIdx.x == 0) gm_check_state(a->st, v, a->tol, a->max_iter, a->hist, a->verify);
  if (a->host) {
    __syncthreads();
    constexpr int W = sizeof(SolveState) / 4;
    if (threadIdx.x < W)
      reinterpret_cast<unsigned*>(a->host)[threadIdx.x] =
          reinterpret_cast<const unsigned*>(a->st)[threadIdx.x];
    __threadfence_system();
  }
}

// b = e_j (length m): the unit vectors a setup applies the V-cycle to.
__global__ void k_basis(double* b, int m, int j) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < m) b[i] = i == j ? 1.0 : 0.0;
}
// Column j of a batch of unit-vector right-hand sides: b_j = e_j, where b_j
// starts at base + j * stride (m entries each, m columns).
__global__ void k_basis_batch(double* base, int64_t stride, int m, int j0) {
  const int j = blockIdx.y;
  double* b = base + (int64_t)j * stride;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < m; i += gridDim.x * blockDim.x)
    b[i] = i == j0 + j ? 1.0 : 0.0;
}
hipError_t launch_basis_batch(double* base, int64_t stride, int m, hipStream_t s, int count,
                              int j0) {
  if (count < 0) count = m;
  if (m < 1 || count < 1 || count > 65535 || j0 < 0 || j0 + count > m) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_basis_batch, dim3((m + 255) / 256, count), 256, 0, s, base, stride, m, j0);
  return hipGetLastError();
}
// M[:, j] = u_j (column-major, ld rows to a column), u_j at base + j * stride.
__global__ void k_gather_columns(double* M, int ld, const double* base, int64_t stride, int m) {
  const int j = blockIdx.y;
  const double* u = base + (int64_t)j * stride;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < m; i += gridDim.x * blockDim.x)
    M[(int64_t)j * ld + i] = u[i];
}
hipError_t launch_gather_columns(double* M, int ld, const double* base, int64_t stride, int m,
                                 hipStream_t s) {
  if (m < 1 || m > 65535 || ld < m) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_gather_columns, dim3((m + 255) / 256, m), 256, 0, s, M, ld, base, stride, m);
  return hipGetLastError();
}

hipError_t launch_basis(double* b, int m, int j, hipStream_t s) {
  hipLaunchKernelGGL(k_basis, (m + 255) / 256, 256, 0, s, b, m, j);
  return hipGetLastError();
}

__global__ void k_copy_f2d(const float* a, double* b, int64_t m) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < m) b[i] = (double)a[i];
}

// Band product bc = B x of a level's tridiagonal part (block-ordered vector).
template <typename T>
__global__ __launch_bounds__(kVecNT) void k_band_mv(LevelDev<T> lv, const T* x) {
  const int m = 2 * lv.n + 1;
  const int i = blockIdx.x * kVecNT + threadIdx.x;
  if (i >= m) return;
  T y = lv.bmain[i] * x[i];
  if (i > 0) y += lv.bsub[i] * x[i - 1];
  if (i + 1 < m) y += lv.bsup[i] * x[i + 1];
  lv.bc[i] = y;
}

template <typename T>
hipError_t launch_band_mv(const LevelDev<T>& lv, const T* x, hipStream_t s) {
  const int m = 2 * lv.n + 1;
  hipLaunchKernelGGL(k_band_mv<T>, (m + kVecNT - 1) / kVecNT, kVecNT, 0, s, lv, x);
  return hipGetLastError();
}
template hipError_t launch_band_mv<double>(const LevelDev<double>&, const double*, hipStream_t);
template hipError_t launch_band_mv<float>(const LevelDev<float>&, const float*, hipStream_t);

// BDF4 history combination of eq. (bdf4), one element per thread
__global__ __launch_bounds__(kVecNT) void k_bdf4_rhs(const double* u1, const double* u2,
                                                     const double* u3, const double* u4,
                                                     const double* src, double* b, int64_t m) {
  const int64_t i = (int64_t)blockIdx.x * kVecNT + threadIdx.x;
  if (i >= m) return;
  double v = 4.0 * u1[i] - 3.0 * u2[i] + (4.0 / 3.0) * u3[i] - 0.25 * u4[i];
  if (src) v += src[i];
  b[i] = v;
}

template <typename TZ>
__global__ __launch_bounds__(kVecNT) void k_cg_dir(const SolveState* st, double* p, const TZ* z,
                                                   int64_t m, int first) {
  if (st->done) return;
  const int64_t i = (int64_t)blockIdx.x * kVecNT + threadIdx.x;
  if (i >= m) return;
  p[i] = first ? (double)z[i] : (double)z[i] + st->beta * p[i];
}
template <typename TZ>
__global__ __launch_bounds__(kVecNT) void k_cg_dir_b(const CgArgs* __restrict__ args) {
  const CgArgs* g = args + blockIdx.y;
  if (gate_skip(g->st, g->gate)) return;
  const int64_t i = (int64_t)blockIdx.x * kVecNT + threadIdx.x;
  if (i >= g->m) return;
  const TZ* z = static_cast<const TZ*>(g->z);
  const SolveState* st = g->st;
  g->p[i] = st->cg_first ? (double)z[i] : (double)z[i] + st->beta * g->p[i];
}

// ---------------------------------------------------------------------------
// Near field of the split residual.  A workgroup owns kNearTS consecutive
// collocation positions s (units of h/2: nodes at even s, midpoints at odd
// s) and stages x at s - M .. s + kNearTS - 1 + M, read from the block
// order, in LDS; each output sums W(k) (x_{s+k} - x_s) over 0 < |k| <= M in
// (k, -k) pairs in a fixed order and adds R_s x_s.  Only the first and last
// workgroups hold positions whose stencil leaves 1..2N-1; they test every
// column (out-of-range columns are not in the matrix).
// ---------------------------------------------------------------------------
constexpr int kNearTS = 1024;
constexpr int kNearNT = 256;

__device__ __forceinline__ int64_t near_block(int64_t s, int64_t n) {
  // block-order index of position s: node s = 2(i+1) -> i; midpoint s = 2k+1 -> n + k
  return (s & 1) ? n + (s >> 1) : (s >> 1) - 1;
}

__global__ __launch_bounds__(kNearNT) void k_near(const double* x, double* y, int64_t N,
                                                 const double* w, const double* rl,
                                                 const double* rr, double rin_n, double rin_m) {
  constexpr int M = kNearM;
  __shared__ double zs[kNearTS + 2 * M];
  __shared__ double ws[2 * (2 * M + 1)];
  const int64_t last = 2 * N - 1, n = N - 1;
  const int64_t s0 = 1 + (int64_t)blockIdx.x * kNearTS;
  // workgroups with a position within M of either end test every column
  const bool edge = s0 <= M || s0 + kNearTS - 1 > last - M;
  for (int i = threadIdx.x; i < kNearTS + 2 * M; i += kNearNT) {
    const int64_t s = s0 - M + i;
    zs[i] = (s >= 1 && s <= last) ? x[near_block(s, n)] : 0.0;
  }
  for (int i = threadIdx.x; i < 2 * (2 * M + 1); i += kNearNT) ws[i] = w[i];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < kNearTS / kNearNT; ++e) {
    const int t = threadIdx.x + e * kNearNT;
    const int64_t s = s0 + t;
    if (s > last) break;
    const double* W = ws + ((s & 1) ? (2 * M + 1) : 0) + M;
    const int c = t + M;
    const double zc = zs[c];
    double acc = 0.0;
    double R = (s & 1) ? rin_m : rin_n;
    if (!edge) {
#pragma unroll 8
      for (int k = 1; k <= M; ++k) acc += W[k] * (zs[c + k] - zc) + W[-k] * (zs[c - k] - zc);
    } else {
      for (int k = 1; k <= M; ++k) {
        if (s + k <= last) acc += W[k] * (zs[c + k] - zc);
        if (s - k >= 1) acc += W[-k] * (zs[c - k] - zc);
      }
      if (s <= M) R = rl[s - 1];
      else if (s > last - M) R = rr[s - (last - M + 1)];
    }
    y[near_block(s, n)] = acc + R * zc;
  }
}

hipError_t launch_near(const double* x, double* y, int64_t N, const double* w, const double* rl,
                       const double* rr, double rin_n, double rin_m, hipStream_t s) {
  const int64_t m = 2 * N - 1;
  const int64_t grid = (m + kNearTS - 1) / kNearTS;
  // the edge test of the kernel assumes a tile longer than the near reach
  static_assert(kNearTS > kNearM, "near tile");
  if (N <= kNearM || grid > ((int64_t)1 << 30)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_near, dim3((unsigned)grid), dim3(kNearNT), 0, s, x, y, N, w, rl, rr, rin_n,
                     rin_m);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
template <typename T>
hipError_t launch_tail_matvec(const LevelDev<T>& lv, const ColIn<T>& in, const EpiOut<T>& out,
                              const Twiddles<T>& tw, hipStream_t s) {
  if (lv.logL < 3 || lv.logL > kTailLog) return hipErrorInvalidValue;
  const size_t lds = tail_mv_lds_bytes(sizeof(T), lv.logL);
  return launch_lds(k_tail_matvec<T, COL_MV, EPI_MV>, 1, kNTT, lds, s, lv, in, out, tw,
                    (double*)nullptr);
}

hipError_t launch_tail_outer(int colmode, const LevelDev<double>& lv, const ColIn<double>& in,
                             const EpiOut<double>& out, const Twiddles<double>& tw, double* part,
                             const StopTest& stop, hipStream_t s) {
  if (lv.logL < 3 || lv.logL > kTailLog) return hipErrorInvalidValue;
  const size_t lds = tail_mv_lds_bytes(sizeof(double), lv.logL);
  if (colmode == COL_MV)
    return launch_lds(k_tail_outer<COL_MV>, 1, kNTT, lds, s, lv, in, out, tw, part, stop);
  if (colmode == COL_OUTER_UPDATE)
    return launch_lds(k_tail_outer<COL_OUTER_UPDATE>, 1, kNTT, lds, s, lv, in, out, tw, part, stop);
  return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_tail_vcycle(const LevelDev<T>* levels_dev, int first, int last, const T* rf,
                              int m1, int m2, T wpre, T wpost, const CoarseLU& lu,
                              const Twiddles<T>& tw, int maxL, int variant, hipStream_t s) {
  if (maxL > (1 << kTailLog) || !coarse_ok(lu.m) || first < 0 ||
      last - first + 1 > kTailMaxLev || last < first)
    return hipErrorInvalidValue;
  const size_t lds = tail_lds_bytes(sizeof(T));
  switch (variant) {
    case 0: return launch_lds(k_tail_vcycle<T, false, false>, 1, kNTT, lds, s, levels_dev, first,
                              last, rf, m1, m2, wpre, wpost, lu, tw);
    case TAIL_SYM: return launch_lds(k_tail_vcycle<T, false, true>, 1, kNTT, lds, s, levels_dev,
                                     first, last, rf, m1, m2, wpre, wpost, lu, tw);
    case TAIL_BAND: return launch_lds(k_tail_vcycle<T, true, false>, 1, kNTT, lds, s, levels_dev,
                                      first, last, rf, m1, m2, wpre, wpost, lu, tw);
    case TAIL_BAND | TAIL_SYM:
      return launch_lds(k_tail_vcycle<T, true, true>, 1, kNTT, lds, s, levels_dev, first, last,
                        rf, m1, m2, wpre, wpost, lu, tw);
    default: return hipErrorInvalidValue;
  }
}

template <typename T>
hipError_t launch_tail_program(const LevelDev<T>* levels_dev, int first, int last, const T* rf,
                               const TailOp* ops, int nops, T wpre, T wpost, const CoarseLU& lu,
                               const Twiddles<T>& tw, int maxL, int variant, hipStream_t s) {
  if (maxL > (1 << kTailLog) || !coarse_ok(lu.m) || first < 0 ||
      last - first + 1 > kTailMaxLev || last < first)
    return hipErrorInvalidValue;
  const size_t lds = tail_lds_bytes(sizeof(T));
  switch (variant) {
    case 0: return launch_lds(k_tail_program<T, false, false>, 1, kNTT, lds, s, levels_dev, first,
                              last, rf, ops, nops, wpre, wpost, lu, tw);
    case TAIL_SYM: return launch_lds(k_tail_program<T, false, true>, 1, kNTT, lds, s, levels_dev,
                                     first, last, rf, ops, nops, wpre, wpost, lu, tw);
    case TAIL_BAND: return launch_lds(k_tail_program<T, true, false>, 1, kNTT, lds, s, levels_dev,
                                      first, last, rf, ops, nops, wpre, wpost, lu, tw);
    case TAIL_BAND | TAIL_SYM:
      return launch_lds(k_tail_program<T, true, true>, 1, kNTT, lds, s, levels_dev, first, last,
                        rf, ops, nops, wpre, wpost, lu, tw);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_tail_spectra(const std::vector<TailSpectra>& lv, const Twiddles<double>& tw,
                               hipStream_t s) {
  for (size_t i = 0; i < lv.size(); i += kTailSpectraMax) {
    const int cnt = (int)std::min(lv.size() - i, (size_t)kTailSpectraMax);
    TailSpectraTable t{};
    int logm = 0;
    for (int k = 0; k < cnt; ++k) {
      t.lv[k] = lv[i + k];
      if (t.lv[k].logL < 3 || t.lv[k].logL > kTailLog) return hipErrorInvalidValue;
      logm = std::max(logm, t.lv[k].logL);
    }
    const hipError_t e =
        launch_lds(k_tail_spectra, cnt, kNTT, tail_mv_lds_bytes(sizeof(double), logm), s, t, tw);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_combine(int logL, int logL1, int logL2, const cplx<double>* z1,
                          const cplx<double>* z2, int sym, double* g1, double* g2, float* g1f,
                          float* g2f, hipStream_t s) {
  const int64_t L = int64_t(1) << logL;
  const int grid = (int)((L + 255) / 256);
  hipLaunchKernelGGL(k_combine, grid, 256, 0, s, logL, logL1, logL2, z1, z2, sym, g1, g2, g1f, g2f);
  return hipGetLastError();
}

hipError_t launch_finish(const StopTest& t, const double* part, int npart, hipStream_t s) {
  hipLaunchKernelGGL(k_finish, 1, 256, 0, s, t, part, npart);
  return hipGetLastError();
}

hipError_t launch_copy_d2f(const double* a, float* b, int64_t m, hipStream_t s) {
  const int grid = (int)((m + 255) / 256);
  hipLaunchKernelGGL(k_copy_d2f, grid, 256, 0, s, a, b, m);
  return hipGetLastError();
}

template <typename TZ>
hipError_t launch_vdot(const double* a, const TZ* z, const double* c, int64_t m, double* part,
                       hipStream_t s) {
  hipLaunchKernelGGL(k_vdot<TZ>, vec_blocks(m), kVecNT, 0, s, a, z, c, m, vec_chunk(m), part);
  return hipGetLastError();
}

hipError_t launch_cg_scalar(SolveState* st, const double* part, int nb, int stage, hipStream_t s) {
  hipLaunchKernelGGL(k_cg_scalar, 1, kVecNT, 0, s, st, part, nb, stage);
  return hipGetLastError();
}

hipError_t launch_cg_update(const SolveState* st, double* x, const double* p, double* r,
                            double* r_old, const double* q, float* r32, int64_t m, double* npart,
                            hipStream_t s) {
  hipLaunchKernelGGL(k_cg_update, vec_blocks(m), kVecNT, 0, s, st, x, p, r, r_old, q, r32, m,
                     vec_chunk(m), npart);
  return hipGetLastError();
}

template <typename TZ>
hipError_t launch_cg_dir(const SolveState* st, double* p, const TZ* z, int64_t m, int first,
                         hipStream_t s) {
  const int grid = (int)((m + kVecNT - 1) / kVecNT);
  hipLaunchKernelGGL(k_cg_dir<TZ>, grid, kVecNT, 0, s, st, p, z, m, first);
  return hipGetLastError();
}

hipError_t launch_gm_start(const SolveState* st, const double* r, double* v0, double* g, int64_t m,
                           double* vin64, float* vin32, hipStream_t s) {
  const int grid = (int)((m + kVecNT - 1) / kVecNT);
  hipLaunchKernelGGL(k_gm_start, grid, kVecNT, 0, s, st, r, v0, g, m, vin64, vin32);
  return hipGetLastError();
}

hipError_t launch_gm_dot(const double* V, int cnt, const double* w, int64_t m, double* part,
                         hipStream_t s) {
  const dim3 grid(vec_blocks(m), (cnt + kGmGroup - 1) / kGmGroup);
  hipLaunchKernelGGL(k_gm_dot, grid, kVecNT, 0, s, V, cnt, w, m, vec_chunk(m), part);
  return hipGetLastError();
}

hipError_t launch_gm_reduce(const SolveState* st, const double* part, int nb, int cnt,
                            double* hcur, double* hcol, int accumulate, hipStream_t s) {
  hipLaunchKernelGGL(k_gm_reduce, 1, kVecNT, 0, s, st, part, nb, cnt, hcur, hcol, accumulate);
  return hipGetLastError();
}

hipError_t launch_gm_axpy(const SolveState* st, double* w, const double* V, const double* hcur,
                          int cnt, int64_t m, double* npart, hipStream_t s) {
  hipLaunchKernelGGL(k_gm_axpy, vec_blocks(m), kVecNT, 0, s, st, w, V, hcur, cnt, m, vec_chunk(m),
                     npart);
  return hipGetLastError();
}

hipError_t launch_gm_givens(const StopTest& t, double* H, int j, double* cs, double* sn, double* g,
                            double* hn, const double* npart, int nb, int restart, hipStream_t s) {
  hipLaunchKernelGGL(k_gm_givens, 1, kVecNT, 0, s, t, H, j, cs, sn, g, hn, npart, nb, restart);
  return hipGetLastError();
}

hipError_t launch_gm_scale(const SolveState* st, double* w, const double* hn, int64_t m,
                           double* vin64, float* vin32, hipStream_t s) {
  const int grid = (int)((m + kVecNT - 1) / kVecNT);
  hipLaunchKernelGGL(k_gm_scale, grid, kVecNT, 0, s, st, w, hn, m, vin64, vin32);
  return hipGetLastError();
}

hipError_t launch_gm_update(const SolveState* st, const double* H, const double* g, int k,
                            double* y, double* x, const double* Z, int64_t m, hipStream_t s) {
  hipLaunchKernelGGL(k_gm_solve, 1, 64, 0, s, st, H, g, k, y);
  const int grid = (int)((m + kVecNT - 1) / kVecNT);
  hipLaunchKernelGGL(k_gm_xupdate, grid, kVecNT, 0, s, st, x, Z, y, k, m);
  return hipGetLastError();
}

hipError_t launch_copy_f2d(const float* a, double* b, int64_t m, hipStream_t s) {
  const int grid = (int)((m + 255) / 256);
  hipLaunchKernelGGL(k_copy_f2d, grid, 256, 0, s, a, b, m);
  return hipGetLastError();
}

hipError_t launch_bdf4_rhs(const double* u1, const double* u2, const double* u3,
                           const double* u4, const double* src, double* b, int64_t m,
                           hipStream_t s) {
  const int grid = (int)((m + kVecNT - 1) / kVecNT);
  hipLaunchKernelGGL(k_bdf4_rhs, grid, kVecNT, 0, s, u1, u2, u3, u4, src, b, m);
  return hipGetLastError();
}

// ---- batched launchers ------------------------------------------------------
template <typename T>
hipError_t launch_tail_vcycle_batch(const TailArgs<T>* args, int count, int variant,
                                    const Twiddles<T>& tw, hipStream_t s) {
  if (count < 1) return hipErrorInvalidValue;
  const size_t lds = tail_lds_bytes(sizeof(T));
  switch (variant) {
    case 0: return launch_lds(k_tail_vcycle_b<T, false, false>, count, kNTT, lds, s, args, tw);
    case TAIL_SYM: return launch_lds(k_tail_vcycle_b<T, false, true>, count, kNTT, lds, s, args, tw);
    case TAIL_BAND: return launch_lds(k_tail_vcycle_b<T, true, false>, count, kNTT, lds, s, args, tw);
    case TAIL_BAND | TAIL_SYM:
      return launch_lds(k_tail_vcycle_b<T, true, true>, count, kNTT, lds, s, args, tw);
    default: return hipErrorInvalidValue;
  }
}

// ---------------------------------------------------------------------------
// The folded V-cycle below the four-step levels (its matrix formed at setup
// from the unit vectors) as one product over many workgroups: every block
// restricts the fine residual into LDS (FP64), then each wavefront takes
// rows, lanes striding the row (coalesced), four partial sums per lane in a
// fixed order and a butterfly over the wavefront.
// ---------------------------------------------------------------------------
constexpr int kFoldNT = 512;
constexpr int kFoldRows = 8;  // one row per wavefront

template <typename T, typename MT>
__device__ __forceinline__ void fold_gemv_body(const T* __restrict__ rf, int m,
                                               const MT* __restrict__ M, T* __restrict__ u,
                                               int block) {
  extern __shared__ double fb[];  // m values of R rf
  for (int i = threadIdx.x; i < m; i += kFoldNT) fb[i] = (double)restrict_at(rf, i);
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int rr = wave; rr < kFoldRows; rr += kFoldNT / 64) {
    const int row = block * kFoldRows + rr;
    if (row >= m) break;  // uniform in the wavefront
    const MT* a = M + (size_t)row * (size_t)m;
    // U loads in flight per lane (a row of 4095 in two batches of FP32 or
    // four of FP64), four partial sums
    constexpr int U = sizeof(MT) == 4 ? 32 : 16;
    double acc[4] = {0, 0, 0, 0};
    int j = lane;
    for (; j + 64 * (U - 1) < m; j += 64 * U) {
      MT av[U];
#pragma unroll
      for (int k = 0; k < U; ++k) av[k] = a[j + 64 * k];
#pragma unroll
      for (int k = 0; k < U; ++k) acc[k & 3] += (double)av[k] * fb[j + 64 * k];
    }
    {
      // the rest (fewer than U per lane): clamped loads, masked terms
      MT av[U];
#pragma unroll
      for (int k = 0; k < U; ++k) av[k] = a[min(j + 64 * k, m - 1)];
#pragma unroll
      for (int k = 0; k < U; ++k)
        if (j + 64 * k < m) acc[k & 3] += (double)av[k] * fb[j + 64 * k];
    }
    double v = (acc[0] + acc[1]) + (acc[2] + acc[3]);
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if (lane == 0) u[row] = (T)v;
  }
}

template <typename T, typename MT>
__global__ __launch_bounds__(kFoldNT) void k_fold_gemv(const T* rf, int m, const MT* M, T* u) {
  fold_gemv_body<T, MT>(rf, m, M, u, blockIdx.x);
}

template <typename T>
__global__ __launch_bounds__(kFoldNT) void k_fold_gemv_b(const FoldArgs<T>* __restrict__ args) {
  const FoldArgs<T>* a = args + blockIdx.y;
  if (gate_skip(a->st, a->gate)) return;
  if ((int)blockIdx.x * kFoldRows >= a->m) return;
  fold_gemv_body<T, T>(a->rf, a->m, a->M, a->u, blockIdx.x);
}

template <typename T, typename MT>
hipError_t launch_fold_gemv(const T* rf, int m, const MT* M, T* u, hipStream_t s) {
  if (m < 1 || m > kFoldMax) return hipErrorInvalidValue;
  const int grid = (m + kFoldRows - 1) / kFoldRows;
  return launch_lds(k_fold_gemv<T, MT>, grid, kFoldNT, (size_t)m * sizeof(double), s, rf, m, M, u);
}

template <typename T>
hipError_t launch_fold_gemv_batch(const FoldArgs<T>* args, int count, int m, hipStream_t s) {
  if (count < 1 || m < 1 || m > kFoldMax) return hipErrorInvalidValue;
  const dim3 grid((m + kFoldRows - 1) / kFoldRows, count);
  return launch_lds(k_fold_gemv_b<T>, grid, kFoldNT, (size_t)m * sizeof(double), s, args);
}

// 32 x 32 tiles through LDS: reads along the source vectors, writes along
// the matrix rows.
__global__ __launch_bounds__(256) void k_gather_rows(double* M, const double* src, int64_t stride,
                                                     int m, int j0, int count) {
  __shared__ double tile[32][33];
  const int ib = blockIdx.x * 32, kb = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int r = ty; r < 32; r += 8) {
    const int k = kb + r, i = ib + tx;
    tile[r][tx] = (k < count && i < m) ? src[(int64_t)k * stride + i] : 0.0;
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const int i = ib + r, k = kb + tx;
    if (i < m && k < count) M[(int64_t)i * m + j0 + k] = tile[tx][r];
  }
}

hipError_t launch_gather_rows(double* M, const double* src, int64_t stride, int m, int j0,
                              int count, hipStream_t s) {
  if (m < 1 || count < 1 || j0 < 0 || j0 + count > m) return hipErrorInvalidValue;
  const dim3 grid((m + 31) / 32, (count + 31) / 32);
  hipLaunchKernelGGL(k_gather_rows, grid, 256, 0, s, M, src, stride, m, j0, count);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_tail_matvec_batch(int colmode, int epimode, const PassArgs<T>* args, int count,
                                    const Twiddles<T>& tw, hipStream_t s) {
  if (count < 1) return hipErrorInvalidValue;
  const size_t lds = tail_mv_lds_bytes(sizeof(T), kTailLog);
  if (colmode == COL_MV && epimode == EPI_MV)
    return launch_lds(k_tail_matvec_b<T, COL_MV, EPI_MV>, count, kNTT, lds, s, args, tw);
  if (colmode == COL_MV && epimode == EPI_OUTER)
    return launch_lds(k_tail_matvec_b<T, COL_MV, EPI_OUTER>, count, kNTT, lds, s, args, tw);
  if (colmode == COL_OUTER_UPDATE && epimode == EPI_OUTER)
    return launch_lds(k_tail_matvec_b<T, COL_OUTER_UPDATE, EPI_OUTER>, count, kNTT, lds, s, args,
                      tw);
  return hipErrorInvalidValue;
}

template <typename TZ>
hipError_t launch_vdot_batch(const VdotArgs* args, int count, int64_t mmax, hipStream_t s) {
  if (count < 1 || count > 65535) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_vdot_b<TZ>, dim3(vec_blocks(mmax), count), kVecNT, 0, s, args);
  return hipGetLastError();
}
hipError_t launch_cg_scalar_batch(const CgArgs* args, int count, int stage, hipStream_t s) {
  if (count < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_cg_scalar_b, count, kVecNT, 0, s, args, stage);
  return hipGetLastError();
}
template <typename TZ>
hipError_t launch_cg_dir_batch(const CgArgs* args, int count, int64_t mmax, hipStream_t s) {
  if (count < 1 || count > 65535) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_cg_dir_b<TZ>, dim3((unsigned)((mmax + kVecNT - 1) / kVecNT), count), kVecNT,
                     0, s, args);
  return hipGetLastError();
}
hipError_t launch_cg_update_batch(const CgArgs* args, int count, int64_t mmax, hipStream_t s) {
  if (count < 1 || count > 65535) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_cg_update_b, dim3(vec_blocks(mmax), count), kVecNT, 0, s, args);
  return hipGetLastError();
}
hipError_t launch_finish_batch(const FinishArgs* args, int count, hipStream_t s) {
  if (count < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_finish_b, count, 256, 0, s, args);
  return hipGetLastError();
}
hipError_t launch_gm_check_batch(const FinishArgs* args, int count, hipStream_t s) {
  if (count < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_gm_check_b, count, kVecNT, 0, s, args);
  return hipGetLastError();
}
template hipError_t launch_vdot_batch<double>(const VdotArgs*, int, int64_t, hipStream_t);
template hipError_t launch_vdot_batch<float>(const VdotArgs*, int, int64_t, hipStream_t);
template hipError_t launch_cg_dir_batch<double>(const CgArgs*, int, int64_t, hipStream_t);
template hipError_t launch_cg_dir_batch<float>(const CgArgs*, int, int64_t, hipStream_t);

template hipError_t launch_vdot<double>(const double*, const double*, const double*, int64_t,
                                        double*, hipStream_t);
template hipError_t launch_vdot<float>(const double*, const float*, const double*, int64_t,
                                       double*, hipStream_t);
template hipError_t launch_cg_dir<double>(const SolveState*, double*, const double*, int64_t, int,
                                          hipStream_t);
template hipError_t launch_cg_dir<float>(const SolveState*, double*, const float*, int64_t, int,
                                         hipStream_t);
#define AMG_INSTANTIATE(T)                                                                      \
  template hipError_t launch_tail_matvec<T>(const LevelDev<T>&, const ColIn<T>&,               \
                                            const EpiOut<T>&, const Twiddles<T>&, hipStream_t);                                      \
  template hipError_t launch_tail_vcycle<T>(const LevelDev<T>*, int, int, const T*, int, int,  \
                                            T, T, const CoarseLU&, const Twiddles<T>&, int,    \
                                            int, hipStream_t);                                 \
  template hipError_t launch_tail_program<T>(const LevelDev<T>*, int, int, const T*,           \
                                             const TailOp*, int, T, T, const CoarseLU&,        \
                                             const Twiddles<T>&, int, int, hipStream_t);
AMG_INSTANTIATE(double)
AMG_INSTANTIATE(float)
template hipError_t launch_fold_gemv<double, double>(const double*, int, const double*, double*,
                                                     hipStream_t);
template hipError_t launch_fold_gemv<float, float>(const float*, int, const float*, float*,
                                                   hipStream_t);
template hipError_t launch_fold_gemv_batch<double>(const FoldArgs<double>*, int, int, hipStream_t);
template hipError_t launch_fold_gemv_batch<float>(const FoldArgs<float>*, int, int, hipStream_t);
template hipError_t launch_tail_vcycle_batch<double>(const TailArgs<double>*, int, int,
                                                     const Twiddles<double>&, hipStream_t);
template hipError_t launch_tail_vcycle_batch<float>(const TailArgs<float>*, int, int,
                                                    const Twiddles<float>&, hipStream_t);
template hipError_t launch_tail_matvec_batch<double>(int, int, const PassArgs<double>*, int,
                                                     const Twiddles<double>&, hipStream_t);
template hipError_t launch_tail_matvec_batch<float>(int, int, const PassArgs<float>*, int,
                                                    const Twiddles<float>&, hipStream_t);

}  // namespace amg
