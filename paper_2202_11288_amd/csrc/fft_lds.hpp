// Device building blocks of the circulant-embedding FFTs (Sec. 3.2,
// eq. (ccs3.4)): complex arithmetic, in-register DFTs of size 2/4/8/16, and a
// Stockham autosort FFT over signals held in LDS.  gfx950 (CDNA4), wave64.
#pragma once

#include <hip/hip_runtime.h>

namespace amg {

template <typename T>
struct alignas(2 * sizeof(T)) cplx {
  T x, y;
};

template <typename T>
__device__ __forceinline__ cplx<T> operator+(cplx<T> a, cplx<T> b) { return {a.x + b.x, a.y + b.y}; }
template <typename T>
__device__ __forceinline__ cplx<T> operator-(cplx<T> a, cplx<T> b) { return {a.x - b.x, a.y - b.y}; }
template <typename T>
__device__ __forceinline__ cplx<T> cmul(cplx<T> a, cplx<T> b) {
  return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
template <typename T>
__device__ __forceinline__ cplx<T> conj(cplx<T> a) { return {a.x, -a.y}; }
template <typename T>
__device__ __forceinline__ cplx<T> scale(cplx<T> a, T s) { return {a.x * s, a.y * s}; }
// Global loads / stores of one complex value as a single 2-wide vector access
// (keeps register staging arrays of complex values in registers).
template <typename T>
__device__ __forceinline__ cplx<T> ldg(const cplx<T>* p) {
  using V = T __attribute__((ext_vector_type(2)));
  const V v = *reinterpret_cast<const V*>(p);
  return {v.x, v.y};
}
template <typename T>
__device__ __forceinline__ void stg(cplx<T>* p, cplx<T> a) {
  using V = T __attribute__((ext_vector_type(2)));
  *reinterpret_cast<V*>(p) = V{a.x, a.y};
}

// multiply by -i (forward) or +i (inverse)
template <typename T, bool INV>
__device__ __forceinline__ cplx<T> rot(cplx<T> a) {
  return INV ? cplx<T>{-a.y, a.x} : cplx<T>{a.y, -a.x};
}

// ---- in-register DFTs: X_k = sum_j a_j e^{-+2 pi i jk/R} (natural order) ----

template <typename T, bool INV>
__device__ __forceinline__ void dft2(cplx<T>& a0, cplx<T>& a1) {
  const cplx<T> t = a0 - a1;
  a0 = a0 + a1;
  a1 = t;
}

template <typename T, bool INV>
__device__ __forceinline__ void dft4(cplx<T>& a0, cplx<T>& a1, cplx<T>& a2, cplx<T>& a3) {
  const cplx<T> t0 = a0 + a2, t1 = a0 - a2, t2 = a1 + a3, t3 = rot<T, INV>(a1 - a3);
  a0 = t0 + t2;
  a2 = t0 - t2;
  a1 = t1 + t3;
  a3 = t1 - t3;
}

// (1 -+ i)/sqrt2 * a and (-1 -+ i)/sqrt2 * a without a general complex product
template <typename T, bool INV>
__device__ __forceinline__ cplx<T> w8_1(cplx<T> a) {
  const T s = T(0.70710678118654752440);
  return INV ? cplx<T>{s * (a.x - a.y), s * (a.x + a.y)} : cplx<T>{s * (a.x + a.y), s * (a.y - a.x)};
}
template <typename T, bool INV>
__device__ __forceinline__ cplx<T> w8_3(cplx<T> a) {
  const T s = T(0.70710678118654752440);
  return INV ? cplx<T>{-s * (a.x + a.y), s * (a.x - a.y)} : cplx<T>{s * (a.y - a.x), -s * (a.x + a.y)};
}

template <typename T, bool INV>
__device__ __forceinline__ void dft8(cplx<T>* a) {
  // radix-2 decimation in time: even/odd DFT4s, twiddles e^{-+2 pi i k/8}
  cplx<T> e0 = a[0], e1 = a[2], e2 = a[4], e3 = a[6];
  cplx<T> o0 = a[1], o1 = a[3], o2 = a[5], o3 = a[7];
  dft4<T, INV>(e0, e1, e2, e3);
  dft4<T, INV>(o0, o1, o2, o3);
  o1 = w8_1<T, INV>(o1);
  o2 = rot<T, INV>(o2);
  o3 = w8_3<T, INV>(o3);
  a[0] = e0 + o0; a[4] = e0 - o0;
  a[1] = e1 + o1; a[5] = e1 - o1;
  a[2] = e2 + o2; a[6] = e2 - o2;
  a[3] = e3 + o3; a[7] = e3 - o3;
}

template <typename T, bool INV>
__device__ __forceinline__ void dft16(cplx<T>* a) {
  cplx<T> e[8], o[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    e[j] = a[2 * j];
    o[j] = a[2 * j + 1];
  }
  dft8<T, INV>(e);
  dft8<T, INV>(o);
  // e^{-+2 pi i k/16}: k = 2, 4, 6 reuse the eighth roots; 1, 3, 5, 7 need a product
  const T c1 = T(0.92387953251128675613), s1 = T(0.38268343236508977173);
  const cplx<T> w1 = INV ? cplx<T>{c1, s1} : cplx<T>{c1, -s1};
  const cplx<T> w3 = INV ? cplx<T>{s1, c1} : cplx<T>{s1, -c1};
  const cplx<T> w5 = INV ? cplx<T>{-s1, c1} : cplx<T>{-s1, -c1};
  const cplx<T> w7 = INV ? cplx<T>{-c1, s1} : cplx<T>{-c1, -s1};
  o[1] = cmul(o[1], w1);
  o[2] = w8_1<T, INV>(o[2]);
  o[3] = cmul(o[3], w3);
  o[4] = rot<T, INV>(o[4]);
  o[5] = cmul(o[5], w5);
  o[6] = w8_3<T, INV>(o[6]);
  o[7] = cmul(o[7], w7);
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    a[k] = e[k] + o[k];
    a[k + 8] = e[k] - o[k];
  }
}

template <typename T, int R, bool INV>
__device__ __forceinline__ void dft(cplx<T>* a) {
  if constexpr (R == 2) dft2<T, INV>(a[0], a[1]);
  else if constexpr (R == 4) dft4<T, INV>(a[0], a[1], a[2], a[3]);
  else if constexpr (R == 8) dft8<T, INV>(a);
  else dft16<T, INV>(a);
}

// ---- LDS view with a one-in-sixteen skew -------------------------------------
// Element i lives at slot i + i/16: the power-of-two strides of the Stockham
// stores (R*16 B, R*T*16 B) then fall on distinct 16-byte bank groups.
template <typename T>
struct Lds {
  cplx<T>* p;
  __device__ __forceinline__ cplx<T>& operator[](int i) const { return p[i + (i >> 4)]; }
};
// Slot of element i, and the distance in slots of elements 2^q apart (q >= 4):
// slot(i + r 2^q) = lds_slot(i) + r lds_step(q), so that an access at a
// compile-time r takes one base register and an immediate offset.
__device__ __forceinline__ int lds_slot(int i) { return i + (i >> 4); }
__host__ __device__ constexpr int lds_step(int q) { return (1 << q) + (1 << q >> 4); }
__host__ __device__ constexpr int lds_slots(int count) { return count + (count >> 4) + 1; }

// Twiddles w_r = e^{-2 pi i r step / 2^logtw} for r = 1..15 from four table loads
// (w1, w2, w4, w8) and products of two or three of them.
template <typename T>
__device__ __forceinline__ void twiddle16_set(const cplx<T>* __restrict__ tw, int step,
                                              cplx<T>* w) {
  w[1] = tw[step];
  w[2] = tw[2 * step];
  w[3] = cmul(w[1], w[2]);
  w[4] = tw[4 * step];
  w[5] = cmul(w[1], w[4]);
  w[6] = cmul(w[2], w[4]);
  w[7] = cmul(w[3], w[4]);
  w[8] = tw[8 * step];
#pragma unroll
  for (int r = 9; r < 16; ++r) w[r] = cmul(w[r - 8], w[8]);
}

// a[r] *= w_r (conjugated for the inverse), r = 1..15, with the same products
// as twiddle16_set formed just before use (conj(x) conj(y) = conj(xy) exactly),
// so that at most eight twiddles are live at a time.
template <typename T, bool INV>
__device__ __forceinline__ void twiddle16_mul(cplx<T> (&a)[16], cplx<T> w1, cplx<T> w2, cplx<T> w4,
                                              cplx<T> w8) {
  if (INV) {
    w1 = conj(w1);
    w2 = conj(w2);
    w4 = conj(w4);
    w8 = conj(w8);
  }
  const cplx<T> w3 = cmul(w1, w2), w5 = cmul(w1, w4), w6 = cmul(w2, w4), w7 = cmul(w3, w4);
  a[1] = cmul(a[1], w1);
  a[2] = cmul(a[2], w2);
  a[3] = cmul(a[3], w3);
  a[4] = cmul(a[4], w4);
  a[5] = cmul(a[5], w5);
  a[6] = cmul(a[6], w6);
  a[7] = cmul(a[7], w7);
  a[8] = cmul(a[8], w8);
  a[9] = cmul(a[9], cmul(w1, w8));
  a[10] = cmul(a[10], cmul(w2, w8));
  a[11] = cmul(a[11], cmul(w3, w8));
  a[12] = cmul(a[12], cmul(w4, w8));
  a[13] = cmul(a[13], cmul(w5, w8));
  a[14] = cmul(a[14], cmul(w6, w8));
  a[15] = cmul(a[15], cmul(w7, w8));
}
template <typename T, bool INV>
__device__ __forceinline__ void twiddle16_apply(cplx<T> (&a)[16], const cplx<T>* __restrict__ tw,
                                                int step) {
  twiddle16_mul<T, INV>(a, tw[step], tw[2 * step], tw[4 * step], tw[8 * step]);
}

// ---- Stockham passes over signals in LDS --------------------------------------
//
// S = 2^logS signals of length M = 2^logM; element i of signal s lives at
// lds[(s << logss) + (i << loges)].  Twiddles come from a base table
// tw[m] = e^{-2 pi i m/2^logtw} (conjugated for the inverse transform),
// M <= 2^logtw.  sigfast: consecutive threads take consecutive signals (use
// when signals are interleaved), otherwise consecutive butterflies.
struct FftGeom {
  int logM, logS, logss, loges, logtw;
  bool sigfast;
};

// One radix-16 pass in place, in natural order; every thread owns at most one
// butterfly.  (One each where it is used: without the tests on `total`, or with
// the indices formed once for both halves, the compiler mixes the pass with what
// surrounds it: up to 30 registers more, and spills.)
template <typename T, bool INV>
__device__ __forceinline__ void stockham16_pass(Lds<T> lds, const FftGeom& g, int logNs,
                                                const cplx<T>* __restrict__ tw) {
  const int lognbs = g.logM - 4;  // butterflies per signal = M / 16
  const int total = 1 << (lognbs + g.logS);
  const int Ns = 1 << logNs;
  cplx<T> a[16];
  const int bf = threadIdx.x;
  if (bf < total) {
    const int s = g.sigfast ? (bf & ((1 << g.logS) - 1)) : (bf >> lognbs);
    const int j = g.sigfast ? (bf >> g.logS) : (bf & ((1 << lognbs) - 1));
    const int base = s << g.logss;
#pragma unroll
    for (int r = 0; r < 16; ++r) a[r] = lds[base + ((j + (r << lognbs)) << g.loges)];
    if (logNs > 0) {
      // e^{-+2 pi i r k / (16 Ns)}, k = j mod Ns
      const int k = j & (Ns - 1);
      cplx<T> w[16];
      twiddle16_set<T>(tw, k << (g.logtw - logNs - 4), w);
#pragma unroll
      for (int r = 1; r < 16; ++r) a[r] = cmul(a[r], INV ? conj(w[r]) : w[r]);
    }
    dft16<T, INV>(a);
  }
  __syncthreads();
  if (bf < total) {
    const int s = g.sigfast ? (bf & ((1 << g.logS) - 1)) : (bf >> lognbs);
    const int j = g.sigfast ? (bf >> g.logS) : (bf & ((1 << lognbs) - 1));
    const int k = j & (Ns - 1);
    const int out = ((j - k) << 4) + k;
    const int base = s << g.logss;
#pragma unroll
    for (int r = 0; r < 16; ++r) lds[base + ((out + (r << logNs)) << g.loges)] = a[r];
  }
  __syncthreads();
}

// ---- radix-8 FFT of one signal, first and last passes on registers ------------
// Each of M/8 threads owns one radix-8 butterfly of the last pass: on entry
// a[e] = x[j0 + e M/8] (natural order), on exit a[e] = X[j0 + e M/8].  The first
// pass (radix 2^(logM mod 3), or 8) works on the registers and writes LDS, the
// last one reads LDS back: M = 512 takes two LDS exchanges, 1024..4096 three.
// The signal's bins are exchanged through `z`; with M <= 2048 two buffers
// alternate in it (one barrier per exchange instead of two), and where one
// wavefront holds the signal (M <= 512) the exchanges need no barrier at all.
// The inverse transform is conj(F(conj x)), by the caller.
template <bool kWave>
__device__ __forceinline__ void fft_sync() {
  if constexpr (kWave) {
    // one wavefront's LDS accesses are in order: only the compiler is held
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  } else {
    __syncthreads();
  }
}

// Hides a value's origin from the optimiser: what is derived from it inside a
// loop is recomputed there instead of being kept in registers across the
// loop (LDS addresses of every geometry, which spilled).
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Twiddle bases w, w^2, w^4 of the radix-8 passes after the first, from a
// table of e^{-2 pi i m / 2^logtab}, m < 2^(logtab-1): read at each pass (a
// table in LDS) or, FftTw8, all fetched beforehand (a table in memory).
template <typename T>
struct FftTab8 {
  const cplx<T>* tab;
  int logtab;
  __device__ __forceinline__ void get(int, int logNs, int j0, cplx<T> (&w)[3]) const {
    const int step = (j0 & ((1 << logNs) - 1)) << (logtab - logNs - 3);
    w[0] = tab[step];
    w[1] = tab[2 * step];
    w[2] = tab[4 * step];
  }
};
template <typename T>
struct FftTw8 {
  cplx<T> w[3][3];
  __device__ __forceinline__ void load(int logM, int j0, const FftTab8<T>& t) {
    int logNs = logM % 3 == 0 ? 3 : logM % 3;
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      if (logNs < logM) t.get(p, logNs, j0, w[p]);
      logNs += 3;
    }
  }
  __device__ __forceinline__ void get(int p, int, int, cplx<T> (&v)[3]) const {
#pragma unroll
    for (int i = 0; i < 3; ++i) v[i] = w[p][i];
  }
};

template <typename T>
__device__ __forceinline__ void twiddle8_mul(cplx<T> (&a)[8], const cplx<T> (&w)[3]) {
  const cplx<T> w3 = cmul(w[0], w[1]);
  a[1] = cmul(a[1], w[0]);
  a[2] = cmul(a[2], w[1]);
  a[3] = cmul(a[3], w3);
  a[4] = cmul(a[4], w[2]);
  a[5] = cmul(a[5], cmul(w[0], w[2]));
  a[6] = cmul(a[6], cmul(w[1], w[2]));
  a[7] = cmul(a[7], cmul(w3, w[2]));
}

template <typename T, int R0>
__device__ __forceinline__ void first_pass8(const cplx<T> (&a)[8], Lds<T> lds, int j0, int q) {
  constexpr int NB = 8 / R0;
#pragma unroll
  for (int e = 0; e < NB; ++e) {
    cplx<T> b[R0];
#pragma unroll
    for (int r = 0; r < R0; ++r) b[r] = a[e + r * NB];  // x[j + r M/R0], j = j0 + e M/8
    dft<T, R0, false>(b);
    const int j = j0 + (e << q);
#pragma unroll
    for (int r = 0; r < R0; ++r) lds[j * R0 + r] = b[r];
  }
}

// LOGM = 0: 8 <= M = 2^logMr <= 256 at run time.  act: this thread is one of
// the M/8.  Every thread of the workgroup calls it (unless M <= 512, where the
// first wavefront's threads do).  Two buffers of kFft8Half slots in z; after
// the call the second one is free to write where LOGM is 10 or 11.
constexpr int kFft8Half = lds_slots(2048);
template <typename T, int LOGM, typename TW>
__device__ __forceinline__ void fft8(cplx<T> (&a)[8], Lds<T> z, int logMr, int j0, bool act,
                                     const TW& f) {
  constexpr bool kWave = LOGM <= 9;
  constexpr bool kPing = LOGM == 10 || LOGM == 11;
  const int logM = LOGM ? LOGM : logMr;
  const int q = logM - 3, rem = logM % 3;
  static_assert(LOGM == 0 || LOGM >= 7, "lds_step needs q >= 4");
  const int sj = lds_slot(j0);
  if (LOGM == 0 && q == 0) {
    if (act) dft8<T, false>(a);
    return;
  }
  if (act) {
    if (rem == 1) first_pass8<T, 2>(a, z, j0, q);
    else if (rem == 2) first_pass8<T, 4>(a, z, j0, q);
    else first_pass8<T, 8>(a, z, j0, q);
  }
  fft_sync<kWave>();
  int logNs = rem == 0 ? 3 : rem;
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    if (logNs < logM) {
      const Lds<T> cur{z.p + (kPing && (p & 1) ? kFft8Half : 0)};
      if (act) {
#pragma unroll
        for (int r = 0; r < 8; ++r)
          a[r] = LOGM ? cur.p[sj + r * lds_step(q)] : cur[j0 + (r << q)];
        cplx<T> w[3];
        f.get(p, logNs, j0, w);
        twiddle8_mul(a, w);
        dft8<T, false>(a);
      }
      if (logNs + 3 < logM) {
        if constexpr (!kPing && !kWave) __syncthreads();
        if (act) {
          const Lds<T> nxt{z.p + (kPing && !(p & 1) ? kFft8Half : 0)};
          const int k = j0 & ((1 << logNs) - 1);
          const int out = ((j0 - k) << 3) + k;
#pragma unroll
          for (int r = 0; r < 8; ++r) nxt[out + (r << logNs)] = a[r];
        }
        fft_sync<kWave>();
      }
    }
    logNs += 3;
  }
}

// FFT of the signals in LDS with the first and last passes on registers.
// Each thread owns one radix-16 butterfly of the last pass: signal s, index
// j0 < M/16 (M = 2^logM >= 32).  On entry a[e] = x_s[j0 + e M/16] (natural
// order), on exit a[e] = X_s[j0 + e M/16]; the NT threads of the workgroup
// must cover every (s, j0) pair exactly once.  The first pass (radix
// 2^(logM mod 4), or 16) works on the registers and writes LDS, the middle
// radix-16 passes stay in LDS, the last one reads LDS back into registers.
// No barrier at the end: synchronise before the LDS region is written again.
template <typename T, int R0, bool INV>
__device__ __forceinline__ void first_pass_regs(cplx<T> (&a)[16], Lds<T> lds, const FftGeom& g,
                                                int base, int j0, int q) {
  constexpr int NB = 16 / R0;
#pragma unroll
  for (int e = 0; e < NB; ++e) {
    cplx<T> b[R0];
#pragma unroll
    for (int r = 0; r < R0; ++r) b[r] = a[e + r * NB];  // x[j + r M/R0], j = j0 + e M/16
    dft<T, R0, INV>(b);
    const int j = j0 + (e << q);
#pragma unroll
    for (int r = 0; r < R0; ++r) lds[base + ((j * R0 + r) << g.loges)] = b[r];
  }
}

template <typename T, int NT, bool INV>
__device__ __forceinline__ void fft_reg16(cplx<T> (&a)[16], Lds<T> lds, const FftGeom& g, int s,
                                          int j0, const cplx<T>* __restrict__ tw) {
  const int q = g.logM - 4;  // log2(M/16)
  const int base = s << g.logss;
  const int rem = g.logM & 3;
  if (rem == 1) first_pass_regs<T, 2, INV>(a, lds, g, base, j0, q);
  else if (rem == 2) first_pass_regs<T, 4, INV>(a, lds, g, base, j0, q);
  else if (rem == 3) first_pass_regs<T, 8, INV>(a, lds, g, base, j0, q);
  else first_pass_regs<T, 16, INV>(a, lds, g, base, j0, q);
  __syncthreads();
  for (int logNs = rem == 0 ? 4 : rem; logNs < q; logNs += 4)
    stockham16_pass<T, INV>(lds, g, logNs, tw);
  // last pass, Ns = M/16: butterfly j0 (k = j0), outputs j0 + r M/16
#pragma unroll
  for (int r = 0; r < 16; ++r) a[r] = lds[base + ((j0 + (r << q)) << g.loges)];
  twiddle16_apply<T, INV>(a, tw, j0 << (g.logtw - g.logM));
  dft<T, 16, INV>(a);
}

// The radix-8 register FFT for several interleaved or consecutive signals of
// M = 2^LOGM points in one workgroup: element i of the thread's signal lies at
// base + (i << LOGES).  Its exchanges (one for M = 64, two up to 512, three at
// 1024) are numbered from EX0 and alternate between two buffers `half` slots
// apart, one barrier each; with kWave (the workgroup is one wavefront) there is
// one buffer and no barrier.  After the call the buffer of exchange
// EX0 + fft8_exchanges(LOGM) is free to write.
constexpr int fft8_exchanges(int logM) { return (logM - (logM % 3 == 0 ? 3 : logM % 3)) / 3; }
template <typename T, int LOGM, int LOGES, bool kWave, int EX0>
__device__ __forceinline__ void fft8_sig(cplx<T> (&a)[8], Lds<T> z, int half, int base, int j0,
                                         const FftTw8<T>& f) {
  constexpr int q = LOGM - 3, rem = LOGM % 3, R0 = rem == 0 ? 8 : 1 << rem, NB = 8 / R0;
  constexpr int X = fft8_exchanges(LOGM);
  static_assert(LOGM >= 6 && q + LOGES >= 4, "lds_step needs strides of 16");
  auto buf = [&](int ex) { return Lds<T>{z.p + (!kWave && (ex & 1) ? half : 0)}; };
  const int sj = lds_slot(base + (j0 << LOGES));
  {
    const Lds<T> w = buf(EX0);
#pragma unroll
    for (int e = 0; e < NB; ++e) {
      cplx<T> b[R0];
#pragma unroll
      for (int r = 0; r < R0; ++r) b[r] = a[e + r * NB];  // x[j + r M/R0], j = j0 + e M/8
      dft<T, R0, false>(b);
      const int j = j0 + (e << q);
#pragma unroll
      for (int r = 0; r < R0; ++r) w[base + ((j * R0 + r) << LOGES)] = b[r];
    }
  }
  fft_sync<kWave>();
#pragma unroll
  for (int p = 0; p < X; ++p) {
    const int logNs = (rem == 0 ? 3 : rem) + 3 * p;
    const Lds<T> cur = buf(EX0 + p);
#pragma unroll
    for (int r = 0; r < 8; ++r) a[r] = cur.p[sj + r * lds_step(q + LOGES)];
    cplx<T> w[3];
    f.get(p, logNs, j0, w);
    twiddle8_mul(a, w);
    dft8<T, false>(a);
    if (p + 1 < X) {
      const Lds<T> nxt = buf(EX0 + p + 1);
      const int k = j0 & ((1 << logNs) - 1);
      const int out = base + ((((j0 - k) << 3) + k) << LOGES);
#pragma unroll
      for (int r = 0; r < 8; ++r) nxt[out + (r << (logNs + LOGES))] = a[r];
      fft_sync<kWave>();
    }
  }
}

// Sum over the wavefront in lane 63 (a fixed order), by data-parallel moves in
// the register file: the shuffles of wave_sum go through the LDS unit.
template <int CTRL, int ROWS, typename T>
__device__ __forceinline__ T dpp_or_zero(T v) {
  if constexpr (sizeof(T) == 4) {
    const int x = __builtin_bit_cast(int, v);
    return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xf, false));
  } else {
    const long long x = __builtin_bit_cast(long long, v);
    const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xf, false);
    const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(x >> 32), CTRL, ROWS, 0xf, false);
    return __builtin_bit_cast(T, ((unsigned long long)hi << 32) | lo);
  }
}
template <typename T>
__device__ __forceinline__ T wave_sum63(T v) {
  v += dpp_or_zero<0x111, 0xf>(v);  // row_shr 1, 2, 4, 8: lane 15 of each row of 16
  v += dpp_or_zero<0x112, 0xf>(v);
  v += dpp_or_zero<0x114, 0xf>(v);
  v += dpp_or_zero<0x118, 0xf>(v);
  v += dpp_or_zero<0x142, 0xa>(v);  // row_bcast 15 into rows 1 and 3
  v += dpp_or_zero<0x143, 0xc>(v);  // row_bcast 31 into rows 2 and 3
  return v;
}

// Deterministic reduction of one value per thread over a workgroup of NT
// threads: butterfly within each wave (lane 0's fixed order), then the wave
// partials in index order.  Every thread returns the same value.
template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
template <typename T, int NT>
__device__ __forceinline__ T block_sum(T v, T* red /* >= NT/64 entries */) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  T s = red[0];
#pragma unroll
  for (int w = 1; w < NT / 64; ++w) s += red[w];
  __syncthreads();
  return s;
}

}  // namespace amg
