// fft.hpp -- LDS-staged Stockham FFTs for gfx950 (wave64).
//
// The paper moves every field between real and reciprocal space twice per
// step with a library 2D FFT (Appendix B, stage 1b); here the 2D transform is
// split into a real-to-complex transform along each row (x) and a complex
// transform along each column (y), and both halves are fused into the stage
// kernels.  This header holds the building blocks:
//
//   * c2<T>          complex value (T = float or double);
//   * dft_reg        radix-R DFT on R values held in registers (R <= 16);
//   * fft_group      length-L complex FFT done by a group of L/E threads that
//                    each hold E values, exchanging through LDS between the
//                    passes (Stockham autosort: natural order in and out),
//                    its twiddles read from the table pass by pass;
//   * fft_regs       the same for kernels that run several transforms of one
//                    length, the passes' twiddles read once (PassSet);
//   * row_r2c/c2r    real row of 2L values <-> L packed complex values.
//
// Forward transforms are unnormalised, F[a](m) = sum_i a_i exp(-2 pi i m i/n).
#pragma once

#include <hip/hip_runtime.h>

namespace le {

template <typename T>
struct alignas(2 * sizeof(T)) c2 {
  T x, y;
};

// Pointer into device global memory.  The run descriptors hold plain
// pointers; giving them the global address space lets every access compile
// to global_load/store, which (unlike flat accesses) do not share the LDS
// wait counter, so LDS passes do not wait on outstanding memory traffic.
template <typename T>
using gp = __attribute__((address_space(1))) T*;
template <typename T>
__device__ __forceinline__ gp<T> to_global(const void* p) {
  return (gp<T>)(p);
}

// Whole-value load and store of a complex through a global pointer (one
// 8- or 16-byte access).
template <typename T>
using vec2 = T __attribute__((ext_vector_type(2)));
template <typename T>
__device__ __forceinline__ c2<T> ldg(gp<const c2<T>> p) {
  const vec2<T> v = *reinterpret_cast<gp<const vec2<T>>>(p);
  return {v.x, v.y};
}
template <typename T>
__device__ __forceinline__ c2<T> ldg(gp<c2<T>> p) {
  return ldg<T>(static_cast<gp<const c2<T>>>(p));
}
template <typename T>
__device__ __forceinline__ void stg(gp<c2<T>> p, c2<T> a) {
  *reinterpret_cast<gp<vec2<T>>>(p) = vec2<T>{a.x, a.y};
}

template <typename T>
__device__ __forceinline__ c2<T> cadd(c2<T> a, c2<T> b) { return {a.x + b.x, a.y + b.y}; }
template <typename T>
__device__ __forceinline__ c2<T> csub(c2<T> a, c2<T> b) { return {a.x - b.x, a.y - b.y}; }
template <typename T>
__device__ __forceinline__ c2<T> cmul(c2<T> a, c2<T> b) {
  return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
// a * conj(b)
template <typename T>
__device__ __forceinline__ c2<T> cmulc(c2<T> a, c2<T> b) {
  return {a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y};
}

// cos and sin of 2 pi k / 16, k = 0..15, to double precision.
__device__ constexpr double kCos16[16] = {
    1.0, 0.92387953251128675613, 0.70710678118654752440, 0.38268343236508977173,
    0.0, -0.38268343236508977173, -0.70710678118654752440, -0.92387953251128675613,
    -1.0, -0.92387953251128675613, -0.70710678118654752440, -0.38268343236508977173,
    0.0, 0.38268343236508977173, 0.70710678118654752440, 0.92387953251128675613};
__device__ constexpr double kSin16[16] = {
    0.0, 0.38268343236508977173, 0.70710678118654752440, 0.92387953251128675613,
    1.0, 0.92387953251128675613, 0.70710678118654752440, 0.38268343236508977173,
    0.0, -0.38268343236508977173, -0.70710678118654752440, -0.92387953251128675613,
    -1.0, -0.92387953251128675613, -0.70710678118654752440, -0.38268343236508977173};

// d * exp(DIR * 2 pi i * k / R), DIR = -1 forward, +1 inverse.  k is a
// compile-time constant after unrolling, so the trivial cases fold away.
template <typename T, int DIR, int R>
__device__ __forceinline__ c2<T> rot(c2<T> d, int k) {
  k &= (R - 1);
  if (k == 0) return d;
  if (4 * k == R) return DIR < 0 ? c2<T>{d.y, -d.x} : c2<T>{-d.y, d.x};
  if (2 * k == R) return {-d.x, -d.y};
  if (4 * k == 3 * R) return DIR < 0 ? c2<T>{-d.y, d.x} : c2<T>{d.y, -d.x};
  const int i16 = k * (16 / R);
  const T cr = static_cast<T>(kCos16[i16]);
  const T sr = static_cast<T>(DIR * kSin16[i16]);
  return {d.x * cr - d.y * sr, d.x * sr + d.y * cr};
}

constexpr int ilog2(int n) { return n <= 1 ? 0 : 1 + ilog2(n / 2); }
constexpr int bitrev(int i, int bits) {
  int r = 0;
  for (int b = 0; b < bits; ++b) r |= ((i >> b) & 1) << (bits - 1 - b);
  return r;
}

// A pass multiplies its radix-R inputs by powers of a twiddle and transforms
// them, in one of two forms.  Folded: the twiddles go into a decimation-in-time
// DFT's butterflies, six fused multiply-adds each; with R = 16 a pass takes 236
// operations, the twiddles' formation included, the separate form (R - 1
// products, then the DFT) 321 and more registers.  FP64 takes the folded form
// (4096^2 step 840 -> 825 us).  FP32 keeps the separate one: a transform's
// result shrinks by the rounding of the low-order roots, which a run adds up
// step after step, and the folded form shrinks more for R <= 8 (512 points:
// 2.9e-8 per transform against 2.4e-8).  For R = 16 it shrinks less (4096 points:
// 3.2e-8 against 4.7e-8, and 3.0e-8 with R = 8): the column passes, bound by
// these operations, take it there.
template <typename T, int R>
constexpr bool kFolded = sizeof(T) == 8;

// Separate form: radix-2 decimation in frequency, then a compile-time
// bit-reversal rename.
template <typename T, int DIR, int R>
__device__ __forceinline__ void dft_dif(c2<T>* v) {
  if constexpr (R >= 2) {
#pragma unroll
    for (int span = R / 2; span >= 1; span >>= 1) {
#pragma unroll
      for (int start = 0; start < R; start += 2 * span) {
#pragma unroll
        for (int k = 0; k < span; ++k) {
          const c2<T> a = v[start + k];
          const c2<T> b = v[start + k + span];
          v[start + k] = cadd(a, b);
          v[start + k + span] = rot<T, DIR, R>(csub(a, b), k * (R / (2 * span)));
        }
      }
    }
    constexpr int bits = ilog2(R);
    c2<T> tmp[R];
#pragma unroll
    for (int i = 0; i < R; ++i) tmp[i] = v[bitrev(i, bits)];
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = tmp[i];
  }
}

// cos(k pi / 8), k = 0 .. 3 (sin(k pi / 8) is the mirrored entry), to double
// precision.
__device__ constexpr double kCosPi8[5] = {1.0, 0.92387953251128675613, 0.70710678118654752440,
                                          0.38268343236508977173, 0.0};

// Butterfly a, b <- a + c b, a - c b with c = w, or (TURN) w turned by a
// quarter: w exp(DIR i pi / 2).  DIR > 0 takes conj(w).  Six fused
// multiply-adds: the sum by two per component, the difference as 2a minus it.
template <typename T, int DIR, bool TURN>
__device__ __forceinline__ void bfly(c2<T>& a, c2<T>& b, c2<T> w) {
  const T wy = DIR < 0 ? w.y : -w.y;
  T x, y;
  if constexpr (!TURN) {
    x = fma(-wy, b.y, fma(w.x, b.x, a.x));
    y = fma(wy, b.x, fma(w.x, b.y, a.y));
  } else if constexpr (DIR < 0) {  // -i w b
    x = fma(wy, b.x, fma(w.x, b.y, a.x));
    y = fma(wy, b.y, fma(-w.x, b.x, a.y));
  } else {  // +i conj(w) b
    x = fma(-wy, b.x, fma(-w.x, b.y, a.x));
    y = fma(-wy, b.y, fma(w.x, b.x, a.y));
  }
  b = {fma(T(2), a.x, -x), fma(T(2), a.y, -y)};
  a = {x, y};
}
// The same with c = 1, or (TURN) exp(DIR i pi / 2).
template <typename T, int DIR, bool TURN>
__device__ __forceinline__ void bfly1(c2<T>& a, c2<T>& b) {
  const c2<T> t = !TURN ? b : (DIR < 0 ? c2<T>{b.y, -b.x} : c2<T>{-b.y, b.x});
  b = csub(a, t);
  a = cadd(a, t);
}

// The twiddles of a radix-R pass: v[r] is multiplied by w^r before the
// length-R DFT.  Folded into the DFT's butterflies (decimation in time), level
// S = 2, 4, .. R needs w^(R/S) exp(-2 pi i k / S), k < S/4 (k = 0 for S = 2),
// the others being quarter turns of these: R/2 values instead of R - 1
// powers, formed in FP64 and rounded once to T.
//
// PassIn: what they are formed from, w or, TWO (FP64), w and w^Q of the table.
// Each squaring doubles a power's relative rounding: from w alone, w^8 carries
// ten times w's, the larger part of a transform's error (RMS at 2048 points,
// R = 16: 5.1e-16 from w, 2.8e-16 from w and w^4; R = 8: 3.9e-16 and 2.7e-16;
// 256 points, R = 4: 2.3e-16 and, w and w^2, 1.9e-16).
template <typename T, int R, bool TWO_>
struct PassIn {
  static constexpr int Q = R >= 8 ? 4 : 2;
  static constexpr bool TWO = TWO_ && sizeof(T) == 8 && R >= 4;
  c2<double> w, wq;
  // entry i (< n / R) of the table exp(-2 pi i k / n), k < n
  __device__ __forceinline__ void load(gp<const c2<double>> tw, int i) {
    w = ldg<double>(tw + i);
    if constexpr (TWO) wq = ldg<double>(tw + Q * i);
  }
};
template <typename T, int R, bool FOLDED = kFolded<T, R>>
struct PassW {
  static constexpr int N = R >= 4 ? R / 2 : 1;
  c2<T> w[N];  // level R: w[0 .. R/4), level R/2: the next R/8, .., 4: 1, 2: 1
  template <typename In>
  __device__ __forceinline__ void set(const In& in) {
    c2<double> b = in.w;  // w^(R/S)
#pragma unroll
    for (int S = R; S >= 2; S >>= 1) {
      if (In::TWO && In::Q * S == R) b = in.wq;
      const int n = S >= 4 ? S / 4 : 1, o = off(S);
#pragma unroll
      for (int k = 0; k < n; ++k) {
        // exp(-2 pi i k / S) = cos, -sin of (16 k / S) pi / 8
        const int q = 16 * k / S;
        const c2<double> z = k == 0 ? b : cmul(b, c2<double>{kCosPi8[q], -kCosPi8[4 - q]});
        w[o + k] = {static_cast<T>(z.x), static_cast<T>(z.y)};
      }
      b = cmul(b, b);
    }
  }
  static constexpr int off(int S) {
    int o = 0;
    for (int s = R; s > S; s >>= 1) o += s >= 4 ? s / 4 : 1;
    return o;
  }
};
// Separate form: the powers w^r (r = 1 .. R-1) from a product tree of depth <= 3
// in FP64 (error ~1e-15), each rounded once.
template <typename T, int R>
struct PassW<T, R, false> {
  c2<T> w[R];
  __device__ __forceinline__ void put(int r, c2<double> a) {
    w[r] = {static_cast<T>(a.x), static_cast<T>(a.y)};
  }
  template <typename In>
  __device__ __forceinline__ void set(const In& in) {
    const c2<double> w1 = in.w;
    if constexpr (R >= 2) put(1, w1);
    if constexpr (R >= 4) {
      const c2<double> w2 = cmul(w1, w1), w3 = cmul(w2, w1);
      put(2, w2);
      put(3, w3);
      if constexpr (R >= 8) {
        const c2<double> w4 = cmul(w2, w2);
        const c2<double> hi[4] = {w4, cmul(w4, w1), cmul(w4, w2), cmul(w4, w3)};
#pragma unroll
        for (int r = 0; r < 4; ++r) put(4 + r, hi[r]);
        if constexpr (R >= 16) {
          const c2<double> w8 = cmul(w4, w4);
          put(8, w8);
          put(9, cmul(w8, w1));
          put(10, cmul(w8, w2));
          put(11, cmul(w8, w3));
#pragma unroll
          for (int r = 0; r < 4; ++r) put(12 + r, cmul(w8, hi[r]));
        }
      }
    }
  }
};

// Radix-R DFT of v (R = 1, 2, 4, 8, 16; natural order in and out) with the
// pass's twiddles: v[k] <- sum_r w^r v[r] exp(DIR 2 pi i r k / R), w conjugated
// for DIR > 0.
template <typename T, int DIR, int R, bool FOLDED>
__device__ __forceinline__ void dft_tw(c2<T>* v, const PassW<T, R, FOLDED>& pw) {
  if constexpr (!FOLDED) {
#pragma unroll
    for (int r = 1; r < R; ++r) v[r] = DIR < 0 ? cmul(v[r], pw.w[r]) : cmulc(v[r], pw.w[r]);
    dft_dif<T, DIR, R>(v);
  } else {
    constexpr int bits = ilog2(R);
    c2<T> a[R];
#pragma unroll
    for (int i = 0; i < R; ++i) a[i] = v[bitrev(i, bits)];
#pragma unroll
    for (int S = 2; S <= R; S <<= 1) {
#pragma unroll
      for (int g = 0; g < R; g += S) {
#pragma unroll
        for (int k = 0; k < S / 2; ++k) {
          c2<T>& x = a[g + k];
          c2<T>& y = a[g + k + S / 2];
          const int n = S >= 4 ? S / 4 : 1;
          if (k < n)
            bfly<T, DIR, false>(x, y, pw.w[PassW<T, R, FOLDED>::off(S) + k]);
          else
            bfly<T, DIR, true>(x, y, pw.w[PassW<T, R, FOLDED>::off(S) + k - n]);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = a[i];
  }
}

// The same without twiddles.
template <typename T, int DIR, int R, bool FOLDED = kFolded<T, R>>
__device__ __forceinline__ void dft_reg(c2<T>* v) {
  if constexpr (!FOLDED) {
    dft_dif<T, DIR, R>(v);
  } else if constexpr (R >= 2) {
    constexpr int bits = ilog2(R);
    c2<T> a[R];
#pragma unroll
    for (int i = 0; i < R; ++i) a[i] = v[bitrev(i, bits)];
#pragma unroll
    for (int S = 2; S <= R; S <<= 1) {
#pragma unroll
      for (int g = 0; g < R; g += S) {
#pragma unroll
        for (int k = 0; k < S / 2; ++k) {
          c2<T>& x = a[g + k];
          c2<T>& y = a[g + k + S / 2];
          if (k == 0)
            bfly1<T, DIR, false>(x, y);
          else if (4 * k == S)
            bfly1<T, DIR, true>(x, y);
          else {
            const int q = (16 * k / S) & 3;  // angle within the quarter
            const c2<T> w = {static_cast<T>(kCosPi8[q]), static_cast<T>(-kCosPi8[4 - q])};
            if (4 * k < S)
              bfly<T, DIR, false>(x, y, w);
            else
              bfly<T, DIR, true>(x, y, w);
          }
        }
      }
    }
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = a[i];
  }
}

// Radix of the first Stockham pass: L / E^n with 1 < R0 <= E.
constexpr int first_radix(int L, int E) {
  int r = L;
  while (r > E) r /= E;
  return r;
}

// Elements per thread used for a transform of length L.
constexpr int elems_for(int L) { return L >= 1024 ? 16 : (L >= 8 ? 8 : L); }

// Number of LDS passes (twiddled radix-E passes) of a length-L transform.
constexpr int fft_passes(int L, int E) {
  int n = 0;
  for (int Ns = first_radix(L, E); Ns < L; Ns *= E) ++n;
  return n;
}

// LDS slot of element i of a transform's exchange area, a permutation within
// aligned runs of elements (the area keeps its size) that spreads the strided
// accesses of the Stockham passes over the banks.  LDS serves 128 bytes per
// clock: 8 lanes of 16-byte (FP64) complex values or 16 lanes of 8-byte
// (FP32) ones.  FP64: the low three bits XORed by bits 3..5 and 4..6, which
// puts any 8 consecutive lanes of the passes' accesses (first-pass strides of
// 2 to 16 elements, later passes' groups of 2 to 256) and any 8 consecutive
// elements on distinct bank groups.  FP32: the low four bits XORed by the
// next four (lanes 16 or more elements apart).
template <typename T>
__device__ __forceinline__ int lds_slot(int i) {
  if constexpr (sizeof(T) == 8) return i ^ (((i >> 3) ^ (i >> 4)) & 7);
  return i ^ ((i >> 4) & 15);
}

// Orders a group's LDS accesses between the steps of a transform.  WAVE: the
// group lies within one wavefront, whose LDS operations execute in order, so
// only the compiler has to keep them in order; else a block barrier.
template <bool WAVE>
__device__ __forceinline__ void group_sync() {
  if constexpr (WAVE) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  } else {
    __syncthreads();
  }
}

// Length-L complex FFT by a group of P = L/E threads; thread t in [0, P).
// On entry v[q] = x[t + q P]; on exit v[q] = X[t + q P].
// lds: the group's LDS area, element i at lds[lds_slot<T>(i) * LS].  tw: the FP64 table
// exp(-2 pi i k / (2L)), k < 2L.  Pass p (stride Ns = R0 E^p) needs w^r,
// w = exp(-2 pi i k / (Ns E)), k = t mod Ns, r = 1 .. E-1: w is read from
// the table one pass ahead (its latency hides behind the pass before), the
// powers are formed in FP64 and rounded once to T.  Every thread of the
// block must call this with the same L (the passes contain
// __syncthreads()).  On return other threads may still read lds: barrier
// before reusing it.
template <typename T, int L, int E, int DIR>
__device__ __forceinline__ void fft_group(c2<T>* v, c2<T>* lds, int LS,
                                          gp<const c2<double>> __restrict__ tw, int t) {
  constexpr int P = L / E;
  constexpr int R0 = first_radix(L, E);
  constexpr int Q = E / R0;
  static_assert(L % E == 0 && E % R0 == 0, "bad FFT factorisation");
  // pass 0: radix R0, Q butterflies per thread, operands already in registers
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    c2<T> b[R0];
#pragma unroll
    for (int r = 0; r < R0; ++r) b[r] = v[q + r * Q];
    dft_reg<T, DIR, R0>(b);
    if constexpr (L == R0) {
#pragma unroll
      for (int r = 0; r < R0; ++r) v[r] = b[r];
    } else {
      const int j = t + q * P;
#pragma unroll
      for (int r = 0; r < R0; ++r) lds[lds_slot<T>(j * R0 + r) * LS] = b[r];
    }
  }
  if constexpr (L > R0) {
    constexpr int NP = fft_passes(L, E);
    // entry (2L/E)/Ns (t mod Ns): even, below 2L/E, as Ns <= L/E
    typedef PassIn<T, E, false> In;
    In wn;
    wn.load(tw, (2 * L / E) / R0 * (t & (R0 - 1)));
    int Ns = R0;
#pragma unroll
    for (int pass = 0; pass < NP; ++pass) {
      const In w = wn;
      if (pass + 1 < NP) wn.load(tw, (2 * L / E) / (Ns * E) * (t & (Ns * E - 1)));
      __syncthreads();
#pragma unroll
      for (int r = 0; r < E; ++r) v[r] = lds[lds_slot<T>(t + r * P) * LS];
      PassW<T, E> pw;
      pw.set(w);
      dft_tw<T, DIR, E>(v, pw);
      if (pass + 1 == NP) break;
      __syncthreads();
      const int k = t & (Ns - 1);
      const int idxD = (t / Ns) * Ns * E + k;
#pragma unroll
      for (int r = 0; r < E; ++r) lds[lds_slot<T>(idxD + r * Ns) * LS] = v[r];
      Ns *= E;
    }
  }
}

// The passes' twiddles of a kernel that runs several transforms of one length:
// per pass and thread w = exp(-2 pi i (t mod Ns) / (Ns E)) and, TWO, its power,
// read from the table once (fft_regs then touches no global memory).  KEEP: what a
// pass forms from them (PassW) stays in registers (FP32, and up to 8 values in
// FP64 where LDS and grid leave the registers free); else it is formed at each
// use, from registers or, with LDSW (NT threads), from the thread's own place in
// LDS.  SHARED (FP64): one place per t in LDS, filled by the block's first group
// of P threads for all of them (a read of the table by every group costs a
// joined kernel 0.2 us per power); load(), a block barrier, then form().
template <typename T, int L, int E, int LDSW_ = 0, bool FOLDED_ = kFolded<T, E>, bool TWO = true,
          bool SHARED_ = false>
struct PassSet {
  static constexpr bool FOLDED = FOLDED_;
  typedef PassIn<T, E, TWO> In;
  static constexpr int NP = fft_passes(L, E), NPA = NP > 0 ? NP : 1;
  static constexpr bool KEEP = sizeof(T) == 4 || E <= 4 || (E == 8 && L <= 1024);
  static constexpr bool SHARED = SHARED_ && sizeof(T) == 8;
  static constexpr int LDSW = SHARED ? L / E : (KEEP ? 0 : LDSW_);
  static constexpr int NLDS = LDSW > 0 ? (In::TWO ? 2 : 1) * NPA * LDSW : 1;  // values of `area`
  In in[KEEP || LDSW > 0 ? 1 : NPA];
  PassW<T, E, FOLDED> pw[KEEP ? NPA : 1];
  c2<double>* area;
  __device__ __forceinline__ void load(gp<const c2<double>> tw, int t, c2<double>* lds = nullptr) {
    int Ns = first_radix(L, E);
    if constexpr (LDSW > 0) area = lds + (SHARED ? t : (int)threadIdx.x);
    if (SHARED && (int)threadIdx.x >= LDSW) return;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      In a;
      a.load(tw, (2 * L / E) / Ns * (t & (Ns - 1)));
      if constexpr (LDSW > 0) {
        area[p * LDSW] = a.w;
        if constexpr (In::TWO) area[(NPA + p) * LDSW] = a.wq;
      } else if constexpr (KEEP) {
        pw[p].set(a);
      } else {
        in[p] = a;
      }
      Ns *= E;
    }
  }
  __device__ __forceinline__ In get(int p) const {
    In a;
    a.w = area[p * LDSW];
    if constexpr (In::TWO) a.wq = area[(NPA + p) * LDSW];
    return a;
  }
  __device__ __forceinline__ void form() {
    if constexpr (SHARED && KEEP) {
#pragma unroll
      for (int p = 0; p < NP; ++p) pw[p].set(get(p));
    }
  }
  template <int DIR>
  __device__ __forceinline__ void pass(c2<T>* v, int p) const {
    if constexpr (KEEP) {
      dft_tw<T, DIR, E>(v, pw[p]);
    } else {
      In a = LDSW > 0 ? get(p) : in[LDSW > 0 ? 0 : p];
      // opaque, so that the compiler does not keep what it forms from them
      asm volatile("" : "+v"(a.w.x), "+v"(a.w.y));
      if constexpr (In::TWO) asm volatile("" : "+v"(a.wq.x), "+v"(a.wq.y));
      PassW<T, E, FOLDED> f;
      f.set(a);
      dft_tw<T, DIR, E>(v, f);
    }
  }
};

// fft_group's transform with the passes' factors from registers and the
// group's own ordering (WAVE, group_sync).  On return other threads of the
// group may still read lds.
template <typename T, int L, int E, int DIR, bool WAVE, typename TW>
__device__ __forceinline__ void fft_regs(c2<T>* v, c2<T>* lds, int LS, const TW& tw, int t) {
  constexpr int P = L / E;
  constexpr int R0 = first_radix(L, E);
  constexpr int Q = E / R0;
  constexpr int NP = fft_passes(L, E);
  static_assert(L % E == 0 && E % R0 == 0, "bad FFT factorisation");
  // values v[i] to elements dst(i), then v[r] = element t + r P
  auto exchange = [&](auto&& dst) {
#pragma unroll
    for (int i = 0; i < E; ++i) lds[lds_slot<T>(dst(i)) * LS] = v[i];
    group_sync<WAVE>();
#pragma unroll
    for (int r = 0; r < E; ++r) v[r] = lds[lds_slot<T>(t + r * P) * LS];
  };
  // pass 0: value q + r Q is input r of butterfly t + q P
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    c2<T> b[R0];
#pragma unroll
    for (int r = 0; r < R0; ++r) b[r] = v[q + r * Q];
    dft_reg<T, DIR, R0, TW::FOLDED>(b);
#pragma unroll
    for (int r = 0; r < R0; ++r) v[q + r * Q] = b[r];
  }
  if constexpr (L > R0) {
    exchange([&](int i) { return (t + (i % Q) * P) * R0 + i / Q; });
    int Ns = R0;
#pragma unroll
    for (int pass = 0; pass < NP; ++pass) {
      tw.template pass<DIR>(v, pass);
      if (pass + 1 == NP) break;
      group_sync<WAVE>();
      const int d = (t / Ns) * Ns * E + (t & (Ns - 1)), n = Ns;
      exchange([&](int i) { return d + i * n; });
      Ns *= E;
    }
  }
}

// exp(-i pi q / E) for q < E, E a power of two up to 16 (cos and sin of
// multiples of pi/16, correctly rounded).  The table entry m = t + q L/E of
// exp(-2 pi i m / (2L)) is tw[t] times this, so a transform thread that
// needs the E entries t + q L/E reads one and forms the others in FP64.
__device__ constexpr double kCosPi16[9] = {1.0,
                                           0.98078528040323044913,
                                           0.92387953251128675613,
                                           0.83146961230254523708,
                                           0.70710678118654752440,
                                           0.55557023301960222474,
                                           0.38268343236508977173,
                                           0.19509032201612826785,
                                           0.0};
template <int E>
__device__ __forceinline__ c2<double> root_step(int q) {
  static_assert(E >= 1 && E <= 16 && (E & (E - 1)) == 0, "E: power of two up to 16");
  const double* c = kCosPi16;
  const int k = q * (16 / E);  // angle k pi / 16, k < 16
  // cos(k pi/16) = c[k] (k <= 8) or -c[16 - k]; sin(k pi/16) = c[8 - k] or c[k - 8]
  const double cs = k <= 8 ? c[k] : -c[16 - k];
  const double sn = k <= 8 ? c[8 - k] : c[k - 8];
  return {cs, -sn};
}

// Real row x[0 .. 2L) to its packed half spectrum.
// On entry v[q] = (x[2m], x[2m+1]) for m = t + q P.  On exit v[q] = X[m]
// for m >= 1 and v[q] = (X[0], X[L]) for m = 0 (DC and Nyquist are real).
// lds must hold L values (stride 1); tw: the FP64 table exp(-2 pi i k / (2L)),
// k < 2L.
template <typename T, int L, int E>
__device__ __forceinline__ void row_r2c(c2<T>* v, c2<T>* lds, gp<const c2<double>> __restrict__ tw,
                                        int t) {
  constexpr int P = L / E;
  fft_group<T, L, E, -1>(v, lds, 1, tw, t);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < E; ++q) lds[t + q * P] = v[q];
  __syncthreads();
  const c2<double> w0 = ldg<double>(tw + t);  // tw[t + q P] = w0 root_step<E>(q)
#pragma unroll
  for (int q = 0; q < E; ++q) {
    const int m = t + q * P;
    const c2<T> z = v[q];
    if (m == 0) {
      v[q] = {z.x + z.y, z.x - z.y};
    } else {
      const c2<T> zc = lds[L - m];
      const T h = static_cast<T>(0.5);
      const c2<T> e = {h * (z.x + zc.x), h * (z.y - zc.y)};
      const c2<T> o = {h * (z.y + zc.y), -h * (z.x - zc.x)};
      const c2<double> wd = q == 0 ? w0 : cmul(w0, root_step<E>(q));
      v[q] = cadd(e, cmul(o, c2<T>{static_cast<T>(wd.x), static_cast<T>(wd.y)}));
    }
  }
}

// The table entries tw[m], m <= L, as products of two small LDS tables (the
// low entries tw[0 .. LO) and every LO-th entry), for loops that store to
// global memory: a table read from global memory there would wait for the
// loop's earlier stores (a wave's loads and stores share one counter), an
// LDS read does not.  tw_tab_fill (every thread of the block) before a
// barrier, then tw_tab.
template <int L>
struct TwTab {
  static constexpr int LO = L < 64 ? L : 64, NH = L / LO + 1, N = LO + NH;
};
template <int L, int NT>
__device__ __forceinline__ void tw_tab_fill(c2<double>* tab, gp<const c2<double>> __restrict__ tw) {
  using W = TwTab<L>;
  for (int i = threadIdx.x; i < W::N; i += NT)
    tab[i] = ldg<double>(tw + (i < W::LO ? i : (i - W::LO) * W::LO));
}
template <int L>
__device__ __forceinline__ c2<double> tw_tab(const c2<double>* tab, int m) {
  using W = TwTab<L>;
  return cmul(tab[m % W::LO], tab[W::LO + m / W::LO]);
}

// row_r2c split for callers that store the spectrum from LDS: row_r2c_z
// leaves the complex DFT z of the packed row in lds[0 .. L) (stride 1;
// visible to the block after its next barrier), and r2c_mode forms mode m
// (0 .. L) of the half spectrum from it with row_r2c's arithmetic, m = 0 and
// m = L being the real DC and Nyquist values, the twiddle from the LDS
// tables of tw_tab.  This saves the LDS pass that stages row_r2c's result
// for the stores.
template <typename T, int L, int E>
__device__ __forceinline__ void row_r2c_z(c2<T>* v, c2<T>* lds,
                                          gp<const c2<double>> __restrict__ tw, int t) {
  constexpr int P = L / E;
  fft_group<T, L, E, -1>(v, lds, 1, tw, t);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < E; ++q) lds[t + q * P] = v[q];
}
template <typename T, int L>
__device__ __forceinline__ c2<T> r2c_mode(const c2<T>* lds, const c2<double>* wtab, int m) {
  if (m == 0 || m == L) {
    const c2<T> z = lds[0];
    return m == 0 ? c2<T>{z.x + z.y, T(0)} : c2<T>{z.x - z.y, T(0)};
  }
  const c2<T> z = lds[m], zc = lds[L - m];
  const T h = static_cast<T>(0.5);
  const c2<T> e = {h * (z.x + zc.x), h * (z.y - zc.y)};
  const c2<T> o = {h * (z.y + zc.y), -h * (z.x - zc.x)};
  const c2<double> wd = tw_tab<L>(wtab, m);
  return cadd(e, cmul(o, c2<T>{static_cast<T>(wd.x), static_cast<T>(wd.y)}));
}

// Packed half spectrum to the real row, scaled by 1/(2L) so that
// row_c2r(row_r2c(x)) = x.  On entry v[q] = packed X[m], m = t + q P; on exit
// v[q] = (x[2m], x[2m+1]).
template <typename T, int L, int E>
__device__ __forceinline__ void row_c2r(c2<T>* v, c2<T>* lds, gp<const c2<double>> __restrict__ tw,
                                        int t) {
  constexpr int P = L / E;
#pragma unroll
  for (int q = 0; q < E; ++q) lds[t + q * P] = v[q];
  __syncthreads();
  const c2<double> w0 = ldg<double>(tw + t);  // tw[t + q P] = w0 root_step<E>(q)
#pragma unroll
  for (int q = 0; q < E; ++q) {
    const int m = t + q * P;
    const c2<T> X = v[q];
    if (m == 0) {
      v[q] = {X.x + X.y, X.x - X.y};
    } else {
      const c2<T> Xc = lds[L - m];
      const c2<T> a = {X.x + Xc.x, X.y - Xc.y};          // X + conj(Xc)
      const c2<T> d = {X.x - Xc.x, X.y + Xc.y};          // X - conj(Xc)
      const c2<double> wd = q == 0 ? w0 : cmul(w0, root_step<E>(q));
      const c2<T> b = cmulc(d, c2<T>{static_cast<T>(wd.x), static_cast<T>(wd.y)});                   // times exp(+2 pi i m / 2L)
      v[q] = {a.x - b.y, a.y + b.x};                      // a + i b
    }
  }
  __syncthreads();
  fft_group<T, L, E, +1>(v, lds, 1, tw, t);
  const T sc = static_cast<T>(1.0 / (2.0 * L));
#pragma unroll
  for (int q = 0; q < E; ++q) v[q] = {v[q].x * sc, v[q].y * sc};
}

}  // namespace le
