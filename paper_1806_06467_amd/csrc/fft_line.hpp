// LDS-staged Stockham FFT of one line of N complex values held by T = N / E threads.
//
// Register-slot convention: thread t holds slots m = 0..E-1, slot m being element t + T*m.
// That is the coalesced global-load pattern, the input pattern of every Stockham pass
// (butterfly b reads b + r*N/R, with b = t + j*T and slot m = j + r*E/R), and the output
// pattern of the last pass. So a forward FFT, a pointwise product in frequency and a second
// FFT chain without any reordering: the spectrum leaves the first transform with slot m
// holding frequency t + T*m, and the second transform takes it from the same registers.
//
// Pass with radix R after span P (P = product of earlier radices): butterfly b twiddles leg r
// by w_{P R}^{r (b mod P)}, runs DFT_R and writes output r to (b / P) P R + (b mod P) + r P.
// Twiddles come from per-pass tables built in float64 on the host (exact to half an ulp).
#pragma once
#include "dft_small.hpp"

namespace fr {

// one float2 of padding every 16 keeps the power-of-two strides of the exchanges spread
// over the LDS banks
__device__ __forceinline__ int lds_pad(int i) { return i + (i >> 4); }
template <int N>
struct LdsLine {
  static constexpr int size = N + N / 16;
};

// Padded LDS index of output r of butterfly b in a pass of span P and radix R, written as a
// per-thread base plus a compile-time offset per r (so the stores use immediate offsets).
template <int P, int R>
struct PassOut {
  int base;  // padded index of r = 0
  __device__ __forceinline__ explicit PassOut(int b) {
    const int i0 = (b / P) * (P * R) + (b % P);
    base = lds_pad(i0);
  }
  // valid when P % 16 == 0 (the pad of i0 + rP is pad(i0) + 17 rP/16), or P == 1 and 16 % R == 0 with
  // i0 = b R (then (b R + r) / 16 = b R / 16 for r < R)
  __device__ __forceinline__ static constexpr int off(int r) {
    if constexpr (P % 16 == 0) return r * (P + P / 16);
    return r;  // P == 1
  }
  static constexpr bool exact = (P % 16 == 0) || (P == 1 && 16 % R == 0);
};

// Twiddles of one pass for the NB butterflies a thread owns: leg r of butterfly b is
// multiplied by w_{PR}^{r (b mod P)}, read from the pass's float32 (or float64) table laid out
// [r - 1][k], k = b mod P, so that for each leg the lanes of a wavefront read consecutive
// entries (the table is built in float64 on the host; each entry is within half an ulp).
template <int P, int R, int NB, int T, class C = c32, class TW = float2>
struct PassTw {
  C w[NB][R > 1 ? R - 1 : 1];
  __device__ __forceinline__ void load(const TW* __restrict__ tw, int t) {
    if constexpr (P > 1) {
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const int k = (t + j * T) % P;
#pragma unroll
        for (int r = 1; r < R; ++r) {
          const TW q = tw[(r - 1) * P + k];
          w[j][r - 1] = {q.x, q.y};
        }
      }
    }
  }
};

template <int R0, int... Rs>
struct FirstOf {
  static constexpr int value = R0;
};

// Pass with radix R after span P. The twiddles of the next pass are loaded before this
// pass's LDS exchange, so their latency overlaps the exchange.
//
// SPLIT exchanges move the real and then the imaginary parts through one line of reals, half the
// LDS of a line of complex values: the outputs stay in their registers until their turn, so a
// thread holds nothing more than its line's elements.
// C: the element type (c32 or c64d); TW: the twiddle table's (float2 or double2); L: what the LDS
// line holds (C, or its real type for SPLIT)
template <class C, class TW, class L, bool INV, bool SPLIT, int N, int E, int P, int R, int... Rest>
__device__ __forceinline__ void fft_passes(C (&v)[E], L* __restrict__ lds, int t,
                                           const TW* __restrict__ tw,
                                           const PassTw<P, R, E / R, N / E, C, TW>& cur) {
  constexpr int T = N / E;
  constexpr int NB = E / R;
  static_assert(E % R == 0, "radix must divide the elements per thread");
  static_assert(N % (P * R) == 0, "plan does not factor N");
  constexpr bool last = sizeof...(Rest) == 0;
  // write outputs of butterfly b: value(r) to the position of output r
  auto put = [&](int b, auto value) {
    if constexpr (PassOut<P, R>::exact) {
      const PassOut<P, R> o(b);
#pragma unroll
      for (int r = 0; r < R; ++r) lds[o.base + PassOut<P, R>::off(r)] = value(r);
    } else {
      const int base = (b / P) * (P * R) + (b % P);
#pragma unroll
      for (int r = 0; r < R; ++r) lds[lds_pad(base + r * P)] = value(r);
    }
  };
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    C u[R];
#pragma unroll
    for (int r = 0; r < R; ++r) u[r] = v[j + r * NB];
    const int b = t + j * T;
    if constexpr (P > 1) {
      if constexpr (SPLIT) {  // each twiddle read where it is used: the table lies in LDS
        const int k = b % P;
#pragma unroll
        for (int r = 1; r < R; ++r) {
          const TW q = tw[(r - 1) * P + k];
          u[r] = INV ? cmulc(u[r], C{q.x, q.y}) : cmul(u[r], C{q.x, q.y});
        }
      } else {
#pragma unroll
        for (int r = 1; r < R; ++r) u[r] = INV ? cmulc(u[r], cur.w[j][r - 1]) : cmul(u[r], cur.w[j][r - 1]);
      }
    }
    DftDir<R, INV>::run(u);
    if constexpr (last || SPLIT) {
#pragma unroll
      for (int r = 0; r < R; ++r) v[j + r * NB] = u[r];
    } else {
      put(b, [&](int r) { return u[r]; });
    }
  }
  if constexpr (!last) {
    constexpr int R2 = FirstOf<Rest...>::value;
    const TW* tw_next = tw + (P > 1 ? (R - 1) * P : 0);
    PassTw<P * R, R2, E / R2, T, C, TW> nxt;
    if constexpr (!SPLIT) nxt.load(tw_next, t);
    auto at = [&](int m) {
      if constexpr (T % 16 == 0) return lds_pad(t) + m * (T + T / 16);
      else return lds_pad(t + T * m);
    };
    if constexpr (!SPLIT) {
      __syncthreads();
#pragma unroll
      for (int m = 0; m < E; ++m) v[m] = lds[at(m)];
      __syncthreads();
    } else {
#pragma unroll
      for (int j = 0; j < NB; ++j) put(t + j * T, [&](int r) { return v[j + r * NB].x; });
      __syncthreads();
#pragma unroll
      for (int m = 0; m < E; ++m) v[m].x = lds[at(m)];
      __syncthreads();
#pragma unroll
      for (int j = 0; j < NB; ++j) put(t + j * T, [&](int r) { return v[j + r * NB].y; });
      __syncthreads();
#pragma unroll
      for (int m = 0; m < E; ++m) v[m].y = lds[at(m)];
      __syncthreads();
    }
    fft_passes<C, TW, L, INV, SPLIT, N, E, P * R, Rest...>(v, lds, t, tw_next, nxt);
  }
}

// float64-built twiddle table of a plan: for each pass with span P > 1 and radix R, the block
// [r - 1][k] = exp(-2 pi i r k / (P R)), r = 1..R-1, k = 0..P-1 (rounded once to float for a
// float2 table, kept in float64 for a double2 table)
inline void tw_store(float2* p, double c, double s) { *p = make_float2(float(c), float(s)); }
inline void tw_store(double2* p, double c, double s) { *p = make_double2(c, s); }
template <int N, int P, int R, int... Rest>
struct TwiddleTable {
  template <class TW>
  static void build(TW* out) {
    if (P > 1) {
      for (int r = 1; r < R; ++r)
        for (int k = 0; k < P; ++k) {
          const long long num = (long long)r * k % (P * R);
          const double turn = -double(num) / double(P * R);
          tw_store(out + (r - 1) * P + k, __builtin_cos(2.0 * kPi * turn), __builtin_sin(2.0 * kPi * turn));
        }
    }
    if constexpr (sizeof...(Rest) > 0) TwiddleTable<N, P * R, Rest...>::build(out + (P > 1 ? (R - 1) * P : 0));
  }
  static constexpr int size() {
    int s = P > 1 ? (R - 1) * P : 0;
    if constexpr (sizeof...(Rest) > 0) s += TwiddleTable<N, P * R, Rest...>::size();
    return s;
  }
};

// compile-time FFT plan: N = product of Rs, E elements per thread
template <int N_, int E_, int... Rs>
struct Plan {
  static constexpr int N = N_;
  static constexpr int E = E_;
  static constexpr int T = N_ / E_;
  static constexpr int twiddles = TwiddleTable<N_, 1, Rs...>::size();
  static constexpr int R0 = FirstOf<Rs...>::value;
  template <class TW>
  static void build_twiddles(TW* out) { TwiddleTable<N_, 1, Rs...>::build(out); }
  // unnormalised DFT of the line, kernel exp(-2 pi i nk/N); tw = the plan's twiddle table (float2
  // for c32 elements, double2 for c64d). An LDS line of reals selects the split exchanges.
  template <class C, class L, class TW>
  __device__ __forceinline__ static void forward(C (&v)[E_], L* lds, int t, const TW* tw) {
    PassTw<1, R0, E_ / R0, N_ / E_, C, TW> none;
    fft_passes<C, TW, L, false, sizeof(L) != sizeof(C), N_, E_, 1, Rs...>(v, lds, t, tw, none);
  }
  // unnormalised inverse DFT, kernel exp(+2 pi i nk/N)
  template <class C, class L, class TW>
  __device__ __forceinline__ static void inverse(C (&v)[E_], L* lds, int t, const TW* tw) {
    PassTw<1, R0, E_ / R0, N_ / E_, C, TW> none;
    fft_passes<C, TW, L, true, sizeof(L) != sizeof(C), N_, E_, 1, Rs...>(v, lds, t, tw, none);
  }
};

}  // namespace fr
