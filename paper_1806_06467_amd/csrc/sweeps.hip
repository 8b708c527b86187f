// Fresnel plane = two in-place sweeps over an n x n c64 field (Sec. 1.1: angular-spectrum
// propagation; Sec. 1.2: FFTs of large 2-D arrays dominate; Sec. 2.4: fftshift).
//
// The paraxial transfer function factors, H[ky][kx] = h[ky] h[kx], so
//   IDFT2( H . DFT2(U) ) = (column pass: FFT, * h, IFFT) o (row pass: FFT, * h, IFFT)
// and each pass reads and writes the plane once. No fftshift is ever materialised: the
// angular-spectrum step is shift-invariant and h is indexed by the signed frequency.
//
//   row_sweep : load a row (or synthesise it from the pupil optic), optic prologue (amplitude,
//               OPD and mirror phasors of Eq. 3, thin-lens chirp), FFT, * h (scaled 1/n),
//               inverse FFT, store.
//   col_sweep : load a tile of adjacent columns, FFT, * h, inverse FFT, epilogue (the mirror
//               after the step, or the conjugate optic for the adjoint), store. From 2048 rows
//               (col_sweep_pipe) a block walks several tiles and loads the next one while it
//               transforms the present one.
// The column tile is LINES columns wide so that a wavefront reads LINES*8-byte contiguous
// segments; blocks are renumbered so that the blocks resident on one XCD (one L2) work on
// neighbouring columns at the same time.
#include <type_traits>

#include "fft_line.hpp"
#include "fr_internal.h"
#include "fr_exact.h"
#include "../../include/fresnel.h"

namespace fr {

namespace {

__device__ __forceinline__ c32 ld2(const float2 *p) {
  float2 v = *p;
  return {v.x, v.y};
}

// Raw buffer access to one plane: a 32-bit per-lane offset plus a wave-uniform offset held in a
// scalar register, so that the sixteen strided accesses of a thread cost one address VGPR.
// The hardware range check applies to the per-lane offset: lanes whose offset is past the
// buffer read 0 and do not write; every per-lane offset used here is non-negative.
// (The 64-bit results are moved whole with bit casts: extracting single elements of the
// builtin's vector type was observed to address the wrong half.)
struct PlaneBuf {
  __amdgpu_buffer_rsrc_t r;
  typedef unsigned int raw64 __attribute__((__vector_size__(8)));  // the builtin's value type
  __device__ __forceinline__ PlaneBuf(const void *p, unsigned bytes)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, int(bytes), 0x00020000)) {}
  __device__ __forceinline__ c32 load(unsigned vo, unsigned so) const {
    const float2 q = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, vo, so, 0));
    return {q.x, q.y};
  }
  __device__ __forceinline__ void store(unsigned vo, unsigned so, c32 v) const {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(raw64, make_float2(v.x, v.y)), r, vo, so, 0);
  }
};

// Same for float maps (amplitude, OPD, mirror surfaces).
struct MapBuf {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ MapBuf(const void *p, unsigned bytes)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, int(bytes), 0x00020000)) {}
  __device__ __forceinline__ float load(unsigned vo, unsigned so) const {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, vo, so, 0));
  }
};

// The pre optic along one row y for the thread's slots x = t + T m: amplitude, OPD (win x win
// maps centred in the plane), mirror surface (n x n) and thin lens. Returns false when the
// amplitude is zero on the whole row (a row outside the pupil window).
template <int E, int T>
__device__ __forceinline__ bool pre_optic_row(const PlaneArgs &pa, int n, int y, int t, c32 (&ph)[E]) {
  const int win = pa.win;
  const int off = (n - win) >> 1;
  const int wy = y - off;
  const bool row_in = unsigned(wy) < unsigned(win);
  if (pa.amp && !row_in) return false;
  float a[E], turns[E];
#pragma unroll
  for (int m = 0; m < E; ++m) {
    a[m] = 1.0f;
    turns[m] = 0.0f;
  }
  if ((pa.amp || pa.opd) && row_in) {
    // The hardware range check of a raw buffer access looks at the per-lane (VGPR) offset
    // only, so every per-lane offset here is non-negative and inside the map: full maps use
    // lane offset + per-slot scalar offset; windowed maps clamp the column into the window
    // (lanes outside it are masked after the load).
    const unsigned bytes = unsigned(win) * unsigned(win) * 4u;
    unsigned vo[E], so[E];
    if (win == n) {
#pragma unroll
      for (int m = 0; m < E; ++m) {
        vo[m] = unsigned(wy * win + t) * 4u;
        so[m] = unsigned(T * m) * 4u;
      }
    } else {
#pragma unroll
      for (int m = 0; m < E; ++m) {
        const int wx = min(max(t + T * m - off, 0), win - 1);
        vo[m] = unsigned(wy * win + wx) * 4u;
        so[m] = 0u;
      }
    }
    if (pa.amp) {
      const MapBuf mb(pa.amp, bytes);
#pragma unroll
      for (int m = 0; m < E; ++m) a[m] = mb.load(vo[m], so[m]);
    }
    if (pa.opd) {
      const MapBuf mb(pa.opd, bytes);
#pragma unroll
      for (int m = 0; m < E; ++m) turns[m] = mb.load(vo[m], so[m]) * pa.inv_lambda;
    }
    if (win < n) {
#pragma unroll
      for (int m = 0; m < E; ++m) {
        const bool in = unsigned(t + T * m - off) < unsigned(win);
        a[m] = in ? a[m] : (pa.amp ? 0.0f : 1.0f);
        turns[m] = in ? turns[m] : 0.0f;
      }
    }
  }
  if (pa.pre_surf) {
    const MapBuf sb(pa.pre_surf, unsigned(n) * unsigned(n) * 4u);
    const unsigned vo = unsigned(y * n + t) * 4u;
#pragma unroll
    for (int m = 0; m < E; ++m) turns[m] += 2.0f * sb.load(vo, unsigned(T * m) * 4u) * pa.inv_lambda;
  }
  if (pa.opd || pa.pre_surf) {
#pragma unroll
    for (int m = 0; m < E; ++m) {
      float sn, cs;
      sincos_turns(turns[m], &sn, &cs);
      ph[m] = {a[m] * cs, a[m] * sn};
    }
  } else {
#pragma unroll
    for (int m = 0; m < E; ++m) ph[m] = {a[m], 0.0f};
  }
  if (pa.lens) {
    const c32 ly = ld2(pa.lens + y);
#pragma unroll
    for (int m = 0; m < E; ++m) ph[m] = cmul(ph[m], cmul(ld2(pa.lens + t + T * m), ly));
  }
  return true;
}

// v times the post optic exp(2 pi i 2 post_surf / lambda) (its conjugate for the adjoint) at rows
// y = t + T m of column x: the map (4-column tiles) is read for a group of G slots before their
// phasors are formed (the pipelined column sweep holds two tiles' elements and takes a few at a time)
template <int G, int E, int T>
__device__ __forceinline__ void post_optic_col(const PlaneArgs &pa, int n, int t, int x, bool adj, c32 (&v)[E]) {
  const MapBuf map(pa.post_surf, unsigned(post_tiled_size(n)) * 4u);
#pragma unroll
  for (int m0 = 0; m0 < E; m0 += G) {
    if constexpr (G < E) __builtin_amdgcn_sched_barrier(0);
    float sv[G];
#pragma unroll
    for (int m = 0; m < G; ++m) sv[m] = map.load(unsigned(post_tiled_index(n, t + T * (m0 + m), x)) * 4u, 0u);
    c32 ph[G];
#pragma unroll
    for (int m = 0; m < G; ++m) {
      float s, c;
      sincos_turns(2.0f * sv[m] * pa.inv_lambda, &s, &c);
      ph[m] = {c, s};
    }
#pragma unroll
    for (int m = 0; m < G; ++m) v[m0 + m] = adj ? cmulc(v[m0 + m], ph[m]) : cmul(v[m0 + m], ph[m]);
  }
}

__device__ __forceinline__ bool has_pre(const PlaneArgs &pa) {
  return pa.amp || pa.opd || pa.pre_surf || pa.lens;
}

// frequency product of the pass: Y h (forward) or Y conj(h) (adjoint, AS over -z); slot m
// holds frequency t + T m. h carries the 1/n of the inverse transform.
template <int E, int T>
__device__ __forceinline__ void freq_product(c32 (&v)[E], const float2 *h, int t, bool adj) {
  if (adj) {
#pragma unroll
    for (int m = 0; m < E; ++m) v[m] = cmulc(v[m], ld2(h + t + T * m));
  } else {
#pragma unroll
    for (int m = 0; m < E; ++m) v[m] = cmul(v[m], ld2(h + t + T * m));
  }
}

// DIRECT: the row half of the direct (single-transform) Fresnel step: the prologue applies the
// optic times the input quadratic phase (held in the lens slot), then the forward transform only;
// for its adjoint the inverse transform, then the conjugate of both
// Up to 4096, at most 128 VGPRs (four waves per SIMD): at 4096 four 256-thread row blocks then
// share a compute unit (their LDS lines allow four) instead of three (measured 1 % faster per
// plane, bit-identical results); the 8192 row would spill under that cap.
template <class PL, int LINES, bool DIRECT = false>
__global__ void __launch_bounds__(PL::T *LINES) __attribute__((amdgpu_waves_per_eu(PL::N <= 4096 ? 4 : 1)))
row_sweep(BatchArgs args, const float2 *tw) {
  constexpr int N = PL::N, E = PL::E, T = PL::T;
  __shared__ c32 lds[LINES * LdsLine<N>::size];
  const PlaneArgs &pa = args.p[blockIdx.y];
  const int line = threadIdx.x / T;
  const int t = threadIdx.x - line * T;
  const int y = blockIdx.x * LINES + line;
  const bool adj = pa.flags & FR_ADJOINT;
  if (adj && (pa.flags & kWindowRowsOnly)) {
    // rows of this block all outside the rows wanted from the step (block-uniform)
    const int y0 = blockIdx.x * LINES, off = (N - pa.win) >> 1;
    if (y0 + LINES <= off || y0 >= off + pa.win) return;
  }
  const PlaneBuf buf(pa.field, unsigned(N) * N * 8u);
  const unsigned vo = unsigned(y * N + t) * 8u;
  c32 v[E];
  if (!adj && has_pre(pa)) {
    c32 ph[E];
    const bool nonzero = pre_optic_row<E, T>(pa, N, y, t, ph);
    if constexpr (LINES == 1) {
      // a whole row outside the amplitude window stays zero through the row transform
      // (block-uniform); the column sweep takes it as zero without reading it, so it is not
      // stored
      if (!nonzero) return;
    }
    if (!nonzero) {
#pragma unroll
      for (int m = 0; m < E; ++m) ph[m] = {0.0f, 0.0f};
    }
    if (pa.flags & kSourceOptic) {
#pragma unroll
      for (int m = 0; m < E; ++m) v[m] = ph[m];
    } else {
#pragma unroll
      for (int m = 0; m < E; ++m) v[m] = cmul(buf.load(vo, unsigned(T * m) * 8u), ph[m]);
    }
  } else if (pa.flags & kSourceOptic) {
#pragma unroll
    for (int m = 0; m < E; ++m) v[m] = {1.0f, 0.0f};
  } else {
#pragma unroll
    for (int m = 0; m < E; ++m) v[m] = buf.load(vo, unsigned(T * m) * 8u);
  }
  c32 *my = lds + line * LdsLine<N>::size;
  if constexpr (DIRECT) {
    // the adjoint direct step runs this sweep second: inverse transform, then the conjugate
    // optic and input phase below
    // the transform's kernel sign: + for the adjoint, flipped again over z < 0
    if (adj != bool(pa.flags & kTowardSource)) PL::inverse(v, my, t, tw);
    else PL::forward(v, my, t, tw);
  } else {
    PL::forward(v, my, t, tw);
    freq_product<E, T>(v, pa.h, t, adj);
    PL::inverse(v, my, t, tw);
  }
  if (adj && has_pre(pa)) {
    c32 ph[E];
    if (!pre_optic_row<E, T>(pa, N, y, t, ph)) {
#pragma unroll
      for (int m = 0; m < E; ++m) ph[m] = {0.0f, 0.0f};
    }
#pragma unroll
    for (int m = 0; m < E; ++m) v[m] = cmulc(v[m], ph[m]);
  }
#pragma unroll
  for (int m = 0; m < E; ++m) buf.store(vo, unsigned(T * m) * 8u, v[m]);
}

// DIRECT: the column half of the direct Fresnel step: the forward transform,
// then the output quadratic phase of both axes (h holds it per index, with the constant's root).
// EXACT (with DIRECT): the column sweep of the exact-transfer-function step (fr_exact.h), 1 with
// H's phase formed per element in float64, 2 in its split form.
template <class PL, int LINES, bool DIRECT = false, int EXACT = 0>
__global__ void __launch_bounds__(PL::T *LINES) col_sweep(BatchArgs args, const float2 *tw) {
  static_assert(!EXACT || DIRECT, "the exact mode is one of the direct kernel");
  constexpr int N = PL::N, E = PL::E, T = PL::T;
  constexpr int G = N / LINES;  // column groups per plane
  // the lines of the LINES columns start 8 float2 apart in the bank pattern (measured: a
  // 3 % faster sweep than 4, 10 % than 1)
  constexpr int LINE = LdsLine<N>::size + 8;
  __shared__ c32 lds[LINES * LINE];
  const PlaneArgs &pa = args.p[blockIdx.y];
  const int c = threadIdx.x % LINES;
  const int t = threadIdx.x / LINES;
  // blocks are dealt round-robin to the 8 XCDs; give each XCD a contiguous run of groups
  int g = blockIdx.x;
  if constexpr (G % 8 == 0) g = (blockIdx.x & 7) * (G / 8) + (blockIdx.x >> 3);
  const int x = g * LINES + c;
  const bool adj = pa.flags & FR_ADJOINT;
  const PlaneBuf buf(pa.field, unsigned(N) * N * 8u);
  const unsigned vo = unsigned(t * N + x) * 8u;
  // the post surface's phasor, unless this tile lies where the surface is 0 (the phasor is 1)
  const int x0 = g * LINES;
  const bool post = pa.post_surf && !(pa.post_hi > pa.post_lo && (x0 + LINES <= pa.post_lo || x0 >= pa.post_hi));
  c32 v[E];
  if (!adj && pa.amp && pa.win < N) {
    // forward plane with a windowed amplitude: the rows outside the window are zero after the
    // row sweep, which did not store them (uniform over a wavefront when the window edges are
    // multiples of the wavefront's rows)
    const int off = (N - pa.win) >> 1;
#pragma unroll
    for (int m = 0; m < E; ++m)
      v[m] = unsigned(t + T * m - off) < unsigned(pa.win) ? buf.load(vo, unsigned(T * m) * unsigned(N) * 8u)
                                                         : c32{0.0f, 0.0f};
  } else {
#pragma unroll
    for (int m = 0; m < E; ++m) v[m] = buf.load(vo, unsigned(T * m) * unsigned(N) * 8u);
  }
  if (adj && post) post_optic_col<E, E, T>(pa, N, t, x, true, v);
  c32 *my = lds + c * LINE;
  if constexpr (DIRECT) {
    if constexpr (EXACT) {
      // exact transfer function of frequency (kx, ky) = (x, t + T m) (signed), with the 1/n^2
      // of the two inverse transforms; conjugated for the adjoint. The spectrum goes through the
      // thread's own LDS slots so that the float64 phase of one element at a time is formed
      // beside no more than the loop's registers (the LDS is free between the transforms: the
      // forward one ends on a barrier after its last read).
      const double *prm = reinterpret_cast<const double *>(pa.h);
      const double zl = prm[0], a2 = prm[1];
      const int kx = x < N / 2 ? x : x - N;
      if constexpr (EXACT == 2) {
        // H = h[kx] h[ky] exp(2 pi i c): the paraxial part from its float64-built table (it
        // carries the 1/n of each inverse transform), the rest c = -(z/lambda) u^2 /
        // (2 (1 + sqrt(1 - u))^2) turns, at most a quarter turn on this grid, in float32
        const float2 *hp = reinterpret_cast<const float2 *>(prm + 4);
        const float zlf = float(zl), a2f = float(a2);
        const c32 hx = ld2(hp + x);
        PL::forward(v, my, t, tw);
#pragma unroll
        for (int m = 0; m < E; ++m) {
          const int k = t + T * m;
          const int ky = k < N / 2 ? k : k - N;
          const float u = a2f * float(kx * kx + ky * ky);
          const float r = 1.0f + sqrtf(1.0f - u);
          float sn, cs;
          sincos_turns(-zlf * u * u / (2.0f * r * r), &sn, &cs);
          const c32 hh = cmul(cmul(hx, ld2(hp + k)), c32{cs, sn});
          v[m] = adj ? cmulc(v[m], hh) : cmul(v[m], hh);
        }
        PL::inverse(v, my, t, tw);
#pragma unroll
        for (int m = 0; m < E; ++m) buf.store(vo, unsigned(T * m) * unsigned(N) * 8u, v[m]);
        return;
      } else {
        PL::forward(v, my, t, tw);
#pragma unroll
        for (int m = 0; m < E; ++m) my[t + T * m] = v[m];
        constexpr float inv_n2 = 1.0f / (float(N) * float(N));
#pragma unroll 1
        for (int m = 0; m < E; ++m) {
          const int k = t + T * m;
          const int ky = k < N / 2 ? k : k - N;
          const double u = a2 * double(kx * kx + ky * ky);  // (lambda f)^2
          float amp = inv_n2, turns;
          if (u < 1.0) {
            const double tr = -zl * u / (sqrt(1.0 - u) + 1.0);
            turns = float(tr - rint(tr));
          } else {
            amp *= float(exp(-2.0 * kPi * fabs(zl) * sqrt(u - 1.0)));
            turns = float(-(zl - rint(zl)));
          }
          float sn, cs;
          sincos_turns(adj ? -turns : turns, &sn, &cs);
          my[k] = cmul(my[k], c32{amp * cs, amp * sn});
        }
#pragma unroll
        for (int m = 0; m < E; ++m) v[m] = my[t + T * m];
        __syncthreads();  // every slot read back before the inverse transform's first exchange
        PL::inverse(v, my, t, tw);
#pragma unroll
        for (int m = 0; m < E; ++m) buf.store(vo, unsigned(T * m) * unsigned(N) * 8u, v[m]);
        return;
      }
    }
    // slot m holds frequency row ky = t + T m of column kx = x (after the forward transform;
    // the adjoint, which runs this sweep first, multiplies the conjugate phases before its
    // inverse transform)
    const c32 px = ld2(pa.h + x);
    const bool inv = adj != bool(pa.flags & kTowardSource);  // kernel sign, as in the row sweep
    if (adj) {
#pragma unroll
      for (int m = 0; m < E; ++m) v[m] = cmulc(v[m], cmul(ld2(pa.h + t + T * m), px));
    }
    if (inv) PL::inverse(v, my, t, tw);
    else PL::forward(v, my, t, tw);
    if (!adj) {
#pragma unroll
      for (int m = 0; m < E; ++m) v[m] = cmul(v[m], cmul(ld2(pa.h + t + T * m), px));
    }
#pragma unroll
    for (int m = 0; m < E; ++m) buf.store(vo, unsigned(T * m) * unsigned(N) * 8u, v[m]);
    return;
  }
  PL::forward(v, my, t, tw);
  freq_product<E, T>(v, pa.h, t, adj);
  PL::inverse(v, my, t, tw);
  if (!adj && post) post_optic_col<E, E, T>(pa, N, t, x, false, v);
  if (adj && (pa.flags & kWindowRowsOnly)) {
    // the row sweep that follows transforms only the rows of the window
    const int off = (N - pa.win) >> 1;
#pragma unroll
    for (int m = 0; m < E; ++m)
      if (unsigned(t + T * m - off) < unsigned(pa.win)) buf.store(vo, unsigned(T * m) * unsigned(N) * 8u, v[m]);
  } else {
#pragma unroll
    for (int m = 0; m < E; ++m) buf.store(vo, unsigned(T * m) * unsigned(N) * 8u, v[m]);
  }
}

// The column sweep of long lines, where a tile fills a compute unit: one block per compute unit
// walks `tiles` tiles of a plane and loads the next tile while it transforms the current one, so
// that the loads, the transforms and the stores overlap. Two things make room for that: the
// exchanges move real and imaginary parts in turn through LDS lines of floats (half the LDS of the
// tile), and the twiddles and h are copied to the rest of the LDS once per block, which takes
// their registers and 76 of the 108 vector memory instructions per 16 elements away and leaves no
// load between a tile's transform and the next tile's (vector loads return in order). It was the
// address unit that bound the sweep before (busy 75 % of the time at 4096, the vector units 37 %).
// Measured per plane (forward, adjoint): 4096^2 92 and 115 us to 83 and 100 us, 8192^2 877 us to
// 705 us (16-byte pieces of rows 64 KiB apart: what the 32 compute units of an XCD have in flight
// exceeds its L2, so a line is fetched 1.3 times and written in pieces).
// PF: elements of the next tile loaded before the transform, the others just before the stores.
template <class PL, int LINES, int PF, bool DIRECT = false, int EXACT = 0>
__global__ void __launch_bounds__(PL::T *LINES) __attribute__((amdgpu_waves_per_eu(4))) col_sweep_pipe(BatchArgs args, const float2 *tw, int tiles) {
  static_assert(EXACT != 1, "the float64 phase goes through complex LDS lines");
  constexpr int N = PL::N, E = PL::E, T = PL::T;
  constexpr int LINE = LdsLine<N>::size + 8;
  constexpr bool HTAB = 4 * LINES * LINE + 8 * (PL::twiddles + N) <= 160 * 1024;
  __shared__ float lds[LINES * LINE];
  __shared__ __attribute__((aligned(16))) float2 tab[PL::twiddles + (HTAB ? N : 0)];
  const PlaneArgs &pa = args.p[blockIdx.y];
  const int c = threadIdx.x % LINES;
  const int t = threadIdx.x / LINES;
  const bool adj = pa.flags & FR_ADJOINT;
  const PlaneBuf buf(pa.field, unsigned(N) * N * 8u);
  // rows that the forward row sweep did not store (zero rows outside a windowed amplitude) are not
  // loaded, and rows that the adjoint row sweep does not read are not stored: their offsets are
  // moved past the buffer, whose range check returns 0 and drops the store
  const int lwin = !adj && pa.amp ? pa.win : N, swin = adj && (pa.flags & kWindowRowsOnly) ? pa.win : N;
  auto offset = [](int win, int t, unsigned vo, int m) {
    return unsigned(t + T * m - ((N - win) >> 1)) < unsigned(win) ? vo : 0x80000000u;
  };
  // the thread's place in a tile, formed anew for each tile (kept, it would cost registers that
  // the two tiles need)
  auto place = [](int g, int &t, unsigned &vo) {
    unsigned tid = threadIdx.x;
    asm("" : "+v"(tid));
    t = tid / LINES;
    vo = (unsigned(t) * N + unsigned(g) * LINES + tid % LINES) * 8u;
  };
  const double *prm = reinterpret_cast<const double *>(pa.h);
  const float2 *hg = EXACT ? reinterpret_cast<const float2 *>(prm + 4) : pa.h;
  // tile i of this block: blocks are dealt round-robin to the 8 XCDs; the blocks of one XCD take
  // tiles in runs that fill a 128-byte line of each row, and walk from a line to the next (the
  // adjoint sweep of a 4096^2 plane, which reads from HBM: 100 us, 121-130 us where the lines of
  // one block are 8 or 64 apart)
  constexpr int RUN = LINES < 16 ? 16 / LINES : 1;
  const int slot = blockIdx.x >> 3, q = (blockIdx.x & 7) * ((gridDim.x >> 3) / RUN) + slot / RUN;
  const int first = q * tiles * RUN + slot % RUN, per = RUN;
  auto load = [&](c32 *v, int g, auto m0, auto m1) {
    int tl;
    unsigned vo;
    place(g, tl, vo);
#pragma unroll
    for (int m = m0; m < m1; ++m) v[m] = buf.load(offset(lwin, tl, vo, m), unsigned(T * m) * unsigned(N) * 8u);
  };
  using Zero = std::integral_constant<int, 0>;
  using Mid = std::integral_constant<int, PF>;
  using All = std::integral_constant<int, E>;
  c32 v[E], nxt[E];
  load(v, first, Zero{}, All{});
  {
    static_assert(PL::twiddles % 2 == 0 && N % 2 == 0, "two entries per copy");
    const float4 *src = reinterpret_cast<const float4 *>(tw);
    float4 *dst = reinterpret_cast<float4 *>(tab);
    for (int i = threadIdx.x; i < PL::twiddles / 2; i += PL::T * LINES) dst[i] = src[i];
    if constexpr (HTAB) {
      const float4 *hs = reinterpret_cast<const float4 *>(hg);
      for (int i = threadIdx.x; i < N / 2; i += PL::T * LINES) dst[PL::twiddles / 2 + i] = hs[i];
    }
  }
  __syncthreads();
  // h at the thread's slot m (where it is not in LDS, one address register serves all slots)
  const PlaneBuf hb(hg, N * 8u);
  auto h_at = [&](int m) {
    if constexpr (HTAB) return ld2(tab + PL::twiddles + t + T * m);
    else return hb.load(unsigned(t) * 8u, unsigned(T * m) * 8u);
  };
  auto h_x = [&](int x) { return ld2((HTAB ? tab + PL::twiddles : hg) + x); };
  float *my = lds + c * LINE;
  for (int i = 0; i < tiles; ++i) {
    const int g = first + i * per;
    const int x = g * LINES + c;
    // the post surface's phasor, unless this tile lies where the surface is 0 (the phasor is 1)
    const int x0 = g * LINES;
    const bool post = pa.post_surf && !(pa.post_hi > pa.post_lo && (x0 + LINES <= pa.post_lo || x0 >= pa.post_hi));
    if (adj && post) post_optic_col<4, E, T>(pa, N, t, x, true, v);
    if (i + 1 < tiles) load(nxt, g + per, Zero{}, Mid{});
    if constexpr (EXACT) {
      // the split form of the exact transfer function (see col_sweep)
      const float zlf = float(prm[0]), a2f = float(prm[1]);
      const int kx = x < N / 2 ? x : x - N;
      const c32 hx = h_x(x);
      PL::forward(v, my, t, tab);
#pragma unroll
      for (int m = 0; m < E; ++m) {
        const int k = t + T * m;
        const int ky = k < N / 2 ? k : k - N;
        const float u = a2f * float(kx * kx + ky * ky);
        const float r = 1.0f + sqrtf(1.0f - u);
        float sn, cs;
        sincos_turns(-zlf * u * u / (2.0f * r * r), &sn, &cs);
        const c32 hh = cmul(cmul(hx, h_at(m)), c32{cs, sn});
        v[m] = adj ? cmulc(v[m], hh) : cmul(v[m], hh);
      }
      PL::inverse(v, my, t, tab);
    } else if constexpr (DIRECT) {
      const c32 px = h_x(x);
      const bool inv = adj != bool(pa.flags & kTowardSource);  // kernel sign, as in the row sweep
      if (adj) {
#pragma unroll
        for (int m = 0; m < E; ++m) v[m] = cmulc(v[m], cmul(h_at(m), px));
      }
      if (inv) PL::inverse(v, my, t, tab);
      else PL::forward(v, my, t, tab);
      if (!adj) {
#pragma unroll
        for (int m = 0; m < E; ++m) v[m] = cmul(v[m], cmul(h_at(m), px));
      }
    } else {
      PL::forward(v, my, t, tab);
#pragma unroll
      for (int m = 0; m < E; ++m) {
        // (a few loads of h at a time: two tiles' elements leave no registers for more)
        if (!HTAB && m % 4 == 0) __builtin_amdgcn_sched_barrier(0);
        const c32 q = h_at(m);
        v[m] = adj ? cmulc(v[m], q) : cmul(v[m], q);
      }
      PL::inverse(v, my, t, tab);
      if (!adj && post) post_optic_col<4, E, T>(pa, N, t, x, false, v);
    }
    if constexpr (PF < E) {
      __builtin_amdgcn_sched_barrier(0);
      if (i + 1 < tiles) load(nxt, g + per, Mid{}, All{});
      __builtin_amdgcn_sched_barrier(0);
    }
    int ts;
    unsigned vo;
    place(g, ts, vo);
#pragma unroll
    for (int m = 0; m < E; ++m) buf.store(offset(swin, ts, vo, m), unsigned(T * m) * unsigned(N) * 8u, v[m]);
#pragma unroll
    for (int m = 0; m < E; ++m) v[m] = nxt[m];
  }
}

// blocks per plane of the pipelined column sweep: as many as run at once (1024 threads per compute
// unit at its 128 registers) when `count` planes share the launch, a power of two so that a block's
// tiles are whole runs of 128-byte lines
template <class PL, int LINES>
int pipe_blocks(int count) {
  constexpr int G = PL::N / LINES, kAtOnce = 256 * 1024 / (PL::T * LINES);
  constexpr int kLeast = 8 * (LINES < 16 ? 16 / LINES : 1);
  static_assert(G % kLeast == 0, "a block per XCD and tile of a line");
  int b = kLeast;
  while (b < G && b * count < kAtOnce) b *= 2;
  return b;
}

// Forward planes run the row sweep first (optic prologue on contiguous rows) and the column
// sweep second (mirror epilogue); adjoint planes run the column sweep first (conjugate mirror
// prologue) and the row sweep second (conjugate optic epilogue). The two halves of the
// angular-spectrum step commute, so only the placement of the optics sets the order, and the
// amplitude/OPD maps are always read along rows.
// PF > 0: the column sweep is the pipelined one with PF elements of the next tile in flight
template <class PL, int ROW_LINES, int COL_LINES, int PF = 0, bool DIRECT = false>
hipError_t launch_sweeps(const BatchArgs &fwd, int nf, const BatchArgs &adj, int na,
                         const float2 *tw, hipStream_t s, const LaunchHook &hook) {
  constexpr int N = PL::N;
  static_assert(N % ROW_LINES == 0 && N % COL_LINES == 0, "tile must divide n");
  // timing names carry the direction (the optic maps read differ), tags the planes per launch
  auto rows = [&](const BatchArgs &a, int count, const char *name) {
    hook(s, name, count, 0);
    hipLaunchKernelGGL((row_sweep<PL, ROW_LINES, DIRECT>), dim3(N / ROW_LINES, count),
                       dim3(PL::T * ROW_LINES), 0, s, a, tw);
    hipError_t e = hipGetLastError();
    hook(s, name, count, 1);
    return e;
  };
  auto cols = [&](const BatchArgs &a, int count, const char *name) {
    hook(s, name, count, 0);
    if constexpr (PF > 0) {
      const int blocks = pipe_blocks<PL, COL_LINES>(count);
      hipLaunchKernelGGL((col_sweep_pipe<PL, COL_LINES, PF, DIRECT>), dim3(blocks, count), dim3(PL::T * COL_LINES), 0, s,
                         a, tw, N / COL_LINES / blocks);
    } else {
      hipLaunchKernelGGL((col_sweep<PL, COL_LINES, DIRECT>), dim3(N / COL_LINES, count), dim3(PL::T * COL_LINES), 0, s,
                         a, tw);
    }
    hipError_t e = hipGetLastError();
    hook(s, name, count, 1);
    return e;
  };
  hipError_t e = hipSuccess;
  if (nf && (e = rows(fwd, nf, DIRECT ? "direct_rows" : "row_sweep")) != hipSuccess) return e;
  if (nf && (e = cols(fwd, nf, DIRECT ? "direct_cols" : "col_sweep")) != hipSuccess) return e;
  if (na && (e = cols(adj, na, DIRECT ? "direct_cols_adj" : "col_sweep_adj")) != hipSuccess) return e;
  if (na && (e = rows(adj, na, DIRECT ? "direct_rows_adj" : "row_sweep_adj")) != hipSuccess) return e;
  return e;
}

}  // namespace

bool fresnel_size_supported(int n) {
  switch (n) {
    case 64: case 128: case 256: case 512: case 1024: case 2048: case 4096: case 8192:
      return true;
    default:
      return false;
  }
}

// the twiddle table of the plan the sweeps use for edge n (same Plan types as the launches)
int fresnel_twiddle_count(int n) {
  switch (n) {
    case 64: return Plan<64, 8, 8, 8>::twiddles;
    case 128: return Plan<128, 16, 16, 8>::twiddles;
    case 256: return Plan<256, 16, 16, 16>::twiddles;
    case 512: return Plan<512, 8, 8, 8, 8>::twiddles;
    case 1024: return Plan<1024, 16, 16, 8, 8>::twiddles;
    case 2048: return Plan<2048, 16, 16, 16, 8>::twiddles;
    case 4096: return Plan<4096, 16, 16, 16, 16>::twiddles;
    case 8192: return Plan<8192, 16, 16, 16, 16, 2>::twiddles;
    default: return 0;
  }
}
void fresnel_twiddle_build(int n, float2 *out) {
  switch (n) {
    case 64: Plan<64, 8, 8, 8>::build_twiddles(out); break;
    case 128: Plan<128, 16, 16, 8>::build_twiddles(out); break;
    case 256: Plan<256, 16, 16, 16>::build_twiddles(out); break;
    case 512: Plan<512, 8, 8, 8, 8>::build_twiddles(out); break;
    case 1024: Plan<1024, 16, 16, 8, 8>::build_twiddles(out); break;
    case 2048: Plan<2048, 16, 16, 16, 8>::build_twiddles(out); break;
    case 4096: Plan<4096, 16, 16, 16, 16>::build_twiddles(out); break;
    case 8192: Plan<8192, 16, 16, 16, 16, 2>::build_twiddles(out); break;
    default: break;
  }
}

int fresnel_variants(int n) { return n == 4096 ? 4 : n == 2048 || n == 8192 ? 3 : 1; }

hipError_t launch_fresnel_batch(const PlaneArgs *planes, int count, int n, const float2 *root,
                                hipStream_t s, const LaunchHook &hook, int variant) {
  BatchArgs fwd, adj;
  int nf = 0, na = 0;
  for (int i = 0; i < count; ++i) {
    if (planes[i].flags & FR_ADJOINT)
      adj.p[na++] = planes[i];
    else
      fwd.p[nf++] = planes[i];
  }
  // Tiles: rows per row block, columns per column tile, elements of the next tile in flight. Small
  // tiles keep the chip in blocks: a single 256^2 plane took 20 us with 16 rows and 32 columns (16
  // and 8 blocks) and takes 12 us, a 512^2 plane 27 us with 4 rows and 16 columns and 12 us, 21 of
  // them 87 us and 51 us, a 1024^2 plane 32 us with 4 and 8 and 23 us. From 2048 the column tile
  // fills half a compute unit or more and the pipelined sweep wins: a 2048^2 plane 54 us with 2
  // rows and 8 columns, 45 us; the 4096^2 column sweeps 92 and 115 us to 83 and 100 us (forward,
  // adjoint), the 8192^2 ones 877 us to 705 us. The direct, the exact and the float64 steps take tiles as
  // small up to 1024 (512^2 18, 29 and 21 us with the larger tiles, 12, 15 and 17 us), and so do large
  // batches (42 planes of 1024^2, a paraxial step 441 us and 381 us, an exact one 513 us and 443 us).
#define FR_SWEEPS(...) return launch_sweeps<__VA_ARGS__>(fwd, nf, adj, na, root, s, hook)
  switch (n) {
    case 64: {
      using P = Plan<64, 8, 8, 8>;
      FR_SWEEPS(P, 8, 8);
    }
    case 128: {
      using P = Plan<128, 16, 16, 8>;
      FR_SWEEPS(P, 8, 8);
    }
    case 256: {
      using P = Plan<256, 16, 16, 16>;
      FR_SWEEPS(P, 4, 4);
    }
    case 512: {
      using P = Plan<512, 8, 8, 8, 8>;
      FR_SWEEPS(P, 1, 4);
    }
    case 1024: {
      using P = Plan<1024, 16, 16, 8, 8>;
      FR_SWEEPS(P, 1, 4);
    }
    case 2048: {
      using P2 = Plan<2048, 16, 16, 16, 8>;
      if (variant == 1) FR_SWEEPS(P2, 2, 4, 12);
      if (variant == 2) FR_SWEEPS(P2, 2, 8);
      FR_SWEEPS(P2, 1, 4, 12);
    }
    case 4096: {
      using P4 = Plan<4096, 16, 16, 16, 16>;
      if (variant == 1) FR_SWEEPS(P4, 1, 2, 16);
      if (variant == 2) FR_SWEEPS(P4, 2, 2, 16);
      if (variant == 3) FR_SWEEPS(P4, 2, 4, 16);
      FR_SWEEPS(P4, 1, 4, 16);
    }
    case 8192: {
      using P8 = Plan<8192, 16, 16, 16, 16, 2>;
      if (variant == 1) FR_SWEEPS(P8, 1, 2);
      if (variant == 2) FR_SWEEPS(P8, 2, 1);
      FR_SWEEPS(P8, 1, 2, 16);
    }
    default: return hipErrorInvalidValue;
  }
#undef FR_SWEEPS
}

// the exact-transfer-function step: row FFT (optic prologue, or plain for the adjoint), column
// FFT * H * IFFT, row IFFT (plain, or the conjugate optic epilogue for the adjoint), each sweep
// the direct step's kernel with its own plane arguments
// (planes whose bit is set in `split` have H in its split form: their column sweep is the split
// instance's launch, the others' the float64 one's, so each plane takes the kernels it takes in
// a call of its own)
template <class PL, int RL, int CL, int PF = 0>
hipError_t launch_exact_sweeps(const PlaneArgs *planes, int count, const float2 *tw, hipStream_t s,
                               const LaunchHook &hook, uint64_t split) {
  constexpr int N = PL::N;
  BatchArgs a, b, c, bs;
  int nb = 0, ns = 0;
  for (int i = 0; i < count; ++i) {
    const PlaneArgs &p = planes[i];
    const bool adj = p.flags & FR_ADJOINT;
    PlaneArgs plain = p;
    plain.amp = plain.opd = plain.pre_surf = plain.post_surf = nullptr;
    plain.lens = nullptr;
    a.p[i] = adj ? plain : p;
    a.p[i].flags = 0;                        // forward row transform (optic first when forward)
    PlaneArgs &col = (split >> i) & 1u ? bs.p[ns++] : b.p[nb++];
    col = p;
    col.flags = p.flags & FR_ADJOINT;
    c.p[i] = adj ? p : plain;
    c.p[i].flags = FR_ADJOINT;               // inverse row transform (conjugate optic after when adjoint)
  }
  auto rows = [&](const BatchArgs &x, const char *name) {
    hook(s, name, count, 0);
    hipLaunchKernelGGL((row_sweep<PL, RL, true>), dim3(N / RL, count), dim3(PL::T * RL), 0, s, x, tw);
    hipError_t e = hipGetLastError();
    hook(s, name, count, 1);
    return e;
  };
  hipError_t e = rows(a, "exact_rows_fwd");
  if (e != hipSuccess) return e;
  if (ns) {
    hook(s, "exact_cols", ns, 0);
    if constexpr (PF > 0) {
      const int blocks = pipe_blocks<PL, CL>(ns);
      hipLaunchKernelGGL((col_sweep_pipe<PL, CL, PF, true, 2>), dim3(blocks, ns), dim3(PL::T * CL), 0, s, bs, tw,
                         N / CL / blocks);
    } else {
      hipLaunchKernelGGL((col_sweep<PL, CL, true, 2>), dim3(N / CL, ns), dim3(PL::T * CL), 0, s, bs, tw);
    }
    e = hipGetLastError();
    hook(s, "exact_cols", ns, 1);
    if (e != hipSuccess) return e;
  }
  if (nb) {
    hook(s, "exact_cols_f64", nb, 0);
    hipLaunchKernelGGL((col_sweep<PL, CL, true, 1>), dim3(N / CL, nb), dim3(PL::T * CL), 0, s, b, tw);
    e = hipGetLastError();
    hook(s, "exact_cols_f64", nb, 1);
  }
  if (e != hipSuccess) return e;
  return rows(c, "exact_rows_inv");
}

hipError_t launch_exact_batch(const PlaneArgs *planes, int count, int n, const float2 *root, hipStream_t s,
                              const LaunchHook &hook, uint64_t split) {
  // the split form's column sweep is pipelined where that is faster (2048 32 us plain, 30 us; 4096 117
  // and 109 us; 8192 751 and 792 us)
  switch (n) {
    case 64: return launch_exact_sweeps<Plan<64, 8, 8, 8>, 8, 8>(planes, count, root, s, hook, split);
    case 128: return launch_exact_sweeps<Plan<128, 16, 16, 8>, 8, 8>(planes, count, root, s, hook, split);
    case 256: return launch_exact_sweeps<Plan<256, 16, 16, 16>, 4, 4>(planes, count, root, s, hook, split);
    case 512: return launch_exact_sweeps<Plan<512, 8, 8, 8, 8>, 1, 4>(planes, count, root, s, hook, split);
    case 1024: return launch_exact_sweeps<Plan<1024, 16, 16, 8, 8>, 1, 4>(planes, count, root, s, hook, split);
    case 2048: return launch_exact_sweeps<Plan<2048, 16, 16, 16, 8>, 1, 4, 12>(planes, count, root, s, hook, split);
    case 4096: return launch_exact_sweeps<Plan<4096, 16, 16, 16, 16>, 1, 4, 16>(planes, count, root, s, hook, split);
    case 8192: return launch_exact_sweeps<Plan<8192, 16, 16, 16, 16, 2>, 1, 2>(planes, count, root, s, hook, split);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_direct_batch(const PlaneArgs *planes, int count, int n, const float2 *root, hipStream_t s,
                               const LaunchHook &hook) {
  BatchArgs fwd, adj;
  int nf = 0, na = 0;
  for (int i = 0; i < count; ++i) {
    if (planes[i].flags & FR_ADJOINT)
      adj.p[na++] = planes[i];
    else
      fwd.p[nf++] = planes[i];
  }
  // one transform per sweep: the tables' copy pays where a block walks several tiles (4096 columns 82
  // and 124 us plain, 70 and 97 us pipelined; 2048 23 and 25 us; 8192 686 and 828 us)
#define FR_DIRECT(PL, RL, CL, PF) return launch_sweeps<PL, RL, CL, PF, true>(fwd, nf, adj, na, root, s, hook)
  switch (n) {
    case 64: { using P = Plan<64, 8, 8, 8>; FR_DIRECT(P, 8, 8, 0); }
    case 128: { using P = Plan<128, 16, 16, 8>; FR_DIRECT(P, 8, 8, 0); }
    case 256: { using P = Plan<256, 16, 16, 16>; FR_DIRECT(P, 4, 4, 0); }
    case 512: { using P = Plan<512, 8, 8, 8, 8>; FR_DIRECT(P, 1, 4, 0); }
    case 1024: { using P = Plan<1024, 16, 16, 8, 8>; FR_DIRECT(P, 1, 4, 0); }
    case 2048: { using P = Plan<2048, 16, 16, 16, 8>; FR_DIRECT(P, 1, 4, 0); }
    case 4096: { using P = Plan<4096, 16, 16, 16, 16>; FR_DIRECT(P, 1, 4, 16); }
    case 8192: { using P = Plan<8192, 16, 16, 16, 16, 2>; FR_DIRECT(P, 1, 2, 0); }
    default: return hipErrorInvalidValue;
  }
#undef FR_DIRECT
}

}  // namespace fr
