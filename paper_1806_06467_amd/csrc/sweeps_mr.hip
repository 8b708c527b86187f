// Mixed-radix Fresnel sweeps for plane edges that factor into radices up to 16 (for example the
// per-wavelength grids 3584 ... 4096 of a broadband model, Sec. 1.2), with planes of different
// edges in one persistent launch per sweep.
//
// Same algorithm as the power-of-two sweeps (row pass and column pass, each FFT, * h, inverse
// FFT, with the optics in the prologue/epilogue), but the radix plan is a runtime list and every
// Stockham pass goes through LDS: a thread reads the R inputs of each butterfly it owns, applies
// the twiddles (per-pass float32 tables built in float64 on the host), runs DFT_R, and writes
// the outputs after a barrier. The transfer function is applied while the first inverse pass
// reads its inputs. Blocks loop over a flattened list of (plane, row) or (plane, 4-column tile)
// work items, so one launch covers a whole batch of uneven planes. For some of a broadband
// model's grid edges a register-resident form (MrReg: the line in registers between a
// transform's first and last passes, as in the power-of-two sweeps) runs instead, one row or
// 4-column tile per block, when every plane of the launch has that edge and its plan.
//
// All accesses to fields and maps use raw buffer instructions whose per-lane offset the hardware checks
// against the array (lines past a plane read 0 and store nothing). The tables' buffers (MrTable) carry no
// length of their own: their offsets follow from the plan.
#include <algorithm>
#include <tuple>
#include <type_traits>
#include <utility>

#include "fft_mr.hpp"
#include "fr_internal.h"
#include "../../include/fresnel.h"

namespace fr {

namespace {


struct Buf64 {
  __amdgpu_buffer_rsrc_t r;
  typedef unsigned int raw64 __attribute__((__vector_size__(8)));
  __device__ __forceinline__ Buf64(const void *p, unsigned bytes)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, int(bytes), 0x00020000)) {}
  __device__ __forceinline__ c32 load(unsigned vo) const {
    const float2 q = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, vo, 0u, 0));
    return {q.x, q.y};
  }
  __device__ __forceinline__ void store(unsigned vo, c32 v) const {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(raw64, make_float2(v.x, v.y)), r, vo, 0u, 0);
  }
};

struct Buf32 {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ Buf32(const void *p, unsigned bytes)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, int(bytes), 0x00020000)) {}
  __device__ __forceinline__ float load(unsigned vo) const {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, vo, 0u, 0));
  }
};

// The optic maps of a plane as buffer resources. A missing map gets zero records, so its loads
// return 0 without touching memory: every slot's loads are then issued together, with no
// branch between them, and the selects below drop the missing terms.
struct PreMaps {
  Buf32 amp, opd, pre;
  Buf64 lens;
  int n, win, off;
  float inv_lambda;
  bool has_amp, has_phase, has_lens;
  __device__ __forceinline__ PreMaps(const PlaneArgs &pa, int n_)
      : amp(pa.amp, pa.amp ? unsigned(pa.win) * unsigned(pa.win) * 4u : 0u),
        opd(pa.opd, pa.opd ? unsigned(pa.win) * unsigned(pa.win) * 4u : 0u),
        pre(pa.pre_surf, pa.pre_surf ? unsigned(n_) * unsigned(n_) * 4u : 0u),
        lens(pa.lens, pa.lens ? unsigned(n_) * 8u : 0u),
        n(n_), win(pa.win), off((n_ - pa.win) >> 1), inv_lambda(pa.inv_lambda), has_amp(pa.amp != nullptr),
        has_phase(pa.opd != nullptr || pa.pre_surf != nullptr), has_lens(pa.lens != nullptr) {}
};
struct PreVals {
  float a, o, p;
  c32 lx;
};

// loads of the pre optic at (y, x), both < n
__device__ __forceinline__ PreVals pre_fetch(const PreMaps &m, int y, int x) {
  const int wy = min(max(y - m.off, 0), m.win - 1), wx = min(max(x - m.off, 0), m.win - 1);
  const unsigned o = unsigned(wy * m.win + wx) * 4u;
  PreVals v;
  v.a = m.amp.load(o);
  v.o = m.opd.load(o);
  v.p = m.pre.load(unsigned(y * m.n + x) * 4u);
  v.lx = m.lens.load(unsigned(x) * 8u);
  return v;
}

// pre optic amp exp(2 pi i (opd + 2 pre_surf) / lambda) lens[x] lens[y] at (y, x); ly = lens[y]
__device__ __forceinline__ c32 pre_optic(const PreMaps &m, const PreVals &v, int y, int x, c32 ly) {
  const bool in = unsigned(y - m.off) < unsigned(m.win) && unsigned(x - m.off) < unsigned(m.win);
  const float a = m.has_amp ? (in ? v.a : 0.0f) : 1.0f;
  c32 ph = {a, 0.0f};
  if (m.has_phase) {
    const float turns = (in ? v.o : 0.0f) * m.inv_lambda + 2.0f * v.p * m.inv_lambda;
    float s, c;
    sincos_turns(turns, &s, &c);
    ph = {a * c, a * s};
  }
  if (m.has_lens) ph = cmul(ph, cmul(v.lx, ly));
  return ph;
}

__device__ __forceinline__ bool mr_has_pre(const PlaneArgs &pa) {
  return pa.amp || pa.opd || pa.pre_surf || pa.lens;
}

// The plan policy of a sweep instance: MrRuntime<C> takes each plane's packed plan (any edge of
// class C: at most C, more than C / 2 above the smallest class), MrCt<N, Rs...> one compile-time
// plan (every plane of the launch has edge N and that plan). A class sets the threads per line:
// an eighth of its longest line, so that a radix-8 or larger pass runs one butterfly per thread
// and few slots of the load, the optic and the store lie past the line's end (with 256 threads and
// 16 slots for every edge a 1000^2 plane took 69 us, with 64 and 16 for its class 64 us, with 128
// and 8 39 us); a sixteenth for the largest class, where 512 threads a row are slower (a 3000^2
// row sweep 206 us against 133 us) and would leave no room for four columns.
template <int C>
struct MrRuntime {
  static constexpr int N = 0;
  static constexpr int MAXN = C;
};
template <class F>
struct MrDims {
  static constexpr int MAXN = F::MAXN;
  static constexpr int E = MAXN <= 2048 ? 8 : 16;     // slots per thread for the global load / store
  static constexpr int T = MAXN / E;                  // threads per line
  static constexpr int RL = T < 64 ? 64 / T : 1;      // rows per row block: at least one wavefront
};
template <int N, int... Rs>
struct MrDims<MrCt<N, Rs...>> {
  static constexpr int MAXN = kMrMaxN;
  static constexpr int E = 16;
  static constexpr int T = MAXN / E;
  static constexpr int RL = 1;
};

template <class F, bool INV>
__device__ __forceinline__ void plane_fft(c32 *lds, const MrPlane &mp, int t, const float2 *h, bool hconj) {
  using D = MrDims<F>;
  if constexpr (F::N == 0)
    mr_fft<INV, D::T, D::MAXN>(lds, mp.n, mp.npass, mp.plan, mp.tw, t, h, hconj);
  else
    F::template fft<INV, D::T>(lds, mp.tw, mr_opaque(t), h, hconj);
}

// The batch is the kernel's only argument, so it sits at offset 0 of the kernel-argument
// segment; reading it through that pointer keeps the dynamically indexed plane table in the
// (scalar-loaded, read-only) argument segment instead of a private copy.
__device__ __forceinline__ const MrBatch &kernarg_batch() {
  return *(const MrBatch *)__builtin_amdgcn_kernarg_segment_ptr();
}

// work item -> plane (the batch is at most kMrMaxBatch planes; block-uniform scan)
__device__ __forceinline__ int mr_find(const MrBatch &a, int item) {
  int p = 0;
  while (p + 1 < a.count && item >= a.p[p + 1].first) ++p;
  return p;
}

// blocks are dealt round-robin to the 8 XCDs; inside each round of gridDim items, give every XCD
// a contiguous run of items so that concurrently running neighbours share L2 lines
__device__ __forceinline__ int mr_item(int round) {
  const int g = gridDim.x, b = blockIdx.x;
  const int local = (g % 8 == 0) ? (b & 7) * (g / 8) + (b >> 3) : b;
  return round * g + local;
}

// slots of the global load / store handled per batch of optic loads
constexpr int kOptBatch = 8;

// multiplies v[0..E) of row y by the pre optic (conjugated when CONJ), in batches of
// kOptBatch slots whose loads are issued together
template <bool CONJ, int kT, int kEM>
__device__ __forceinline__ void apply_pre(c32 (&v)[kEM], const PlaneArgs &pa, int n, int y, int t, bool source) {
  const PreMaps pm(pa, n);
  const c32 ly = pm.lens.load(unsigned(y) * 8u);
#pragma unroll
  for (int m0 = 0; m0 < kEM; m0 += kOptBatch) {
    PreVals pv[kOptBatch];
#pragma unroll
    for (int q = 0; q < kOptBatch; ++q) pv[q] = pre_fetch(pm, y, min(t + kT * (m0 + q), n - 1));
#pragma unroll
    for (int q = 0; q < kOptBatch; ++q) {
      const c32 ph = pre_optic(pm, pv[q], y, min(t + kT * (m0 + q), n - 1), ly);
      v[m0 + q] = source ? ph : (CONJ ? cmulc(v[m0 + q], ph) : cmul(v[m0 + q], ph));
    }
  }
}

template <class F>
__global__ void __launch_bounds__(MrDims<F>::T *MrDims<F>::RL) mr_row_sweep(MrBatch) {
  constexpr int kT = MrDims<F>::T, kEM = MrDims<F>::E, RL = MrDims<F>::RL, LINE = LdsLine<MrDims<F>::MAXN>::size;
  const MrBatch &args = kernarg_batch();
  __shared__ c32 lines[RL * LINE];
  const int line = threadIdx.x / kT, t0 = threadIdx.x % kT;
  c32 *lds = lines + line * LINE;
  for (int round = 0;; ++round) {
    const int item = mr_item(round);
    if (round * int(gridDim.x) >= args.total) break;
    if (item < args.total) {
      const MrPlane &mp = args.p[mr_find(args, item)];
      const PlaneArgs &pa = mp.pa;
      const int n = F::N ? F::N : mp.n, y0 = (item - mp.first) * RL + line;
      const int y = RL > 1 ? min(y0, n - 1) : y0;  // a last block's lines past the plane repeat its last row, unstored
      const int t = mr_opaque(t0);
      const bool adj = pa.flags & FR_ADJOINT;
      const bool source = pa.flags & kSourceOptic;
      const bool pre = mr_has_pre(pa);
      const Buf64 fb(pa.field, unsigned(n) * unsigned(n) * 8u);
      c32 v[kEM];
      if (source) {
#pragma unroll
        for (int m = 0; m < kEM; ++m) v[m] = {1.0f, 0.0f};
      } else {
#pragma unroll
        for (int m = 0; m < kEM; ++m) v[m] = fb.load(unsigned(y * n + t + kT * m) * 8u);  // past the line: unused, past the plane: 0
      }
      if (!adj && pre) apply_pre<false, kT, kEM>(v, pa, n, y, t, source);
#pragma unroll
      for (int m = 0; m < kEM; ++m)
        if (t + kT * m < n) lds[lds_pad(t + kT * m)] = v[m];
      __syncthreads();
      plane_fft<F, false>(lds, mp, t, nullptr, false);
      plane_fft<F, true>(lds, mp, t, pa.h, adj);
#pragma unroll
      for (int m = 0; m < kEM; ++m) v[m] = lds[lds_pad(min(t + kT * m, n - 1))];
      if (adj && pre) apply_pre<true, kT, kEM>(v, pa, n, y, t, false);
#pragma unroll
      for (int m = 0; m < kEM; ++m)
        if (t + kT * m < n && (RL == 1 || y0 < n)) fb.store(unsigned(y * n + t + kT * m) * 8u, v[m]);
      __syncthreads();
    }
  }
}

// 4 adjacent columns per item (32-byte row segments), one line of kT threads per column
template <class F>
__global__ void __launch_bounds__(MrDims<F>::T * 4) mr_col_sweep(MrBatch) {
  constexpr int kT = MrDims<F>::T, kEM = MrDims<F>::E, LINE = LdsLine<MrDims<F>::MAXN>::size + 4;
  const MrBatch &args = kernarg_batch();
  __shared__ c32 lds[4 * LINE];
  const int c = threadIdx.x & 3, t0 = threadIdx.x >> 2;
  c32 *my = lds + c * LINE;
  for (int round = 0;; ++round) {
    const int item = mr_item(round);
    if (round * int(gridDim.x) >= args.total) break;
    if (item < args.total) {
      const MrPlane &mp = args.p[mr_find(args, item)];
      const PlaneArgs &pa = mp.pa;
      const int n = F::N ? F::N : mp.n;
      const int t = mr_opaque(t0);
      const int x = (item - mp.first) * 4 + c;
      const bool xin = x < n;
      const int xc = min(x, n - 1);
      const bool adj = pa.flags & FR_ADJOINT;
      const Buf64 fb(pa.field, unsigned(n) * unsigned(n) * 8u);
      // a missing post map has zero records (its loads return 0)
      const Buf32 post(pa.post_surf, pa.post_surf ? unsigned(post_tiled_size(n)) * 4u : 0u);
      const bool has_post = pa.post_surf != nullptr;
      c32 v[kEM];
#pragma unroll
      for (int m = 0; m < kEM; ++m) v[m] = fb.load(unsigned(min(t + kT * m, n - 1) * n + xc) * 8u);
      if (adj && has_post) {
        float sv[kEM];
#pragma unroll
        for (int m = 0; m < kEM; ++m) sv[m] = post.load(unsigned(post_tiled_index(n, min(t + kT * m, n - 1), xc)) * 4u);
#pragma unroll
        for (int m = 0; m < kEM; ++m) {
          float sn, cs;
          sincos_turns(2.0f * sv[m] * pa.inv_lambda, &sn, &cs);
          v[m] = cmulc(v[m], c32{cs, sn});
        }
      }
#pragma unroll
      for (int m = 0; m < kEM; ++m)
        if (t + kT * m < n) my[lds_pad(t + kT * m)] = v[m];
      __syncthreads();
      plane_fft<F, false>(my, mp, t, nullptr, false);
      plane_fft<F, true>(my, mp, t, pa.h, adj);
#pragma unroll
      for (int m = 0; m < kEM; ++m) v[m] = my[lds_pad(min(t + kT * m, n - 1))];
      if (!adj && has_post) {
        float sv[kEM];
#pragma unroll
        for (int m = 0; m < kEM; ++m) sv[m] = post.load(unsigned(post_tiled_index(n, min(t + kT * m, n - 1), xc)) * 4u);
#pragma unroll
        for (int m = 0; m < kEM; ++m) {
          float sn, cs;
          sincos_turns(2.0f * sv[m] * pa.inv_lambda, &sn, &cs);
          v[m] = cmul(v[m], c32{cs, sn});
        }
      }
#pragma unroll
      for (int m = 0; m < kEM; ++m)
        if (t + kT * m < n && xin) fb.store(unsigned((t + kT * m) * n + x) * 8u, v[m]);
      __syncthreads();
    }
  }
}

// ---- register-resident sweeps of the broadband grids' plans ------------------------------
// One row (row sweep) or one 4-column tile (column sweep, 32-byte row segments) per block, the
// line held in registers E elements per thread between a transform's first and last passes and
// from one transform to the next (MrReg); grid (lines, planes) with every plane of the launch of
// the policy's edge and plan.

// the pre optic on the slots x = t + T m of row y (conjugated when CONJ; the source optic itself
// when `source`), loads issued kOptBatch slots at a time
template <int E, int T, bool CONJ>
__device__ __forceinline__ void apply_pre_reg(c32 (&v)[E], const PlaneArgs &pa, int n, int y, int t, bool source) {
  const PreMaps pm(pa, n);
  const c32 ly = pm.lens.load(unsigned(y) * 8u);
#pragma unroll
  for (int m0 = 0; m0 < E; m0 += kOptBatch) {
    constexpr int B = kOptBatch;
    PreVals pv[B];
#pragma unroll
    for (int q = 0; q < B; ++q)
      if (m0 + q < E) pv[q] = pre_fetch(pm, y, t + T * (m0 + q));
#pragma unroll
    for (int q = 0; q < B; ++q)
      if (m0 + q < E) {
        const c32 ph = pre_optic(pm, pv[q], y, t + T * (m0 + q), ly);
        v[m0 + q] = source ? ph : (CONJ ? cmulc(v[m0 + q], ph) : cmul(v[m0 + q], ph));
      }
  }
}

// the frequency product with h (conj(h) for the adjoint); slot m holds frequency t + T m
template <int E, int T>
__device__ __forceinline__ void freq_reg(c32 (&v)[E], const float2 *h, int t, bool adj) {
  const MrTable ht(h);
#pragma unroll
  for (int m = 0; m < E; ++m) {
    if (m % 8 == 0) __builtin_amdgcn_sched_barrier(0);  // eight loads at a time beside the line
    const c32 q = ht.load(unsigned(t) * 8u, unsigned(T * m) * 8u);
    v[m] = adj ? cmulc(v[m], q) : cmul(v[m], q);
  }
}

// (three waves per SIMD: left alone the 3920 plan takes 183 registers, which allow two: 197 us)
template <class F>
__global__ void __launch_bounds__(F::T) __attribute__((amdgpu_waves_per_eu(3))) mrr_row_sweep(MrBatch) {
  constexpr int N = F::N, E = F::E, T = F::T;
  const MrBatch &args = kernarg_batch();
  __shared__ c32 lds[LdsLine<N>::size];
  const MrPlane &mp = args.p[blockIdx.y];
  const PlaneArgs &pa = mp.pa;
  const int y = blockIdx.x, t = threadIdx.x;
  const bool adj = pa.flags & FR_ADJOINT;
  const bool source = pa.flags & kSourceOptic;
  const bool pre = mr_has_pre(pa);
  const Buf64 fb(pa.field, unsigned(N) * unsigned(N) * 8u);
  c32 v[E];
  if (source) {
#pragma unroll
    for (int m = 0; m < E; ++m) v[m] = {1.0f, 0.0f};
  } else {
#pragma unroll
    for (int m = 0; m < E; ++m) v[m] = fb.load(unsigned(y * N + t + T * m) * 8u);
  }
  if (!adj && pre) apply_pre_reg<E, T, false>(v, pa, N, y, t, source);
  F::template fft<false>(v, lds, t, mp.tw);
  freq_reg<E, T>(v, pa.h, t, adj);
  F::template fft<true>(v, lds, t, mp.tw);
  if (adj && pre) apply_pre_reg<E, T, true>(v, pa, N, y, t, false);
#pragma unroll
  for (int m = 0; m < E; ++m) fb.store(unsigned(y * N + t + T * m) * 8u, v[m]);
}

// the post surface phasor exp(2 pi i 2 s / lambda) at rows t + T m of column x (conjugated when
// CONJ), from the 4-column tiled map
template <int E, int T, bool CONJ>
__device__ __forceinline__ void apply_post_reg(c32 (&v)[E], const PlaneArgs &pa, int n, int t, int x) {
  const Buf32 post(pa.post_surf, unsigned(post_tiled_size(n)) * 4u);
  float sv[E];
#pragma unroll
  for (int m = 0; m < E; ++m) sv[m] = post.load(unsigned(post_tiled_index(n, t + T * m, x)) * 4u);
#pragma unroll
  for (int m = 0; m < E; ++m) {
    float sn, cs;
    sincos_turns(2.0f * sv[m] * pa.inv_lambda, &sn, &cs);
    v[m] = CONJ ? cmulc(v[m], c32{cs, sn}) : cmul(v[m], c32{cs, sn});
  }
}

template <class F>
__global__ void __launch_bounds__(4 * F::T) mrr_col_sweep(MrBatch) {
  constexpr int N = F::N, E = F::E, T = F::T;
  static_assert(N % 4 == 0, "4-column tiles");
  constexpr int G = N / 4;  // column tiles per plane
  constexpr int LINE = LdsLine<N>::size + 8;
  const MrBatch &args = kernarg_batch();
  __shared__ c32 lds[4 * LINE];
  const MrPlane &mp = args.p[blockIdx.y];
  const PlaneArgs &pa = mp.pa;
  const int c = threadIdx.x & 3, t = threadIdx.x >> 2;
  // blocks are dealt round-robin to the 8 XCDs: XCD i takes a contiguous run of the tiles
  const int i = blockIdx.x & 7, k = blockIdx.x >> 3;
  const int g = i * (G / 8) + min(i, G % 8) + k;
  const int x = g * 4 + c;
  const bool adj = pa.flags & FR_ADJOINT;
  const Buf64 fb(pa.field, unsigned(N) * unsigned(N) * 8u);
  c32 v[E];
#pragma unroll
  for (int m = 0; m < E; ++m) v[m] = fb.load(unsigned((t + T * m) * N + x) * 8u);
  if (adj && pa.post_surf) apply_post_reg<E, T, true>(v, pa, N, t, x);
  c32 *my = lds + c * LINE;
  F::template fft<false>(v, my, t, mp.tw);
  freq_reg<E, T>(v, pa.h, t, adj);
  F::template fft<true>(v, my, t, mp.tw);
  if (!adj && pa.post_surf) apply_post_reg<E, T, false>(v, pa, N, t, x);
#pragma unroll
  for (int m = 0; m < E; ++m) fb.store(unsigned((t + T * m) * N + x) * 8u, v[m]);
}

}  // namespace

bool mr_plan(int n, int *npass, int *radix) { return mr_plan_build(n, kMrMaxN, kMrMaxPass, npass, radix); }
unsigned mr_pack(int npass, const int *radix) { return mr_plan_pack(npass, radix); }
int mr_plan_orders(int n, int max, unsigned *plans, int *npass) {
  int rad[kMrMaxPass];
  if (!mr_plan_build(n, kMrMaxN, kMrMaxPass, npass, rad)) return 0;
  std::sort(rad, rad + *npass, [](int a, int b) { return a > b; });
  int count = 0;
  do {
    plans[count++] = mr_plan_pack(*npass, rad);
  } while (count < max && std::next_permutation(rad, rad + *npass, [](int a, int b) { return a > b; }));
  return count;
}
int mr_twiddle_count(int npass, const int *radix) { return mr_twiddle_size(npass, radix); }
void mr_twiddle_build(int npass, const int *radix, float2 *out) { mr_twiddle_fill(npass, radix, out); }

// blocks of a persistent kernel that one compute unit holds at once
template <class K>
int resident_blocks(K kernel, int threads, int fallback) {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kernel, threads, 0) != hipSuccess || nb < 1) {
    (void)hipGetLastError();
    return fallback;
  }
  return nb;
}

// compile-time plans: the greedy plans of the 7-smooth grid edges of a broadband model
// (3584 ... 4032, Sec. 1.2); other edges and other pass orders take the runtime plan
using MrCtPlans = std::tuple<MrCt<3584, 16, 16, 14>, MrCt<3600, 16, 15, 15>, MrCt<3840, 16, 16, 15>,
                             MrCt<3888, 16, 9, 9, 3>, MrCt<3920, 16, 7, 7, 5>, MrCt<4000, 16, 10, 5, 5>,
                             MrCt<4032, 16, 14, 9, 2>>;
constexpr int kMrCt = std::tuple_size<MrCtPlans>::value;

// register-resident plans of the same edges: factorisations whose first and last radices divide
// the elements per thread (E), T = N / E threads per line, 4 T per column tile, and whose middle
// passes leave few threads idle. With E = 14 or 15 and every middle radix 16 a middle pass's
// butterflies fit the threads, so 3584, 3600 and 3840 run as the power-of-two sweeps do (measured
// per plane, rows / columns: 3584 81 / 109 us against 113 / 124 us for the greedy compile-time
// plan, 3600 96 / 104 against 117 / 129, 3840 99 / 119 against 118 / 134). 3888, 3920, 4000 and
// 4032 take three passes with two or three butterflies per thread in the middle one (324 on 216
// threads, 392 on 140, 400 on 200, 288 on 168) and large first and last radices: 3888 120 / 121 us
// against 159 / 147 for the greedy compile-time plan, 3920 169 / 130 against 174 / 183, 4000 179 /
// 135 against 180 / 159, 4032 132 / 133 against 165 / 204 for 9.16.14.2.
// The edges are the grids that a broadband model on 4096^2 pads its wavelengths to: every 7-smooth multiple
// of 16 from 7/8 of 4096 up. Other edges run the runtime plan (a rule over all edges that have such a
// factorisation would need instances with the edge at run time).
// These orders are the edges' default plans (mr_default_plan; the last entry of 4032 is the one
// that older tuning files name); a tuning file may choose another.
using MrRegPlans = std::tuple<MrReg<3584, 14, 7, 16, 16, 2>, MrReg<3600, 15, 15, 16, 15>,
                              MrReg<3840, 15, 3, 16, 16, 5>, MrReg<3888, 18, 18, 12, 18>,
                              MrReg<3920, 28, 14, 10, 28>, MrReg<4000, 20, 20, 10, 20>,
                              MrReg<4032, 24, 24, 14, 12>, MrReg<4032, 18, 9, 16, 14, 2>>;
constexpr int kMrReg = std::tuple_size<MrRegPlans>::value;

// calls f(policy) and returns true when a register-resident plan runs edge n with plan `plan`
template <class Fn, int I = 0>
bool with_mr_reg(int n, unsigned plan, Fn &&f) {
  if constexpr (I == kMrReg) {
    return false;
  } else {
    using P = std::tuple_element_t<I, MrRegPlans>;
    if (n == P::N && plan == P::packed()) {
      f(P{});
      return true;
    }
    return with_mr_reg<Fn, I + 1>(n, plan, std::forward<Fn>(f));
  }
}

template <int I = 0>
unsigned mr_reg_plan(int n) {
  if constexpr (I == kMrReg) {
    return 0u;
  } else {
    using P = std::tuple_element_t<I, MrRegPlans>;
    return n == P::N ? P::packed() : mr_reg_plan<I + 1>(n);
  }
}

// calls f(policy) for the instance that runs planes of edge n with packed plan `plan` (the
// runtime policy when no compile-time plan matches)
template <class Fn, int I = 0>
auto with_mr_policy(int n, unsigned plan, int cls, Fn &&f) {
  if constexpr (I == kMrCt) {
    switch (cls) {
      case 0: return f(MrRuntime<256>{});
      case 1: return f(MrRuntime<512>{});
      case 2: return f(MrRuntime<1024>{});
      case 3: return f(MrRuntime<2048>{});
      default: return f(MrRuntime<4096>{});
    }
  } else {
    using P = std::tuple_element_t<I, MrCtPlans>;
    if (n == P::N && plan == P::packed()) return f(P{});
    return with_mr_policy<Fn, I + 1>(n, plan, cls, std::forward<Fn>(f));
  }
}

template <class P>
void resident_of(int *rows, int *cols) {
  using D = MrDims<P>;
  *rows = resident_blocks(mr_row_sweep<P>, D::T * D::RL, 2);
  *cols = resident_blocks(mr_col_sweep<P>, 4 * D::T, 1);
}
template <int I = 0>
void resident_all(int *rows, int *cols) {
  if constexpr (I == 0) {
    resident_of<MrRuntime<256>>(rows + 0, cols + 0);
    resident_of<MrRuntime<512>>(rows + 1, cols + 1);
    resident_of<MrRuntime<1024>>(rows + 2, cols + 2);
    resident_of<MrRuntime<2048>>(rows + 3, cols + 3);
    resident_of<MrRuntime<4096>>(rows + 4, cols + 4);
  }
  if constexpr (I < kMrCt) {
    resident_of<std::tuple_element_t<I, MrCtPlans>>(rows + kMrClasses + I, cols + kMrClasses + I);
    resident_all<I + 1>(rows, cols);
  }
}

// -1 for the runtime plan, else the index of the matching compile-time plan
template <int I = 0>
int mr_policy_index(int n, unsigned plan) {
  if constexpr (I == kMrCt) {
    return -1;
  } else {
    using P = std::tuple_element_t<I, MrCtPlans>;
    if (n == P::N && plan == P::packed()) return I;
    return mr_policy_index<I + 1>(n, plan);
  }
}

unsigned mr_default_plan(int n) { return mr_reg_plan(n); }

int mr_class(int n) {
  int c = 0;
  while (c + 1 < kMrClasses && n > (256 << c)) ++c;
  return c;
}

// A plane's result does not depend on its company: edges share a launch whose instances give the same
// bits, those of all classes but the largest (they differ in threads per line only; the largest has more
// elements per thread, and its arithmetic is contracted differently). A launch for each class left small
// batches waiting for launches: 250 and 270 42 us, together 23 us; 250, 500 and 1000 94 and 46 us; twelve
// edges from 960 to 1100 284 and 287 us. Only the register-resident sweeps know radices past 16: an edge
// that has them goes by itself.
int mr_launch_count(const int *edges, int count) {
  auto shares = [&](int n) {
    const int a = mr_class(edges[0]), b = mr_class(n);
    return !mr_default_plan(edges[0]) && !mr_default_plan(n) && (a == b || std::max(a, b) < kMrClasses - 1);
  };
  int j = 1;
  while (j < count && (edges[j] == edges[0] || shares(edges[j]))) ++j;
  return j;
}

bool mr_past_16(unsigned plan) {
  for (; plan; plan >>= 5)
    if ((plan & 31u) > 16u) return true;
  return false;
}

void mr_resident(int *rows_per_cu, int *cols_per_cu) {
  static_assert(kMrClasses + kMrCt <= kMrPolicies, "residency table size");
  resident_all(rows_per_cu, cols_per_cu);
}

hipError_t launch_mr_batch(const MrBatch &all, const int *rows_per_cu, const int *cols_per_cu, int cus,
                           hipStream_t s, const LaunchHook &hook) {
  // forward planes: rows then columns; adjoint planes: columns then rows (see the power-of-two
  // sweeps: the optic maps are always read along rows)
  MrBatch fwd, adj;
  fwd.count = adj.count = 0;
  fwd.total = adj.total = 0;
  for (int i = 0; i < all.count; ++i) {
    MrBatch &dst = (all.p[i].pa.flags & FR_ADJOINT) ? adj : fwd;
    dst.p[dst.count++] = all.p[i];
  }
  auto rows_list = [](MrBatch &b, int rows_per_item) {
    int acc = 0;
    for (int i = 0; i < b.count; ++i) {
      b.p[i].first = acc;
      acc += (b.p[i].n + rows_per_item - 1) / rows_per_item;
    }
    b.total = acc;
  };
  auto cols_list = [](MrBatch &b) {
    int acc = 0;
    for (int i = 0; i < b.count; ++i) {
      b.p[i].first = acc;
      acc += (b.p[i].n + 3) / 4;
    }
    b.total = acc;
  };
  // one compile-time instance when every plane of the batch has the same edge and its plan
  int pol = all.count ? mr_policy_index(all.p[0].n, all.p[0].plan) : -1;
  int cls = 0;
  for (int i = 0; i < all.count; ++i) {
    if (all.p[i].n != all.p[0].n || all.p[i].plan != all.p[0].plan) pol = -1;
    cls = std::max(cls, mr_class(all.p[i].n));
  }
  // one register-resident instance when every plane has the same edge and its plan; the others know
  // radices up to 16 only
  bool same = all.count > 0;
  for (int i = 1; i < all.count && same; ++i)
    if (all.p[i].n != all.p[0].n || all.p[i].plan != all.p[0].plan) same = false;
  const int nr = same ? all.p[0].n : 0;
  const unsigned planr = same ? all.p[0].plan : 0u;
  if (!with_mr_reg(nr, planr, [](auto) {}))
    for (int i = 0; i < all.count; ++i)
      if (mr_past_16(all.p[i].plan)) return hipErrorInvalidValue;
  const int n0 = pol >= 0 ? all.p[0].n : 0;
  const unsigned plan0 = pol >= 0 ? all.p[0].plan : 0u;
  const int idx = pol >= 0 ? kMrClasses + pol : cls;
  const int blocks_rows = cus * rows_per_cu[idx], blocks_cols = cus * cols_per_cu[idx];
  auto rows = [&](MrBatch b, const char *name) {
    hook(s, name, b.count, 0);
    const bool reg = with_mr_reg(nr, planr, [&](auto p) {
      using P = decltype(p);
      hipLaunchKernelGGL((mrr_row_sweep<P>), dim3(P::N, b.count), dim3(P::T), 0, s, b);
    });
    if (!reg)
      with_mr_policy(n0, plan0, cls, [&](auto p) {
        using D = MrDims<decltype(p)>;
        rows_list(b, D::RL);
        hipLaunchKernelGGL((mr_row_sweep<decltype(p)>), dim3(std::max(1, std::min(blocks_rows, b.total))),
                           dim3(D::T * D::RL), 0, s, b);
      });
    hipError_t e = hipGetLastError();
    hook(s, name, b.count, 1);
    return e;
  };
  auto cols = [&](MrBatch b, const char *name) {
    cols_list(b);
    hook(s, name, b.count, 0);
    const bool reg = with_mr_reg(nr, planr, [&](auto p) {
      using P = decltype(p);
      hipLaunchKernelGGL((mrr_col_sweep<P>), dim3(P::N / 4, b.count), dim3(4 * P::T), 0, s, b);
    });
    if (!reg)
      with_mr_policy(n0, plan0, cls, [&](auto p) {
        hipLaunchKernelGGL((mr_col_sweep<decltype(p)>), dim3(std::max(1, std::min(blocks_cols, b.total))),
                           dim3(4 * MrDims<decltype(p)>::T), 0, s, b);
      });
    hipError_t e = hipGetLastError();
    hook(s, name, b.count, 1);
    return e;
  };
  hipError_t e = hipSuccess;
  if (fwd.count && (e = rows(fwd, "mr_row_sweep")) != hipSuccess) return e;
  if (fwd.count && (e = cols(fwd, "mr_col_sweep")) != hipSuccess) return e;
  if (adj.count && (e = cols(adj, "mr_col_sweep_adj")) != hipSuccess) return e;
  if (adj.count && (e = rows(adj, "mr_row_sweep_adj")) != hipSuccess) return e;
  return e;
}

}  // namespace fr
