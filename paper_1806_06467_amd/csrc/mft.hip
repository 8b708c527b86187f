// Matrix Fourier transform on the matrix cores (Sec. 1.1: the semi-analytic coronagraph of
// Soummer et al. uses matrix DFTs; Sec. 2.3: the sin/cos arrays of that matrix DFT). Unlike the
// FFT sweeps this step really is a dense contraction, so it runs on MFMA.
//
// One transform is two products with the Fourier matrix, one per axis, each
//   out(a) = sum_b in(b) exp(s 2 pi i a b du / n_d),   a, b signed about the axis, s = -1 or +1.
// The matrix is even in its cosine and odd in its sine, so each product runs on the folded input
//   P(j) = in(j) + in(-j),  M(j) = in(j) - in(-j),  j = 1 .. Q/2
// against two real matrices over positive indices only,
//   C(k) = in(0) + sum_j P(j) cos(2 pi k j du/n_d),  S(k) = sum_j M(j) sin(2 pi k j du/n_d),
//   out(+-k) = C(k) +- i s S(k),  k = 1 .. P/2,       out(0) = in(0) + sum_j P(j):
// two real products per complex value over half the inputs and half the outputs, a quarter of
// the 8 P Q real operations of the complex product, and a quarter of its matrix.
//
// The real products run on v_mfma_f32_32x32x16_bf16 from bfloat16 pieces. Every folded float32
// value x is split exactly into x = hi + mid + lo by rounding to nearest: hi = bf16(x),
// mid = bf16(x - hi), lo = x - hi - mid. Both differences are exact in float32 (each operand pair
// is within a factor of two), and lo has at most eight significant bits, so it is a bfloat16 too;
// |mid| <= 2^-8 |x| and |lo| <= 2^-16 |x|. The cosines and sines are split the same way on the
// host from float64 (their three pieces hold 2^-25, more than a float32 table's entry). A real
// product is the sum of the nine piece products, each exact in float32; the kernel forms the six
// down to 2^-16 (hi hi, hi mid, mid hi, mid mid, hi lo, lo hi); the three left out are below
// 2^-23 together and, as round-to-nearest residuals, of either sign. The hi hi products and the
// correction products go to separate float32 sums, so that the corrections are never rounded at
// the scale of the running total; every kFoldDepth pairs the hi hi sums are added into float64 totals
// (the long Fourier sums of the coronagraph cancel to tiny values in the dark hole, so their
// rounding must not grow with the length). The correction sums stay in float32 to the end of a slice:
// their terms are below 2^-7 of the products', so of N pairs they leave about 2^-31 sqrt(5 N / 8) of
// the largest term (2^-26 for 8192 inputs), and taking them along in every fold cost 2 to 5 % of the
// products from 512 outputs on and changed no error by more than 2 %.
//
// The matrix unit rounds with a bias: of each eight products it cuts what lies below 2^-24 of the largest
// towards zero, and where the running sum is the smaller one it cuts that towards minus infinity (a model
// with these cuts gives 99.98 % of 4000 random sums bit for bit). The first product's rows share the second
// cut's bias, and the second product adds it up at frequency 0: with inputs over twelve decades the outputs
// of the axis were six times as far off as the others (4095^2 -> 64^2). So half of every sum runs with the
// opposite sign, by matrix entries of that sign (fold_negated), and the bias cancels between the halves; the
// short sums, which one float32 sum holds, take a sign by free index instead.
//
// The epilogue (alpha, beta, mask, intensity) runs in float64. Products with few tiles and long sums are
// split over j; the float64 partial sums go to the workspace and split_reduce adds them in a fixed order
// (deterministic).
// Measured (MI355X, 4096^2 -> 256^2 and back): 763 us with the complex products on float32 MFMA
// tiles, 214 us folded on the general kernel alone, 154 us with the short sums on their own kernel, the
// loads ordered as below and the split by cost; the result's distance from 64 bits 1.5e-7 before, 7e-8 now.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>

#include "fr_internal.h"

namespace fr {

// Output tiles per block of the short kernel, by the least time: rounds of a block per compute unit, each
// its start (two tiles' worth) and its tiles one per SIMD at a time. (Blocks for every compute unit,
// rounded up, left a nearly empty second round on most edges that are no power of two: 256^2 -> 2050^2
// 60 us, 39 us; 16^2 -> 2600^2 38 us, 27 us, the complex product 29 us.)
int fold_short_tiles(int tiles, int ftiles) {
  auto div_up = [](int x, int y) { return (x + y - 1) / y; };
  int per = tiles, least = div_up(ftiles, 256) * (2 + div_up(tiles, 4));
  for (int chunks = 2; chunks <= tiles; ++chunks) {
    const int p = div_up(tiles, chunks), cost = div_up(div_up(tiles, p) * ftiles, 256) * (2 + div_up(p, 4));
    if (cost < least) {
      least = cost;
      per = p;
    }
  }
  return per;
}

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

struct FoldParams {
  FoldArgs a;
  int split;         // slices of the pairs (gridDim.z)
  int j_per_split;   // multiple of kFoldStage
  double2 *partial;  // split x rows x columns of the output when split > 1
};

// result (i, j) = alpha acc + beta Cin, times mask, in float64; written to C and/or
// accumulated as weight |result|^2 into the float64 intensity map
__device__ __forceinline__ void epilogue(const FoldArgs &a, int i, int j, double cr, double ci) {
  double orr = a.alpha * cr;
  double oi = a.alpha * ci;
  if (a.beta != 0.f) {
    const float2 old = a.Cin ? a.Cin[size_t(i) * a.ldcin + j] : a.C[size_t(i) * a.ldc + j];
    orr += double(a.beta) * double(old.x);
    oi += double(a.beta) * double(old.y);
  }
  if (a.mask) {
    const double mk = a.mask[size_t(i) * a.ldm + j];
    orr *= mk;
    oi *= mk;
  }
  if (!a.skip_c) a.C[size_t(i) * a.ldc + j] = make_float2(float(orr), float(oi));
  if (a.intensity) {
    double *ip = a.intensity + size_t(i) * a.ldi + j;
    *ip += a.weight * (orr * orr + oi * oi);
  }
}

// the same in two steps, what result (i, j) reads and the result: a block that forms several issues
// all their loads ahead of the first store
struct EpilogueIn {
  float2 old;
  float mask;
  double intensity;
  __device__ __forceinline__ void load(const FoldArgs &a, int i, int j) {
    if (a.beta != 0.f) old = a.Cin ? a.Cin[size_t(i) * a.ldcin + j] : a.C[size_t(i) * a.ldc + j];
    if (a.mask) mask = a.mask[size_t(i) * a.ldm + j];
    if (a.intensity) intensity = a.intensity[size_t(i) * a.ldi + j];
  }
  __device__ __forceinline__ void store(const FoldArgs &a, int i, int j, double cr, double ci) const {
    double orr = a.alpha * cr;
    double oi = a.alpha * ci;
    if (a.beta != 0.f) {
      orr += double(a.beta) * double(old.x);
      oi += double(a.beta) * double(old.y);
    }
    if (a.mask) {
      const double mk = mask;
      orr *= mk;
      oi *= mk;
    }
    if (!a.skip_c) a.C[size_t(i) * a.ldc + j] = make_float2(float(orr), float(oi));
    if (a.intensity) a.intensity[size_t(i) * a.ldi + j] = intensity + a.weight * (orr * orr + oi * oi);
  }
};

// Blocks are dealt round-robin to the 8 XCDs (each with its own L2). Renumber them so that each
// XCD runs a contiguous range of tiles; inside a slice the range is walked in groups of
// kGroupRows tile rows, column by column, so that the blocks resident on an XCD at one time share
// a few panels of the data and of the matrix in that XCD's L2.
__device__ __forceinline__ void block_tile(int &bx, int &by, int &bz) {
  constexpr int kGroupRows = 8;
  const int gx = gridDim.x, gy = gridDim.y;
  const int total = gx * gy * gridDim.z;
  const int lin = blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z);
  const int tile = total % 8 == 0 ? (lin & 7) * (total >> 3) + (lin >> 3) : lin;
  bz = tile / (gx * gy);
  const int t = tile % (gx * gy);
  const int g = t / (kGroupRows * gx);             // group of tile rows
  const int rows = min(kGroupRows, gy - g * kGroupRows);
  const int u = t % (kGroupRows * gx);             // position inside the group
  bx = u / rows;
  by = g * kGroupRows + u % rows;
}

// two values as packed bfloat16 pairs of their pieces (first value in the low half), x = hi +
// mid + lo exactly for each (see above)
__device__ __forceinline__ void bf_split2(float x0, float x1, unsigned &hi, unsigned &mid, unsigned &lo) {
  hi = __builtin_bit_cast(unsigned, __builtin_convertvector(floatx2{x0, x1}, bf16x2));
  const float r0 = x0 - __uint_as_float(hi << 16), r1 = x1 - __uint_as_float(hi & 0xffff0000u);
  mid = __builtin_bit_cast(unsigned, __builtin_convertvector(floatx2{r0, r1}, bf16x2));
  const float l0 = r0 - __uint_as_float(mid << 16), l1 = r1 - __uint_as_float(mid & 0xffff0000u);
  lo = __builtin_bit_cast(unsigned, __builtin_convertvector(floatx2{l0, l1}, bf16x2));
}

constexpr int kFoldFree = 32;      // free indices (rows or columns of the data) per block
constexpr int kFoldStage = 64;     // pairs per stage: four 16-deep MFMA steps
constexpr int kFoldThreads = 512;  // eight waves
constexpr int kFoldDepth = 64;     // pairs a float32 sum runs over before it goes to float64
constexpr int kFoldPieces = 12;    // P.re, P.im, M.re, M.im, each hi, mid, lo
// a piece of one stage in LDS: 16-byte units of eight consecutive pairs of one free index, unit
// (pair / 8) * 32 + free index, so that a wave's fragment read is 1 KiB contiguous; the free
// index is xored with twice the group of eight pairs, so that half a wave's 8-byte stores along
// the pairs (eight groups of two free indices) fall on 32 different bank pairs
__device__ __forceinline__ int fold_unit(int g8, int f) { return g8 * kFoldFree + (f ^ ((g8 & 7) << 1)); }

constexpr int kPieceUnits = kFoldFree * kFoldStage / 8;  // 16-byte units of a piece of one stage

// A thread's share of the folding: four consecutive pairs of one free index per stage.
template <bool COLS>
struct FoldLoader {
  struct Regs {
    float2 p[4], m[4];
  };
  const float2 *centre;  // element 0 of this thread's free index (clamped to the last)
  ptrdiff_t step;        // elements between consecutive indices
  int half, full_pairs;  // pairs j = 1 .. half; in(+j) exists up to full_pairs (one less for even Q)
  int lf, jq, wunit, wbyte;
  bool zero_tile;        // keep the sum of P for out(0)
  double zero_re = 0.0, zero_im = 0.0;
  // the block's free indices as a raw buffer, when its bytes fit 32-bit offsets: this thread's
  // offsets of in(+j) and in(-j - 3) (rows) or in(-j) (columns), j its first pair of stage 0
  __amdgpu_buffer_rsrc_t rsrc;
  unsigned row_bytes, vp, vm;
  bool fits;

  __device__ __forceinline__ FoldLoader(const FoldArgs &a, int tid, int f0, bool zero) {
    half = a.Q / 2;
    full_pairs = a.Q - 1 - half;
    lf = COLS ? tid & 31 : tid >> 4;
    jq = COLS ? tid >> 5 : tid & 15;
    const int f = min(f0 + lf, a.F - 1);
    step = COLS ? a.ldd : 1;
    centre = COLS ? a.data + size_t(half) * a.ldd + f : a.data + size_t(f) * a.ldd + half;
    wunit = fold_unit(jq >> 1, lf);
    wbyte = (jq & 1) * 8;
    zero_tile = zero;
    const float2 *base = COLS ? a.data + f0 : a.data + size_t(f0) * a.ldd;
    const int nf = min(kFoldFree, a.F - f0);
    const size_t bytes = (COLS ? size_t(a.Q - 1) * a.ldd + nf : size_t(nf - 1) * a.ldd + a.Q) * 8;
    fits = bytes < (size_t(1) << 31);
    rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float2 *>(base), (short)0, int(fits ? bytes : 0), 0x00020000);
    row_bytes = unsigned(a.ldd) * 8u;
    const unsigned at = COLS ? unsigned(half) * row_bytes + unsigned(f - f0) * 8u
                             : unsigned(f - f0) * row_bytes + unsigned(half) * 8u;
    const unsigned j = 4u * jq + 1u;
    vp = at + (COLS ? j * row_bytes : j * 8u);
    vm = at - (COLS ? j * row_bytes : (j + 3u) * 8u);
  }
  // a whole stage of pairs j0 + 1 .. j0 + kFoldStage <= half. An even Q has no in(+half): what its
  // slot reads (the next row's start, or 0 past the buffer, whose range check sees the whole
  // per-lane offset) is replaced by 0.
  __device__ __forceinline__ void load(Regs &r, int j0) const {
    typedef float f4 __attribute__((ext_vector_type(4)));
    const unsigned d = unsigned(j0) * (COLS ? row_bytes : 8u);
    if constexpr (COLS) {
#pragma unroll
      for (unsigned q = 0; q < 4; ++q) {
        r.p[q] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rsrc, vp + d + q * row_bytes, 0, 0));
        r.m[q] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rsrc, vm - d - q * row_bytes, 0, 0));
      }
    } else {
      const f4 p0 = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, vp + d, 0, 0));
      const f4 p1 = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, vp + d + 16u, 0, 0));
      const f4 m1 = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, vm - d, 0, 0));
      const f4 m0 = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, vm - d + 16u, 0, 0));
      r.p[0] = make_float2(p0[0], p0[1]);
      r.p[1] = make_float2(p0[2], p0[3]);
      r.p[2] = make_float2(p1[0], p1[1]);
      r.p[3] = make_float2(p1[2], p1[3]);
      r.m[0] = make_float2(m0[2], m0[3]);
      r.m[1] = make_float2(m0[0], m0[1]);
      r.m[2] = make_float2(m1[2], m1[3]);
      r.m[3] = make_float2(m1[0], m1[1]);
    }
  }
  __device__ __forceinline__ void trim(Regs &r, int j0) const {
    if (j0 + 4 * jq + 4 > full_pairs) r.p[3] = make_float2(0.f, 0.f);
  }
  // any stage, element by element, zero past the last pair
  __device__ __forceinline__ void load_any(Regs &r, int j0) const {
    const int j = j0 + 4 * jq + 1;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      r.p[q] = j + q <= full_pairs ? centre[(j + q) * step] : make_float2(0.f, 0.f);
      r.m[q] = j + q <= half ? centre[-(j + q) * step] : make_float2(0.f, 0.f);
    }
  }
  __device__ __forceinline__ void scale(Regs &r, float w) const {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      r.p[q] = make_float2(w * r.p[q].x, w * r.p[q].y);
      r.m[q] = make_float2(w * r.m[q].x, w * r.m[q].y);
    }
  }
  // the largest magnitude's bits
  __device__ __forceinline__ unsigned peak(const Regs &r) const {
    unsigned k = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      k = max(max(max(k, __float_as_uint(r.p[q].x) & 0x7fffffffu), __float_as_uint(r.p[q].y) & 0x7fffffffu),
              max(__float_as_uint(r.m[q].x) & 0x7fffffffu, __float_as_uint(r.m[q].y) & 0x7fffffffu));
    return k;
  }
  __device__ __forceinline__ void put_part(uint4 *dst, float v0, float v1, float v2, float v3) const {
    unsigned h[2], m[2], l[2];
    bf_split2(v0, v1, h[0], m[0], l[0]);
    bf_split2(v2, v3, h[1], m[1], l[1]);
    unsigned char *d = reinterpret_cast<unsigned char *>(dst + wunit) + wbyte;
    *reinterpret_cast<uint2 *>(d) = make_uint2(h[0], h[1]);
    *reinterpret_cast<uint2 *>(d + kPieceUnits * 16) = make_uint2(m[0], m[1]);
    *reinterpret_cast<uint2 *>(d + 2 * kPieceUnits * 16) = make_uint2(l[0], l[1]);
  }
  // fold the real (imaginary) parts of the four pairs, split them and write their six pieces to
  // the stage buffer [kFoldPieces][kPieceUnits]; `count`: add to the sum for out(0)
  __device__ __forceinline__ void put_re(const Regs &r, uint4 *buf, bool count) {
    const float s0 = r.p[0].x + r.m[0].x, s1 = r.p[1].x + r.m[1].x, s2 = r.p[2].x + r.m[2].x, s3 = r.p[3].x + r.m[3].x;
    if (zero_tile && count) zero_re += double((s0 + s1) + (s2 + s3));
    put_part(buf, s0, s1, s2, s3);
    put_part(buf + 6 * kPieceUnits, r.p[0].x - r.m[0].x, r.p[1].x - r.m[1].x, r.p[2].x - r.m[2].x, r.p[3].x - r.m[3].x);
  }
  __device__ __forceinline__ void put_im(const Regs &r, uint4 *buf, bool count) {
    const float s0 = r.p[0].y + r.m[0].y, s1 = r.p[1].y + r.m[1].y, s2 = r.p[2].y + r.m[2].y, s3 = r.p[3].y + r.m[3].y;
    if (zero_tile && count) zero_im += double((s0 + s1) + (s2 + s3));
    put_part(buf + 3 * kPieceUnits, s0, s1, s2, s3);
    put_part(buf + 9 * kPieceUnits, r.p[0].y - r.m[0].y, r.p[1].y - r.m[1].y, r.p[2].y - r.m[2].y, r.p[3].y - r.m[3].y);
  }
};

// data fragment times matrix fragment; COLS: the output tile is transposed (the free index along
// the lanes) by swapping the operands
template <bool COLS>
__device__ __forceinline__ floatx16 fold_mfma(bf16x8 d, bf16x8 t, floatx16 c) {
  if constexpr (COLS) return __builtin_amdgcn_mfma_f32_32x32x16_bf16(t, d, c, 0, 0, 0);
  else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(d, t, c, 0, 0, 0);
}

// one 16-deep step of one parity: re and im, each into its hi hi and its correction sum. The five
// corrections smallest first (mid mid, lo hi, hi lo, mid hi, hi mid), then hi hi
template <bool COLS>
__device__ __forceinline__ void fold_step(const bf16x8 (&d)[6], const bf16x8 (&b)[3], floatx16 &rh, floatx16 &rc,
                                          floatx16 &ih, floatx16 &ic) {
  constexpr int lx[5] = {1, 2, 0, 1, 0}, ly[5] = {1, 0, 2, 0, 1};
#pragma unroll
  for (int q = 0; q < 5; ++q) {
    rc = fold_mfma<COLS>(d[lx[q]], b[ly[q]], rc);
    ic = fold_mfma<COLS>(d[3 + lx[q]], b[ly[q]], ic);
  }
  rh = fold_mfma<COLS>(d[0], b[0], rh);
  ih = fold_mfma<COLS>(d[3], b[0], ih);
}

// What a block's magnitudes are, from the largest bit pattern each lane saw: flags per wave, and after a
// barrier those of the block
enum { kSmall = 1, kWithin = 2, kBeyond = 4 };  // some not zero, some from `low` on, some from `high` on
__device__ __forceinline__ void range_mark(int *range, int wave, int lane, unsigned peak, unsigned low, unsigned high) {
  const int mine = (__any(peak != 0u) ? kSmall : 0) | (__any(peak >= low) ? kWithin : 0) | (__any(peak >= high) ? kBeyond : 0);
  if (lane == 0) range[wave] = mine;
}
__device__ __forceinline__ int range_seen(const int *range) {
  int all = 0;
#pragma unroll
  for (int w = 0; w < kFoldThreads / 64; ++w) all |= range[w];
  return __builtin_amdgcn_readfirstlane(all);
}

// One folded product. A block forms 32 free indices by 64 positive outputs (both signs of each):
// eight waves, each one parity (cosine or sine), one 32-wide output tile and one half of every
// stage's pairs (the halves are added in the epilogue). The data are loaded two stages ahead,
// folded and split by all threads into the other LDS buffer while the current stage is
// multiplied; the matrix comes fragment by fragment (1 KiB, L2-resident) straight from its table,
// a stage ahead. Vector loads return in order, so each stage issues its matrix loads before its
// data loads: a wait for the matrix then never waits for data still on their way from HBM.
template <bool COLS>
__global__ void __launch_bounds__(kFoldThreads) __attribute__((amdgpu_waves_per_eu(2)))
fold_kernel(FoldParams gp) {
  constexpr int KT = 2, KS = 2;  // output tiles per block, halves of a stage
  using Loader = FoldLoader<COLS>;
  const FoldArgs &a = gp.a;
  __shared__ __attribute__((aligned(16))) unsigned char lds[8 * 16 * 64 * 16 + 16 * kFoldFree * 16];
  __shared__ float2 in0[kFoldFree];  // the unpaired element of each free index (slice 0 adds it)
  __shared__ __attribute__((aligned(16))) int range[kFoldThreads / 64];
  uint4 *pieces = reinterpret_cast<uint4 *>(lds);  // [2][kFoldPieces][kPieceUnits]
  constexpr int kBuf = kFoldPieces * kPieceUnits;
  static_assert(2 * kBuf * 16 <= 8 * 16 * 64 * 16, "stage buffers fit the exchange area");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int par = wave & 1, kt = (wave >> 1) % KT, ks = (wave >> 1) / KT;
  int bx, by, bz;
  block_tile(bx, by, bz);
  const int f0 = by * kFoldFree;
  Loader ld(a, tid, f0, bx == 0);
  const int half = ld.half;
  const int jbeg = bz * gp.j_per_split;
  const int jend = min(half, jbeg + gp.j_per_split);
  const int nst = jend > jbeg ? (jend - jbeg + kFoldStage - 1) / kFoldStage : 0;

  // this wave's matrix fragments: [parity][output tile][step][piece], 64 lanes of eight values
  const int out_half = a.P / 2;
  const int tiles = fold_tiles(a.P), steps = fold_steps(a.Q);
  const int ktile = bx * KT + kt;
  const bf16x8 *tab = reinterpret_cast<const bf16x8 *>(a.table) +
                      (size_t(par) * tiles + min(ktile, tiles - 1)) * steps * 3 * 64 + lane;
  auto load_tab = [&](bf16x8 (&b)[2][3], int step) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int q = 0; q < 3; ++q) b[t][q] = tab[(size_t(step + t) * 3 + q) * 64];
  };

  // float32 sums of the current group (re and im, each as hi hi and correction sums; the corrections'
  // run on to the end, see the head of this file)
  floatx16 rh = floatx16{0.f}, rc = floatx16{0.f}, ih = floatx16{0.f}, ic = floatx16{0.f};
  double totr[16], toti[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) totr[r] = toti[r] = 0.0;
  auto multiply = [&](int buf, int sub, const bf16x8 (&b)[3]) {
    const int g8 = sub * 2 + (lane >> 5);
    const uint4 *src = pieces + buf * kBuf + 6 * par * kPieceUnits + fold_unit(g8, lane & 31);
    bf16x8 d[6];
#pragma unroll
    for (int q = 0; q < 6; ++q) d[q] = __builtin_bit_cast(bf16x8, src[q * kPieceUnits]);
    fold_step<COLS>(d, b, rh, rc, ih, ic);
  };
  auto fold = [&] {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      totr[r] += double(rh[r]);
      toti[r] += double(ih[r]);
    }
    rh = floatx16{0.f};
    ih = floatx16{0.f};
  };

  constexpr int kStagesPerFold = kFoldDepth / 32;
  typename Loader::Regs r0, r1;
  bf16x8 tb[2][2][3];
  const int step0 = jbeg / 16 + 2 * ks;  // the steps are padded to whole stages
  // (a slice past the last pair, where whole stages leave too few for every slice, has no stage)
  const int nfull = ld.fits ? max(jend - jbeg, 0) / kFoldStage : 0;
  int pending = 0;
  if (nfull > 0) {
    ld.load(r0, jbeg);
    load_tab(tb[0], step0);
    ld.load(r1, jbeg + min(1, nfull - 1) * kFoldStage);
    ld.trim(r0, jbeg);
    ld.put_re(r0, pieces, true);
    ld.put_im(r0, pieces, true);
    __syncthreads();
    // stage s: multiply LDS buffer `buf` while `ready` (stage s + 1) is split into the other
    // buffer and `fill` receives stage s + 2 (the last stages reload the last one; their split
    // goes to a buffer nobody reads again)
    auto stage = [&](int s, int buf, typename Loader::Regs &fill, typename Loader::Regs &ready) {
      uint4 *other = pieces + (buf ^ 1) * kBuf;
      const int next = min(s + 1, nfull - 1);
      load_tab(tb[buf ^ 1], step0 + 4 * next);
      __builtin_amdgcn_sched_barrier(0);
      ld.load(fill, jbeg + min(s + 2, nfull - 1) * kFoldStage);
      __builtin_amdgcn_sched_barrier(0);
      multiply(buf, 2 * ks, tb[buf][0]);
      __builtin_amdgcn_sched_barrier(0);  // half a stage more for the loads of stage s + 1
      ld.trim(ready, jbeg + next * kFoldStage);
      multiply(buf, 2 * ks + 1, tb[buf][1]);
      ld.put_re(ready, other, s + 1 < nfull);
      ld.put_im(ready, other, s + 1 < nfull);
      if (++pending == kStagesPerFold) {
        fold();
        pending = 0;
      }
      __syncthreads();
    };
    // (one exit at the end of both halves keeps the register sets in place: with another in the
    // middle the compiler moved them at the loop's head, waiting for the loads under way)
    int s = 0;
    for (; s + 2 <= nfull; s += 2) {
      stage(s, 0, r0, r1);
      stage(s + 1, 1, r1, r0);
    }
    if (s < nfull) stage(s, 0, r0, r1);
  }
  // The ends of float32's range lie outside the pieces': a value from 2^128 - 2^119 on rounds to an
  // infinite piece and a sum of two may be infinite from 2^127 on, so that the totals are not finite;
  // below 2^-110 the last piece is cut. A block whose totals are not finite, or all below 2^-100,
  // repeats its sums on data scaled by 2^-16 or 2^32 (unscaled again if that was too much, where larger
  // values had cancelled). The look at the totals costs at most 1 % of a transform.
  constexpr float kDown = 0x1p-16f, kUp = 0x1p32f;
  float scale = 1.f;
  double2 *ex = reinterpret_cast<double2 *>(lds);
  double2 *zs = ex + 8 * 16 * 64;  // [16 groups of pairs][free index]
  float2 unpaired = make_float2(0.f, 0.f);
  if (bz == 0 && tid < kFoldFree) {
    // (the address is formed here: kept across the products it costs registers they need)
    unsigned f = tid;
    asm("" : "+v"(f));
    f = min(f0 + int(f), a.F - 1);
    unpaired = COLS ? a.data[size_t(half) * a.ldd + f] : a.data[size_t(f) * a.ldd + half];
  }
  for (int first = nfull, repeats = 0;; first = 0, ++repeats) {
    // a last partial stage (every stage where the data's bytes do not fit 32-bit offsets, or repeated)
    for (int s = first; s < nst; ++s) {
      ld.load_any(r0, jbeg + s * kFoldStage);
      if (scale != 1.f) ld.scale(r0, scale);
      load_tab(tb[0], step0 + 4 * s);
      ld.put_re(r0, pieces, true);
      ld.put_im(r0, pieces, true);
      __syncthreads();
      multiply(0, 2 * ks, tb[0][0]);
      multiply(0, 2 * ks + 1, tb[0][1]);
      if (++pending == kStagesPerFold) {
        fold();
        pending = 0;
      }
      __syncthreads();
    }
    // exchange: every wave's totals, then each wave of a tile (2 parities x KS halves) forms both
    // signs of its share of the tile's outputs (every stage ended on a barrier: the buffers are free)
    double sum[2] = {0.0, 0.0};
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      totr[r] += double(rh[r]) + double(rc[r]);
      toti[r] += double(ih[r]) + double(ic[r]);
      ex[(wave * 16 + r) * 64 + lane] = make_double2(totr[r], toti[r]);
      sum[0] += fabs(totr[r]);
      sum[1] += fabs(toti[r]);
    }
    zs[ld.jq * kFoldFree + ld.lf] = make_double2(ld.zero_re, ld.zero_im);
    if (tid < kFoldFree) in0[tid] = unpaired;
    range_mark(range, wave, lane, unsigned(__double2hiint(sum[0] + sum[1])), unsigned(1023 - 100) << 20, 0x7ff00000u);
    __syncthreads();
    const int seen = range_seen(range);
    float next = scale;
    if (repeats == 0) next = seen & kBeyond ? kDown : seen == kSmall ? kUp : 1.f;
    else if (scale == kUp && (seen & kBeyond)) next = 1.f;
    if (next == scale) break;
    __syncthreads();
    scale = next;
    pending = 0;
    ld.zero_re = ld.zero_im = 0.0;
    rh = rc = ih = ic = floatx16{0.f};
#pragma unroll
    for (int r = 0; r < 16; ++r) totr[r] = toti[r] = 0.0;
  }
  const double back = 1.0 / double(scale);
  const int rows = COLS ? a.P : a.F, cols = COLS ? a.F : a.P;
  // A column product, the second of a transform, may add a background and apply a mask: its eight
  // results' loads go out ahead of the stores (one after the other, each behind the last one's wait,
  // they were up to 2 us of the 1024-edge products: the 21-wavelength train 12.58 ms, 12.40 ms). A row product
  // only stores, and there the two steps cost 1 us.
  auto load_in = [&](EpilogueIn &in, int o, int ff) {
    if (COLS && gp.split == 1) in.load(a, o, ff);
  };
  auto emit = [&](int o, int ff, double re, double im, const EpilogueIn &in) {
    const int i = COLS ? o : ff, j = COLS ? ff : o;
    if (gp.split > 1) gp.partial[(size_t(bz) * rows + i) * cols + j] = make_double2(re, im);
    else if (COLS) in.store(a, i, j, re, im);
    else epilogue(a, i, j, re, im);
  };
  constexpr int SHARE = 16 / (2 * KS);
  const int share = (par * KS + ks) * SHARE;
  const double sg = a.sign;
  // item r of lane l sits at row (r/4)*8 + (l/32)*4 + r%4, column l%32 of a 32 x 32 tile
  auto item = [&](int rr, int &lf, int &k) {
    const int r = share + rr, trow = (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3), tcol = lane & 31;
    lf = COLS ? tcol : trow;
    k = ktile * 32 + (COLS ? trow : tcol) + 1;
    return f0 + lf < a.F && k <= out_half;
  };
  EpilogueIn plus[SHARE], minus[SHARE];
#pragma unroll
  for (int rr = 0; rr < SHARE; ++rr) {
    int lf, k;
    if (!item(rr, lf, k)) continue;
    if (k < a.P - out_half) load_in(plus[rr], out_half + k, f0 + lf);
    load_in(minus[rr], out_half - k, f0 + lf);
  }
#pragma unroll
  for (int rr = 0; rr < SHARE; ++rr) {
    const int r = share + rr;
    double2 c = make_double2(0.0, 0.0), s = make_double2(0.0, 0.0);
#pragma unroll
    for (int h = 0; h < KS; ++h) {
      const double2 cv = ex[(((h * KT + kt) * 2) * 16 + r) * 64 + lane];
      const double2 sv = ex[(((h * KT + kt) * 2 + 1) * 16 + r) * 64 + lane];
      const double w = fold_negated(2 * h) ? -back : back;  // (the sign of the half's matrix entries)
      c.x += w * cv.x;
      c.y += w * cv.y;
      s.x += w * sv.x;
      s.y += w * sv.y;
    }
    int lf, k;
    if (!item(rr, lf, k)) continue;
    const float2 z = in0[lf];
    c.x += double(z.x);
    c.y += double(z.y);
    if (k < a.P - out_half) emit(out_half + k, f0 + lf, c.x - sg * s.y, c.y + sg * s.x, plus[rr]);
    emit(out_half - k, f0 + lf, c.x + sg * s.y, c.y - sg * s.x, minus[rr]);
  }
  if (bx == 0 && tid < kFoldFree && f0 + tid < a.F) {
    EpilogueIn in;
    load_in(in, out_half, f0 + tid);
    double2 z = make_double2(in0[tid].x, in0[tid].y);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const double2 v = zs[q * kFoldFree + tid];
      z.x += back * v.x;
      z.y += back * v.y;
    }
    emit(out_half, f0 + tid, z.x, z.y, in);
  }
}

// the sign with which a free index's data go through the short kernel (see the head of this file),
// mixed so that it has no frequency of its own
__device__ __forceinline__ float short_sign(int f) {
  unsigned h = unsigned(f) * 0x9e3779b1u;
  h = (h ^ (h >> 15)) * 0x2c1b3c6du;
  return h >> 31 ? -1.f : 1.f;
}

// The same for at most kShortPairs pairs, where the general kernel's blocks spend their time
// filling and draining (two stages, then the exchange of the totals). Here the block folds and
// splits its 32 free indices once, keeps all their pieces in LDS (96 KiB) and its waves walk the
// output tiles on their own, without barriers: a wave forms both parities of a tile in one float32
// group, so the outputs of either sign come straight from its registers, and its stores overlap
// the other waves' products. (256^2 -> 4096^2: 60 us against 120 us on the general kernel.)
constexpr int kShortPairs = 2 * kFoldStage;
template <bool COLS>
__global__ void __launch_bounds__(kFoldThreads) __attribute__((amdgpu_waves_per_eu(2)))
fold_short_kernel(FoldArgs a, int tiles_per_block) {
  using Loader = FoldLoader<COLS>;
  constexpr int kBuf = kFoldPieces * kPieceUnits;
  __shared__ __attribute__((aligned(16))) uint4 pieces[2 * kBuf];  // [stage][kFoldPieces][kPieceUnits]
  __shared__ double2 zs[16 * kFoldFree];                           // [group of pairs][free index]
  __shared__ float2 in0[kFoldFree];
  __shared__ __attribute__((aligned(16))) int range[kFoldThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int f0 = blockIdx.y * kFoldFree;
  const int out_half = a.P / 2, tiles = fold_tiles(a.P), steps = fold_steps(a.Q);
  Loader ld(a, tid, f0, blockIdx.x == 0);
  const int used = (ld.half + 31) / 32 * 2;  // steps with a pair, in twos (both stages end on zeros)
  const int top = max(used - 2, 0);          // the first two that are summed
  double back = 1.0;
  {
    typename Loader::Regs r0, r1;
    auto load = [&](typename Loader::Regs &r, int j0) {
      if (ld.fits && ld.half >= j0 + kFoldStage) {
        ld.load(r, j0);
        ld.trim(r, j0);
      } else {
        ld.load_any(r, j0);
      }
    };
    load(r0, 0);
    load(r1, kFoldStage);
    // the block's data in the range of the pieces (see fold_kernel; here the values themselves tell)
    const unsigned peak = max(ld.peak(r0), ld.peak(r1));
    range_mark(range, wave, lane, peak, unsigned(127 - 70) << 23, unsigned(127 + 100) << 23);
    __syncthreads();
    const int seen = range_seen(range);
    const float scale = seen & kBeyond ? 0x1p-32f : seen == kSmall ? 0x1p64f : 1.f;
    back = 1.0 / double(scale);
    // the sign of the free index, and of the matrix entries of the thread's step
    const float sgn = short_sign(f0 + ld.lf) * (fold_negated(ld.jq >> 2) ? -1.f : 1.f);
    ld.scale(r0, sgn * scale);
    ld.scale(r1, sgn * scale);
    ld.put_re(r0, pieces, true);
    ld.put_im(r0, pieces, true);
    ld.put_re(r1, pieces + kBuf, true);
    ld.put_im(r1, pieces + kBuf, true);
    if (ld.jq == 0) in0[ld.lf] = *ld.centre;
    zs[ld.jq * kFoldFree + ld.lf] = make_double2(sgn * back * ld.zero_re, sgn * back * ld.zero_im);
  }
  __syncthreads();
  const double sg = a.sign;
  auto emit = [&](int o, int ff, double re, double im) { epilogue(a, COLS ? o : ff, COLS ? ff : o, re, im); };
  const int last = min(tiles, int(blockIdx.x + 1) * tiles_per_block);
  bf16x8 tb[2][2][3];  // [step parity][parity][piece]
  auto load_tab = [&](bf16x8 (&b)[2][3], int tile, int step) {
#pragma unroll
    for (int q = 0; q < 6; ++q)
      b[q / 3][q % 3] = reinterpret_cast<const bf16x8 *>(
          a.table)[(((size_t(q / 3) * tiles + tile) * steps + step) * 3 + q % 3) * 64 + lane];
  };
  int tile = blockIdx.x * tiles_per_block + wave;
  if (tile < last) {
    load_tab(tb[0], tile, top);
    load_tab(tb[1], tile, top + 1);
  }
  for (; tile < last; tile += 8) {
    const int next = tile + 8 < last ? tile + 8 : tile;
    floatx16 s[2][4];  // [parity][re hi hi, re corrections, im hi hi, im corrections]
#pragma unroll
    for (int q = 0; q < 8; ++q) s[q >> 2][q & 3] = floatx16{0.f};
    auto multiply = [&](int step, const bf16x8 (&b)[2][3]) {
      const int g8 = (step & 3) * 2 + (lane >> 5);
      const uint4 *src = pieces + (step >> 2) * kBuf + fold_unit(g8, lane & 31);
#pragma unroll
      for (int par = 0; par < 2; ++par) {
        bf16x8 d[6];
#pragma unroll
        for (int q = 0; q < 6; ++q) d[q] = __builtin_bit_cast(bf16x8, src[(6 * par + q) * kPieceUnits]);
        fold_step<COLS>(d, b[par], s[par][0], s[par][1], s[par][2], s[par][3]);
      }
    };
    // from the outermost pairs inward: a focal field is largest about the axis, and what is added after
    // its peak is rounded at the peak's scale (256^2 -> 4096^2, largest error over the largest result of
    // a field falling off as 1 / r^2: outward 3.3e-7, inward 1.1e-7, the float32 matrix unit 1.8e-7).
    // The last steps load the next tile's first ones: they are on their way before the stores
    for (int step = used - 2; step >= 0; step -= 2) {
      const bool more = step > 0;
      multiply(step, tb[0]);
      load_tab(tb[0], more ? tile : next, more ? step - 2 : top);
      multiply(step + 1, tb[1]);
      load_tab(tb[1], more ? tile : next, more ? step - 1 : top + 1);
    }
    int fbase = f0;
    asm("" : "+s"(fbase));  // the rows' addresses are formed here, not kept across the products
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int trow = (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3), tcol = lane & 31;
      const int lf = COLS ? tcol : trow, ff = fbase + lf;
      const int k = tile * 32 + (COLS ? trow : tcol) + 1;
      if (ff >= a.F || k > out_half) continue;
      const float2 z = in0[lf];
      const double w = short_sign(ff) * back;
      const double cx = w * (double(s[0][0][r]) + double(s[0][1][r])) + double(z.x);
      const double cy = w * (double(s[0][2][r]) + double(s[0][3][r])) + double(z.y);
      const double sx = w * (double(s[1][0][r]) + double(s[1][1][r]));
      const double sy = w * (double(s[1][2][r]) + double(s[1][3][r]));
      if (k < a.P - out_half) emit(out_half + k, ff, cx - sg * sy, cy + sg * sx);
      emit(out_half - k, ff, cx + sg * sy, cy - sg * sx);
      if ((r & 3) == 3) __builtin_amdgcn_sched_barrier(0);  // four items' addresses and loads at a time
    }
  }
  if (blockIdx.x == 0 && tid < kFoldFree && f0 + tid < a.F) {
    double2 z = make_double2(in0[tid].x, in0[tid].y);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const double2 v = zs[q * kFoldFree + tid];
      z.x += v.x;
      z.y += v.y;
    }
    emit(out_half, f0 + tid, z.x, z.y);
  }
}

// Products of at most kFewPairs pairs (one matrix step) with a small output, where the kernels above are a
// chain of waits around one stage. Here the loads of the data and of the matrix go out together, then come
// vector multiply-adds in float64 on the folded pairs and the entries (the sum of their pieces, rounded to
// float32), and the stores. Along columns a lane holds a column's pairs and a wave walks `per_wave` (at most
// kFewOut) positive outputs, their entries in LDS; along rows a lane holds an output's entries and a wave a
// row, its pairs in LDS. (Both products of a transform in a recorded graph: 16^2 -> 512^2 14.4 us above, 6.3 us
// here, 10.1 us as complex products of 64 x 64 tiles; 33^2 -> 512^2 14.7, 7.7 and 17.4 us.)
constexpr int kFewPairs = 16;
constexpr int kFewOut = 8;
// four entries from their pieces' words
__device__ __forceinline__ float4 few_entries(uint2 hi, uint2 mid, uint2 lo) {
  auto sum = [](unsigned h, unsigned m, unsigned l) {
    return (__uint_as_float(h) + __uint_as_float(m)) + __uint_as_float(l);
  };
  constexpr unsigned kTop = 0xffff0000u;
  return make_float4(sum(hi.x << 16, mid.x << 16, lo.x << 16), sum(hi.x & kTop, mid.x & kTop, lo.x & kTop),
                     sum(hi.y << 16, mid.y << 16, lo.y << 16), sum(hi.y & kTop, mid.y & kTop, lo.y & kTop));
}
struct FewPair {
  double px, py, mx, my;  // folded pair
};
template <bool COLS, int PAIRS>
__global__ void __launch_bounds__(256) fold_few_kernel(FoldArgs a, int per_wave) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = a.Q / 2, full_pairs = a.Q - 1 - half, out_half = a.P / 2;
  const int tiles = fold_tiles(a.P), steps = fold_steps(a.Q);
  const double sg = a.sign;
  // words of four pieces of pairs 4 q + 1 .. 4 q + 4 of positive output k + 1
  auto entries = [&](int par, int k, int q) {
    const int kc = min(k, tiles * 32 - 1);
    const uint2 *t = static_cast<const uint2 *>(a.table) +
                     ((size_t(par * tiles + kc / 32) * steps * 3 * 64) + kc % 32 + 32 * (q >> 1)) * 2 + (q & 1);
    return few_entries(t[0], t[128], t[256]);
  };
  auto fold = [](float2 p, float2 m) {
    return FewPair{double(p.x) + double(m.x), double(p.y) + double(m.y), double(p.x) - double(m.x), double(p.y) - double(m.y)};
  };
  struct Sums {
    double cx, cy, sx, sy;
    __device__ __forceinline__ void add(const FewPair &v, float c, float s) {
      cx = fma(v.px, double(c), cx);
      cy = fma(v.py, double(c), cy);
      sx = fma(v.mx, double(s), sx);
      sy = fma(v.my, double(s), sy);
    }
  };
  auto emit = [&](int o, int f, double re, double im) { epilogue(a, COLS ? o : f, COLS ? f : o, re, im); };
  auto both = [&](int k, int f, const Sums &v) {
    if (k + 1 < a.P - out_half) emit(out_half + k + 1, f, v.cx - sg * v.sy, v.cy + sg * v.sx);
    emit(out_half - k - 1, f, v.cx + sg * v.sy, v.cy - sg * v.sx);
  };
  if constexpr (COLS) {
    __shared__ float4 w[4 * kFewOut][2][PAIRS / 4];
    const int f = blockIdx.y * 64 + lane, first = (blockIdx.x * 4 + wave) * per_wave;
    const float2 *c = a.data + size_t(half) * a.ldd + min(f, a.F - 1);
    const float2 in0 = *c;
    float2 p[PAIRS], m[PAIRS];
#pragma unroll
    for (int j = 1; j <= PAIRS; ++j) {
      p[j - 1] = c[ptrdiff_t(min(j, full_pairs)) * a.ldd];
      m[j - 1] = c[-ptrdiff_t(min(j, half)) * a.ldd];
    }
    constexpr int QUADS = PAIRS / 4;
    if (tid < 8 * QUADS * per_wave) {
      const int q = tid % QUADS, par = tid / QUADS % 2, i = tid / (2 * QUADS);
      w[i][par][q] = entries(par, blockIdx.x * 4 * per_wave + i, q);
    }
    FewPair v[PAIRS];
#pragma unroll
    for (int j = 1; j <= PAIRS; ++j)
      v[j - 1] = fold(j <= full_pairs ? p[j - 1] : make_float2(0.f, 0.f), j <= half ? m[j - 1] : make_float2(0.f, 0.f));
    __syncthreads();
    if (f >= a.F) return;
    for (int k = first; k < min(out_half, first + per_wave); ++k) {
      Sums s{in0.x, in0.y, 0.0, 0.0};
#pragma unroll
      for (int q = 0; q < PAIRS / 4; ++q) {
        const float4 cw = w[wave * per_wave + k - first][0][q], sw = w[wave * per_wave + k - first][1][q];
        s.add(v[4 * q], cw.x, sw.x);
        s.add(v[4 * q + 1], cw.y, sw.y);
        s.add(v[4 * q + 2], cw.z, sw.z);
        s.add(v[4 * q + 3], cw.w, sw.w);
      }
      both(k, f, s);
    }
    if (first == 0) {
      double zx = in0.x, zy = in0.y;
#pragma unroll
      for (int j = 0; j < PAIRS; ++j) {
        zx += v[j].px;
        zy += v[j].py;
      }
      emit(out_half, f, zx, zy);
    }
  } else {
    __shared__ FewPair v[4][PAIRS];
    const int f = blockIdx.y * 4 + wave, k = blockIdx.x * 64 + lane, j = (lane & (PAIRS - 1)) + 1;
    const float2 *c = a.data + size_t(min(f, a.F - 1)) * a.ldd + half;
    const float2 in0 = *c, p = c[min(j, full_pairs)], m = c[-min(j, half)];
    float4 cw[PAIRS / 4], sw[PAIRS / 4];
#pragma unroll
    for (int q = 0; q < PAIRS / 4; ++q) {
      cw[q] = entries(0, k, q);
      sw[q] = entries(1, k, q);
    }
    if (lane < PAIRS) v[wave][lane] = fold(j <= full_pairs ? p : make_float2(0.f, 0.f), j <= half ? m : make_float2(0.f, 0.f));
    __syncthreads();
    if (f >= a.F) return;
    Sums s{in0.x, in0.y, 0.0, 0.0};
    double zx = in0.x, zy = in0.y;
#pragma unroll
    for (int q = 0; q < PAIRS / 4; ++q) {
      s.add(v[wave][4 * q], cw[q].x, sw[q].x);
      s.add(v[wave][4 * q + 1], cw[q].y, sw[q].y);
      s.add(v[wave][4 * q + 2], cw[q].z, sw[q].z);
      s.add(v[wave][4 * q + 3], cw[q].w, sw[q].w);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        zx += v[wave][4 * q + i].px;
        zy += v[wave][4 * q + i].py;
      }
    }
    if (k < out_half) both(k, f, s);
    if (k == 0) emit(out_half, f, zx, zy);
  }
}

// output rows over blockIdx.y, columns over blockIdx.x and the threads (no index division),
// the partials added in slice order
__global__ void __launch_bounds__(256) split_reduce(FoldParams gp, int rows, int cols) {
  const FoldArgs &a = gp.a;
  const size_t total = size_t(rows) * cols;
  for (int i = blockIdx.y; i < rows; i += gridDim.y) {
    for (int j = blockIdx.x * 256 + threadIdx.x; j < cols; j += gridDim.x * 256) {
      const size_t e = size_t(i) * cols + j;
      double sr = 0.0, si = 0.0;
      // four slices' loads at a time: one by one they are a chain of waits where the output is small
      // (sixteen slices of 256 x 256: 8.6 us, 6.6 us)
      int s = 0;
      for (; s + 4 <= gp.split; s += 4) {
        double2 v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = gp.partial[size_t(s + q) * total + e];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          sr += v[q].x;
          si += v[q].y;
        }
      }
      for (; s < gp.split; ++s) {
        const double2 v = gp.partial[size_t(s) * total + e];
        sr += v.x;
        si += v.y;
      }
      epilogue(a, i, j, sr, si);
    }
  }
}

int div_up(int x, int y) { return (x + y - 1) / y; }

template <bool COLS>
hipError_t launch_fold_kernel(const FoldParams &gp, hipStream_t stream) {
  const FoldArgs &a = gp.a;
  const dim3 grid(div_up(fold_tiles(a.P), 2), div_up(a.F, kFoldFree), gp.split);
  hipLaunchKernelGGL((fold_kernel<COLS>), grid, dim3(kFoldThreads), 0, stream, gp);
  return hipGetLastError();
}

template <bool COLS>
hipError_t launch_short_kernel(const FoldArgs &a, hipStream_t stream) {
  const int tiles = fold_tiles(a.P), ftiles = div_up(a.F, kFoldFree), per = fold_short_tiles(tiles, ftiles);
  hipLaunchKernelGGL((fold_short_kernel<COLS>), dim3(div_up(tiles, per), ftiles), dim3(kFoldThreads), 0, stream, a, per);
  return hipGetLastError();
}

template <bool COLS>
hipError_t launch_few_kernel(const FoldArgs &a, hipStream_t stream) {
  // along columns as many outputs per wave as leave every compute unit a block (33^2 -> 1400^2 with 8, 4 and 2
  // outputs 14.7, 17.0 and 21.5 us; 33^2 -> 512^2 with 2, a block per compute unit, and 4 7.8 and 8.6 us)
  int per = kFewOut;
  while (per > 1 && div_up(a.P / 2, 4 * per) * div_up(a.F, 64) < 256) per /= 2;
  const dim3 grid(std::max(div_up(a.P / 2, COLS ? 4 * per : 64), 1), div_up(a.F, COLS ? 64 : 4));
  if (a.Q / 2 <= kFewPairs / 2) hipLaunchKernelGGL((fold_few_kernel<COLS, kFewPairs / 2>), grid, dim3(256), 0, stream, a, per);
  else hipLaunchKernelGGL((fold_few_kernel<COLS, kFewPairs>), grid, dim3(256), 0, stream, a, per);
  return hipGetLastError();
}

}  // namespace

// Which kernel runs a product. Short sums go to the kernel of their own where the output is large enough
// that every wave walks tiles: below that the general kernel's two halves of every stage on different waves
// are faster (256^2 -> 1024^2 with mask and background 16 us general, 37 us short; 256^2 -> 2048^2 43 and
// 25 us). One matrix step over a smaller output goes to the vector units (over a larger one the matrix
// unit's work hides behind the stores).
int fold_kind(int F, int P, int Q) {
  const int half = Q / 2;
  if (half <= kShortPairs && (long long)fold_tiles(P) * div_up(F, kFoldFree) >= 1024) return kFoldShort;
  return half <= kFewPairs ? kFoldFew : kFoldGeneral;
}

// slices of the pairs: the power of two with the least time by what the kernels measured over
// edges of 256 to 4096 and 64 to 512 (one block per compute unit at a time): 1.6 us a stage of a
// round of blocks, and for a split 4 us for the pass that adds the slices and the slices' bytes
// written and read at 3 TB/s. A slice for every idle compute unit, at least 128 pairs deep, was
// too many for the middle sizes (us at 1, 2, 4 slices, input length 1024: 1024 x 512 outputs 22,
// 26, 33; 1024 x 256 21, 25, 25; length 512: 512 x 1024 17, 26, 29); over the 96 products of
// those edges that the general kernel runs this choice is at most 2 % behind that one and 5 % ahead of it
// in sum (2469 us against 2589 us, the best choice of each 2458 us).
int fold_split_for(const FoldArgs &a) {
  if (fold_kind(a.F, a.P, a.Q) != kFoldGeneral) return 1;
  const double blocks = double(div_up(fold_tiles(a.P), 2)) * div_up(a.F, kFoldFree);
  const int stages = div_up(a.Q / 2, kFoldStage);
  int best = 1;
  double least = 0.0;
  for (int s = 1; s <= kMaxSplit && (s == 1 || s <= stages); s *= 2) {
    double us = 1.6 * div_up(stages, s) * std::ceil(blocks * s / 256.0);
    if (s > 1) us += 4.0 + double(s) * a.F * a.P * 16.0 / 3.0e6;
    if (s == 1 || us < least) {
      least = us;
      best = s;
    }
  }
  return best;
}

hipError_t launch_fold(const FoldArgs &a, int split, void *partial, hipStream_t stream, const LaunchHook &hook) {
  const int kind = fold_kind(a.F, a.P, a.Q);
  if (kind != kFoldGeneral) split = 1;  // one group of pairs: nothing to slice
  FoldParams gp;
  gp.a = a;
  gp.split = split;
  gp.j_per_split = std::max(div_up(div_up(a.Q / 2, split), kFoldStage), 1) * kFoldStage;
  gp.partial = static_cast<double2 *>(partial);
  const int rows = a.cols ? a.P : a.F, cols = a.cols ? a.F : a.P;
  char name[64];
  std::snprintf(name, sizeof name, "fold%s_%dx%dx%d_s%d", a.cols ? "C" : "R", a.F, a.P, a.Q, split);
  hook(stream, name, a.Q, 0);
  hipError_t e = kind == kFoldShort ? (a.cols ? launch_short_kernel<true>(a, stream) : launch_short_kernel<false>(a, stream))
                 : kind == kFoldFew ? (a.cols ? launch_few_kernel<true>(a, stream) : launch_few_kernel<false>(a, stream))
                                    : (a.cols ? launch_fold_kernel<true>(gp, stream) : launch_fold_kernel<false>(gp, stream));
  hook(stream, name, a.Q, 1);
  if (e != hipSuccess || split == 1) return e;
  hook(stream, "split_reduce", a.Q, 0);
  hipLaunchKernelGGL(split_reduce, dim3(std::min((cols + 255) / 256, 16), std::min(rows, 65535)), dim3(256), 0, stream,
                     gp, rows, cols);
  e = hipGetLastError();
  hook(stream, "split_reduce", a.Q, 1);
  return e;
}

}  // namespace fr
