// The matrix Fourier transform in float64 (Sec. 1.1, after Soummer et al.; Sec. 2.3 for the
// precision the paper benchmarks): out = (du / n_d) W in W^T and its adjoint
// (du / n_d) W^H in conj(W), each as two products along one axis, folded about it and formed in
// float64 on the matrix cores (on gfx950 their dense float64 peak, 78.6 TFLOP/s, equals the vector
// units').
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "../../include/fresnel.h"
#include "fr_runtime.h"

namespace fr {
namespace {

struct z64 {
  double x, y;
};

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

constexpr int kFree = 32;      // free indices (rows or columns of the data) per block
constexpr int kStage = 32;     // pairs per stage
constexpr int kThreads = 256;  // four waves

struct ZFold {
  int F, P, Q;       // free indices, output length, input length
  double sign;       // -1 (W) or +1 (conj(W))
  const z64 *data;   // row stride ldd
  int ldd;
  const d2 *table;   // ztable_bytes
  z64 *out;          // split == 1: the output (rows of ldc); else partials of ldc x rows each
  int ldc;
  double scale;
  int j_per_split;   // pairs per slice, a multiple of kStage
  size_t split_stride;
};

// cosines (parity 0) and sines (parity 1) of 2 pi k j du / n_d, k = 1 .. P/2, j = 1 .. Q/2, as
// MFMA fragments [parity][tile of 32 k][step of 8 j][16 k][lane][2]: lane l holds k = l % 16 and
// j = l / 16 and l / 16 + 4 of the step; zero past P/2 and Q/2, the steps padded to whole stages
__host__ __device__ inline int ztiles(int P) { return P / 2 > 0 ? (P / 2 + 31) / 32 : 1; }
__host__ __device__ inline int zsteps(int Q) { return Q / 2 > 0 ? (Q / 2 + kStage - 1) / kStage * 4 : 4; }

// One product with the Fourier matrix along one axis, folded about it: with P(j) = in(j) + in(-j)
// and M(j) = in(j) - in(-j), out(+-k) = in(0) + sum_j P(j) cos(2 pi k j du / n_d)
// +- i sign sum_j M(j) sin(2 pi k j du / n_d), j = 1 .. Q/2, k = 1 .. P/2, a quarter of the complex
// product's operations, and out(0) = in(0) + sum_j P(j).
//
// Bound by the float64 matrix cores (a 16 x 16 x 4 product holds its SIMD's unit for 64 cycles;
// the folds, the LDS and the loads need far less). A block of four waves forms 32 free indices by
// KT * 32 positive outputs (both signs): each wave one parity, a 32 x 32 tile and, for KT = 1, one
// half of every stage's pairs (added in the epilogue); 68 KiB of LDS and under 256 registers, so
// two blocks share a compute unit and one's loads, folds and stores overlap the other's products.
// Stages are double-buffered in LDS: the next stage's data and matrix fragments are on their way
// while the current one is multiplied. COLS: the transform runs along the columns (the free index
// is the column), so the tile is transposed by swapping the MFMA operands. Fragment layouts
// (checked on gfx950 with one-hot operands): lane l holds A[l % 16][l / 16] and B[l / 16][l % 16]
// of the 16 x 4 and 4 x 16 operands, and item r of the result D[4 r + l / 16][l % 16].
// Measured (MI355X, 4096^2 -> 256^2 and back): 1198 us as complex products of 64 x 64 tiles, 409 us
// folded (the long products 223 us and 204 us, 38 and 42 TFLOP/s on the folded operations).
template <int KT, bool COLS>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) zfold_kernel(ZFold a) {
  constexpr int KS = 2 / KT;
  constexpr int STEPS = 4 / KS;  // 8-deep steps per wave and stage
  constexpr int kVal = kFree * kStage;
  // [buffer][P.re, P.im, M.re, M.im][pair][free index, xored with the pair's low four bits so that
  // stores along the pairs spread over the banks]; later the waves' sums, [wave][item][lane]
  __shared__ double lds[2 * 4 * kVal];
  __shared__ z64 zs[8 * kFree];
  static_assert(sizeof(lds) >= 4 * 16 * 64 * sizeof(z64), "the exchange fits the stage buffers");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int par = wave & 1, kt = KT == 2 ? wave >> 1 : 0, ks = KT == 2 ? 0 : wave >> 1;
  // an XCD's blocks walk a contiguous range of tiles, eight tiles of free indices at a time and all
  // their output tiles, so that they share the data in its L2
  const int gx = gridDim.x, gy = gridDim.y, total = gx * gy * gridDim.z;
  const int lin = blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z);
  const int tile = total % 8 == 0 ? (lin & 7) * (total >> 3) + (lin >> 3) : lin;
  const int bz = tile / (gx * gy), in_z = tile % (gx * gy);
  const int grp = in_z / (8 * gx), rows_g = min(8, gy - grp * 8), u = in_z % (8 * gx);
  const int bx = u / rows_g, f0 = (grp * 8 + u % rows_g) * kFree;

  const int half = a.Q / 2, full_pairs = a.Q - 1 - half;
  const int jbeg = bz * a.j_per_split, jend = min(half, jbeg + a.j_per_split);
  const int nst = jend > jbeg ? (jend - jbeg + kStage - 1) / kStage : 0;
  const bool zero_tile = bx == 0;

  // four (free index, pair) items per thread and stage, 8 apart in the index the lanes do not walk
  const ptrdiff_t step = COLS ? a.ldd : 1, fstep = COLS ? 1 : a.ldd;
  const int walk = tid & 31, other = tid >> 5;
  z64 p[4], m[4], zero[COLS ? 1 : 4];
#pragma unroll
  for (int i = 0; i < (COLS ? 1 : 4); ++i) zero[i] = {0.0, 0.0};
  auto load = [&](int j0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int lf = COLS ? walk : other + 8 * i, j = j0 + (COLS ? other + 8 * i : walk) + 1;
      const z64 *c = a.data + half * step + min(f0 + lf, a.F - 1) * fstep;
      p[i] = j <= full_pairs ? c[j * step] : z64{0.0, 0.0};
      m[i] = j <= half ? c[-j * step] : z64{0.0, 0.0};
    }
  };
  auto put = [&](int buf, bool count) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int lf = COLS ? walk : other + 8 * i, j = COLS ? other + 8 * i : walk;
      double *d = lds + buf * 4 * kVal + j * kFree + (lf ^ (j & 15));
      const double sx = p[i].x + m[i].x, sy = p[i].y + m[i].y;
      d[0] = sx;
      d[kVal] = sy;
      d[2 * kVal] = p[i].x - m[i].x;
      d[3 * kVal] = p[i].y - m[i].y;
      if (count && zero_tile) {
        zero[COLS ? 0 : i].x += sx;
        zero[COLS ? 0 : i].y += sy;
      }
    }
  };
  const int tiles = ztiles(a.P), steps = zsteps(a.Q), out_half = a.P / 2;
  const int ktile = bx * KT + kt;
  const d2 *tab = a.table + (size_t(par) * tiles + min(ktile, tiles - 1)) * steps * 128 + lane;
  d2 tc[STEPS][2], tn[STEPS][2];
  auto load_tab = [&](d2 (&t)[STEPS][2], int s) {
    const int st = jbeg / 8 + s * 4 + ks * STEPS;
#pragma unroll
    for (int q = 0; q < STEPS; ++q)
#pragma unroll
      for (int h = 0; h < 2; ++h) t[q][h] = tab[(size_t(st + q) * 2 + h) * 64];
  };
  d4 re[2][2], im[2][2];  // [16 free indices][16 outputs]
#pragma unroll
  for (int i = 0; i < 4; ++i) re[i >> 1][i & 1] = im[i >> 1][i & 1] = d4{0.0, 0.0, 0.0, 0.0};
  auto mm = [](double d, double t, d4 c) {
    if constexpr (COLS) return __builtin_amdgcn_mfma_f64_16x16x4f64(t, d, c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f64_16x16x4f64(d, t, c, 0, 0, 0);
  };
  const int fl = lane & 15, fk = lane >> 4;
  if (nst > 0) {
    load_tab(tc, 0);
    load(jbeg);
    put(0, true);
    __syncthreads();
    for (int s = 0; s < nst; ++s) {
      // the last stage loads and stores itself again, to a buffer nobody reads
      const int next = min(s + 1, nst - 1);
      load_tab(tn, next);
      load(jbeg + next * kStage);
      const double *src = lds + (s & 1) * 4 * kVal + 2 * par * kVal;
#pragma unroll
      for (int q = 0; q < STEPS; ++q)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int j = ((ks * STEPS + q) * 2 + e) * 4 + fk;
          double dr[2], di[2];
#pragma unroll
          for (int ft = 0; ft < 2; ++ft) {
            const double *d = src + j * kFree + ft * 16 + (fl ^ (j & 15));
            dr[ft] = d[0];
            di[ft] = d[kVal];
          }
#pragma unroll
          for (int ft = 0; ft < 2; ++ft)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              re[ft][h] = mm(dr[ft], tc[q][h][e], re[ft][h]);
              im[ft][h] = mm(di[ft], tc[q][h][e], im[ft][h]);
            }
        }
      put((s & 1) ^ 1, s + 1 < nst);
#pragma unroll
      for (int q = 0; q < STEPS; ++q)
#pragma unroll
        for (int h = 0; h < 2; ++h) tc[q][h] = tn[q][h];
      __syncthreads();
    }
  }

  // exchange: every wave's sums, then each wave of a tile (2 parities x KS halves) forms both signs
  // of its share of the tile's outputs. Item t = (16 free indices, 16 outputs, r).
  z64 *ex = reinterpret_cast<z64 *>(lds);
  __syncthreads();
#pragma unroll
  for (int t = 0; t < 16; ++t)
    ex[(wave * 16 + t) * 64 + lane] = {re[t >> 3][(t >> 2) & 1][t & 3], im[t >> 3][(t >> 2) & 1][t & 3]};
  if (zero_tile) {
    if constexpr (COLS) {
      zs[other * kFree + walk] = zero[0];
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        for (int o = 16; o > 0; o >>= 1) {
          zero[i].x += __shfl_xor(zero[i].x, o);
          zero[i].y += __shfl_xor(zero[i].y, o);
        }
        if (walk == 0) zs[other + 8 * i] = zero[i];
      }
    }
  }
  __syncthreads();
  z64 *out = a.out + bz * a.split_stride;
  auto emit = [&](int o, int f, double x, double y) {
    out[COLS ? size_t(o) * a.ldc + f : size_t(f) * a.ldc + o] = {a.scale * x, a.scale * y};
  };
  auto in0 = [&](int f) { return bz == 0 ? a.data[half * step + f * fstep] : z64{0.0, 0.0}; };
  constexpr int SHARE = 16 / (2 * KS);
#pragma unroll
  for (int tt = 0; tt < SHARE; ++tt) {
    const int t = (par * KS + ks) * SHARE + tt;
    z64 c = {0.0, 0.0}, sn = {0.0, 0.0};
#pragma unroll
    for (int h = 0; h < KS; ++h) {
      const int w = KT == 2 ? 2 * kt : 2 * h;
      const z64 cv = ex[(w * 16 + t) * 64 + lane], sv = ex[((w + 1) * 16 + t) * 64 + lane];
      c.x += cv.x;
      c.y += cv.y;
      sn.x += sv.x;
      sn.y += sv.y;
    }
    const int row = 4 * (t & 3) + fk, col = fl;
    const int f = f0 + (t >> 3) * 16 + (COLS ? col : row);
    const int k = ktile * 32 + ((t >> 2) & 1) * 16 + (COLS ? row : col) + 1;
    if (f >= a.F || k > out_half) continue;
    const z64 z = in0(f);
    c.x += z.x;
    c.y += z.y;
    if (k < a.P - out_half) emit(out_half + k, f, c.x - a.sign * sn.y, c.y + a.sign * sn.x);
    emit(out_half - k, f, c.x + a.sign * sn.y, c.y - a.sign * sn.x);
  }
  if (zero_tile && tid < kFree && f0 + tid < a.F) {
    z64 z = in0(f0 + tid);
#pragma unroll
    for (int q = 0; q < (COLS ? 8 : 1); ++q) {
      z.x += zs[q * kFree + tid].x;
      z.y += zs[q * kFree + tid].y;
    }
    emit(out_half, f0 + tid, z.x, z.y);
  }
}

// Products of at most kFewPairs pairs, where a stage of the kernel above is mostly padding (three of its four
// steps) and its exchange comes with every 64 outputs. A large output along columns is bound by its bytes,
// the others by the chain of loads, sums and stores. Along columns a lane holds a column's folded pairs and
// a wave forms `per_wave` (at most kFewOut) outputs of either sign by vector multiply-adds, their matrix
// entries in LDS; along rows a lane holds an output's entries and a wave a row, its pairs in LDS. (Both
// products of a transform in a recorded graph: 16^2 -> 4096^2 80 us above, 48 us here, 57 us as complex
// products of 64 x 64 tiles; 16^2 -> 200^2 12.1, 5.5 and 9.7 us.)
constexpr int kFewPairs = 8;
constexpr int kFewOut = 16;
struct ZPair {
  z64 sum, diff;
};
template <bool COLS>
__global__ void __launch_bounds__(256) zfew_kernel(ZFold a, int per_wave) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = a.Q / 2, full_pairs = a.Q - 1 - half, out_half = a.P / 2;
  const int steps = zsteps(a.Q), kmax = ztiles(a.P) * 32 - 1;
  const size_t par = size_t(ztiles(a.P)) * steps * 128;
  // entries of pairs i + 1 and i + 5 of positive output k + 1
  auto entry = [&](int sine, int k, int i) {
    const int kc = min(k, kmax);
    return a.table[sine * par + (size_t(kc / 32) * steps * 2 + kc % 32 / 16) * 64 + kc % 16 + 16 * i];
  };
  auto fold = [](z64 p, z64 m) { return ZPair{{p.x + m.x, p.y + m.y}, {p.x - m.x, p.y - m.y}}; };
  struct Sums {
    z64 c, s;
    __device__ __forceinline__ void add(const ZPair &v, double wc, double ws) {
      c.x = fma(v.sum.x, wc, c.x);
      c.y = fma(v.sum.y, wc, c.y);
      s.x = fma(v.diff.x, ws, s.x);
      s.y = fma(v.diff.y, ws, s.y);
    }
  };
  auto emit = [&](int o, int f, double x, double y) {
    a.out[COLS ? size_t(o) * a.ldc + f : size_t(f) * a.ldc + o] = {a.scale * x, a.scale * y};
  };
  auto both = [&](int k, int f, const Sums &v) {
    if (k + 1 < a.P - out_half) emit(out_half + k + 1, f, v.c.x - a.sign * v.s.y, v.c.y + a.sign * v.s.x);
    emit(out_half - k - 1, f, v.c.x + a.sign * v.s.y, v.c.y - a.sign * v.s.x);
  };
  constexpr z64 none = {0.0, 0.0};
  if constexpr (COLS) {
    __shared__ d2 w[4 * kFewOut][2][kFewPairs / 2];
    const int f = blockIdx.y * 64 + lane, first = (blockIdx.x * 4 + wave) * per_wave;
    const z64 *c = a.data + size_t(half) * a.ldd + min(f, a.F - 1);
    z64 p[kFewPairs], m[kFewPairs];
    const z64 in0 = *c;
#pragma unroll
    for (int j = 1; j <= kFewPairs; ++j) {
      p[j - 1] = c[ptrdiff_t(min(j, full_pairs)) * a.ldd];
      m[j - 1] = c[-ptrdiff_t(min(j, half)) * a.ldd];
    }
    for (int i = tid; i < 32 * per_wave; i += 256)
      w[i >> 3][(i >> 2) & 1][i & 3] = entry((i >> 2) & 1, blockIdx.x * 4 * per_wave + (i >> 3), i & 3);
    ZPair v[kFewPairs];
#pragma unroll
    for (int j = 1; j <= kFewPairs; ++j) v[j - 1] = fold(j <= full_pairs ? p[j - 1] : none, j <= half ? m[j - 1] : none);
    __syncthreads();
    if (f >= a.F) return;
    for (int k = first; k < min(out_half, first + per_wave); ++k) {
      Sums s{in0, none};
#pragma unroll
      for (int i = 0; i < kFewPairs / 2; ++i) {
        const d2 wc = w[wave * per_wave + k - first][0][i], ws = w[wave * per_wave + k - first][1][i];
        s.add(v[i], wc[0], ws[0]);
        s.add(v[i + 4], wc[1], ws[1]);
      }
      both(k, f, s);
    }
    if (first == 0) {
      z64 z = in0;
#pragma unroll
      for (int j = 0; j < kFewPairs; ++j) z = {z.x + v[j].sum.x, z.y + v[j].sum.y};
      emit(out_half, f, z.x, z.y);
    }
  } else {
    __shared__ ZPair v[4][kFewPairs];
    const int f = blockIdx.y * 4 + wave, k = blockIdx.x * 64 + lane, j = (lane & (kFewPairs - 1)) + 1;
    const z64 *c = a.data + size_t(min(f, a.F - 1)) * a.ldd + half;
    const z64 in0 = *c, p = c[min(j, full_pairs)], m = c[-min(j, half)];
    d2 wc[kFewPairs / 2], ws[kFewPairs / 2];
#pragma unroll
    for (int i = 0; i < kFewPairs / 2; ++i) {
      wc[i] = entry(0, k, i);
      ws[i] = entry(1, k, i);
    }
    if (lane < kFewPairs) v[wave][lane] = fold(j <= full_pairs ? p : none, j <= half ? m : none);
    __syncthreads();
    if (f >= a.F) return;
    Sums s{in0, none};
    z64 z = in0;
#pragma unroll
    for (int i = 0; i < kFewPairs / 2; ++i) {
      s.add(v[wave][i], wc[i][0], ws[i][0]);
      s.add(v[wave][i + 4], wc[i][1], ws[i][1]);
    }
#pragma unroll
    for (int i = 0; i < kFewPairs; ++i) z = {z.x + v[wave][i].sum.x, z.y + v[wave][i].sum.y};
    if (k < out_half) both(k, f, s);
    if (k == 0) emit(out_half, f, z.x, z.y);
  }
}

// most partials zsum_kernel adds
constexpr int kMaxZsum = 32;

// most slices that the workspace holds for the forward transform's two products: 4 and 32 where
// their outputs are small and the pupil is large
int f64_split(int n, int m) {
  const long tiles = long((n + 63) / 64) * long((m + 63) / 64);
  return tiles < 1024 && n >= 1024 ? 4 : 1;
}
int f64_split2(int n, int m) {
  const long tiles = long((m + 63) / 64) * long((m + 63) / 64);
  return tiles < 1024 && n >= 1024 ? kMaxZsum : 1;
}

// out[i] = s sum_p part[p stride + i], the partials added in order (np <= kMaxZsum; every
// partial's load is issued before the first addition)
__global__ void __launch_bounds__(256) zsum_kernel(const z64 *__restrict__ part, size_t stride, int np,
                                                   z64 *__restrict__ out, size_t count, double s) {
  const size_t i = size_t(blockIdx.x) * 256 + threadIdx.x;
  if (i >= count) return;
  z64 v[kMaxZsum];
#pragma unroll
  for (int p = 0; p < kMaxZsum; ++p)
    if (p < np) v[p] = part[p * stride + i];
  z64 acc = v[0];
#pragma unroll
  for (int p = 1; p < kMaxZsum; ++p)
    if (p < np) {
      acc.x += v[p].x;
      acc.y += v[p].y;
    }
  out[i] = {s * acc.x, s * acc.y};
}

// part[i] = sum_p part[p stride + i], the partials added in order (in place into the first)
__global__ void __launch_bounds__(256) zsum_inplace_kernel(z64 *part, size_t stride, int np, size_t count) {
  const size_t i = size_t(blockIdx.x) * 256 + threadIdx.x;
  if (i >= count) return;
  z64 acc = part[i];
  for (int p = 1; p < np; ++p) {
    const z64 v = part[p * stride + i];
    acc.x += v.x;
    acc.y += v.y;
  }
  part[i] = acc;
}

int div_up(int x, int y) { return (x + y - 1) / y; }
// one output tile per block unless two still give every compute unit two blocks
int zblocks(const ZFold &a, int kt) { return div_up(ztiles(a.P), kt) * div_up(a.F, kFree); }

// slices of the pairs, at most `most`, so that every compute unit gets two blocks, each slice at
// least 128 pairs deep
int zsplit(const ZFold &a, int most) {
  int s = 1;
  while (zblocks(a, 1) * s < 512 && 2 * s <= most && a.Q / 2 / (2 * s) >= 128) s *= 2;
  return s;
}

template <bool COLS>
hipError_t zfold(ZFold a, hipStream_t st, const LaunchHook &hook, const char *name, int split = 1) {
  hook(st, name, 1, 0);
  a.j_per_split = std::max(div_up(div_up(a.Q / 2, split), kStage), 1) * kStage;
  const int ftiles = div_up(a.F, kFree);
  if (a.Q / 2 <= kFewPairs) {
    // along columns as many outputs per wave as leave every compute unit two blocks
    int per = kFewOut;
    while (per > 1 && div_up(a.P / 2, 4 * per) * div_up(a.F, 64) < 512) per /= 2;
    const dim3 grid(std::max(div_up(a.P / 2, COLS ? 4 * per : 64), 1), div_up(a.F, COLS ? 64 : 4));
    hipLaunchKernelGGL((zfew_kernel<COLS>), grid, dim3(256), 0, st, a, per);
  } else if (zblocks(a, 2) * split >= 512)
    hipLaunchKernelGGL((zfold_kernel<2, COLS>), dim3(div_up(ztiles(a.P), 2), ftiles, split), dim3(kThreads), 0, st, a);
  else
    hipLaunchKernelGGL((zfold_kernel<1, COLS>), dim3(ztiles(a.P), ftiles, split), dim3(kThreads), 0, st, a);
  hipError_t e = hipGetLastError();
  hook(st, name, 1, 1);
  return e;
}

uint64_t dbits(double v) {
  uint64_t u;
  std::memcpy(&u, &v, sizeof u);
  return u;
}

// the table of ztiles / zsteps for an output of length p and an input of length q; the index
// product is an exact integer, its turns reduced to [-1/2, 1/2] before the cosine and sine. A
// transform and its adjoint read the same entries in two orders: both are built with the first of
// them, so that the other can be recorded into a graph, where no table can be built.
int mft64_table(Ctx *ctx, int p, int q, double n_d, double du, hipStream_t s, const d2 **out) {
  const TableKey key{kMft64, p, uint64_t(q), dbits(n_d), dbits(du), 0}, other{kMft64, q, uint64_t(p), dbits(n_d), dbits(du), 0};
  if (auto it = ctx->tables.find(key); it != ctx->tables.end()) {
    *out = static_cast<const d2 *>(it->second);
    return FR_OK;
  }
  auto entries = [](int tiles, int steps) { return size_t(tiles) * steps * 256; };  // of one parity
  auto at = [](int steps, int k, int j) {
    const int lane = k % 16 + 16 * (j % 4);
    return (((size_t(k / 32) * steps + j / 8) * 2 + k % 32 / 16) * 64 + lane) * 2 + j % 8 / 4;
  };
  const int steps = zsteps(q), steps2 = zsteps(p);
  const size_t par = entries(ztiles(p), steps), par2 = entries(ztiles(q), steps2);
  const bool both = p != q && ctx->tables.find(other) == ctx->tables.end();
  std::vector<double> w(2 * par, 0.0), w2(both ? 2 * par2 : 0, 0.0);
  const double r = du / n_d;
  for (int k = 0; k < p / 2; ++k)
    for (int j = 0; j < q / 2; ++j) {
      double t = double(int64_t(k + 1) * int64_t(j + 1)) * r;
      t -= std::rint(t);
      const double c = std::cos(2.0 * M_PI * t), sn = std::sin(2.0 * M_PI * t);
      const size_t i = at(steps, k, j);
      w[i] = c;
      w[par + i] = sn;
      if (both) {
        const size_t i2 = at(steps2, j, k);
        w2[i2] = c;
        w2[par2 + i2] = sn;
      }
    }
  void *d = nullptr;
  int st = ctx->upload(key, w.data(), w.size() * sizeof(double), s, &d);
  *out = static_cast<const d2 *>(d);
  if (st == FR_OK && both) {
    st = ctx->upload(other, w2.data(), w2.size() * sizeof(double), s, &d);
    if (st == FR_ENOMEM) st = FR_OK;  // (this call does not need it)
  }
  return st;
}

}  // namespace
}  // namespace fr

extern "C" size_t mft_f64_workspace_bytes(int32_t n_pupil, int32_t m_focal) {
  if (n_pupil <= 0 || m_focal <= 0) return 0;
  const int s2 = fr::f64_split2(n_pupil, m_focal);
  return sizeof(fr_c128) * (size_t(n_pupil) * size_t(m_focal) * size_t(fr::f64_split(n_pupil, m_focal)) +
                            (s2 > 1 ? size_t(m_focal) * size_t(m_focal) * size_t(s2) : 0));
}

extern "C" int mft_f64(fr_ctx *ctx_, const fr_c128 *in, fr_c128 *out, int32_t n_pupil, int32_t m_focal,
                       double n_d, double du, int32_t flags, fr_c128 *ws, size_t ws_bytes, void *stream) {
  if (!in || !out || !ws || n_pupil <= 0 || m_focal <= 0 || (flags & ~FR_ADJOINT)) return FR_EINVAL;
  if (!(n_d > 0) || !std::isfinite(n_d) || !(du > 0) || !std::isfinite(du)) return FR_EINVAL;
  if (ws_bytes < mft_f64_workspace_bytes(n_pupil, m_focal)) return FR_EWORKSPACE;
  fr::Ctx *ctx = reinterpret_cast<fr::Ctx *>(ctx_);
  if (!ctx) return FR_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipError_t e = hipSetDevice(ctx->device);
  if (e != hipSuccess) return fr::record_hip(e);
  if (int st = ctx->begin_call(); st != FR_OK) return st;
  const int n = n_pupil, m = m_focal;
  const bool adj = flags & FR_ADJOINT;
  // forward: T = in W^T (n x m), out = scale W T (m x m); adjoint: T = in conj(W) (m x n),
  // out = scale W^H T (n x n); both read one table, of the output's and the input's length
  const int p = adj ? n : m, q = adj ? m : n;
  const fr::d2 *w;
  int st = fr::mft64_table(ctx, p, q, n_d, du, s, &w);
  if (st != FR_OK) return st;
  const fr::LaunchHook hook = ctx->hook();
  auto *t = reinterpret_cast<fr::z64 *>(ws);
  fr::ZFold g;
  std::memset(&g, 0, sizeof g);
  g.F = q; g.P = p; g.Q = q;
  g.sign = adj ? 1.0 : -1.0;
  g.data = reinterpret_cast<const fr::z64 *>(in); g.ldd = q;
  g.table = w;
  g.out = t; g.ldc = p;
  g.scale = 1.0;
  // the forward's products may be split over the pairs: the first into partials that are added in
  // place into T, the second into partials after them (the adjoint's sums are short)
  const size_t part = size_t(m) * size_t(n), part2 = size_t(m) * size_t(m);
  const int most = adj ? 1 : fr::f64_split(n, m), most2 = adj ? 1 : fr::f64_split2(n, m);
  const int split = fr::zsplit(g, most);
  g.split_stride = part;
  e = fr::zfold<false>(g, s, hook, adj ? "zfold_mft64_adj_1" : "zfold_mft64_1", split);
  if (e == hipSuccess && split > 1) {
    hook(s, "zsum_mft64_t", 1, 0);
    hipLaunchKernelGGL(fr::zsum_inplace_kernel, dim3(unsigned((part + 255) / 256)), dim3(256), 0, s, t, part, split,
                       part);
    e = hipGetLastError();
    hook(s, "zsum_mft64_t", 1, 1);
  }
  if (e == hipSuccess) {
    g.F = p;
    g.data = t; g.ldd = p;
    g.out = reinterpret_cast<fr::z64 *>(out);
    g.scale = du / n_d;
    const int split2 = fr::zsplit(g, most2);
    if (split2 > 1) {
      g.out = t + part * most;
      g.scale = 1.0;
      g.split_stride = part2;
    }
    e = fr::zfold<true>(g, s, hook, adj ? "zfold_mft64_adj_2" : "zfold_mft64_2", split2);
    if (e == hipSuccess && split2 > 1) {
      hook(s, "zsum_mft64", 1, 0);
      hipLaunchKernelGGL(fr::zsum_kernel, dim3(unsigned((part2 + 255) / 256)), dim3(256), 0, s, g.out, part2, split2,
                         reinterpret_cast<fr::z64 *>(out), part2, du / n_d);
      e = hipGetLastError();
      hook(s, "zsum_mft64", 1, 1);
    }
  }
  if (e != hipSuccess) return fr::record_hip(e);
  return FR_OK;
}
