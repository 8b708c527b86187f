// Internal interfaces between the host runtime (api.cpp) and the kernel launchers.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace fr {

struct c32;

// Optional per-launch callback (kernel timing): phase 0 just before a kernel launch on `s`,
// phase 1 just after it. `tag` distinguishes launches of one kernel (e.g. the plane edge).
struct LaunchHook {
  void (*fn)(void *user, hipStream_t s, const char *name, int tag, int phase) = nullptr;
  void *user = nullptr;
  void operator()(hipStream_t s, const char *name, int tag, int phase) const {
    if (fn) fn(user, s, name, tag, phase);
  }
};

// One plane of a Fresnel batch, as the sweep kernels see it (device pointers).
// Forward:  field <- post(x,y) * AS_z( src * pre(x,y) ),   src = field or 1 (kSourceOptic)
// Adjoint:  field <- conj(pre) * AS_{-z}( conj(post) * field )
//   pre  = amp * exp(2 pi i (opd + 2 pre_surf) / lambda) * lens[x] lens[y]
//   post = exp(2 pi i 2 post_surf / lambda)               (reflective DM after the step)
// amp and opd are win x win maps centred in the plane (offset (n - win)/2); outside the
// window amp is 0 when given. pre_surf is an n x n surface map [m], row-major; post_surf is the
// same kind of map stored in 4-column tiles (post_tiled_index) so that the column sweep, which
// applies it, reads it contiguously.
// A forward plane with a windowed amplitude (win < n) has zero rows outside the window after
// the optic; the power-of-two sweeps neither store them (row sweep) nor load them (column sweep).
constexpr int kSourceOptic = 2;  // forward only: the input field is 1 (it is not read)
constexpr int kTowardSource = 4;  // direct step over z < 0: the transforms' kernel sign flips
// adjoint planes: only the centred win rows of the output are needed (the others are left
// unspecified): the power-of-two column sweep, which runs first, stores only those rows, and
// the row sweep skips the blocks whose rows all lie outside them
constexpr int kWindowRowsOnly = 8;
struct PlaneArgs {
  float2 *field;             // n x n, in place
  const float *amp;          // win x win or null
  const float *opd;          // win x win OPD [m] or null
  const float *pre_surf;     // n x n or null
  const float *post_surf;    // n x n or null
  const float2 *h;           // n: exp(-i pi lambda z k^2/(n dx)^2) / n over signed index k
  const float2 *lens;        // n: exp(-i pi c^2 dx^2 / (lambda f)) or null
  float inv_lambda;          // 1 / lambda [1/m]
  int n;                     // plane edge
  int win;                   // window edge of amp / opd (n for full maps)
  int flags;                 // FR_ADJOINT | kSourceOptic | kTowardSource | kWindowRowsOnly
  int post_lo, post_hi;      // when post_hi > post_lo: post_surf is 0 outside columns [post_lo, post_hi)
};

// element (y, x) of an n x n map stored in 4-column tiles: tile x/4 holds rows 0..n-1 of its
// 4 columns, row-major within the tile (post_tiled_size(n) floats in all)
__host__ __device__ inline size_t post_tiled_index(int n, int y, int x) {
  return (size_t(x >> 2) * size_t(n) + size_t(y)) * 4 + size_t(x & 3);
}
__host__ __device__ inline size_t post_tiled_size(int n) { return size_t((n + 3) / 4) * 4 * size_t(n); }

constexpr int kMaxBatch = 64;
struct BatchArgs {
  PlaneArgs p[kMaxBatch];
};

// Row sweep then column sweep over `count` planes of edge n (count <= kMaxBatch).
// tw: the plan's twiddle table (fresnel_twiddle_build). Returns a hipError_t.
// `variant` selects a tile configuration (row lines per block, column tile width); every
// variant computes the same result. fresnel_variants(n) = number of variants for edge n.
hipError_t launch_fresnel_batch(const PlaneArgs *planes, int count, int n, const float2 *tw,
                                hipStream_t stream, const LaunchHook &hook, int variant);
// The direct (single-transform) Fresnel step of `count` planes of power-of-two edge n
// (count <= kMaxBatch): the row sweep applies the optic times the input quadratic phase (lens
// slot) and the forward transform, the column sweep the forward transform and the output
// quadratic phase (h slot). Same tiles as variant 0 of launch_fresnel_batch.
hipError_t launch_direct_batch(const PlaneArgs *planes, int count, int n, const float2 *tw, hipStream_t s,
                               const LaunchHook &hook);
int fresnel_variants(int n);
int fresnel_twiddle_count(int n);
void fresnel_twiddle_build(int n, float2 *out);  // host
bool fresnel_size_supported(int n);  // power-of-two edges with register-resident plans
bool plane_size_supported(int n);    // those or any mixed-radix edge

// ---- mixed-radix sweeps (any edge up to kMrMaxN that factors into radices <= 16) ----------
constexpr int kMrMaxN = 4096;
constexpr int kMrMaxPass = 6;
constexpr int kMrMaxBatch = 24;
struct MrPlane {
  PlaneArgs pa;
  int n, npass, first;  // first: index of the plane's first work item (set by the launcher)
  unsigned plan;        // radices, 5 bits per pass
  const float2 *tw;     // mr_twiddle_build table of the plan
};
struct MrBatch {
  int count, total;
  MrPlane p[kMrMaxBatch];
};
bool mr_plan(int n, int *npass, int *radix);
// distinct orders of the greedy plan's radices (the first is the greedy plan), at most `max`
int mr_plan_orders(int n, int max, unsigned *plans, int *npass);
unsigned mr_pack(int npass, const int *radix);
int mr_twiddle_count(int npass, const int *radix);
void mr_twiddle_build(int npass, const int *radix, float2 *out);  // host
// rows then columns for forward planes, columns then rows for adjoint planes; persistent grids
// of cus x the resident blocks per compute unit of the instance that runs them (a compile-time
// plan when every plane has the same edge and one of the broadband grids' plans, else the
// runtime plan of the largest edge's class; mr_launch_count says which edges keep their bits in one
// launch)
hipError_t launch_mr_batch(const MrBatch &all, const int *rows_per_cu, const int *cols_per_cu, int cus,
                           hipStream_t s, const LaunchHook &hook);
// classes of the runtime plan's instances by the longest line they hold: 256, 512, 1024, 2048, 4096
constexpr int kMrClasses = 5;
int mr_class(int n);
// of planes ordered by edge, how many from the first on may share a launch
int mr_launch_count(const int *edges, int count);
// a packed plan with a radix that the runtime plan's sweeps do not have (launch_mr_batch refuses a
// launch that would run one)
bool mr_past_16(unsigned plan);
// blocks of each instance of the two persistent sweeps that one compute unit holds at once
// (the runtime plan's classes, then the compile-time plans); a device query, made at context
// creation
constexpr int kMrPolicies = 12;
void mr_resident(int *rows_per_cu, int *cols_per_cu);

// ---- MFT: one product with the Fourier matrix, folded about its axis, on MFMA ------------
// out(a) = alpha sum_b in(b) exp(sign 2 pi i a b c) (+ beta Cin) (* mask) along one axis of the
// data, a and b signed indices about P/2 and Q/2; the other axis is free.
struct FoldArgs {
  int F, P, Q;         // free indices, output length, input length
  int cols;            // 0: along each row (data F x Q, out F x P); 1: along each column (Q x F, P x F)
  double sign;         // -1 (W) or +1 (conj(W))
  const float2 *data;  // row stride ldd
  int ldd;
  const void *table;   // fold_table_build(P, Q, c)
  float2 *C;           // row stride ldc
  int ldc;
  double alpha;        // applied in float64 in the epilogue
  float beta;          // the beta term reads Cin (row stride ldcin), or C when Cin is null
  const float2 *Cin;
  int ldcin;
  const float *mask;   // like the output (row stride ldm) or null: multiplies the result
  int ldm;
  double *intensity;   // like the output (row stride ldi) or null: intensity += weight |result|^2 (float64)
  int ldi;
  double weight;
  int skip_c;          // 1: do not write C (only the intensity)
};
// The table: bfloat16 pieces of cos (parity 0) and sin (parity 1) of 2 pi k j c, k = 1 .. P/2,
// j = 1 .. Q/2, as MFMA fragments [parity][tile of 32 k][step of 16 j][piece][lane][8]: lane l
// holds k = l % 32 of the tile, j = 8 (l / 32) .. + 7 of the step; zero past P/2 and Q/2. The
// steps are padded to whole stages of four.
__host__ __device__ inline int fold_tiles(int P) { return (P / 2 + 31) / 32 > 0 ? (P / 2 + 31) / 32 : 1; }
__host__ __device__ inline int fold_steps(int Q) { return (Q / 2 + 63) / 64 > 0 ? (Q / 2 + 63) / 64 * 4 : 4; }
// every second pair of steps holds the entries with the opposite sign: the pairs that one of the two
// halves of the general kernel's waves sums, so that the rounding bias of the halves cancels
__host__ __device__ inline bool fold_negated(int step) { return step & 2; }
inline size_t fold_table_bytes(int P, int Q) { return size_t(2) * fold_tiles(P) * fold_steps(Q) * 3 * 64 * 8 * 2; }
// split > 1 slices the pairs; the slices' partial sums go to `partial` (split x output complex
// float64, 16-byte aligned) and are added in a fixed order by a second kernel.
constexpr int kMaxSplit = 16;
// tile numbers a tuning file may carry (they name complex tiles that the folded product, which
// picks its tile by shape, has replaced; the split factor beside them is used)
constexpr int kGemmTiles = 7;
enum { kFoldGeneral, kFoldShort, kFoldFew };
int fold_kind(int F, int P, int Q);
int fold_split_for(const FoldArgs &a);
int fold_short_tiles(int tiles, int ftiles);
hipError_t launch_fold(const FoldArgs &a, int split, void *partial, hipStream_t stream, const LaunchHook &hook);

}  // namespace fr
