// Internal helpers shared by the HIP sources of libkmq (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/kmq.h"

namespace kmq {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

constexpr int kWave = 64;

// Launch-facing description of the points (validated copy of km_points).
struct Points {
  int fmt;
  int d;          // logical dims
  int64_t n;
  const void *data;
  int64_t ld;     // F32: floats, SQ8: bytes, 1-bit: words (= d/32)
  const float *alpha;
  const float *center;
  const float *front;  // hybrid: n x d_front
  int d_front;
  const float *raw;    // nullable: fp32 rows in the clustering space (last update of a fit)
  int64_t raw_ld;
  const float *vparams;  // LVQ4: per-vector (s, b, A, N)
  bool fit;              // one pass among others: the kernels wait for each other and not for their launches
  bool split;            // F32, HYBRID: assignments take the fp16 matrix cores (split.hpp) where the data allow
};

// 1-bit point formats (codes + one scale per point)
__host__ __device__ constexpr bool is_bits_fmt(int fmt) {
  return fmt == KM_SIGN1 || fmt == KM_HYBRID || fmt == KM_RABITQ;
}

// What the preparation decides for one pass on the fp16 matrix cores (in device memory).
struct SplitRoute {
  int ok;    // 0: the fp32 kernel takes the pass
  float s;   // power of two that scales points and centroids
  float m2;  // -2 / s^2
  int pad;
};

// The centroids for the fp16 matrix cores (split.hip), rebuilt with CentroidPrep.
struct SplitPrep {
  SplitRoute *route;  // NULL: not used
  uint32_t *rmax;     // [k] bit pattern of the row's largest |c|
  float *seed;        // [k + pad] -s^2 ||c||^2 / 2, then -inf
  int *tflag;         // point tiles the fp32 kernel has to redo
  float *tail;        // HYBRID: -T (int bits), u and 2 sigma times -s^2 / 2, k + pad each; else NULL
  uint8_t *img;       // stage-major: 64 bytes (16 hi, 16 lo halves) of every row per 16 dims
  int64_t cstage;     // bytes of one stage of img
  unsigned long long *keys;  // few tiles (split_small; route is NULL): the points' (score, index) keys
};

// Per-centroid data rebuilt before each assignment pass.
struct CentroidPrep {
  const float *cn;     // F32/HYBRID/BF16: ||c'||^2 over the fp32 dims; RABITQ, LVQ4: bias b
  const int *qsum;     // SQ8: -||c~||^2 ; SIGN1/HYBRID/RABITQ: T_j = sum q ; LVQ4: S_j = sum of codes
  const float *u;      // SIGN1/HYBRID: (sigma*sigma)*Q ; RABITQ: ||c||^2 ; LVQ4: N_j
  const float *sig2;   // SIGN1/HYBRID: 2*sigma ; RABITQ, LVQ4: scale s
  const int8_t *q;     // SIGN1/HYBRID: int8 residual codes, k x dt ; RABITQ: codes 0..15, k x d ; LVQ4: codes
                       // 0..15, k x d, each 8 dims ordered 0 2 4 6 1 3 5 7 (the unpacked point order)
  const uint16_t *cb;  // BF16: centroids rounded to bfloat16, k x d
  unsigned long long *keys;  // centroid-tile groups (F32/HYBRID/SQ8/BF16/LVQ4): per-point (score, index) keys
  SplitPrep sp;              // F32 and HYBRID with Points::split
};

// Host-side error plumbing.
void set_error(const char *fmt, ...);
km_status hip_fail(hipError_t e, const char *what);

#define KMQ_HIP(call)                                         \
  do {                                                        \
    hipError_t _e = (call);                                   \
    if (_e != hipSuccess) return ::kmq::hip_fail(_e, #call);  \
  } while (0)

#define KMQ_LAUNCH_CHECK(what)                                \
  do {                                                        \
    hipError_t _e = hipGetLastError();                        \
    if (_e != hipSuccess) return ::kmq::hip_fail(_e, what);   \
  } while (0)

__host__ __device__ static inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ---- launchers implemented in the kernel sources ---------------------------

// pca.hip: compute units of the current device (256 if the query fails)
int cu_count();

// assign.hip
km_status launch_prep(const Points &P, const void *C, int k, void *ws_prep, CentroidPrep *out,
                      hipStream_t s);
size_t prep_bytes(const Points &P, int k);
// whether the fp16 matrix cores are the faster ones for these points and k centroids (P.split says that they can)
bool split_pays(const Points &P, int k);
// aoff is added to every stored centroid index (C and cp may be a slice of a larger set)
// One launch for many (row range, centroid range) segments of fp32, SQ8 or bf16
// points: segment i is rows [segs[i].x, + segs[i].y) against centroids
// [segs[i].z, + segs[i].w) of C and of the prepared constants; workgroup b takes
// point tile tiles[b].y of segment tiles[b].x (tiles of assign_segment_rows(P) rows;
// 0 = not supported for these points).  Centroid indices are absolute; assign and
// score are indexed by absolute row.  fp32: row i of the segments is row prow[i] of
// the points and of assign (score stays in segment order).  tile_c: centroids per tile
// of every segment of the launch (segment_tile_centroids picks it per segment).
int assign_segment_rows(const Points &P);
// 128 for a segment of at most 128 centroids, else 256: the 256-centroid kernel does
// more MFMA work per stage, which outweighs its extra padding from 129 on.  fp32
// segments of at most 64 take 64: the fp32 matrix work that a 128-centroid tile spends
// on padding is the pass's time (1M x 1024 in 63 segments of about 63 centroids: 2.2 ms per
// pass on 128-centroid tiles, 0.7 + 1.3 ms on tiles of 64 and of 128).
int segment_tile_centroids(const Points &P, int k_seg);
km_status launch_assign_segments(const Points &P, const void *C, const CentroidPrep &cp, const int4 *segs,
                                 const int2 *tiles, int64_t ntiles, int tile_c, int32_t *assign, float *score,
                                 const int *prow, hipStream_t s);
km_status launch_assign(const Points &P, const void *C, const CentroidPrep &cp, int k, int32_t *assign,
                        float *score, hipStream_t s, int aoff = 0);
// cp restricted to centroids [off, ...) and, for the per-point keys, to points [pstart, ...)
CentroidPrep prep_slice(const Points &P, const CentroidPrep &cp, int off, int64_t pstart);
// prow (nullable): entry i is of row prow[i]
km_status launch_xconst(const Points &P, float *xc, hipStream_t s, const int *prow = nullptr);
km_status launch_objective(const Points &P, const float *xc, const float *score, int64_t n, double *out,
                           double *partials, int nblk_max, hipStream_t s, const double *xsum = nullptr);
int objective_blocks(int64_t n);
// the same sum for fp32 and hybrid points from the distances (direct_objective_bytes of partials)
km_status launch_direct_objective(const Points &P, const float *C, const CentroidPrep &cp, int k,
                                  const int32_t *assign, double *out, double *partials, hipStream_t s);
size_t direct_objective_bytes();
km_status launch_gather_init(const Points &P, const int64_t *idx, int k, void *C, hipStream_t s);
km_status launch_cost(const float *X, int64_t n, int d, int64_t ldx, const float *C, int k,
                      const int32_t *assign, double *out, double *partials, hipStream_t s);

// split.hip: fp32 points on the fp16 matrix cores
struct SplitArgs {
  const float *x;  // n x ldx
  int64_t ldx;
  int d;
  SplitPrep sp;
  int kall;  // rows in sp (its seed[kall] is -inf)
  int k;
  int64_t n;
  int32_t *assign;
  float *score;
  int aoff;
  int ngroups;
  int64_t n_ptiles;
  unsigned long long *keys;
  // HYBRID: the points' 1-bit codes (words per row, first tail word), the centroids' codes, tail dims
  const uint32_t *pbits;
  int64_t pbw;
  int pbw0;
  const int8_t *ci8;
  int64_t cild;
  int di;
  const float *alpha;
  // projection: d dims to k outputs, Y n x k
  const float *mean;
  float *Y;
  // pruning: front norms, thresholds, previous centroids, survivor bits (W4 words a row), partial counts
  const float *xn, *tau;
  float r0;
  const int32_t *prev;
  uint32_t *mask;
  int W4;
  unsigned long long *cnt;  // nullable, [2 ncnt]: two per 128 points
  int64_t ncnt;
};
enum { kSplitAssign = 0, kSplitHybrid = 1, kSplitProject = 2, kSplitPrune = 3 };
constexpr int kSplitProjMaxD = 4096;  // the mean's place in LDS
// Y = (X - mean) W on the fp16 matrix cores; out: the route and the point tiles (of 256) left to the fp32 kernel
size_t split_project_bytes(int64_t n, int d, int d_out);
km_status launch_split_project(const float *X, int64_t n, int d, int64_t ldx, const float *mean, const float *W,
                               int d_out, float *Y, void *ws, SplitPrep *out, hipStream_t s);
constexpr int kSplitTailWords = 20;  // resident tail words per point (640 tail dims)
size_t split_bytes(int64_t n, int k, int d, bool tail);
SplitPrep split_layout(int64_t n, int k, int d, bool tail, void *ws);
km_status launch_split_prep(const float *C, int64_t ldc, int64_t n, int k, int d, const CentroidPrep &cp,
                            hipStream_t s);
km_status launch_split(const SplitArgs &A, int64_t grid, int tile_c, hipStream_t s);

// split_small.hip: fp32 points and centroids of few tiles
struct SmallArgs {
  const float *x, *C;  // points (rows ldx floats apart), centroids (k x d)
  int64_t ldx;
  const float *cn;
  const uint32_t *rmax;
  int64_t n;
  int k, d;
  int ngroups;  // centroid tiles
  int64_t n_ptiles;
  unsigned long long *keys;  // ngroups > 1
  int *count;
  int32_t *assign;
  float *score;  // nullable
  int aoff;
};
bool split_small(int64_t n, int k);
size_t split_small_bytes(int64_t n, int k);
// fills cn; one assignment per preparation
km_status launch_split_small_prep(const float *C, int64_t n, int k, int d, float *cn, void *ws, SplitPrep *out,
                                  hipStream_t s);
km_status launch_split_small(const float *X, int64_t ldx, const float *C, const CentroidPrep &cp, int64_t n, int k,
                             int d, int32_t *assign, float *score, int aoff, hipStream_t s);

// update.hip
size_t update_bytes(const Points &P, int k);
// seg_lo / seg_hi (nullable, int[k]): the split takes the donor of empty cluster j
// from clusters [seg_lo[j], seg_hi[j]) only.  objective (nullable, DEVICE, F32 only): the
// sum of the points' squared distances to the centroids passed in; with norms the sum of
// the squared norms of all points but those with assign = -1.
km_status launch_update(const Points &P, const int32_t *assign, int k, void *C, int64_t *counts,
                        int policy, void *ws, hipStream_t s, const int *seg_lo = nullptr,
                        const int *seg_hi = nullptr, double *objective = nullptr, bool norms = false);
struct SortOut {
  const int *perm;    // [n]: point indices ordered by cluster, point order kept inside a cluster
  const int *cnt;     // [k]: members per cluster (ids outside [0, k) are left out)
  const int *cstart;  // [k]: first position of each cluster in perm
};
size_t sort_bytes(int64_t n, int k);
km_status launch_cluster_sort(const int32_t *assign, int64_t n, int k, void *ws, SortOut *out, hipStream_t s);

// hier.hip: contiguous per-meso-cluster copies of the points and the write-back
size_t permuted_bytes(const Points &P, int64_t nrows);
km_status launch_permute_points(const Points &P, const int *perm, int64_t nrows, void *ws, Points *out,
                                hipStream_t s);
Points slice_points(const Points &P, int64_t start, int64_t count);
// idx[j] = perm[idx[j]], j < k
km_status launch_map_index(const int *perm, int64_t *idx, int k, hipStream_t s);
// a[i] = v, i < n
km_status launch_fill_assign(int32_t *a, int64_t n, int32_t v, hipStream_t s);
km_status launch_scatter_assign(const int *perm, const int32_t *a_perm, int64_t nsel, int64_t n, int32_t *assign,
                                hipStream_t s);

// skm.hip: dimension pruning inside STEP 2
double prune_factor(int D, int d, double eps0);
int prune_front_default(int d);
size_t pruned_bytes(const Points &P, int k, int D0);
km_status launch_assign_pruned(const Points &P, const void *C, int k, const int32_t *prev, int32_t *assign,
                               double *dist, double *objective, double eps0, int D0,
                               unsigned long long *cnt, void *ws, hipStream_t s);
km_status launch_zero_counters(unsigned long long *c, hipStream_t s);

// quantize.hip
size_t quantize_bytes(int64_t n, int d, int fmt);
km_status launch_quantize(const float *X, int64_t n, int d, int64_t ldx, int fmt, void *codes,
                          float *params, float *alpha, int d_front, float *front, int flags, void *ws,
                          hipStream_t s);

// split: the rotation on the fp16 matrix cores (project_split allowing)
size_t rabitq_encode_bytes(int64_t n, int d, bool y_given, bool split);
km_status launch_rabitq_encode(const float *X, int64_t n, int d, int64_t ldx, const float *P, float *m,
                               uint32_t *bits, float *alpha, float *Y, int flags, void *ws, bool split,
                               hipStream_t s);
size_t colmean_bytes(int64_t n, int d, bool ranges = false);
// top (nullable): each column's largest |x - mean| (workspace with ranges)
km_status launch_colmean(const float *X, int64_t n, int d, int64_t ldx, float *m, void *ws, hipStream_t s,
                         float *top = nullptr);

// pca.hip
size_t pca_cov_bytes(int64_t n, int d);
km_status launch_pca_cov(const float *X, int64_t n, int d, float *mean, float *cov, void *ws,
                         hipStream_t s);
// whether the fp16 matrix cores take a projection of these rows (split below)
bool project_split(int64_t n, int d, int d_out, int64_t ldx);
km_status launch_pca_project(const float *X, int64_t n, int d, int64_t ldx, const float *mean, const float *W,
                             int d_out, float *Y, void *ws, bool split, hipStream_t s);
size_t pca_project_bytes(int64_t n, int d, int d_out, bool split);

// ---- device helpers ---------------------------------------------------------

__device__ __forceinline__ int lane_id() { return __lane_id(); }

// Nearest bfloat16 of x, ties to the even significand, as its 16-bit pattern.
// bfloat16 keeps the top 16 bits of the fp32 pattern; adding 0x7FFF plus the
// lowest kept bit carries into the kept half exactly when the discarded half
// exceeds 0x8000, or equals it and the kept half is odd.  A carry out of the
// significand steps the exponent (up to infinity), which is the correct result.
// NaN keeps its sign and top payload bits and is made quiet.
__device__ __forceinline__ uint32_t bf16_bits(float x) {
  const uint32_t u = __float_as_uint(x);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
  return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

__device__ __forceinline__ uint32_t spread4(uint32_t b4) {
  // 4 bits -> 4 bytes holding 0 or 1 (bit j -> byte j)
  return (b4 * 0x00204081u) & 0x01010101u;
}

// A word of 1-bit codes for the matrix cores: bit 16 h + 4 q + j goes to bit 8 j + 4 h + q.
__device__ __forceinline__ uint32_t regroup_bits(uint32_t w) {
  uint32_t o = 0;
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int q = 0; q < 4; ++q) o |= spread4((w >> (16 * h + 4 * q)) & 15u) << (4 * h + q);
  return o;
}

// x: a regrouped word shifted right by 4h.  Register q takes bit 8j + q of x as
// byte j with the value 0 or 2, so the products sum to 2D; seeded with -T the
// accumulator ends at 2D - T.
__device__ __forceinline__ i32x4 widen_regrouped2(uint32_t x) {
  constexpr uint32_t M2 = 0x02020202u;
  return i32x4{(int)((x << 1) & M2), (int)(x & M2), (int)((x >> 1) & M2), (int)((x >> 2) & M2)};
}

__device__ __forceinline__ float bf16_value(uint32_t b) { return __uint_as_float(b << 16); }

// Deterministic block-wide sum of doubles (fixed tree order). blockDim.x == 256.
__device__ __forceinline__ double block_sum_f64(double v, double *sh) {
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  if (t < 64) {  // the halving tree over 256 values, its last six levels inside a wave
    v = (sh[t] + sh[t + 128]) + (sh[t + 64] + sh[t + 192]);
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) v += __shfl_down(v, s);
    if (t == 0) sh[0] = v;
  }
  __syncthreads();
  const double r = sh[0];
  __syncthreads();
  return r;
}

}  // namespace kmq
