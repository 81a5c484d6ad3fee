// PCA before clustering (Sec. 3.1 "PCA"; Sec. 4.2): covariance of the centred
// points and the projection onto the leading principal directions, both as
// MFMA contractions.
//
// Covariance: the d x d output is cut into 256 x 256 tiles (upper triangle only,
// mirrored at the end) and the n rows are split across workgroups; every workgroup's
// fp64 partial tile is folded in split order.
// Projection: on the fp16 matrix cores (split.hip); the fp32 kernels below take the
// tiles and shapes it leaves, with the rows centred as they are read and W
// pre-transposed so that both MFMA operands are 16 contiguous bytes per lane.
#include <algorithm>
#include <type_traits>

#include "split.hpp"

namespace kmq {
namespace {

constexpr int kT = 128;           // projection tile
constexpr int kCT = 256;          // covariance output tile

__device__ __forceinline__ void tile_ij(int t, int T, int &ti, int &tj) {
  // enumerate the upper triangle row by row
  ti = 0;
  while (t >= T - ti) {
    t -= T - ti;
    ++ti;
  }
  tj = ti + t;
}

// Direct copy of 16 bytes per lane from global memory into LDS: the wave's 64 lanes
// fill 1 KB at LDS byte address lds (wave-uniform) in lane order, from a
// wave-uniform base plus a 32-bit per-lane byte offset.  Inline assembly, so that
// the compiler does not wait for the copy before the LDS reads of the other stage
// buffer; the caller waits (vmcnt) before the barrier that publishes the data.
typedef __attribute__((address_space(3))) uint8_t lds_u8;
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void lds_copy16(const void *base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds)
               : "memory", "m0");
}
#pragma clang diagnostic pop

// Covariance on the fp16 matrix cores (split.hpp).  One workgroup per (256 x 256 output
// tile, split of the rows): 8 waves, two per SIMD, each owning 128 x 64 of the tile as
// 4 x 2 blocks of 32 x 32; the rows of X are the contraction index, 16 per stage.
//
// Every thread owns a column of the two blocks (a tile of the diagonal has one block:
// half the rows of a column each).  It loads 8 rows of it at a time into registers two
// stages ahead, centres and scales them as it splits them (the column's own power of
// two, from its largest |x - mean|, which the mean's pass over X finds: no value leaves
// fp16's range, and a column's relative precision does not depend on the others), and
// stores hi and lo as MFMA operand chunks: 8 consecutive rows of a column are 16
// contiguous bytes.  The chunks lie as in split_kernel (two 32-column blocks share
// 128-byte rows, chunk c in slot c ^ ((r >> 1) & 7)).  Three buffers and one barrier
// per stage: step i multiplies stage i from registers while it reads stage i + 1 into
// them and splits stage i + 2.
//
// The fp32 accumulators are added into this workgroup's fp64 partial tile in global
// memory every 4096 rows: the instruction's rounding, and the little it cuts, grow with
// the number of additions (at 8192 rows the relative error of the covariance was that
// of the fp32 kernel's, 2.1e-7).  2M x 1024:
// 20.5 -> 8.8 ms against v_mfma_f32_32x32x2_f32 tiles centred as they were read; three
// matrix products of 2.6 TFLOP take 6.1 ms at the rate of a large library product.
// Workgroups of one split are neighbours on one XCD, whose L2 then serves the rows
// that its tiles share.
constexpr int kCovThreads = 512;
constexpr int kCovSD = 16;                        // rows per stage
constexpr int kCovBlk = kCT * 64;                 // bytes of one column block of a stage
constexpr int kCovStage = 2 * kCovBlk;
constexpr int kCovFlush = 4096 / kCovSD;          // stages per fp32 accumulation run

// the power of two that puts a column's largest |x - mean| at [2^14, 2^15)
__device__ __forceinline__ float cov_scale(float top) {
  if (!(top > 0.f)) return 1.0f;
  const int e = (int)(__float_as_uint(top) >> 23) - 127;
  return ldexpf(1.0f, min(14 - e, 100));
}

template <bool DIAG>
__device__ __forceinline__ void cov_tile(const float *X, int d, const float *mean, const float *top, int ti, int tj,
                                         int64_t rb, int64_t re, uint8_t *ring, double *out);

__global__ __launch_bounds__(kCovThreads, 1) void cov_kernel(const float *X, int64_t n, int d, const float *mean,
                                                             const float *top, int T, int ntiles, int nsplit,
                                                             int64_t rows_per_split, double *partial) {
  __shared__ __align__(16) uint8_t ring[3 * kCovStage];
  const int per = (int)(gridDim.x >> 3);  // workgroups of one XCD: neighbours in (split, tile)
  const int id = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if (id >= ntiles * nsplit) return;  // whole workgroup, before any barrier
  const int tile = id % ntiles, split = id / ntiles;
  int ti, tj;
  tile_ij(tile, T, ti, tj);
  const int64_t rb = (int64_t)split * rows_per_split;
  const int64_t re = min<int64_t>(n, rb + rows_per_split);
  double *out = partial + ((int64_t)split * ntiles + tile) * (kCT * kCT);
  if (re <= rb) {  // no rows: the partial tile is zero
    for (int e = threadIdx.x; e < kCT * kCT; e += kCovThreads) out[e] = 0.0;
  } else if (ti == tj) {
    cov_tile<true>(X, d, mean, top, ti, tj, rb, re, ring, out);
  } else {
    cov_tile<false>(X, d, mean, top, ti, tj, rb, re, ring, out);
  }
}

template <bool DIAG>
__device__ __forceinline__ void cov_tile(const float *X, int d, const float *mean, const float *top, int ti, int tj,
                                         int64_t rb, int64_t re, uint8_t *ring, double *out) {
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int r = lane & 31, h = lane >> 5;
  const int wi = wave & 1, wj = wave >> 1;
  const int len = (int)(re - rb);  // rows of a split: below 2^31 as n is
  const int nst = (len + kCovSD - 1) / kCovSD;
  // this thread's column, its centre and scale, and its place in a stage
  const int lc = t & 255;  // column within its block
  const int gc = min((!DIAG && t >= 256 ? tj : ti) * kCT + lc, d - 1);
  const float sc = cov_scale(top[gc]), ms = mean[gc] * sc;
  constexpr int NU = DIAG ? 1 : 2;              // units of 8 rows per stage
  const int half0 = DIAG ? wave >> 2 : 0;       // the first unit's half of the stage's rows
  const uint32_t ring0 = (uint32_t)(size_t)(lds_byte *)ring;
  const uint32_t lrow = (uint32_t)((!DIAG && t >= 256 ? kCovBlk : 0) + (lc >> 6) * 4096 + (lc & 31) * 128);
  const uint32_t lkx = (uint32_t)(lc >> 1) & 7u;
  auto place = [&](int c) -> uint32_t { return lrow + 16u * ((4u * ((lc >> 5) & 1) + c) ^ lkx); };
  typedef __attribute__((address_space(3))) i32x4 lds_i32x4;
  auto st16 = [&](uint32_t off, i32x4 v) { *(lds_i32x4 *)(size_t)(ring0 + off) = v; };
  auto rd16 = [&](uint32_t off) -> i32x4 { return *(const lds_i32x4 *)(size_t)(ring0 + off); };

  float raw[2][NU][8];  // two stages in flight
  const float *xrow = X + rb * d;
  const int nfull = len / kCovSD;
  // wave-uniform row addresses; rows past the split read the mean and count as zero
  auto load = [&](int st, int set, auto full_) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int row = st * kCovSD + 8 * (half0 + u);
      const float *p = xrow + (int64_t)row * d;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        raw[set][u][i] = (decltype(full_)::value || row + i < len ? p : mean)[(uint32_t)gc];
        p += d;
      }
    }
  };
  uint32_t hi[4], lo[4];
  float one = 1.0f;  // not seen through by the compiler: keeps split2's mixed instructions
  asm volatile("" : "+s"(one));
  auto conv = [&](int set, int u, int q) {  // pair q of unit u
    split2(__builtin_fmaf(raw[set][u][2 * q], sc, -ms), __builtin_fmaf(raw[set][u][2 * q + 1], sc, -ms), one, hi[q],
           lo[q]);
    asm volatile("" : "+v"(hi[q]), "+v"(lo[q]));
  };
  auto put = [&](uint32_t buf, int u) {
    st16(buf + place(half0 + u), i32x4{(int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]});
    st16(buf + place(2 + half0 + u), i32x4{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3]});
  };

  const uint32_t orow = (uint32_t)(r * 128), kx = (uint32_t)((r >> 1) & 7);
  auto at = [&](int b, int c) -> uint32_t {
    return (uint32_t)(b >> 1) * 4096u + orow + 16u * ((4u * (b & 1) + c) ^ kx);
  };
  const uint32_t breg = DIAG ? 0u : (uint32_t)kCovBlk;
  f32x16 acc[4][2];
  h16x8 ah[4], al[4], bh[2], bl[2];
  auto read_a = [&](int cb, int c, uint32_t buf) { return __builtin_bit_cast(h16x8, rd16(buf + at(wi * 4 + cb, c + h))); };
  auto read_b = [&](int pb, int c, uint32_t buf) {
    return __builtin_bit_cast(h16x8, rd16(buf + breg + at(wj * 2 + pb, c + h)));
  };
  auto pin = [&]() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto next = [](uint32_t b) { return b == 2u * kCovStage ? 0u : b + kCovStage; };
  uint32_t b0 = 0, b1 = kCovStage, b2 = 2 * kCovStage;  // buffers of stages i, i + 1, i + 2
  auto step = [&](int i, auto set_, auto full_) {
    constexpr int SET = decltype(set_)::value;  // where stage i + 2 waits (and stage i + 4 will)
#pragma unroll
    for (int pb = 0; pb < 2; ++pb)
#pragma unroll
      for (int j = 0; j < 12; ++j) {
        const int pr = j / 4, cb = j % 4;
        acc[cb][pb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(pr == 0 ? al[cb] : ah[cb], pr == 1 ? bl[pb] : bh[pb],
                                                             acc[cb][pb], 0, 0, 0);
        if (pb == 0) {
          if (j == 0) bh[1] = read_b(1, 0, b0);
          if (j == 1) bl[1] = read_b(1, 2, b0);
          // unit 0 of stage i + 2
          if (j >= 2 && j < 10 && j % 2 == 0) conv(SET, 0, (j - 2) / 2);
          if (j == 10) put(b2, 0);
        } else {
          if constexpr (NU == 2) {
            if (j < 8 && j % 2 == 0) conv(SET, 1, j / 2);
            if (j == 7) put(b2, 1);
          }
          if (j >= 1 && j <= 4) al[j - 1] = read_a(j - 1, 2, b1);
          if (j == 5) bh[0] = read_b(0, 0, b1);
          if (j == 6) bl[0] = read_b(0, 2, b1);
          if (j == 8) load(i + 4, SET, full_);
          if (j >= 9) ah[j - 9] = read_a(j - 9, 0, b1);
        }
        pin();
      }
    ah[3] = read_a(3, 0, b1);
    // the stores are complete when only the four reads after them are out
    asm volatile("s_waitcnt lgkmcnt(4)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    b0 = b1;
    b1 = b2;
    b2 = next(b2);
  };
  auto zero = [&]() {
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
  };
  bool first = true;
  auto flush = [&]() {
    // the lane's offset passes through an empty asm statement so that the element
    // addresses are formed here, not hoisted out of the loop
    int boff = (wi * 128 + 4 * h) * kCT + wj * 64 + r;
    asm volatile("" : "+v"(boff));
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int pb = 0; pb < 2; ++pb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          double *o = out + boff + (cb * 32 + 8 * (v >> 2) + (v & 3)) * kCT + pb * 32;
          *o = (first ? 0.0 : *o) + (double)acc[cb][pb][v];
        }
    first = false;
  };

  // stages 0 and 1 into their buffers, 2 and 3 into registers, stage 0's operands
  constexpr std::true_type T{};
  constexpr std::false_type F{};
  load(0, 0, F);
  load(1, 1, F);
#pragma unroll
  for (int st = 0; st < 2; ++st) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
#pragma unroll
      for (int q = 0; q < 4; ++q) conv(st, u, q);
      put(st * kCovStage, u);
    }
    load(st + 2, st, F);
  }
  zero();
  __syncthreads();
#pragma unroll
  for (int cb = 0; cb < 4; ++cb) {
    al[cb] = read_a(cb, 2, 0);
    ah[cb] = read_a(cb, 0, 0);
  }
  bh[0] = read_b(0, 0, 0);
  bl[0] = read_b(0, 2, 0);
  std::integral_constant<int, 0> S0;
  std::integral_constant<int, 1> S1;
  for (int i = 0; i < nst; i += kCovFlush) {
    const int e = min(nst, i + kCovFlush);
    int s = i;
    for (; s + 1 < e && s + 5 < nfull; s += 2) {
      step(s, S0, T);
      step(s + 1, S1, T);
    }
    for (; s < e; s += 2) {
      step(s, S0, F);
      if (s + 1 < e) step(s + 1, S1, F);
    }
    flush();
    zero();
  }
}

// The partial tiles in split order, back from the columns' scales; an element per thread
// (d = 1024, 10 tiles: 0.34 ms with 16 workgroups per tile, 0.04 so).
__global__ __launch_bounds__(256) void cov_reduce_kernel(const double *partial, int ntiles, int nsplit, int T, int d,
                                                         int64_t n, const float *top, float *cov) {
  const int tile = blockIdx.x;
  int ti, tj;
  tile_ij(tile, T, ti, tj);
  for (int e = blockIdx.y * 256 + threadIdx.x; e < kCT * kCT; e += gridDim.y * 256) {
    const int il = e / kCT, jl = e % kCT;
    const int i = ti * kCT + il, j = tj * kCT + jl;
    // (the two halves of a diagonal tile are rounded in different orders: one of them counts)
    if (i >= d || j >= d || i > j) continue;
    double s = 0.0;
#pragma unroll 8
    for (int sp = 0; sp < nsplit; ++sp) s += partial[((int64_t)sp * ntiles + tile) * (kCT * kCT) + e];
    const float v = (float)(s / ((double)cov_scale(top[i]) * cov_scale(top[j])) / (double)n);
    cov[(int64_t)i * d + j] = v;
    cov[(int64_t)j * d + i] = v;
  }
}

__global__ void transpose_kernel(const float *W, int d, int d_out, float *Wt) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= (int64_t)d * d_out) return;
  const int i = (int)(e / d_out), o = (int)(e % d_out);
  Wt[(int64_t)o * d + i] = W[e];
}

constexpr int kPStride = 32 + 4;  // floats per LDS row of a projection stage

// Workgroups are numbered so that the output tiles of one point tile land on the
// same XCD one after another (consecutive ids are spread over the 8 XCDs), so the
// point rows come from HBM once and from that XCD's L2 for the other tiles.
__global__ __launch_bounds__(256) void project_staged_kernel(const float *X, int64_t n, int d, int64_t ldx,
                                                      const float *mean, const float *Wt, int d_out, float *Y,
                                                      int n_ptiles, int n_otiles) {
  __shared__ float Xs[2][kT * kPStride];
  __shared__ float Ws[2][kT * kPStride];
  const int64_t b = blockIdx.x;
  const int64_t group = b / (8 * (int64_t)n_otiles);      // 8 point tiles per group
  const int rem = (int)(b % (8 * (int64_t)n_otiles));
  const int64_t ptile = group * 8 + rem % 8;
  const int otile = rem / 8;
  if (ptile >= n_ptiles) return;
  const int64_t p0 = ptile * kT;
  const int o0 = otile * kT;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int r = lane & 31, h = lane >> 5;
  const int wm = wave & 1, wn = wave >> 1;
  f32x16 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

  const int nst = (d + 31) / 32;
  f32x4 rx[4], rw[4];
  const int prmax = (int)min<int64_t>(n - 1 - p0, kT - 1);
  const int ormax = min(d_out - 1 - o0, kT - 1);
  auto load = [&](int st) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int idx = t + 256 * q;
      const int row = idx >> 3, c4 = idx & 7;
      const int dim = 32 * st + 4 * c4;
      const int dimc = dim < d ? dim : 0;
      rx[q] = *reinterpret_cast<const f32x4 *>(X + (p0 + min(row, prmax)) * ldx + dimc);
      rw[q] = *reinterpret_cast<const f32x4 *>(Wt + (int64_t)(o0 + min(row, ormax)) * d + dimc);
    }
  };
  // centring and zero-fill at store time, one stage after the loads were issued
  auto store = [&](int st, int buf) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int idx = t + 256 * q;
      const int row = idx >> 3, c4 = idx & 7;
      const int dim = 32 * st + 4 * c4;
      const bool ok = dim < d;
      const f32x4 m = *reinterpret_cast<const f32x4 *>(mean + (ok ? dim : 0));
      const f32x4 z = {0.f, 0.f, 0.f, 0.f};
      *reinterpret_cast<f32x4 *>(&Xs[buf][row * kPStride + 4 * c4]) = ok ? rx[q] - m : z;
      *reinterpret_cast<f32x4 *>(&Ws[buf][row * kPStride + 4 * c4]) = ok ? rw[q] : z;
    }
  };
  load(0);
  store(0, 0);
  __syncthreads();
  for (int st = 0; st < nst; ++st) {
    const bool nxt = st + 1 < nst;
    if (nxt) load(st + 1);
    const float *A = Xs[st & 1];
    const float *B = Ws[st & 1];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      f32x4 a[2], b[2];
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
        a[cb] = *reinterpret_cast<const f32x4 *>(&A[(wm * 64 + cb * 32 + r) * kPStride + 8 * g + 4 * h]);
#pragma unroll
      for (int pb = 0; pb < 2; ++pb)
        b[pb] = *reinterpret_cast<const f32x4 *>(&B[(wn * 64 + pb * 32 + r) * kPStride + 8 * g + 4 * h]);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
#pragma unroll
          for (int pb = 0; pb < 2; ++pb)
            acc[cb][pb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[cb][e], b[pb][e], acc[cb][pb], 0, 0, 0);
    }
    if (nxt) store(st + 1, (st + 1) & 1);
    __syncthreads();
  }
#pragma unroll
  for (int cb = 0; cb < 2; ++cb)
#pragma unroll
    for (int pb = 0; pb < 2; ++pb)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int64_t p = p0 + wm * 64 + cb * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
        const int o = o0 + wn * 64 + pb * 32 + r;
        if (p < n && o < d_out) Y[p * d_out + o] = acc[cb][pb][v];
      }
}

struct CovPlan {
  int T, ntiles, nsplit;
  int64_t rows_per_split;
};

// Projection, direct-copy design (d <= kProjMaxD, ldx % 4 == 0, 256 rows of X
// within 2 GB): the 8-wave shape of the fp32 assignment kernel with the points as
// the first MFMA operand and the rows of W^T as the second, so a lane's outputs
// are consecutive output dims of one point and the stores are coalesced.  A
// workgroup computes 256 points x 256 outputs; stages of 32 dims (128 bytes of
// every row: 256 point rows, then 256 rows of W^T) are copied straight from global
// memory into LDS in the XOR slot layout (chunk c of row R in slot c ^ ((R >> 1) &
// 7)), two stage buffers, one workgroup per CU.  The mean sits in LDS (zero past
// d) and the point operands are centred as they are read (x - mean in fp32, the
// value a centring copy would store).  Chunks past d are zero-filled; rows past n
// or d_out are clamped to the last one and their outputs are not stored.
constexpr int kProjMaxD = 4096;
constexpr int kPT = 256;  // points and outputs per workgroup

__global__ __launch_bounds__(512, 1) void project_kernel(const float *X, int64_t n, int d, int64_t ldx,
                                                         const float *mean, const float *Wt, int d_out, float *Y,
                                                         int n_ptiles, int n_otiles, const SplitRoute *route,
                                                         const int *tflag) {
  constexpr int NCP = kPT / 64;            // point copies per thread and stage
  constexpr int NCOPY = 2 * kPT / 64;      // all copies per thread and stage
  constexpr int STAGE = 2 * kPT * 128;     // bytes: point rows, then W^T rows
  __shared__ __align__(16) uint8_t pst0[STAGE];
  __shared__ __align__(16) uint8_t pst1[STAGE];
  __shared__ __align__(16) float msh[kProjMaxD + 32];
  // workgroup ids, tiles and bases are wave-uniform: computed in 32 bits and
  // pinned to scalar registers (the copies take their bases there)
  const int b = (int)blockIdx.x;
  const int group = __builtin_amdgcn_readfirstlane(b / (8 * n_otiles));  // 8 point tiles per group
  const int rem = __builtin_amdgcn_readfirstlane(b % (8 * n_otiles));
  const int ptile = group * 8 + rem % 8;
  const int otile = rem / 8;
  if (ptile >= n_ptiles) return;  // whole workgroup, before any barrier
  if (route && route->ok && !tflag[ptile]) return;  // done on the fp16 matrix cores
  const int64_t p0 = (int64_t)ptile * kPT;
  const int o0 = otile * kPT;
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int r = lane & 31, h = lane >> 5;
  const int wc = wave & 1, wp = wave >> 1;  // 128-point half, 64-output quarter
  const int prmax = (int)min<int64_t>(n - 1 - p0, kPT - 1);
  const int ormax = min(d_out - 1 - o0, kPT - 1);
  const int S = (d + 31) / 32;
  for (int i = t; i < 32 * S; i += 512) msh[i] = i < d ? mean[i] : 0.f;
  const float *xbase = X + p0 * ldx;
  const float *wbase = Wt + (int64_t)o0 * d;

  // copy i of a wave fills slots (8 i + wave) 64 .. + 63: rows 0 .. 255 are points,
  // rows 256 .. 511 rows of W^T; byte offsets from the stage's first dim
  uint32_t soff[NCOPY];
#pragma unroll
  for (int i = 0; i < NCOPY; ++i) {
    const int slot = (i * 8 + wave) * 64 + lane;
    const int row = slot >> 3;
    const int chunk = (slot & 7) ^ ((row >> 1) & 7);
    soff[i] = i < NCP ? (uint32_t)(min(row, prmax) * (int)ldx * 4 + 16 * chunk)
                      : (uint32_t)(min(row - kPT, ormax) * d * 4 + 16 * chunk);
  }
  auto copy = [&](int st, uint8_t *dst, int i) {
    const int slot = (i * 8 + wave) * 64 + lane;
    const int row = slot >> 3;
    const int chunk = (slot & 7) ^ ((row >> 1) & 7);
    lds_u8 *w = (lds_u8 *)dst + (i * 8 + wave) * 1024;
    // the stage's first dim of the points or of W^T, pinned to scalar registers
    const float *src = (i < NCP ? xbase : wbase) + 32 * st;
    const uint64_t su = (uint64_t)(size_t)src;
    const void *base = (const void *)(size_t)(((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(su >> 32)) << 32) |
                                              (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)su));
    if (32 * st + 4 * chunk < d) {
      lds_copy16(base, soff[i], (uint32_t)(size_t)w);
    } else {
      __attribute__((address_space(3))) uint32_t *z = (__attribute__((address_space(3))) uint32_t *)(w + 16 * lane);
      z[0] = z[1] = z[2] = z[3] = 0u;
    }
  };
  auto land = [&]() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };

  f32x16 acc[4][2];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[a][c][v] = 0.f;
  // one stage: four steps of 8 dims; the operand reads of step g + 1 and two of
  // the next stage's copies go out before step g's MFMAs
  auto mfma_stage = [&](int st, const uint8_t *buf, bool copying, uint8_t *nxt) {
    f32x4 av[2][4], bv[2][2];
    auto read = [&](int g, int set) {
      const int so = 16 * ((2 * g + h) ^ ((r >> 1) & 7));
      const f32x4 m4 = *reinterpret_cast<const f32x4 *>(&msh[32 * st + 8 * g + 4 * h]);
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
        av[set][cb] = *reinterpret_cast<const f32x4 *>(buf + (wc * 128 + cb * 32 + r) * 128 + so) - m4;
#pragma unroll
      for (int pb = 0; pb < 2; ++pb)
        bv[set][pb] = *reinterpret_cast<const f32x4 *>(buf + (kPT + wp * 64 + pb * 32 + r) * 128 + so);
    };
    read(0, 0);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int cur = g & 1;
      if (g + 1 < 4) read(g + 1, cur ^ 1);
      __builtin_amdgcn_sched_barrier(0);
      if (copying) {
        copy(st + 1, nxt, 2 * g);
        copy(st + 1, nxt, 2 * g + 1);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
          for (int pb = 0; pb < 2; ++pb)
            acc[cb][pb] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[cur][cb][e], bv[cur][pb][e], acc[cb][pb], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

#pragma unroll
  for (int i = 0; i < NCOPY; ++i) copy(0, pst0, i);
  land();
  __syncthreads();  // also publishes the mean
  for (int st = 0; st < S; ++st) {
    const bool nxt = st + 1 < S;
    mfma_stage(st, (st & 1) ? pst1 : pst0, nxt, (st & 1) ? pst0 : pst1);
    if (nxt) land();
    __syncthreads();
  }
  // lane (r, h) of block (cb, pb) holds points wc 128 + cb 32 + 8 i4 + 4 h + e of
  // output wp 64 + pb 32 + r
#pragma unroll
  for (int cb = 0; cb < 4; ++cb)
#pragma unroll
    for (int pb = 0; pb < 2; ++pb) {
      const int o = o0 + wp * 64 + pb * 32 + r;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int64_t p = p0 + wc * 128 + cb * 32 + 8 * (v >> 2) + 4 * h + (v & 3);
        if (p < n && o < d_out) Y[p * d_out + o] = acc[cb][pb][v];
      }
    }
}

// One covariance workgroup fills a CU (LDS), so the number of (tile, split)
// workgroups is kept just under a whole number of passes over the CUs.
CovPlan cov_plan(int64_t n, int d) {
  CovPlan p;
  p.T = (int)cdiv(d, kCT);
  p.ntiles = p.T * (p.T + 1) / 2;
  const int cus = cu_count();
  int want = std::max(1, (2 * cus) / p.ntiles);
  if (want * p.ntiles < cus) want = std::max(1, cus / p.ntiles);
  want = (int)std::min<int64_t>(want, std::max<int64_t>(1, cdiv(n, 4096)));
  p.rows_per_split = cdiv(n, want);
  p.nsplit = (int)cdiv(n, p.rows_per_split);
  return p;
}

}  // namespace

int cu_count() {
  static int cus = 0;
  if (cus == 0) {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
        v > 0)
      cus = v;
    else
      cus = 256;
  }
  return cus;
}

// workspace: the partial tiles, and before them the column sums and ranges in their place |
// the columns' largest |x - mean|
static size_t cov_partial_bytes(int64_t n, int d) {
  const CovPlan p = cov_plan(n, d);
  return (std::max((size_t)p.nsplit * p.ntiles * kCT * kCT * sizeof(double), colmean_bytes(n, d, true)) + 255) &
         ~(size_t)255;
}

size_t pca_cov_bytes(int64_t n, int d) { return cov_partial_bytes(n, d) + 4 * (size_t)d; }

km_status launch_pca_cov(const float *X, int64_t n, int d, float *mean, float *cov, void *ws, hipStream_t s) {
  const CovPlan p = cov_plan(n, d);
  double *partial = static_cast<double *>(ws);
  float *top = reinterpret_cast<float *>(static_cast<uint8_t *>(ws) + cov_partial_bytes(n, d));
  km_status st = launch_colmean(X, n, d, d, mean, ws, s, top);
  if (st != KM_OK) return st;
  hipLaunchKernelGGL(cov_kernel, dim3((unsigned)(8 * cdiv(p.ntiles * p.nsplit, 8))), dim3(kCovThreads), 0, s, X, n, d,
                     mean, top, p.T, p.ntiles, p.nsplit, p.rows_per_split, partial);
  hipLaunchKernelGGL(cov_reduce_kernel, dim3(p.ntiles, kCT * kCT / 256), dim3(256), 0, s, partial, p.ntiles, p.nsplit, p.T, d, n,
                     top, cov);
  KMQ_LAUNCH_CHECK("pca_fit_cov");
  return KM_OK;
}

// The fp16 matrix cores can take the rows whose 256 span less than 2 GB (as the fp32
// kernel's do), from two stages of 16 dims on.  They cost three launches more, 13 us of a
// call shorter than that, so a CU's chain of 256 x 256 tiles and stages of 32 dims has to be long
// enough, and where the outputs bound a pass (tiles of 256, 32 or 64 dims) they gain nothing.
// us per call, fp32 kernel first: to 16 outputs 50k x 64 (two stages) 33 / 47, 100k x 64 (four) 51 / 47,
// 1000 x 160 (five) 53 / 48, 1M x 64 (32) 345 / 198; to 256 outputs 100k x 64 (four) 59 / 71, 100k x 96 (six)
// 76 / 78, 20k x 128 (four) 49 / 51, 1000 x 192 (six, one tile) 62 / 52, 100k x 128 (eight) 92 / 82, 1M x 64
// 437 / 460, 1M x 48 452 / 427.
bool project_split(int64_t n, int d, int d_out, int64_t ldx) {
  if (d < 32 || d > kSplitProjMaxD || ldx % 4 != 0 || (int64_t)kPT * ldx * 4 >= ((int64_t)1 << 31)) return false;
  const int64_t rounds = cdiv(cdiv(n, kPT) * cdiv(d_out, kPT), cu_count()), chain = rounds * cdiv(d, 32);
  if (d_out <= 128) return chain >= 4 && (d > 32 || d_out <= 64);
  const int64_t steps = cdiv(d, 16);
  return chain >= (rounds == 1 ? 5 : 8) && steps != 2 && steps != 4;
}

size_t pca_project_bytes(int64_t n, int d, int d_out, bool split) {
  return (((size_t)d * d_out * sizeof(float) + 255) & ~(size_t)255) + 256 + (split ? split_project_bytes(n, d, d_out) : 0);
}

km_status launch_pca_project(const float *X, int64_t n, int d, int64_t ldx, const float *mean, const float *W,
                             int d_out, float *Y, void *ws, bool split, hipStream_t s) {
  float *Wt = static_cast<float *>(ws);
  const int64_t e = (int64_t)d * d_out;
  hipLaunchKernelGGL(transpose_kernel, dim3((unsigned)cdiv(e, 256)), dim3(256), 0, s, W, d, d_out, Wt);
  if (d <= kProjMaxD && ldx % 4 == 0 && (int64_t)kPT * ldx * 4 < ((int64_t)1 << 31)) {
    const int n_ptiles = (int)cdiv(n, kPT), n_otiles = (int)cdiv(d_out, kPT);
    const int64_t nblk = cdiv(n_ptiles, 8) * 8 * n_otiles;
    SplitPrep sp{};
    if (split) {
      uint8_t *w = static_cast<uint8_t *>(ws) + ((e * sizeof(float) + 255) & ~(size_t)255);
      const km_status st = launch_split_project(X, n, d, ldx, mean, W, d_out, Y, w, &sp, s);
      if (st != KM_OK) return st;
    }
    hipLaunchKernelGGL(project_kernel, dim3((unsigned)nblk), dim3(512), 0, s, X, n, d, ldx, mean, Wt, d_out, Y,
                       n_ptiles, n_otiles, sp.route, sp.tflag);
  } else {
    const int n_ptiles = (int)cdiv(n, kT), n_otiles = (int)cdiv(d_out, kT);
    const int64_t nblk = cdiv(n_ptiles, 8) * 8 * n_otiles;
    hipLaunchKernelGGL(project_staged_kernel, dim3((unsigned)nblk), dim3(256), 0, s, X, n, d, ldx, mean, Wt, d_out,
                       Y, n_ptiles, n_otiles);
  }
  KMQ_LAUNCH_CHECK("pca_project");
  return KM_OK;
}

}  // namespace kmq
