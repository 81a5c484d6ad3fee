// STEP 2 for few fp32 points and centroids, on the fp16 matrix cores (split.hpp).
#include <float.h>
#include <limits.h>

#include <algorithm>
#include <type_traits>

#include "split.hpp"

namespace kmq {
namespace {

constexpr int kSmallT = 64;    // points and centroids of a tile
constexpr int kSmallThr = 512;  // 8 waves
constexpr int kSmallRing = 4;   // stage buffers

// ||c||^2 and the largest |c| of every centroid, one wave each, and the start of the keys.
__global__ __launch_bounds__(256) void small_prep_kernel(const float *C, int k, int d, float *cn, uint32_t *rmax,
                                                         unsigned long long *keys, int64_t n, int *count,
                                                         int64_t npt) {
  const int64_t g0 = (int64_t)blockIdx.x * 256 + threadIdx.x, gs = (int64_t)gridDim.x * 256;
  if (keys) {
    for (int64_t i = g0; i < n; i += gs) keys[i] = ~0ull;
    for (int64_t i = g0; i < npt; i += gs) count[i] = 0;
  }
  const int lane = threadIdx.x & 63;
  const int j = (int)(g0 >> 6);
  if (j >= k) return;
  const float *c = C + (int64_t)j * d;
  double s = 0.0;
  uint32_t mx = 0;
  for (int i = 4 * lane; i < d; i += 256) {  // d % 4 == 0
    const f32x4 v = *reinterpret_cast<const f32x4 *>(c + i);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s += (double)v[e] * (double)v[e];
      mx = max(mx, __float_as_uint(v[e]) & 0x7fffffffu);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    s += __shfl_xor(s, off);
    mx = max(mx, (uint32_t)__shfl_xor((int)mx, off));
  }
  if (lane == 0) {
    cn[j] = (float)s;
    rmax[j] = mx;
  }
}

// One tile of 64 points x 64 centroids per workgroup: with few tiles the time is what one
// workgroup takes, so the tile is a quarter of split_kernel's side and 8 waves share it: 2 x
// 2 blocks of 32 x 32, two waves per block, one for the even 16 dims of a stage, one for
// the odd (their sums meet at the end).  Stages are 32 floats of every row, points and
// centroids alike, straight into LDS (16-byte chunk c of row R in slot c ^ ((R >> 1) & 7)),
// two multiplied between barriers while the next two are copied; 66 KB, so that two
// workgroups share a CU where there are that many.  Both operands are split as they are
// read, which saves the launch that would make the centroids' image.  The scale is the
// tile's own: the rule of split_prep_kernel on its 64 rows.  What the parts do not hold
// (that rule, or a point without a score that is a number) the workgroup does again with
// fp32 MFMA from the same stages.  With several centroid tiles the points' (score, index)
// keys meet in an atomic, and the last workgroup of a point tile writes the results.
//
// What bounds it is the chain of one tile (768 dims: 12 barriers, each with the copies'
// latency behind it), not a rate.  A pass with its preparation, against split_kernel with
// its: 1024 x 768, k = 1000 66 -> 21 us; 1 x 768, k = 1000 65 -> 17; 20k x 128, k = 64 18.2 -> 10.8.
// One stage per barrier took 21 us instead of 17 (one point), a ring of 8 buffers 18.
__global__ __launch_bounds__(kSmallThr) void assign_small_kernel(SmallArgs A) {
  constexpr int STAGE = 2 * kSmallT * 128;  // centroid rows, then point rows
  __shared__ __align__(16) uint8_t ring[kSmallRing * STAGE];
  __shared__ float msc[kSmallT];
  __shared__ int mix[kSmallT];
  __shared__ int last;
  const int t = threadIdx.x;
  const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int r = lane & 31, h = lane >> 5;
  const int wc = wave & 1, wp = (wave >> 1) & 1, kh = wave >> 2;
  const int pt = (int)(blockIdx.x % (unsigned)A.n_ptiles), g = (int)(blockIdx.x / (unsigned)A.n_ptiles);
  const int64_t p0 = (int64_t)pt * kSmallT;
  const int c0 = g * kSmallT;
  const int prmax = (int)min<int64_t>(A.n - 1 - p0, kSmallT - 1), crmax = min(A.k - 1 - c0, kSmallT - 1);
  const int S = (A.d + 31) / 32;
  const float *xbase = A.x + p0 * A.ldx, *cbase = A.C + (int64_t)c0 * A.d;

  // the tile's scale: 2^7 <= s max|c| < 2^8, and max|c| <= 2^8 ||c|| for every row but zero ones
  bool ok;
  float s;
  {
    const int j = c0 + min(lane, crmax);
    uint32_t m = A.rmax[j];
    const float c = A.cn[j];
    float lo = c != 0.f ? c : FLT_MAX;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      m = max(m, (uint32_t)__shfl_xor((int)m, off));
      lo = fminf(lo, __shfl_xor(lo, off));
    }
    const int e = (int)(m >> 23) - 127;
    ok = e >= -50 && e <= 50 && lo >= ldexpf(1.0f, 2 * e - 16);
    s = ldexpf(1.0f, 7 - (ok ? e : 0));
  }

  // a wave copies 8 rows of the centroids and 8 of the points per stage
  const int crow = wave * 8 + (lane >> 3);
  const int chunk = (lane & 7) ^ ((crow >> 1) & 7);
  const uint32_t co = (uint32_t)min(crow, crmax) * (uint32_t)A.d * 4u + 16u * chunk;
  const uint32_t xo = (uint32_t)min(crow, prmax) * (uint32_t)A.ldx * 4u + 16u * chunk;
  const uint32_t ring0 = (uint32_t)(size_t)(lds_byte *)ring;
  auto copy = [&](int st) {
    const uint32_t b = (uint32_t)(st & (kSmallRing - 1)) * STAGE + wave * 1024;
    if (32 * st + 4 * chunk < A.d) {  // true for some lane of every wave: two copies each
      lds_copy16_at(cbase + 32 * st, co, ring0 + b);
      lds_copy16_at(xbase + 32 * st, xo, ring0 + b + kSmallT * 128);
    } else {  // chunks past the last dim hold zeros
      *reinterpret_cast<uint4 *>(ring + b + 16 * lane) = uint4{0u, 0u, 0u, 0u};
      *reinterpret_cast<uint4 *>(ring + b + kSmallT * 128 + 16 * lane) = uint4{0u, 0u, 0u, 0u};
    }
  };
  const uint32_t crd = (uint32_t)((wc * 32 + r) * 128), xrd = (uint32_t)((kSmallT + wp * 32 + r) * 128);
  const uint32_t kx = (uint32_t)((r >> 1) & 7);

  f32x16 acc;
  float best;
  int bidx;
  auto run = [&](auto split_c) {
    constexpr bool SPLIT = decltype(split_c)::value;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    auto mul = [&](int st) {
      const uint8_t *b = ring + (st & (kSmallRing - 1)) * STAGE;
      if constexpr (SPLIT) {  // this wave's 16 dims, 8 per lane half
        f32x4 cv[2], xv[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const uint32_t o = 16u * ((uint32_t)(4 * kh + 2 * h + q) ^ kx);
          cv[q] = *reinterpret_cast<const f32x4 *>(b + crd + o);
          xv[q] = *reinterpret_cast<const f32x4 *>(b + xrd + o);
        }
        uint32_t ch[4], cl[4], xh[4], xl[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          split2(cv[q >> 1][2 * (q & 1)], cv[q >> 1][2 * (q & 1) + 1], s, ch[q], cl[q]);
          split2(xv[q >> 1][2 * (q & 1)], xv[q >> 1][2 * (q & 1) + 1], s, xh[q], xl[q]);
        }
        auto v8 = [](const uint32_t *u) {
          return __builtin_bit_cast(h16x8, i32x4{(int)u[0], (int)u[1], (int)u[2], (int)u[3]});
        };
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(v8(cl), v8(xh), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(v8(ch), v8(xl), acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(v8(ch), v8(xh), acc, 0, 0, 0);
      } else {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const uint32_t o = 16u * ((uint32_t)(4 * kh + 2 * q + h) ^ kx);
          const f32x4 cv = *reinterpret_cast<const f32x4 *>(b + crd + o);
          const f32x4 xv = *reinterpret_cast<const f32x4 *>(b + xrd + o);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(cv[e], xv[e], acc, 0, 0, 0);
        }
      }
    };
    // stages st and st + 1 have landed, for all waves, and all have read the two before
    auto step_begin = [&]() {
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    };
    copy(0);
    if (S > 1) copy(1);
    int st = 0;
    for (; st + 1 < S; st += 2) {
      step_begin();
      if (st + 2 < S) copy(st + 2);
      if (st + 3 < S) copy(st + 3);
      mul(st);
      mul(st + 1);
    }
    if (st < S) {
      step_begin();
      mul(st);
    }
    __syncthreads();
    // the odd dims' sums to the wave with the even ones, 4 KB per block
    float *sums = reinterpret_cast<float *>(ring) + (wave & 3) * 1024;
    if (kh == 1) {
#pragma unroll
      for (int i = 0; i < 16; ++i) sums[i * 64 + lane] = acc[i];
    }
    __syncthreads();
    best = INFINITY;
    bidx = INT_MAX;
    if (kh == 0) {
      const float m2 = SPLIT ? -2.0f / (s * s) : -2.0f;
      const int j0 = c0 + wc * 32 + 4 * h;
#pragma unroll
      for (int i = 0; i < 16; ++i) {  // rows ascend with i: the strict comparison keeps the smallest index
        const int j = j0 + 8 * (i >> 2) + (i & 3);
        const float cn = j < A.k ? A.cn[j] : INFINITY;
        const float sc = fmaf(m2, acc[i] + sums[i * 64 + lane], cn);
        const bool take = sc < best;
        best = take ? sc : best;
        bidx = take ? j : bidx;
      }
      auto merge = [&](float os, int oi) {
        if (os < best || (os == best && oi < bidx)) {
          best = os;
          bidx = oi;
        }
      };
      merge(__shfl_xor(best, 32), __shfl_xor(bidx, 32));
      if (wc == 1 && h == 0) {
        msc[wp * 32 + r] = best;
        mix[wp * 32 + r] = bidx;
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    __syncthreads();
    if (kh == 0 && wc == 0) {
      const float os = msc[wp * 32 + r];
      const int oi = mix[wp * 32 + r];
      if (os < best || (os == best && oi < bidx)) {
        best = os;
        bidx = oi;
      }
    }
    __syncthreads();
  };
  const bool owner = kh == 0 && wc == 0 && h == 0;  // lanes with a point's result
  bool redo = !ok;
  if (ok) {
    run(std::true_type{});
    redo = __syncthreads_or(owner && bidx == INT_MAX);  // only NaN scores
  }
  if (redo) run(std::false_type{});

  const int64_t p = p0 + wp * 32 + r;
  if (A.ngroups == 1) {
    if (owner && p < A.n) {
      A.assign[p] = bidx + A.aoff;
      if (A.score) A.score[p] = best;
    }
    return;
  }
  // The keys and the count are only touched by atomics at device scope, and the keys' have
  // returned before the count's goes out: no cache needs writing back (a fence that does, in
  // every workgroup, took most of this kernel's time).
  if (owner && p < A.n) {
    unsigned long long old =
        __hip_atomic_fetch_min(A.keys + p, split_key(best, bidx), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" : "+v"(old)::"memory");
  }
  __syncthreads();
  if (t == 0)
    last = __hip_atomic_fetch_add(A.count + pt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == A.ngroups - 1;
  __syncthreads();
  if (!last) return;
  if (owner && p < A.n) {
    const unsigned long long key = __hip_atomic_load(A.keys + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    A.assign[p] = (int32_t)(uint32_t)key + A.aoff;
    if (A.score) {
      const uint32_t u = (uint32_t)(key >> 32);
      A.score[p] = __uint_as_float((u & 0x80000000u) ? u & 0x7fffffffu : ~u);
    }
  }
}

}  // namespace

// Up to 4 tiles per CU, where the workgroups still run at once or nearly so; beyond,
// split_kernel's 256 x 256 tiles move a quarter of the bytes per product.  At 768 dims and
// 1000 centroids, split_kernel against this: 512 tiles 66 / 27 us, 1024 tiles 66 / 45, 2048 tiles 67 / 82; at
// 128 dims 1024 tiles (64 centroids) 20.2 / 15.1, 2500 tiles (256 centroids, 64 dims) 19.3 / 29.4.
bool split_small(int64_t n, int k) {
  return cdiv(n, kSmallT) * cdiv(k, kSmallT) <= 4 * cu_count();
}

size_t split_small_bytes(int64_t n, int k) {
  auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
  return al(4 * (size_t)k) + al(8 * (size_t)n) + al(4 * (size_t)cdiv(n, kSmallT));
}

km_status launch_split_small_prep(const float *C, int64_t n, int k, int d, float *cn, void *ws, SplitPrep *out,
                                  hipStream_t s) {
  auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
  uint8_t *w = static_cast<uint8_t *>(ws);
  *out = SplitPrep{};
  out->rmax = reinterpret_cast<uint32_t *>(w);
  w += al(4 * (size_t)k);
  out->keys = reinterpret_cast<unsigned long long *>(w);
  w += al(8 * (size_t)n);
  out->tflag = reinterpret_cast<int *>(w);  // workgroups of a point tile that have ended
  hipLaunchKernelGGL(small_prep_kernel, dim3((unsigned)cdiv(k, 4)), dim3(256), 0, s, C, k, d, cn, out->rmax,
                     k > kSmallT ? out->keys : nullptr, n, out->tflag, cdiv(n, kSmallT));
  KMQ_LAUNCH_CHECK("small_prep_kernel");
  return KM_OK;
}

km_status launch_split_small(const float *X, int64_t ldx, const float *C, const CentroidPrep &cp, int64_t n, int k,
                             int d, int32_t *assign, float *score, int aoff, hipStream_t s) {
  SmallArgs A{};
  A.x = X;
  A.ldx = ldx;
  A.C = C;
  A.cn = cp.cn;
  A.rmax = cp.sp.rmax;
  A.n = n;
  A.k = k;
  A.d = d;
  A.ngroups = (int)cdiv(k, kSmallT);
  A.n_ptiles = cdiv(n, kSmallT);
  A.keys = cp.sp.keys;
  A.count = cp.sp.tflag;
  A.assign = assign;
  A.score = score;
  A.aoff = aoff;
  hipLaunchKernelGGL(assign_small_kernel, dim3((unsigned)(A.n_ptiles * A.ngroups)), dim3(kSmallThr), 0, s, A);
  KMQ_LAUNCH_CHECK("assign_small_kernel");
  return KM_OK;
}

}  // namespace kmq
