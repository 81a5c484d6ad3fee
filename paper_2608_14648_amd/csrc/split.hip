// STEP 2 for fp32 points on the fp16 matrix cores (split.hpp), and the preparation
// of the centroids for it.
#include <float.h>
#include <limits.h>

#include <algorithm>
#include <type_traits>

#include "split.hpp"

namespace kmq {
namespace {

constexpr int kTP = 256;       // points per workgroup
constexpr int kThr = 512;      // 8 waves
constexpr int kSD = 16;        // dims per stage
constexpr int kRow = 4 * kSD;  // bytes of a row per stage: 16 floats, or 16 hi then 16 lo halves
constexpr int kRing = 4;       // stage buffers
constexpr int kSeedPad = 256;  // -inf seeds past the last centroid

// ---- centroid preparation ------------------------------------------------------
// From every row's largest |c| (bit pattern) and ||c||^2: the common scale, whether
// the split holds for these centroids, the split image and the accumulator seeds.
// Each workgroup reads all k maxima itself (k floats from L2): the launch that
// would reduce them first costs more.
//
// The scale puts the largest |c| of all centroids at [2^7, 2^8): every coordinate is
// held to 2^-32 of that maximum or 2^-23 of itself, and points up to 2^7 times larger
// always stay below fp16's 65504, up to 2^8 times larger mostly (what does not, infinities
// and NaN give NaN scores, which flag their tile for the fp32 kernel).  The absolute part
// stays at the fp32 rounding of ||c||^2 (2^-24 of it) as long as no centroid is tiny beside
// that maximum: ||c|| >= 2^-8 max|c| is asked of every centroid (or ||c|| = 0, whose products
// are exact).  Centroids with NaN or infinities, or so large or small that the
// scale's square leaves fp32's range, take the fp32 kernel as well.
__global__ __launch_bounds__(256) void split_prep_kernel(const float *C, int64_t ldc, int k, int d,
                                                         const uint32_t *rmax, const float *cn, const int *qsum,
                                                         const float *u, const float *sig2, SplitPrep sp,
                                                         int64_t ntflag) {
  __shared__ uint32_t shm[256];
  __shared__ float shn[256];
  const int t = threadIdx.x;
  uint32_t m = 0;
  float lo = FLT_MAX;
  for (int j = t; j < k; j += 256) {
    m = max(m, rmax[j]);
    const float c = cn[j];
    if (c != 0.f) lo = fminf(lo, c);
  }
  shm[t] = m;
  shn[t] = lo;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (t < st) {
      shm[t] = max(shm[t], shm[t + st]);
      shn[t] = fminf(shn[t], shn[t + st]);
    }
    __syncthreads();
  }
  m = shm[0];
  lo = shn[0];
  const int e = (int)(m >> 23) - 127;
  const bool ok = e >= -50 && e <= 50 && lo >= ldexpf(1.0f, 2 * e - 16);
  const float sc = ldexpf(1.0f, 7 - (ok ? e : 0));
  const int64_t g0 = (int64_t)blockIdx.x * 256 + t, gs = (int64_t)gridDim.x * 256;
  if (g0 == 0) *sp.route = SplitRoute{ok ? 1 : 0, sc, -2.0f / (sc * sc), 0};
  for (int64_t i = g0; i < ntflag; i += gs) sp.tflag[i] = 0;
  if (!ok) return;
  for (int64_t j = g0; j < (int64_t)k + kSeedPad; j += gs) sp.seed[j] = j < k ? cn[j] * (-0.5f * sc * sc) : -INFINITY;
  if (sp.tail) {  // hybrid: -T, and u and 2 sigma times the factor that makes tail scores seeds
    const int64_t kp = k + kSeedPad;
    for (int64_t j = g0; j < kp; j += gs) {
      const bool in = j < k;
      sp.tail[j] = in ? __int_as_float(-qsum[j]) : 0.f;
      sp.tail[kp + j] = in ? u[j] * (-0.5f * sc * sc) : 0.f;
      sp.tail[2 * kp + j] = in ? sig2[j] * (-0.5f * sc * sc) : 0.f;
    }
  }
  // the rows read past the last one are finite (a NaN would flag tiles)
  const int ch = 2 * ((d + kSD - 1) / kSD);
  for (int64_t i = g0; i < 256 * kRow / 16; i += gs)
    *reinterpret_cast<uint4 *>(sp.img + (int64_t)(ch / 2) * sp.cstage + 16 * i) = uint4{0u, 0u, 0u, 0u};
  // one unit: 8 dims of one row
  const int64_t units = (int64_t)k * ch;
  for (int64_t u = g0; u < units; u += gs) {
    const int64_t row = u / ch;
    const int c = (int)(u - row * ch);
    const float *src = C + row * ldc + 8 * c;
    f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = a;
    if (8 * c < d) a = *reinterpret_cast<const f32x4 *>(src);  // d % 4 == 0
    if (8 * c + 4 < d) b = *reinterpret_cast<const f32x4 *>(src + 4);
    uint32_t hi[4], lo[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      split2(q < 2 ? a[2 * q] : b[2 * q - 4], q < 2 ? a[2 * q + 1] : b[2 * q - 3], sc, hi[q], lo[q]);
    uint8_t *dst = sp.img + (int64_t)(c >> 1) * sp.cstage + row * kRow + 16 * (c & 1);
    *reinterpret_cast<uint4 *>(dst) = uint4{hi[0], hi[1], hi[2], hi[3]};
    *reinterpret_cast<uint4 *>(dst + 32) = uint4{lo[0], lo[1], lo[2], lo[3]};
  }
}

// ---- projection: scales and the image of W ------------------------------------------
// Every dim's largest |x - mean| over 1024 rows spread over X, as a bit pattern (NaN and
// infinities are the largest): 16 dims per workgroup, 4 per thread of 4 rows, all loads in
// flight at once.
__global__ __launch_bounds__(1024) void proj_sample_kernel(const float *X, int64_t n, int d, int64_t ldx,
                                                           const float *mean, uint32_t *top, SplitRoute *route) {
  __shared__ uint32_t sh[16][16];
  const int t = threadIdx.x;
  const int c = blockIdx.x * 16 + 4 * (t & 3);
  const int rows = (int)min<int64_t>(n, 1024);
  uint32_t m[4] = {0u, 0u, 0u, 0u};
  if (c < d) {  // d % 4 == 0
    const f32x4 mc = *reinterpret_cast<const f32x4 *>(mean + c);
    f32x4 v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = min((t >> 2) + 256 * q, rows - 1);
      v[q] = *reinterpret_cast<const f32x4 *>(X + (int64_t)((double)i * (double)n / rows) * ldx + c);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) m[e] = max(m[e], __float_as_uint(v[q][e] - mc[e]) & 0x7fffffffu);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
#pragma unroll
    for (int o = 4; o < 64; o <<= 1) m[e] = max(m[e], (uint32_t)__shfl_xor((int)m[e], o));
    if ((t & 63) < 4) sh[t >> 6][4 * (t & 3) + e] = m[e];
  }
  __syncthreads();
  if (t < 16 && (int)blockIdx.x * 16 + t < d) {
    uint32_t a = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) a = max(a, sh[w][t]);
    top[blockIdx.x * 16 + t] = a;
  }
  if (t == 0 && blockIdx.x == 0) route->ok = 1;
}

// 16 columns of W per workgroup: each column's own scale (its largest |w| at
// [2^7, 2^8)), its factor back to Y (in seed) and its rows of the image.  The points'
// scale puts the sample's largest |x - mean| at [2^11, 2^12): eight times more always fits.
// A sample or W with NaN or infinities, or past 2^+-50, leaves the call to the fp32
// kernel: the sample kernel sets the route's ok, whoever sees such a value clears it.
// So does a column that lives on dims far smaller than the largest, as the last
// directions of data whose dims have different units do.  The points are held to 2^-36
// of their largest value M and a column to 2^-32 of its largest weight w, whatever the
// dim; against the column's largest term |w_i| max|x_i| that is 2^-24 and less, an fp32
// product's own rounding, as long as this term is at least 2^-8 M w.
__global__ __launch_bounds__(256) void proj_prep_kernel(const float *W, int d, int d_out, const uint32_t *top,
                                                        SplitPrep sp, int64_t ntflag) {
  __shared__ uint32_t sh[256];
  __shared__ float shg[256];
  __shared__ float scl[16];
  const int t = threadIdx.x, o16 = t & 15, rg = t >> 4;
  const int o = blockIdx.x * 16 + o16;
  uint32_t mt = 0;
  for (int i = t; i < d; i += 256) mt = max(mt, top[i]);
  sh[t] = mt;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (t < st) sh[t] = max(sh[t], sh[t + st]);
    __syncthreads();
  }
  const float mx = __uint_as_float(sh[0]);
  const int ex = (int)(sh[0] >> 23) - 127;
  const bool okx = ex >= -50 && ex <= 50;
  const float sx = ldexpf(1.0f, 11 - (okx ? ex : 0));
  __syncthreads();
  uint32_t m = 0;
  float term = 0.f;
  if (o < d_out)
    for (int i = rg; i < d; i += 16) {
      const float w = fabsf(W[(int64_t)i * d_out + o]);
      m = max(m, __float_as_uint(w));
      term = fmaxf(term, w * __uint_as_float(top[i]));
    }
  sh[t] = m;
  shg[t] = term;
  __syncthreads();
  for (int st = 128; st >= 16; st >>= 1) {
    if (t < st) {
      sh[t] = max(sh[t], sh[t + st]);
      shg[t] = fmaxf(shg[t], shg[t + st]);
    }
    __syncthreads();
  }
  if (t < 16) {
    const int ew = (int)(sh[t] >> 23) - 127;
    const bool zero = sh[t] == 0u, okw = zero || (ew >= -50 && ew <= 50);
    const float s = ldexpf(1.0f, 7 - (zero || !okw ? 0 : ew));
    scl[t] = s;
    if (o < d_out) {
      sp.seed[o] = 1.0f / (s * sx);
      if (!okw || (!zero && shg[t] < 0x1p-8f * mx * __uint_as_float(sh[t]))) sp.route->ok = 0;
    }
  }
  const int64_t g0 = (int64_t)blockIdx.x * 256 + t, gs = (int64_t)gridDim.x * 256;
  if (g0 == 0) {
    sp.route->s = sx;
    if (!okx) sp.route->ok = 0;
  }
  for (int64_t i = g0; i < ntflag; i += gs) sp.tflag[i] = 0;
  __syncthreads();
  if (!okx) return;
  const int ch = 2 * ((d + kSD - 1) / kSD);
  for (int64_t i = g0; i < 256 * kRow / 16; i += gs)  // the rows read past the last one are finite
    *reinterpret_cast<uint4 *>(sp.img + (int64_t)(ch / 2) * sp.cstage + 16 * i) = uint4{0u, 0u, 0u, 0u};
  if (o >= d_out) return;
  const float s = scl[o16];
  for (int c = rg; c < ch; c += 16) {
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = 8 * c + i < d ? W[(int64_t)(8 * c + i) * d_out + o] : 0.f;
    uint32_t hi[4], lo[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) split2(v[2 * q], v[2 * q + 1], s, hi[q], lo[q]);
    uint8_t *dst = sp.img + (int64_t)(c >> 1) * sp.cstage + (int64_t)o * kRow + 16 * (c & 1);
    *reinterpret_cast<uint4 *>(dst) = uint4{hi[0], hi[1], hi[2], hi[3]};
    *reinterpret_cast<uint4 *>(dst + 32) = uint4{lo[0], lo[1], lo[2], lo[3]};
  }
}

// ---- assignment ------------------------------------------------------------------
// 8 waves, 256 points x TC = 64 CB centroids, each wave 32 CB x 64.  A stage is 16
// dims: of every point 16 floats, of every centroid 16 hi and 16 lo halves, both 64
// bytes, copied straight into LDS.  Two 32-row blocks share 128-byte LDS rows
// (block b's row r in half b & 1 of row r), 16-byte chunk c in slot c ^ ((r >> 1) & 7),
// the conflict-free order for 128-byte rows.  Points are split as they are read.
//
// Four buffers and one barrier per stage: step i multiplies stage i from registers
// while it reads stage i + 1 into them and the copies of stages i + 2 and i + 3 fly
// (stage i + 3 goes where stage i - 1 was, whose last reads were used in step i - 1).
// Within a step the points' first block is multiplied while the second is split,
// and the second while the first of the next stage is read and split and every
// centroid operand is replaced as it is used: nothing waits behind the barrier.  The
// largest of acc - s^2 ||c||^2 / 2 wins; the first block's argmax of a tile runs under
// the second block's MFMAs, the second's under the next tile's first.  (Starting the
// accumulators at -s^2 ||c||^2 / 2 would save an addition per pair, but then every
// partial sum rounds at that magnitude: points far from all centroids came out 5 times
// less exact.)
//
// Measured against the fp32 kernel: 10M x 256, k = 4096 158.9 -> 59.5 ms (352 TFLOP/s of
// fp32 products, 1057 of fp16 ones); 1M x 768, k = 1000 11.6 -> 4.1 ms (few tiles:
// split_small.hip).  What bounds it is power: on random data the chip runs this
// kernel at 1.6 - 1.8 GHz, and a large f16 library product reaches 1290 - 1310 TFLOP/s;
// with constant data (few bits toggling) the same pass at 2M points takes 8.9 instead
// of 11.8 ms.  The matrix cores are busy 56 % of the cycles.
//
// HYB (fp32 front dims plus 1-bit tail): a tile begins with stages of the tail, 128
// bytes of every centroid's int8 residual codes (32 KB for 256 centroids, as a front
// stage), multiplied with the points' bits, which stay in LDS for the whole workgroup,
// regrouped so that widening to {0, 2} bytes is a shift and a mask.  The accumulators
// start at -T and end at the exact 2D - T; in fp32, in the order of Eq. 4 that the
// oracle uses, that becomes the tail score ts = fmaf(-(alpha 2 sigma), 2D - T,
// sigma^2 Q), and -s^2 ts / 2 (the factor, a power of two, is in the constants) starts
// the front's accumulators.  2M points, front 384 + tail 640, k = 4096:
// 54.4 -> 22.5 ms per pass against the fp32 front (assign_hyb_kernel)
//
// PROJ (Y = (X - mean) W): the columns of W in the place of the centroids, points and
// centroids exchanged in the MFMA so that a lane holds one output of many points and
// the stores are coalesced; s (x - mean) is formed as the points are read, and the
// values go out with their column's scale instead of into an argmax.
// 2M x 1024 -> 256: 8.6 -> 3.5 ms against project_kernel (10.2 GB read and written:
// 2.1 ms at the rate of a large copy); 500k x 1024 x 1024 (RabitQ's rotation): 8.5 -> 3.4.
//
// PRUNE (the first test of a pruned pass, at d' dims): the threshold test of every pair,
// acc - s^2 ||c'||^2 / 2 < (||x'||^2 - tau r(d')) s^2 / 2 drops it, and a point's survivors as
// one bit per centroid.  1M points, d' = 96, k = 1000: 1.95 -> 0.75 ms against skm_front_kernel
// (0.56 ms of it products at the rate of the assignment; six steps a tile do not hide the
// epilogue that turns scores into bits).
template <int CB, int MODE>
__global__ __launch_bounds__(kThr, 1) void split_kernel(SplitArgs A) {
  constexpr bool HYB = MODE == kSplitHybrid, PROJ = MODE == kSplitProject, PRUNE = MODE == kSplitPrune;
  constexpr int TC = 64 * CB;
  constexpr int NCONST = HYB ? 4 : 1;  // constants per centroid: seed; -T, u, 2 sigma
  // Tiles of constants, and the stage of a tile that they are copied with.  A hybrid tile has 3 stages or more
  // and ends its argmax after its last barrier, so the next tile's first step may run while other waves still
  // read the seeds: the copies into their slot wait for that tile's second step or a later one.
  constexpr int CRING = HYB ? 2 : 4, CSTAGE = HYB ? 1 : 0;
  constexpr int NCC = CB / 2;  // centroid copies per wave and stage
  constexpr int CREG = TC * kRow, STAGE = CREG + kTP * kRow;
  if (!A.sp.route->ok) return;  // every workgroup: the fp32 kernel takes this call
  __shared__ __align__(16) uint8_t ring[kRing * STAGE];
  __shared__ __align__(16) float seeds[PROJ ? 1 : CRING][NCONST][PROJ ? 1 : TC];
  __shared__ __align__(16) float msh[PROJ ? kSplitProjMaxD + kSD : 1];  // s mean, 0 past d
  __shared__ uint32_t bitsT[HYB ? kSplitTailWords * kTP : 1];
  __shared__ float alp[HYB ? kTP : 1];
  __shared__ __align__(16) uint32_t mrow[PRUNE ? kTP : 1][TC / 32];  // PRUNE: a tile's mask words of every point
  const int t = threadIdx.x;
  const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int r = lane & 31, h = lane >> 5;
  const int wc = wave & 1, wp = wave >> 1;
  const int NG = A.ngroups;
  int64_t pt = blockIdx.x;
  int g = 0;
  if (NG > 1) {
    const int64_t l = blockIdx.x >> 3;
    pt = (l / NG) * 8 + (blockIdx.x & 7);
    g = (int)(l % NG);
    if (pt >= A.n_ptiles) return;  // whole workgroup, before any barrier
  }
  const int64_t p0 = pt * kTP;
  const int SI = HYB ? (A.di + 127) / 128 : 0;  // tail stages of a tile
  const int S = SI + (A.d + kSD - 1) / kSD;     // all its stages
  const bool ragged = A.d % kSD != 0;
  const int nct = (A.k + TC - 1) / TC;
  const int nmy = (nct - g + NG - 1) / NG;
  const int prmax = (int)min<int64_t>(A.n - 1 - p0, kTP - 1);
  const float sx = A.sp.route->s;
  const float *pbase = A.x + p0 * A.ldx;

  // copy j of a region fills its slots 64 j .. 64 j + 63; wave w makes copies w and
  // w + 8 of the points, and w (and w + 8 for CB = 4) of the centroids.  Copy w + 8
  // lies 128 rows further on.
  uint32_t xoff[2], coff;
  int xchunk;
  {
    const int slot = wave * 64 + lane;
    const int sr = (slot >> 3) & 31, c8 = (slot & 7) ^ ((sr >> 1) & 7);
    const int row = ((slot >> 8) * 2 + (c8 >> 2)) * 32 + sr;
    xchunk = c8 & 3;
    coff = (uint32_t)(row * kRow + 16 * xchunk);
    xoff[0] = (uint32_t)(min(row, prmax) * (int)A.ldx * 4 + 16 * xchunk);
    xoff[1] = (uint32_t)(min(row + 128, prmax) * (int)A.ldx * 4 + 16 * xchunk);
  }
  const uint32_t ring0 = (uint32_t)(size_t)(lds_byte *)ring;
  const uint32_t seeds0 = (uint32_t)(size_t)(lds_byte *)seeds;
  // hybrid: resident tail bits, word-major and regrouped; words past the tail up to the
  // last stage's end are zero (so are their products with whatever codes are there)
  if constexpr (HYB) {
    const int TW = A.di / 32;
    for (int e = t; e < 4 * SI * kTP; e += kThr) {
      const int w = e / kTP, pp = e - w * kTP;
      uint32_t v = 0u;
      if (w < TW) v = regroup_bits(A.pbits[(p0 + min(pp, prmax)) * A.pbw + A.pbw0 + w]);
      bitsT[w * kTP + pp] = v;
    }
    if (t < kTP) alp[t] = A.alpha[p0 + min(t, prmax)];
  }
  if constexpr (PROJ) {
    for (int i = t; i < kSD * S + kSD; i += kThr) msh[i] = i < A.d ? A.mean[i] * sx : 0.f;
  }
  int kc_s = 0, kc_t = 0;  // stage (dims) and tile of the next copy
  uint32_t kbuf = 0;       // its buffer's offset
  // the copies of one stage: NCC + 2, and the tile's constants with its stage CSTAGE
  auto copy_stage = [&]() {
    const int c0 = (g + kc_t * NG) * TC;
    const uint32_t l0 = ring0 + kbuf + wave * 1024;
    if (HYB && kc_s < SI) {  // rows of codes as 128-byte LDS rows, chunk c in slot c ^ ((row >> 1) & 7)
      const int crmax = A.k - 1 - c0;
#pragma unroll
      for (int i = 0; i < NCC + 2; ++i) {
        const int ii = i % CB;  // CB = 2: the third copy is the first again (all stages have as many)
        const int row = (ii * 8 + wave) * 8 + (lane >> 3);
        const int b = 128 * kc_s + 16 * ((lane & 7) ^ ((row >> 1) & 7));
        lds_copy16_at(A.ci8 + (int64_t)c0 * A.cild, (uint32_t)(min(row, crmax) * (int)A.cild + (b < A.di ? b : 0)),
                      l0 + 8192u * ii);
      }
    } else {
      const int fs = kc_s - SI;
      const uint8_t *cb = A.sp.img + (int64_t)fs * A.sp.cstage + (int64_t)c0 * kRow;
      const float *xb = pbase + kSD * fs;
#pragma unroll
      for (int i = 0; i < NCC; ++i) lds_copy16_at(cb, coff + 8192u * i, l0 + 8192u * i);
      if (ragged && kc_s == S - 1) {  // chunks past the last dim hold zeros
        const bool in = kSD * fs + 4 * xchunk < A.d;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          if (in) {
            lds_copy16_at(xb, xoff[i], l0 + CREG + 8192u * i);
          } else {
            *reinterpret_cast<uint4 *>(ring + kbuf + wave * 1024 + CREG + 8192 * i + 16 * lane) = uint4{0u, 0u, 0u, 0u};
          }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      } else {
#pragma unroll
        for (int i = 0; i < 2; ++i) lds_copy16_at(xb, xoff[i], l0 + CREG + 8192u * i);
      }
    }
    if (!PROJ && kc_s == CSTAGE) {
      // wave w copies rows 64 (w mod TC / 64) .. of its constants, so that all waves have
      // the same number of copies in flight; rows past the last centroid read a -inf seed
      const int seg = wave & (TC / 64 - 1);
      const int row = seg * 64 + lane;
      const int j = c0 + row < A.k ? c0 + row : A.kall;
      const uint32_t ls = seeds0 + 4u * (uint32_t)((kc_t & (CRING - 1)) * NCONST * TC + seg * 64);
      if constexpr (HYB) {
        const int kp = A.kall + kSeedPad;
        const int q0 = wave / (TC / 64);  // CB = 4: waves 0-3 and 4-7 share the four; CB = 2: one each
#pragma unroll
        for (int i = 0; i < CB / 2; ++i) {
          const int q = q0 + i * (8 / (TC / 64));
          const float *src = q == 0 ? A.sp.seed : A.sp.tail + (int64_t)(q - 1) * kp;
          lds_copy4_at(src, 4u * (uint32_t)j, ls + 4u * (uint32_t)(q * TC));
        }
      } else {
        lds_copy4_at(A.sp.seed, 4u * (uint32_t)j, ls);
      }
    }
    if (++kc_s == S) {
      kc_s = 0;
      ++kc_t;
      kc_t = min(kc_t, nmy - 1);  // past the end the last tile again: valid copies that nothing reads
    }
    kbuf = kbuf == (kRing - 1) * STAGE ? 0 : kbuf + STAGE;
  };

  // LDS byte offsets of this lane's operands inside a stage: chunk c of block b is at
  // (b >> 1) * 4096 + r * 128 + 16 * ((4 (b & 1) + c) ^ ((r >> 1) & 7))
  const uint32_t lrow = (uint32_t)(r * 128), kx = (uint32_t)((r >> 1) & 7);
  auto at = [&](int b, int c) -> uint32_t {
    return (uint32_t)(b >> 1) * 4096u + lrow + 16u * ((4u * (b & 1) + c) ^ kx);
  };
  typedef __attribute__((address_space(3))) const i32x4 lds_i32x4;
  auto rd16 = [&](uint32_t off) -> i32x4 { return *(lds_i32x4 *)(size_t)(ring0 + off); };

  f32x16 acc[CB][2];
  h16x8 ch[CB], cl[CB];
  uint32_t xh[2][4], xl[2][4];  // the two point blocks of the stage, split
  f32x4 w[2][2];                // those of the next stage, as floats
  float best[2];
  int code[2];  // 64 * tile + row id of the best, -1 while there is none
#pragma unroll
  for (int pb = 0; pb < 2; ++pb) {
    best[pb] = -INFINITY;
    code[pb] = -1;
  }
  auto read_ch = [&](int cb, uint32_t buf) { ch[cb] = __builtin_bit_cast(h16x8, rd16(buf + at(wc * CB + cb, h))); };
  auto read_cl = [&](int cb, uint32_t buf) { cl[cb] = __builtin_bit_cast(h16x8, rd16(buf + at(wc * CB + cb, 2 + h))); };
  auto read_x = [&](int pb, int q, uint32_t buf) {
    w[pb][q] = __builtin_bit_cast(f32x4, rd16(buf + CREG + at(wp * 2 + pb, 2 * h + q)));
  };
  f32x4 mreg[2];                // PROJ: s mean of this lane's dims
  uint32_t seen[2] = {0u, 0u};  // PROJ: the bits of every value of the point, together
  // a 1 the compiler does not see through: fma(t, 1, ..) keeps split2's mixed instructions
  float one = 1.0f;
  if constexpr (PROJ) asm volatile("" : "+s"(one));
  // pair q of a point block; past: a block past the last stage, which nothing multiplies and seen leaves out
  auto conv = [&](int pb, int q, bool past = false) {
    if constexpr (PROJ) {
      const f32x4 v = w[pb][q >> 1], m = mreg[q >> 1];
      const int e = 2 * (q & 1);
      const float t0 = __builtin_fmaf(v[e], sx, -m[e]), t1 = __builtin_fmaf(v[e + 1], sx, -m[e + 1]);
      if (!past) seen[pb] |= __float_as_uint(t0) | __float_as_uint(t1);
      split2(t0, t1, one, xh[pb][q], xl[pb][q]);
      asm volatile("" : "+v"(xh[pb][q]), "+v"(xl[pb][q]), "+v"(seen[pb]));
      return;
    }
    split2(w[pb][q >> 1][2 * (q & 1)], w[pb][q >> 1][2 * (q & 1) + 1], sx, xh[pb][q], xl[pb][q]);
    asm volatile("" : "+v"(xh[pb][q]), "+v"(xl[pb][q]));
  };
  auto op = [&](const uint32_t (&v)[4]) {
    const i32x4 q = {(int)v[0], (int)v[1], (int)v[2], (int)v[3]};
    return __builtin_bit_cast(h16x8, q);
  };

  // The largest value acc + seed of one point block of a tile and the first row that
  // has it (rows ascend with (cb, i) in a lane, and only a larger value takes over,
  // so the smallest index wins ties).  Maxima first, half an instruction per value,
  // then the row: the first centroid block that holds the maximum, its 16 values, the
  // first equal one; with the seeds 2.9 instructions per value where adding,
  // comparing and two selects take 4.  In twelve pieces, to run between MFMAs.
  f32x16 z;
  float mb[CB], mx = 0.f;
  int id = 0, pos = 0;
  auto argmax_piece = [&](int j, int pb, int ct) {
    auto seeds_of = [&](int cb) {
      const float *sd = seeds[ct & (CRING - 1)][0] + wc * 32 * CB + 4 * h + 32 * cb;
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const f32x4 v = *reinterpret_cast<const f32x4 *>(sd + 8 * m);
#pragma unroll
        for (int e = 0; e < 4; ++e) z[4 * m + e] = v[e];
      }
    };
    if (j < CB) {
      if (j == 0) seeds_of(0);
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[j][pb][i] += z[i];
      float m = acc[j][pb][0];
#pragma unroll
      for (int i = 1; i < 15; i += 2) m = __builtin_fmaxf(__builtin_fmaxf(m, acc[j][pb][i]), acc[j][pb][i + 1]);
      mb[j] = __builtin_fmaxf(m, acc[j][pb][15]);
      asm volatile("" : "+v"(mb[j]));
      if (j + 1 < CB) seeds_of(j + 1);
    } else if (j == 4) {
      mx = mb[0];
#pragma unroll
      for (int cb = 1; cb < CB; ++cb) mx = __builtin_fmaxf(mx, mb[cb]);
      id = 16 * (CB - 1);
#pragma unroll
      for (int b = 1; b < CB; ++b) id = mb[CB - 1 - b] == mx ? 16 * (CB - 1 - b) : id;
      pos = 15;
      asm volatile("" : "+v"(mx), "+v"(id));
    } else if (j >= 5 && j < 9) {
#pragma unroll
      for (int i = 4 * (j - 5); i < 4 * (j - 4); ++i) {
        float v = acc[CB - 1][pb][i];
#pragma unroll
        for (int b = 1; b < CB; ++b) v = mb[CB - 1 - b] == mx ? acc[CB - 1 - b][pb][i] : v;
        asm volatile("" : "+v"(v));
        z[i] = v;
      }
    } else if (j == 9 || j == 10) {
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        const int i = (j == 9 ? 15 : 7) - b;
        pos = z[i] == mx ? i : pos;
      }
      asm volatile("" : "+v"(pos));
    } else if (j == 11) {
      const bool take = mx > best[pb];
      best[pb] = take ? mx : best[pb];
      code[pb] = take ? 64 * ct + id + pos : code[pb];
      asm volatile("" : "+v"(best[pb]), "+v"(code[pb]));
    }
  };

  uint32_t nbuf = 0;  // offset of the buffer that step i reads ahead from (stage i + 1)
  // One step: 2 x 3 CB slots of one MFMA and what runs beside it, in this order (the
  // scheduling barriers keep the compiler from gathering the reads, which then wait
  // for LDS, and the conversions).
  constexpr int NM = 3 * CB;
  auto pin = [&]() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  auto next_buf = [&]() { nbuf = nbuf == (kRing - 1) * STAGE ? 0 : nbuf + STAGE; };
  auto end_step = [&]() {
    // stage i + 2 has landed when only the copies of stage i + 3 are out (a tile's
    // constants may be among them: then the wait is for a little more)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NCC + 2) : "memory");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    next_buf();
  };
  auto step = [&](int ct, auto first_, auto last_) {
    constexpr bool FIRST = decltype(first_)::value, LAST = decltype(last_)::value;
    copy_stage();
    pin();
#pragma unroll
    for (int pb = 0; pb < 2; ++pb) {
#pragma unroll
      for (int j = 0; j < NM; ++j) {
        const int pr = j / CB, cb = j % CB;
        const h16x8 a = pr == 0 ? cl[cb] : ch[cb];
        const h16x8 b = pr == 1 ? op(xl[pb]) : op(xh[pb]);
        if constexpr (PROJ) {
          acc[cb][pb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(b, a, acc[cb][pb], 0, 0, 0);
        } else if (!HYB && !PRUNE && FIRST && pr == 0) {
          const f32x16 zero = {0.f};
          acc[cb][pb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, zero, 0, 0, 0);
        } else {
          acc[cb][pb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, acc[cb][pb], 0, 0, 0);
        }
        // the next stage's floats of this block, over two slots
        if (j < 2) read_x(pb, j, nbuf);
        if (PROJ && pb == 1 && j < 2) mreg[j] = *reinterpret_cast<const f32x4 *>(&msh[kSD * ct + 8 * h + 4 * j]);
        // the other block's conversion, a pair at a time: the second block of this
        // stage, then the first of the next
        constexpr int CS = CB == 4 ? 2 : 1;
        if (j >= CS && (j - CS) % CS == 0 && (j - CS) / CS < 4) conv(1 - pb, (j - CS) / CS, LAST && pb == 1);
        if (pb == 1) {  // operands used for the last time are replaced
          if (j >= 1 && j <= CB) read_cl(j - 1, nbuf);
          if (j >= 2 * CB + 1) read_ch(j - 2 * CB - 1, nbuf);
        }
        if (!PROJ && !PRUNE && ((!HYB && FIRST && pb == 0) || (LAST && pb == 1))) {
          if constexpr (CB == 4) {
            argmax_piece(j, FIRST && pb == 0 ? 1 : 0, FIRST && pb == 0 ? ct - 1 : ct);
          } else {
            argmax_piece(2 * j, FIRST && pb == 0 ? 1 : 0, FIRST && pb == 0 ? ct - 1 : ct);
            argmax_piece(2 * j + 1, FIRST && pb == 0 ? 1 : 0, FIRST && pb == 0 ? ct - 1 : ct);
          }
        }
        pin();
      }
    }
    read_ch(CB - 1, nbuf);
    end_step();
  };

  // one tail stage: four steps of 32 dims, operands read as they are needed
  [[maybe_unused]] auto tail_step = [&](int s) {
    copy_stage();
    pin();
    const uint32_t buf = nbuf, hsh = 4u * (uint32_t)h;
    const uint32_t row0 = buf + (uint32_t)((wc * 32 * CB + r) * 128);
    i32x4 av[2][CB];
    auto read = [&](int gg, int set) {
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) av[set][cb] = rd16(row0 + 4096u * cb + 16u * ((uint32_t)(2 * gg + h) ^ kx));
    };
    read(0, 0);
#pragma unroll
    for (int gg = 0; gg < 4; ++gg) {
      i32x4 bv[2];
#pragma unroll
      for (int pb = 0; pb < 2; ++pb) bv[pb] = widen_regrouped2(bitsT[(4 * s + gg) * kTP + wp * 64 + pb * 32 + r] >> hsh);
      if (gg < 3) read(gg + 1, (gg + 1) & 1);
      pin();
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int pb = 0; pb < 2; ++pb)
          acc[cb][pb] = __builtin_bit_cast(f32x16, __builtin_amdgcn_mfma_i32_32x32x32_i8(
                                                       av[gg & 1][cb], bv[pb], __builtin_bit_cast(i32x16, acc[cb][pb]),
                                                       0, 0, 0));
    }
    end_step();
  };
  // constant q of this lane's rows of block cb: rows 8 m + 4 h + e at [4 m + e]
  [[maybe_unused]] auto consts_of = [&](int q, int cb, int ct, float (&v)[16]) {
    const float *p = seeds[ct & (CRING - 1)][HYB ? q : 0] + wc * 32 * CB + 32 * cb + 4 * h;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const f32x4 x = *reinterpret_cast<const f32x4 *>(p + 8 * m);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[4 * m + e] = x[e];
    }
  };

  if constexpr (PROJ) {
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int pb = 0; pb < 2; ++pb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[cb][pb][i] = 0.f;
  } else if constexpr (!HYB && !PRUNE) {
    // before the first tile there is none whose second block's argmax is due: -inf
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[cb][1][i] = -INFINITY;
    // the slot of tile -1, and of tile 3, copied no sooner than in tile 0's first step
    if (t < TC) seeds[CRING - 1][0][t] = 0.f;
  }
  for (int i = 0; i < kRing - 1; ++i) copy_stage();
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  // the operands of the stage at nbuf, with nothing before them to read ahead
  auto open_front = [&]() {
#pragma unroll
    for (int pb = 0; pb < 2; ++pb) {
      read_x(pb, 0, nbuf);
      read_x(pb, 1, nbuf);
    }
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      read_cl(cb, nbuf);
      read_ch(cb, nbuf);
    }
    if constexpr (PROJ) {
      mreg[0] = *reinterpret_cast<const f32x4 *>(&msh[8 * h]);
      mreg[1] = *reinterpret_cast<const f32x4 *>(&msh[8 * h + 4]);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) conv(0, q);
    next_buf();
  };
  constexpr std::true_type T{};
  constexpr std::false_type F{};
  if constexpr (PRUNE) {
    const float half_s2 = 0.5f * sx * sx;
    float thr[2];
    int pj[2];
    bool nan = false;
    unsigned tested = 0, passed = 0;  // per lane
#pragma unroll
    for (int pb = 0; pb < 2; ++pb) {
      const int64_t pc = p0 + min(wp * 64 + pb * 32 + r, prmax);
      thr[pb] = (A.xn[pc] - A.tau[pc] * A.r0) * half_s2;
      pj[pb] = A.prev[pc];
    }
    open_front();
    for (int ct = 0; ct < nmy; ++ct) {
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int pb = 0; pb < 2; ++pb)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[cb][pb][i] = 0.f;
      for (int st = 0; st < S; ++st) step(ct, F, F);
      const int c0 = ct * TC;
#pragma unroll
      for (int pb = 0; pb < 2; ++pb) {
        nan |= acc[0][pb][0] != acc[0][pb][0];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
          float sd[16];
          consts_of(0, cb, ct, sd);
          uint32_t m16 = 0;  // bit i: row 8 (i >> 2) + 4 h + (i & 3) of the block stays
#pragma unroll
          for (int i = 15; i >= 0; --i) m16 = 2 * m16 + !(acc[cb][pb][i] + sd[i] < thr[pb]);
          uint32_t m = (m16 & 15u) | (m16 & 0xf0u) << 4 | (m16 & 0xf00u) << 8 | (m16 & 0xf000u) << 12;
          m <<= 4 * h;
          m |= __shfl_xor((int)m, 32);
          const int jb = c0 + wc * 32 * CB + cb * 32;  // first centroid of the block
          const int nvalid = A.k - jb;
          uint32_t valid = nvalid >= 32 ? 0xffffffffu : nvalid > 0 ? (1u << nvalid) - 1u : 0u;
          if (wp * 64 + pb * 32 + r > prmax) valid = 0u;
          const int rel = pj[pb] - jb;
          if (rel >= 0 && rel < 32) valid &= ~(1u << rel);
          if (h == 0) {
            mrow[wp * 64 + pb * 32 + r][wc * CB + cb] = m & valid;
            if (A.r0 == INFINITY) continue;  // no test
            tested += (unsigned)__popc(valid);
            passed += (unsigned)__popc(m & valid);
          }
        }
      }
      __syncthreads();
      // 16 bytes of a point's words per thread; rows hold whole groups of four words
      for (int e = t; e < kTP * (TC / 128); e += kThr) {
        const int row = e / (TC / 128), q = e % (TC / 128);
        if (row <= prmax && c0 / 32 + 4 * q < A.W4)
          *reinterpret_cast<uint4 *>(A.mask + (p0 + row) * A.W4 + c0 / 32 + 4 * q) =
              *reinterpret_cast<const uint4 *>(&mrow[row][4 * q]);
      }
      __syncthreads();  // the next tile's words
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (nan) A.sp.tflag[pt] = 1;
    if (A.cnt) {  // two partial counts per half of the tile (the fp32 kernel's tiles), here all in the first
      unsigned long long *sh = reinterpret_cast<unsigned long long *>(&mrow[0][0]);
      unsigned long long a = tested, b = passed;
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_xor(a, off);
        b += __shfl_xor(b, off);
      }
      if (lane == 0) {
        sh[2 * wave] = a;
        sh[2 * wave + 1] = b;
      }
      __syncthreads();
      if (t < 2) {
        unsigned long long v = 0;
        for (int w8 = 0; w8 < 8; ++w8) v += sh[2 * w8 + t];
        A.cnt[4 * pt + t] = v;
        if (2 * pt + 1 < A.ncnt) A.cnt[4 * pt + 2 + t] = 0;
      }
    }
    return;
  } else if constexpr (PROJ) {
    open_front();
    for (int st = 1; st < S; ++st) step(st, F, F);  // st: the stage read ahead
    step(S, F, T);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    // rows with a value past fp16's range, NaN or infinities give NaN, and rows whose
    // values are all small (below 2 where the sample's largest is 2^11 .. 2^12) lose bits:
    // the fp32 kernel redoes their tile
    bool redo = false;
#pragma unroll
    for (int pb = 0; pb < 2; ++pb) {
      const uint32_t sn = seen[pb] | __shfl_xor((int)seen[pb], 32);
      if ((sn & 0x40000000u) == 0u && (sn & 0x7fffffffu) != 0u) redo = true;
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (!(fabsf(acc[0][pb][i]) <= FLT_MAX)) redo = true;
    }
    if (redo) A.sp.tflag[pt] = 1;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const int o = g * TC + wc * 32 * CB + cb * 32 + r;
      if (o >= A.k) continue;
      const float f = A.sp.seed[o];
#pragma unroll
      for (int pb = 0; pb < 2; ++pb)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int64_t p = p0 + wp * 64 + pb * 32 + 8 * (i >> 2) + 4 * h + (i & 3);
          if (p < A.n) A.Y[p * A.k + o] = acc[cb][pb][i] * f;
        }
    }
    return;
  } else if constexpr (HYB) {
    for (int ct = 0; ct < nmy; ++ct) {
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        float nt[16];
        consts_of(1, cb, ct, nt);
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[cb][0][i] = acc[cb][1][i] = nt[i];
      }
      for (int s = 0; s < SI; ++s) tail_step(s);
      float al[2];
#pragma unroll
      for (int pb = 0; pb < 2; ++pb) al[pb] = alp[wp * 64 + pb * 32 + r];
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        float u16[16], s16[16];
        consts_of(2, cb, ct, u16);
        consts_of(3, cb, ct, s16);
#pragma unroll
        for (int i = 0; i < 16; ++i)
#pragma unroll
          for (int pb = 0; pb < 2; ++pb)
            acc[cb][pb][i] = fmaf(-(al[pb] * s16[i]), (float)__float_as_int(acc[cb][pb][i]), u16[i]);
        pin();
      }
      open_front();
      for (int s = SI + 1; s < S; ++s) step(ct, F, F);
      step(ct, F, T);
#pragma unroll
      for (int j = 0; j < 12; ++j) argmax_piece(j, 1, ct);
      // step moved nbuf one stage ahead of the tail stage that comes next
      nbuf = nbuf == 0 ? (kRing - 1) * STAGE : nbuf - STAGE;
    }
  } else {
    open_front();
    for (int ct = 0; ct < nmy; ++ct) {
      step(ct, T, F);
      for (int s = 2; s < S; ++s) step(ct, F, F);
      step(ct, F, T);
    }
#pragma unroll
    for (int j = 0; j < 12; ++j) argmax_piece(j, 1, nmy - 1);
  }

  // the copies past the end are still under way, into the LDS that the merge uses
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  // row ids to centroid indices, then merge the lane halves and the wave halves
  int bidx[2];
#pragma unroll
  for (int pb = 0; pb < 2; ++pb) {
    const int id = code[pb] & 63;
    const int row = wc * 32 * CB + (id >> 4) * 32 + ((id >> 2) & 3) * 8 + (id & 3) + 4 * h;
    bidx[pb] = code[pb] < 0 ? INT_MAX : (g + (code[pb] >> 6) * NG) * TC + row;
    const float os = __shfl_xor(best[pb], 32);
    const int oi = __shfl_xor(bidx[pb], 32);
    if (os > best[pb] || (os == best[pb] && oi < bidx[pb])) {
      best[pb] = os;
      bidx[pb] = oi;
    }
  }
  float *ms = reinterpret_cast<float *>(ring);
  int *mi = reinterpret_cast<int *>(ring + kTP * sizeof(float));
  if (wc == 1 && h == 0) {
#pragma unroll
    for (int pb = 0; pb < 2; ++pb) {
      ms[wp * 64 + pb * 32 + r] = best[pb];
      mi[wp * 64 + pb * 32 + r] = bidx[pb];
    }
  }
  __syncthreads();
  if (wc == 0 && h == 0) {
    const float m2 = A.sp.route->m2;
#pragma unroll
    for (int pb = 0; pb < 2; ++pb) {
      const int pc = wp * 64 + pb * 32 + r;
      const float os = ms[pc];
      const int oi = mi[pc];
      if (os > best[pb] || (os == best[pb] && oi < bidx[pb])) {
        best[pb] = os;
        bidx[pb] = oi;
      }
      const int64_t p = p0 + pc;
      if (p < A.n) {
        if (bidx[pb] == INT_MAX) {  // only NaN scores: the fp32 kernel redoes this tile
          A.sp.tflag[pt] = 1;
        } else if (A.keys) {
          atomicMin(A.keys + p, split_key(best[pb] * m2, bidx[pb]));
        } else {
          A.assign[p] = bidx[pb] + A.aoff;
          if (A.score) A.score[p] = best[pb] * m2;
        }
      }
    }
  }
}

}  // namespace

size_t split_bytes(int64_t n, int k, int d, bool tail) {
  auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
  const size_t S = (size_t)cdiv(d, kSD);
  return (tail ? al(12 * ((size_t)k + kSeedPad)) : 0) + 256 + al(4 * (size_t)k) + al(4 * ((size_t)k + kSeedPad)) + al(4 * (size_t)cdiv(n, kTP)) +
         al(S * k * kRow + 256 * kRow);
}

SplitPrep split_layout(int64_t n, int k, int d, bool tail, void *ws) {
  auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
  uint8_t *w = static_cast<uint8_t *>(ws);
  SplitPrep sp{};
  sp.route = reinterpret_cast<SplitRoute *>(w);
  w += 256;
  sp.rmax = reinterpret_cast<uint32_t *>(w);
  w += al(4 * (size_t)k);
  sp.seed = reinterpret_cast<float *>(w);
  w += al(4 * ((size_t)k + kSeedPad));
  sp.tflag = reinterpret_cast<int *>(w);
  w += al(4 * (size_t)cdiv(n, kTP));
  if (tail) {
    sp.tail = reinterpret_cast<float *>(w);
    w += al(12 * ((size_t)k + kSeedPad));
  }
  sp.img = w;
  sp.cstage = (int64_t)k * kRow;
  return sp;
}

km_status launch_split_prep(const float *C, int64_t ldc, int64_t n, int k, int d, const CentroidPrep &cp,
                            hipStream_t s) {
  const SplitPrep &sp = cp.sp;
  const int64_t units = (int64_t)k * 2 * cdiv(d, kSD);
  // every workgroup reads k maxima first: fewer, longer workgroups as k grows
  const int64_t grid = std::min<int64_t>(std::max<int64_t>(1, cdiv(units, 256)), 512);
  hipLaunchKernelGGL(split_prep_kernel, dim3((unsigned)grid), dim3(256), 0, s, C, ldc, k, d, sp.rmax, cp.cn, cp.qsum,
                     cp.u, cp.sig2, sp,
                     cdiv(n, kTP));
  KMQ_LAUNCH_CHECK("split_prep_kernel");
  return KM_OK;
}

km_status launch_split(const SplitArgs &A, int64_t grid, int tile_c, hipStream_t s) {
  const dim3 gr((unsigned)grid), th(kThr);
  if (A.mask) {
    if (tile_c == 128)
      hipLaunchKernelGGL((split_kernel<2, kSplitPrune>), gr, th, 0, s, A);
    else
      hipLaunchKernelGGL((split_kernel<4, kSplitPrune>), gr, th, 0, s, A);
  } else if (A.Y) {
    if (tile_c == 128)
      hipLaunchKernelGGL((split_kernel<2, kSplitProject>), gr, th, 0, s, A);
    else
      hipLaunchKernelGGL((split_kernel<4, kSplitProject>), gr, th, 0, s, A);
  } else if (A.pbits) {
    if (tile_c == 128)
      hipLaunchKernelGGL((split_kernel<2, kSplitHybrid>), gr, th, 0, s, A);
    else
      hipLaunchKernelGGL((split_kernel<4, kSplitHybrid>), gr, th, 0, s, A);
  } else {
    if (tile_c == 128)
      hipLaunchKernelGGL((split_kernel<2, kSplitAssign>), gr, th, 0, s, A);
    else
      hipLaunchKernelGGL((split_kernel<4, kSplitAssign>), gr, th, 0, s, A);
  }
  KMQ_LAUNCH_CHECK("split_kernel");
  return KM_OK;
}

size_t split_project_bytes(int64_t n, int d, int d_out) {  // with the sample's maxima
  return split_bytes(n, d_out, d, false) + 4 * (size_t)d;
}

km_status launch_split_project(const float *X, int64_t n, int d, int64_t ldx, const float *mean, const float *W,
                               int d_out, float *Y, void *ws, SplitPrep *out, hipStream_t s) {
  const SplitPrep sp = split_layout(n, d_out, d, false, ws);
  uint32_t *top = reinterpret_cast<uint32_t *>(static_cast<uint8_t *>(ws) + split_bytes(n, d_out, d, false));
  hipLaunchKernelGGL(proj_sample_kernel, dim3((unsigned)cdiv(d, 16)), dim3(1024), 0, s, X, n, d, ldx, mean, top,
                     sp.route);
  hipLaunchKernelGGL(proj_prep_kernel, dim3((unsigned)cdiv(d_out, 16)), dim3(256), 0, s, W, d, d_out, top, sp,
                     cdiv(n, kTP));
  KMQ_LAUNCH_CHECK("projection scales");
  SplitArgs A{};
  A.x = X;
  A.ldx = ldx;
  A.d = d;
  A.sp = sp;
  A.k = d_out;
  A.n = n;
  A.mean = mean;
  A.Y = Y;
  const int tile_c = d_out <= 128 ? 128 : 256;
  A.ngroups = (int)cdiv(d_out, tile_c);  // one tile of outputs per workgroup
  A.n_ptiles = cdiv(n, kTP);
  *out = sp;
  return launch_split(A, A.ngroups > 1 ? cdiv(A.n_ptiles, 8) * 8 * A.ngroups : A.n_ptiles, tile_c, s);
}

}  // namespace kmq
