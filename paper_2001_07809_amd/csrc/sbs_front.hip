// The step before the disparity search (arXiv 2001.07809, Sec. III): from a
// left image to the ascending list of its refined segment-boundary pixels.
//   lightness      CIE L* of each pixel, scaled to 8 bits ("Colour Space
//                  Conversion"); gray images pass through
//   histogram      256 bins of lightness ("Segmentation")
//   k-means        on the bins, distance |a - b|, exact rational centres
//   labels         each pixel takes its bin's cluster, renumbered by
//                  ascending centre
//   refinement     configured: 3x3 open then close on the labels; paper:
//                  Moore-neighbour boundary, then 'fill', then 'remove'
//                  ("Segment Boundary Detection", "Refinement")
//   components     8-connected components of the boundary map by lock-free
//                  union-find; each root is its component's smallest raster
//                  index
//   filter         configured: keep components of at least min_cc pixels;
//                  paper: drop the smallest components (ties by raster order)
//                  while the dropped total stays within 4% of all boundary
//                  pixels
//   list           left and right border columns plus the kept pixels, in
//                  ascending raster order ("Disparity Measurement": pixels on
//                  the left/right borders of the map count as boundary)
// Declared in include/sbs.h.
#include <hip/hip_runtime.h>
#include <cstring>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>

#include "../../include/sbs.h"
#include "sbs_internal.h"

namespace sbs_front {

constexpr int kBlock = 256;
constexpr int kMaxK = 64;
constexpr int kMaxPasses = 1000;
constexpr int kN1Parts = 64;        // partial counts of kept pixels (fraction control)
constexpr int kMiscBytes = 2048;    // small device state of one call, cleared at its start

// ---------------------------------------------------------------------------
// Lightness. sRGB decode of each channel, luminance Y = 0.2126 R + 0.7152 G +
// 0.0722 B on linear values, L* = 116 f(Y) - 16 with f the CIE cube-root law
// (linear below (6/29)^3), scaled by 255/100 and rounded half away from zero.
// fp64 without contraction: every product and sum is rounded on its own.
__device__ __forceinline__ double srgb_linear(int v) {
#pragma clang fp contract(off)
  const double c = v / 255.0;
  return c <= 0.04045 ? c / 12.92 : pow((c + 0.055) / 1.055, 2.4);
}

// L8 as a function of Y is a non-decreasing step function, so a pixel's
// value is the number of steps at or below its Y: t[v] (v = 1 .. 255) is the
// smallest Y whose L8 is at least v (+inf if none). The table comes from the
// host (light_steps below).
struct LightSteps {
  double t[256];
};

// A block's histogram: LDS adds into 16 copies of the bins (lane l uses copy
// l % 16; copies are 257 words apart, so equal values in different copies
// fall in different banks), then one global add per bin and block, into one
// of kHistParts copies in turn: adds to the same 128 bytes are served one
// after another, some 10 ns each, and would be most of a small image's time.
constexpr int kHistCopies = 16, kHistParts = 16;
struct BlockHist {
  uint32_t h[kHistCopies][257];
  __device__ __forceinline__ void clear() {
    for (int i = threadIdx.x; i < kHistCopies * 257; i += kBlock) (&h[0][0])[i] = 0u;
  }
  __device__ __forceinline__ void add(uint32_t v) { atomicAdd(&h[threadIdx.x & (kHistCopies - 1)][v], 1u); }
  __device__ __forceinline__ void store(uint32_t* hist) const {
    uint32_t t = 0;
#pragma unroll
    for (int c = 0; c < kHistCopies; ++c) t += h[c][threadIdx.x];
    if (t) atomicAdd(&hist[(blockIdx.x % kHistParts) * 256 + threadIdx.x], t);
  }
};

// RGB: four pixels per thread from 12 bytes of a row (at any alignment), two
// such groups in flight; rows end in a group of fewer, read by bytes. HIST:
// the values are counted on the way.
// The value comes from Y in fp32 and the hardware's log2 and exp2. That is
// within 2e-4 of 255/100 L* (3 roundings of 2^-24 on Y, a third of them left
// by the cube root; log2 within 2^-21 of values up to 7, a third of that
// left; exp2 within 2^-23: 296 times 2.6e-7, and 2^-16 of the last sums), so
// a value nearer than kLightEps to where it changes is decided on Y in fp64
// and the steps, as any other would be: one pixel in 500, with one branch for
// a thread's four (a branch per pixel kept their LDS reads one after another:
// 19 us at 4096x2304, 17 us so). Y in fp64 and the steps' search for every
// pixel were bound by LDS reads of 8 bytes: 17 us and the histogram's own pass
// 15 us; 1390x1110, rows not word-aligned: 17 -> 5.9 us; 640x480: 5.7 + 3.8 ->
// 5.3 us.
constexpr float kLightEps = 0x1p-10f;
template <bool HIST>
__global__ __launch_bounds__(kBlock) void k_light(const uint8_t* __restrict__ img, int32_t W, int32_t H, int64_t pitch,
                                                  uint8_t* __restrict__ L8, LightSteps steps, uint32_t* hist) {
#pragma clang fp contract(off)
  __shared__ double lin[256], t[257];
  __shared__ float linf[256];
  __shared__ BlockHist bh[1];
  {
    const double l = srgb_linear((int)threadIdx.x);
    lin[threadIdx.x] = l;
    linf[threadIdx.x] = (float)l;
    t[threadIdx.x] = steps.t[threadIdx.x];
    if (threadIdx.x == 0) t[256] = HUGE_VAL;
  }
  if constexpr (HIST) bh[0].clear();
  __syncthreads();
  constexpr double e = 6.0 / 29.0;
  constexpr float kE3 = (float)(e * e * e), kLinear = (float)(295.8 / (3 * e * e));
  const uint32_t gpr = ((uint32_t)W + 3u) / 4u;   // groups per row (gpr H < 2^31)
  const uint32_t groups = gpr * (uint32_t)H, stride = gridDim.x * kBlock;
  struct Group {
    int64_t at;   // of its first pixel in L8
    int n;        // its pixels
    uint32_t w[3];
  };
  auto fetch = [&](uint32_t g) {
    const uint32_t y = H == 1 ? 0u : g / gpr, x = 4u * (g - y * gpr);
    Group q;
    q.at = (int64_t)y * W + x;
    q.n = min((int)(W - x), 4);
    const uint8_t* p = img + (int64_t)y * pitch + 3 * (int64_t)x;
    if (q.n == 4) {
      __builtin_memcpy(q.w, p, 12);
    } else {
      uint8_t c[12];
#pragma unroll
      for (int k = 0; k < 12; ++k) c[k] = k < 3 * q.n ? p[k] : (uint8_t)0;
#pragma unroll
      for (int k = 0; k < 3; ++k)
        q.w[k] = c[4 * k] | (uint32_t)c[4 * k + 1] << 8 | (uint32_t)c[4 * k + 2] << 16 | (uint32_t)c[4 * k + 3] << 24;
    }
    return q;
  };
  auto take = [&](const Group& q) {
    const uint32_t px[4][3] = {{q.w[0] & 0xFFu, (q.w[0] >> 8) & 0xFFu, (q.w[0] >> 16) & 0xFFu},
                               {q.w[0] >> 24, q.w[1] & 0xFFu, (q.w[1] >> 8) & 0xFFu},
                               {(q.w[1] >> 16) & 0xFFu, q.w[1] >> 24, q.w[2] & 0xFFu},
                               {(q.w[2] >> 8) & 0xFFu, (q.w[2] >> 16) & 0xFFu, q.w[2] >> 24}};
    int v[4];
    bool near[4], any = false;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float Y = __builtin_fmaf(0.0722f, linf[px[k][2]], __builtin_fmaf(0.7152f, linf[px[k][1]], 0.2126f * linf[px[k][0]]));
      const float root = __builtin_amdgcn_exp2f(__builtin_amdgcn_logf(Y) * (1.0f / 3.0f));
      const float s = Y > kE3 ? __builtin_fmaf(295.8f, root, -40.3f) : __builtin_fmaf(kLinear, Y, 0.5f);
      v[k] = (int)s;
      near[k] = fabsf(s - (float)v[k] - 0.5f) > 0.5f - kLightEps;
      any |= near[k];
    }
    // one branch for the four of them: theirs are worked out side by side
    if (any) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (!near[k]) continue;
        const double Y = 0.2126 * lin[px[k][0]] + 0.7152 * lin[px[k][1]] + 0.0722 * lin[px[k][2]];
        const int up = Y >= t[v[k] + 1] ? 1 : 0, down = Y < t[v[k]] ? 1 : 0;
        v[k] += up - down;
      }
    }
    if (q.n == 4) {
      const uint32_t o = (uint32_t)(v[0] | v[1] << 8 | v[2] << 16 | v[3] << 24);
      __builtin_memcpy(L8 + q.at, &o, 4);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (k >= q.n) break;
      if (q.n != 4) L8[q.at + k] = (uint8_t)v[k];
      if constexpr (HIST) bh[0].add((uint32_t)v[k]);
    }
  };
  for (uint32_t g = blockIdx.x * kBlock + threadIdx.x; g < groups; g += 2u * stride) {
    const bool two = g + stride < groups;
    const Group q0 = fetch(g);
    Group q1 = q0;
    if (two) q1 = fetch(g + stride);
    take(q0);
    if (two) take(q1);
  }
  if constexpr (HIST) {
    __syncthreads();
    bh[0].store(hist);
  }
}

// Gray images, 16 pixels of a row per thread (at any alignment), the rest of
// a row by bytes: L8 is the image itself (COPY: its rows gathered from the
// pitch). HIST: the values are counted.
template <bool COPY, bool HIST>
__global__ __launch_bounds__(kBlock) void k_gray(const uint8_t* __restrict__ img, int32_t W, int32_t H, int64_t pitch,
                                                 uint8_t* __restrict__ L8, uint32_t* hist) {
  __shared__ BlockHist bh[1];
  if constexpr (HIST) {
    bh[0].clear();
    __syncthreads();
  }
  const uint32_t gpr = ((uint32_t)W + 15u) / 16u;
  const uint32_t groups = gpr * (uint32_t)H, stride = gridDim.x * kBlock;   // (groups < 2^31, stride at most 2^21)
  for (uint32_t g = blockIdx.x * kBlock + threadIdx.x; g < groups; g += stride) {
    const uint32_t y = g / gpr, x = 16u * (g - y * gpr);
    const uint8_t* p = img + (int64_t)y * pitch + x;
    uint8_t* o = L8 + (int64_t)y * W + x;
    if (x + 16u <= (uint32_t)W) {
      uint32_t w[4];
      __builtin_memcpy(w, p, 16);
      if constexpr (COPY) __builtin_memcpy(o, w, 16);
      if constexpr (HIST) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int b = 0; b < 4; ++b) bh[0].add((w[j] >> (8 * b)) & 0xFFu);
      }
    } else {
      for (uint32_t k = 0; x + k < (uint32_t)W; ++k) {
        const uint8_t v = p[k];
        if constexpr (COPY) o[k] = v;
        if constexpr (HIST) bh[0].add(v);
      }
    }
  }
  if constexpr (HIST) {
    __syncthreads();
    bh[0].store(hist);
  }
}

// Lightness of an image on `s` (L8 null: a gray image without gaps, only
// counted); hist null: not counted.
void launch_light(const uint8_t* img, int32_t W, int32_t H, int32_t C, int64_t pitch, uint8_t* L8, uint32_t* hist,
                  hipStream_t s);

// n bytes of zeros (16-byte aligned, a multiple of 16), by a kernel: no
// memset nodes if the caller captures the stream.
__global__ __launch_bounds__(kBlock) void k_clear(uint4* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n / 16; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = uint4{0u, 0u, 0u, 0u};
}

// K-means on the occupied bins, one block, thread b owns bin b. Centres are
// S_k / N_k (exact rationals); start c_k = Lmin + floor((2k+1)(Lmax-Lmin+1) /
// 2K) with N_k = 1; a bin goes to the nearest centre, ties to the lower k; an
// empty cluster keeps its centre; passes stop when no bin changes (at most
// 1000). Clusters are then renumbered by ascending centre (ties by index).
// Output: lut[b] = label of bin b (0 for empty bins).
// On a line a centre's bins are an interval (two centres part at their
// midpoint, and equal ones leave all to the lower k), so a cluster's sums are
// differences of the histogram's prefix sums at its ends; 64-bit LDS adds of
// every bin to a few words queued up lane by lane, five barriers a pass (K = 10
// at 1390x1110: 44 us; K = 4 at 4096x2304: 13 us), three so (31 and 9 us), and
// none where one wavefront can do it (8.5 and 4.5 us).
__global__ __launch_bounds__(256) void k_kmeans(const uint32_t* __restrict__ hist, int32_t K,
                                                uint8_t* __restrict__ lut, int32_t* __restrict__ passes_out) {
  __shared__ long long S[kMaxK], Nn[kMaxK];
  __shared__ double M[kMaxK + 4];   // S / N rounded to double, then far away values
  __shared__ long long pn[257], pw[257];   // pixels and their values in the bins below
  __shared__ long long wn[4], ww[4];
  __shared__ int asg[256], from[kMaxK], to[kMaxK];
  __shared__ int lo_s, hi_s, changed;
  __shared__ int rank[kMaxK];
  const int b = threadIdx.x, lane = b & 63;
  long long hb = 0;
  {
    uint32_t v[kHistParts];
#pragma unroll
    for (int q = 0; q < kHistParts; ++q) v[q] = hist[q * 256 + b];
#pragma unroll
    for (int q = 0; q < kHistParts; ++q) hb += v[q];
  }
  if (b == 0) { lo_s = 256; hi_s = -1; }
  long long cn = hb, cw = b * hb;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const long long n = __shfl_up(cn, off), w = __shfl_up(cw, off);
    if (lane >= off) { cn += n; cw += w; }
  }
  if (lane == 63) { wn[b >> 6] = cn; ww[b >> 6] = cw; }
  __syncthreads();
  const unsigned long long occ = __builtin_amdgcn_ballot_w64(hb > 0);
  if (lane == 0 && occ) {
    atomicMin(&lo_s, b + __builtin_ctzll(occ));
    atomicMax(&hi_s, b + 63 - __builtin_clzll(occ));
  }
  for (int j = 0; j < (b >> 6); ++j) { cn += wn[j]; cw += ww[j]; }
  pn[b + 1] = cn;
  pw[b + 1] = cw;
  if (b == 0) pn[0] = pw[0] = 0;
  if (b < kMaxK + 4) M[b] = 1e9;
  __syncthreads();
  const int lo = lo_s, hi = hi_s;
  if (hi < 0) {   // empty image cannot occur (N >= 1), kept for completeness
    lut[b] = 0;
    if (b == 0) *passes_out = 0;
    return;
  }
  if (hi - lo + 1 >= K) {
    // The first centres ascend strictly, and then they always do: a bin lies
    // at or below its centre's midpoint with the next one and above that with
    // the one before, so means keep their order, and so does a centre without
    // bins (its neighbours' means stay on their side of it). A pass is then
    // the K - 1 midpoints, the last bin at or below each, and the prefix sums
    // there; no bin changes where the pixels below the midpoints are the same.
    // One wavefront, lane = centre, no barriers.
    if (b < 64) {
      const bool mine = b < K;
      long long s = lo + ((long long)(2 * b + 1) * (hi - lo + 1)) / (2 * K), n = 1;
      long long below = -1;   // pixels at or below the midpoint above this centre
      int t = 255;            // the last bin of this centre
      int pass = 0;
      for (; pass < kMaxPasses; ++pass) {
        const double m = (double)s / (double)n;   // s < 2^40 and n < 2^32: both exact, the quotient rounded once
        const double next = __shfl_down(m, 1);
        t = 255;
        if (b < K - 1) {
          // |error| < 2^-44: where an integer lies closer, whether that bin is
          // at or below the midpoint is decided exactly
          const double mid = 0.5 * (m + next), r = rint(mid);
          t = (int)floor(mid);
          if (fabs(mid - r) < 0x1p-40) t = -1 - (int)r;
        }
        if (__builtin_amdgcn_ballot_w64(t < 0)) {
          const long long s1 = __shfl_down(s, 1), n1 = __shfl_down(n, 1);
          if (t < 0) {
            const int r = -1 - t;
            t = (__int128)(2LL * r * n) * n1 <= (__int128)s * n1 + (__int128)s1 * n ? r : r - 1;
          }
        }
        const long long up = pn[t + 1], uw = pw[t + 1];
        const bool moved = mine && up != below;
        below = up;
        if (!__builtin_amdgcn_ballot_w64(moved) && pass > 0) break;
        long long dn = __shfl_up(up, 1), dw = __shfl_up(uw, 1);
        if (b == 0) dn = dw = 0;
        if (mine && up - dn > 0) { s = uw - dw; n = up - dn; }
      }
      if (mine) to[b] = t;
      if (b == 0) *passes_out = pass + 1;
    }
    __syncthreads();
    int k = 0;
    for (int j = 0; j < K - 1; ++j) k += b > to[j] ? 1 : 0;
    lut[b] = hb > 0 ? (uint8_t)k : 0;
    return;
  }
  // fewer grey levels than clusters: equal centres, each bin by itself
  if (b < K) { S[b] = lo + ((long long)(2 * b + 1) * (hi - lo + 1)) / (2 * K); Nn[b] = 1; }
  int assign = -1;
  int pass = 0;
  for (; pass < kMaxPasses; ++pass) {
    if (b == 0) changed = 0;
    if (b < K) {
      from[b] = to[b] = 0;
      M[b] = (double)S[b] / (double)Nn[b];   // S < 2^40 and N < 2^32: both exact, the quotient rounded once
    }
    __syncthreads();
    // |b - S_k/N_k| < |b - S_best/N_best|, decided on the rounded means where
    // they differ by more than their rounding (|error| < 2^-44 for means in
    // [0, 255]); where two came closer than that, all over again exactly:
    //   |b N_k - S_k| N_best < |b N_best - S_best| N_k
    int best = 0;
    double db = fabs((double)b - M[0]);
    bool close = false;
    for (int k = 1; k < K; k += 4) {
      double d[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) d[j] = fabs((double)b - M[k + j]);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bool less = d[j] < db - 0x1p-40;
        close |= !less && d[j] <= db + 0x1p-40;
        best = less ? k + j : best;
        db = less ? d[j] : db;
      }
    }
    if (close) {
      best = 0;
      long long Sb = S[0], Nb = Nn[0];
      for (int k = 1; k < K; ++k) {
        const long long Sk = S[k], Nk = Nn[k];
        if ((__int128)llabs((long long)b * Nk - Sk) * Nb < (__int128)llabs((long long)b * Nb - Sb) * Nk) {
          best = k; Sb = Sk; Nb = Nk;
        }
      }
    }
    asg[b] = best;
    if (hb > 0 && assign != best) changed = 1;
    assign = best;
    __syncthreads();
    const int ch = changed;
    if (!ch && pass > 0) break;
    if (b == 0 || asg[b - 1] != best) from[best] = b;
    if (b == 255 || asg[b + 1] != best) to[best] = b + 1;
    __syncthreads();
    if (b < K) {
      const long long n = pn[to[b]] - pn[from[b]];
      if (n > 0) { S[b] = pw[to[b]] - pw[from[b]]; Nn[b] = n; }
    }
    if (!ch) break;
  }
  __syncthreads();
  if (b < K) {
    int rk = 0;
    for (int j = 0; j < K; ++j) {
      const __int128 a = (__int128)S[j] * Nn[b], c = (__int128)S[b] * Nn[j];
      rk += (a < c) || (a == c && j < b);
    }
    rank[b] = rk;
  }
  __syncthreads();
  lut[b] = hb > 0 ? (uint8_t)rank[assign] : 0;
  if (b == 0) *passes_out = pass + 1;
}

__global__ __launch_bounds__(kBlock) void k_label(const uint8_t* __restrict__ L8, int64_t N,
                                                  const uint8_t* __restrict__ lut, uint8_t* __restrict__ lab) {
  __shared__ uint8_t t[256];
  t[threadIdx.x] = lut[threadIdx.x];
  __syncthreads();
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (int64_t)gridDim.x * blockDim.x)
    lab[i] = t[L8[i]];
}

// ---------------------------------------------------------------------------
// The 3x3 refinement on bit planes: 32 pixels of a row are one 32-bit word,
// so a step on them is a handful of ands or ors.
//   erosion (min) and dilation (max) with replicate borders;
//   Moore boundary: 1 iff an in-image 8-neighbour differs;
//   'fill': a 0 whose eight neighbours are all 1 becomes 1 (outside = 0);
//   'remove': a 1 whose four 4-neighbours are all 1 becomes 0 (outside = 0).
// MODE 0 (open, close, boundary of the labels): the planes are the
// thresholds label >= t, t = 1 .. K - 1. Minimum and maximum of labels are
// the ands and ors of their threshold planes, a neighbour that the replicate
// border repeats is one the window holds anyway (so cells outside the image
// are left out: ones to an and, zeros to an or), and two labels differ where
// some plane does. MODE 1 (boundary, fill, remove): the planes are the bits
// of the label.
// A wavefront takes kRfCols columns x (64 - 2 halo) rows: lane = row, four
// words per plane in registers, a word of halo columns on either side (six
// words waste fewer columns but leave the chip with half the wavefronts:
// 26 us at 4096x2304 against 20 us); the
// rows above and below are the neighbouring lanes (DPP). No LDS and no
// barriers but for the table that spreads a lightness value's label over
// four planes: a byte each, so that eight pixels gather in one register and
// four of those transpose to a word of each plane. Planes go four at a time
// (one group up to K = 5, or K = 16 in MODE 1). Bound by the latency of one
// wavefront's chain (row loads, table lookups, the steps), so all row loads
// go out first (20 -> 17 us). Against label bytes with a byte-packed minimum
// per word in LDS tiles and a pass of its own for the labels: MODE 0, K = 4:
// 71 -> 17 us at 4096x2304, 28 -> 6 us at 640x480; MODE 1, K = 10: 24 -> 11
// us at 1390x1110.
constexpr int kRfWords = 4;
constexpr int kRfCols = 32 * (kRfWords - 2);
template <int MODE> constexpr int kRfHalo = MODE == 0 ? 5 : 3;
template <int MODE> constexpr int kRfRows = 64 - 2 * kRfHalo<MODE>;

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const u32x4 g_u32x4;

// Pixels x .. x + 15 of a row (those outside the row come out as anything).
// words: rows start on 4-byte boundaries and hold whole words; else the words
// from the boundary below are shifted into place, and a group within 4 pixels
// of the row's ends is read byte by byte.
__device__ __forceinline__ void load16(const uint8_t* row, int x, int W, bool words, uint32_t (&v)[4]) {
  if (words) {
    if (x >= 0 && x + 16 <= W) {
      const u32x4 q = *(g_u32x4*)(row + x);
      v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = x + 4 * j >= 0 && x + 4 * j + 4 <= W ? *(const uint32_t*)(row + x + 4 * j) : 0u;
    }
  } else if (x >= 4 && x + 20 <= W) {
    const uint32_t sh = (uint32_t)(uintptr_t)(row + x) & 3u;
    const uint8_t* p = row + x - sh;
    const u32x4 q = *(g_u32x4*)p;
    const uint32_t e = *(const uint32_t*)(p + 16);
    v[0] = __builtin_amdgcn_alignbyte(q.y, q.x, sh);
    v[1] = __builtin_amdgcn_alignbyte(q.z, q.y, sh);
    v[2] = __builtin_amdgcn_alignbyte(q.w, q.z, sh);
    v[3] = __builtin_amdgcn_alignbyte(e, q.w, sh);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[j] = 0u;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int xx = x + 4 * j + b;
        if (xx >= 0 && xx < W) v[j] |= (uint32_t)row[xx] << (8 * b);
      }
    }
  }
}

// The row above (the lane below) and the row below; the wavefront's first and
// last rows get their own value.
__device__ __forceinline__ uint32_t row_up(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x138, 0xf, 0xf, false);   // wave_shr:1
}
__device__ __forceinline__ uint32_t row_down(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x130, 0xf, 0xf, false);   // wave_shl:1
}
// the pixels to the left and right of a word's (the outermost words take their own edge pixel)
__device__ __forceinline__ uint32_t px_left(const uint32_t (&w)[kRfWords], int i) {
  return __builtin_amdgcn_alignbit(w[i], w[i > 0 ? i - 1 : 0], 31);
}
__device__ __forceinline__ uint32_t px_right(const uint32_t (&w)[kRfWords], int i) {
  return __builtin_amdgcn_alignbit(w[i < kRfWords - 1 ? i + 1 : i], w[i], 1);
}

// One erosion (kMin) or dilation of a plane, in place.
template <bool kMin>
__device__ __forceinline__ void plane_step(uint32_t (&w)[kRfWords], const uint32_t (&valid)[kRfWords]) {
  uint32_t a[kRfWords];
#pragma unroll
  for (int i = 0; i < kRfWords; ++i) a[i] = kMin ? w[i] | ~valid[i] : w[i] & valid[i];
#pragma unroll
  for (int i = 0; i < kRfWords; ++i) {
    const uint32_t l = px_left(a, i), r = px_right(a, i);
    const uint32_t h = kMin ? a[i] & l & r : a[i] | l | r;
    w[i] = kMin ? h & row_up(h) & row_down(h) : h | row_up(h) | row_down(h);
  }
}

// out |= pixels of the plane with an in-image neighbour that differs
__device__ __forceinline__ void plane_boundary(const uint32_t (&w)[kRfWords], const uint32_t (&valid)[kRfWords],
                                               uint32_t (&out)[kRfWords]) {
  uint32_t lo[kRfWords], hi[kRfWords];
#pragma unroll
  for (int i = 0; i < kRfWords; ++i) { lo[i] = w[i]; hi[i] = w[i]; }
  plane_step<true>(lo, valid);
  plane_step<false>(hi, valid);
#pragma unroll
  for (int i = 0; i < kRfWords; ++i) out[i] |= hi[i] & ~lo[i] & valid[i];
}

// Boundary map as bits: word wpr * y + (x >> 6), bit x & 63. `closed`
// (optional, MODE 0) receives the labels after the close.
template <int MODE>
__global__ __launch_bounds__(64) void k_refine(const uint8_t* __restrict__ lum, int32_t W, int32_t H, int32_t K,
                                               const uint8_t* __restrict__ lut, unsigned long long* __restrict__ B,
                                               int32_t wpr, uint8_t* __restrict__ closed, int32_t words) {
  __shared__ uint32_t code[256];
  const int lane = threadIdx.x;
  const int x0 = blockIdx.x * kRfCols, gx = x0 - 32;        // first output column, first column held
  const int gy = (int)blockIdx.y * kRfRows<MODE> - kRfHalo<MODE> + lane;
  const bool row_in = gy >= 0 && gy < H;
  const uint8_t* row = lum + (int64_t)min(max(gy, 0), H - 1) * W;
  uint32_t valid[kRfWords];
#pragma unroll
  for (int i = 0; i < kRfWords; ++i) {
    const int lo = max(0, -(gx + 32 * i)), hi = min(32, W - (gx + 32 * i));   // columns of the word inside the image
    const uint32_t m = hi <= lo ? 0u : (hi == 32 ? ~0u : (1u << hi) - 1u) & ~((1u << lo) - 1u);
    valid[i] = row_in ? m : 0u;
  }
  // planes: MODE 0 label >= 1 .. K - 1, MODE 1 the label's bits
  const int np = MODE == 0 ? K - 1 : 32 - __builtin_clz(max(K - 1, 1));
  uint32_t acc[kRfWords];
#pragma unroll
  for (int i = 0; i < kRfWords; ++i) acc[i] = 0u;
  // the lane's pixels, all loads in flight together (and under the table's making)
  uint32_t px[kRfWords][8];
#pragma unroll
  for (int i = 0; i < kRfWords; ++i) {
    uint32_t q[4];
    load16(row, gx + 32 * i, W, words, q);
    px[i][0] = q[0]; px[i][1] = q[1]; px[i][2] = q[2]; px[i][3] = q[3];
    load16(row, gx + 32 * i + 16, W, words, q);
    px[i][4] = q[0]; px[i][5] = q[1]; px[i][6] = q[2]; px[i][7] = q[3];
  }
  // `closed`: the number of planes each pixel is set in, bit by bit (a label
  // read back and written for every four planes: 292x206, K = 64, 323 us a
  // call, 132 so)
  constexpr int kLabelBits = 6;
  static_assert(kMaxK <= 1 << kLabelBits, "labels below kMaxK");
  uint32_t count[kRfWords - 2][kLabelBits];
#pragma unroll
  for (int i = 0; i < kRfWords - 2; ++i)
#pragma unroll
    for (int b = 0; b < kLabelBits; ++b) count[i][b] = 0u;
  for (int g = 0; g == 0 || 4 * g < np; ++g) {
    __syncthreads();
    for (int b = lane; b < 256; b += 64) {
      const int lab = lut[b];
      uint32_t c = 0u;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const int t = 4 * g + p;
        if (t < np && (MODE == 0 ? lab > t : (lab >> t) & 1)) c |= 1u << (8 * p);
      }
      code[b] = c;
    }
    __syncthreads();
    uint32_t P[4][kRfWords];
#pragma unroll
    for (int i = 0; i < kRfWords; ++i) {
      const uint32_t (&v)[8] = px[i];
      uint32_t a[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        a[q] = 0u;
#pragma unroll
        for (int b = 0; b < 8; ++b) a[q] |= code[(v[2 * q + (b >> 2)] >> (8 * (b & 3))) & 0xFFu] << b;
      }
      const uint32_t t0 = __builtin_amdgcn_perm(a[1], a[0], 0x05010400u), t1 = __builtin_amdgcn_perm(a[1], a[0], 0x07030602u);
      const uint32_t t2 = __builtin_amdgcn_perm(a[3], a[2], 0x05010400u), t3 = __builtin_amdgcn_perm(a[3], a[2], 0x07030602u);
      P[0][i] = __builtin_amdgcn_perm(t2, t0, 0x05040100u);
      P[1][i] = __builtin_amdgcn_perm(t2, t0, 0x07060302u);
      P[2][i] = __builtin_amdgcn_perm(t3, t1, 0x05040100u);
      P[3][i] = __builtin_amdgcn_perm(t3, t1, 0x07060302u);
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      if (4 * g + p >= np) continue;
      if constexpr (MODE == 0) {
        plane_step<true>(P[p], valid);    // open
        plane_step<false>(P[p], valid);
        plane_step<false>(P[p], valid);   // close
        plane_step<true>(P[p], valid);
      }
      plane_boundary(P[p], valid, acc);
    }
    if constexpr (MODE == 0) {
      // the closed label of a pixel is the number of planes it is set in
      if (closed) {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          if (4 * g + p >= np) continue;
#pragma unroll
          for (int i = 1; i < kRfWords - 1; ++i) {
            uint32_t carry = P[p][i];
#pragma unroll
            for (int b = 0; b < kLabelBits; ++b) {
              const uint32_t c = count[i - 1][b] & carry;
              count[i - 1][b] ^= carry;
              carry = c;
            }
          }
        }
      }
    }
  }
  if constexpr (MODE == 0) {
    if (closed && row_in && lane >= kRfHalo<MODE> && lane < 64 - kRfHalo<MODE>) {
      uint8_t* crow = closed + (int64_t)gy * W;
#pragma unroll
      for (int i = 1; i < kRfWords - 1; ++i)
#pragma unroll 4
        for (int j = 0; j < 32; j += 4) {
          const int x = gx + 32 * i + j;
          uint32_t four = 0u;   // a byte per pixel
#pragma unroll
          for (int b = 0; b < kLabelBits; ++b) {
            const uint32_t n = count[i - 1][b] >> j & 0xFu;
            four |= (n * 0x00204081u & 0x01010101u) << b;
          }
          if (x + 4 <= W) {
            __builtin_memcpy(crow + x, &four, 4);
          } else {
            for (int k = 0; x + k < W; ++k) crow[x + k] = (uint8_t)(four >> (8 * k));
          }
        }
    }
  }
  if constexpr (MODE == 1) {
    // 'fill', then 'remove'; acc is 0 outside the image
    uint32_t f[kRfWords];
#pragma unroll
    for (int i = 0; i < kRfWords; ++i) {
      const uint32_t l = px_left(acc, i), r = px_right(acc, i), h = acc[i] & l & r;
      f[i] = (acc[i] | (l & r & row_up(h) & row_down(h))) & valid[i];
    }
#pragma unroll
    for (int i = 0; i < kRfWords; ++i)
      acc[i] = f[i] & ~(px_left(f, i) & px_right(f, i) & row_up(f[i]) & row_down(f[i]));
  }
  if (!row_in || lane < kRfHalo<MODE> || lane >= 64 - kRfHalo<MODE>) return;
  unsigned long long* out = B + (int64_t)gy * wpr + (x0 >> 6);
#pragma unroll
  for (int i = 1; i < kRfWords - 1; i += 2)
    if ((x0 >> 6) + i / 2 < wpr) out[i / 2] = (unsigned long long)acc[i] | (unsigned long long)acc[i + 1] << 32;
}

// ---------------------------------------------------------------------------
// Maps held as bits: word y * wpr + (x >> 6), bit x & 63, the words of a row
// ending with it. Words in order are pixels in raster order.
struct Bits {
  int32_t W, H, wpr;
  int64_t words;   // H * wpr
  int64_t per;     // words per block of the passes that number the list (a multiple of kSelWords)
};
constexpr int kSelWords = 64;       // words a block takes at a time: 16 per wavefront
constexpr int kSelBlocks = 1024;    // most blocks of those passes, so that each can add up the counts before its own

struct WordPos {
  int c, y, i;                // word column, row, and raster index of its first pixel (W * H < 2^31)
  unsigned long long border;  // its pixels in the image's first and last column
};
__device__ __forceinline__ void word_border(const Bits& b, WordPos& p) {
  p.border = (p.c == 0 ? 1ull : 0ull) | (p.c == b.wpr - 1 ? 1ull << ((b.W - 1) & 63) : 0ull);
}
__device__ __forceinline__ WordPos word_pos(const Bits& b, int64_t wi) {
  WordPos p;
  p.y = (int)((uint32_t)wi / (uint32_t)b.wpr);   // words < 2^31
  p.c = (int)((uint32_t)wi - (uint32_t)p.y * (uint32_t)b.wpr);
  p.i = p.y * b.W + 64 * p.c;
  word_border(b, p);
  return p;
}
// kWaveWords words of a map from w0 on (zeros from w_end on): lane j holds
// word j, its first pixel and its border pixels; word(j) and first(j) give
// them to every lane as scalars. One load and one division for all of them
// (a division per word, and words a few at a time with a round trip to memory
// for each step, made k_kept 29 us at 4096x2304, 20 us so).
constexpr int kWaveWords = kSelWords / (kBlock / 64);   // 16
struct WaveWords {
  unsigned long long v, border;
  int i;
  __device__ __forceinline__ unsigned long long word(int j) const {
    return (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, j) |
           (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), j) << 32;
  }
  __device__ __forceinline__ unsigned long long border_of(int j) const {
    return (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)border, j) |
           (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(border >> 32), j) << 32;
  }
  __device__ __forceinline__ int first(int j) const { return __builtin_amdgcn_readlane(i, j); }
};
__device__ __forceinline__ WaveWords wave_words(const Bits& b, const unsigned long long* map, int64_t w0, int64_t w_end) {
  const int lane = threadIdx.x & 63;
  WaveWords r{0ull, 0ull, 0};
  if (lane < kWaveWords && w0 + lane < w_end) {
    r.v = map[w0 + lane];
    const WordPos p = word_pos(b, w0 + lane);
    r.i = p.i;
    r.border = p.border;
  }
  return r;
}
// a[node] at the lanes that start a horizontal run of word j (word w0 + j of
// the map), `none` elsewhere. Node 32 w + k is the k-th run of word w.
__device__ __forceinline__ int node_of(int64_t wi, unsigned long long starts) {
  return (int)(32 * wi) + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(starts >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)starts, 0u));
}
__device__ __forceinline__ void at_run_starts(const WaveWords& w, int64_t w0, const int32_t* a, int32_t none,
                                              int32_t (&v)[kWaveWords]) {
#pragma unroll
  for (int j = 0; j < kWaveWords; ++j) {
    v[j] = none;
    const unsigned long long m = w.word(j), st = m & ~(m << 1);
    if (!m) continue;
    if (__builtin_amdgcn_inverse_ballot_w64(st)) v[j] = a[node_of(w0 + j, st)];
  }
}
// The same for the runs of `kept`, a map of some of the runs of `w` (whose
// numbers in their words are those in `w`).
__device__ __forceinline__ void at_kept_runs(const WaveWords& kept, const WaveWords& w, int64_t w0, const int32_t* a,
                                             int32_t (&v)[kWaveWords]) {
#pragma unroll
  for (int j = 0; j < kWaveWords; ++j) {
    v[j] = 0;
    const unsigned long long k = kept.word(j);
    if (!k) continue;
    const unsigned long long m = w.word(j);
    if (__builtin_amdgcn_inverse_ballot_w64(k & ~(k << 1))) v[j] = a[node_of(w0 + j, m & ~(m << 1))];
  }
}
// The bits of the horizontal run of w that starts at bit a.
__device__ __forceinline__ unsigned long long run_from(unsigned long long w, int a) {
  const unsigned long long m = 1ull << a;
  return w & ~(w + m) & ~(m - 1ull);   // adding the start bit clears exactly its run
}

// Pixel (x, y) of a map.
__device__ __forceinline__ bool map_bit(const unsigned long long* map, int32_t wpr, int x, int y) {
  return (map[(int64_t)y * wpr + (x >> 6)] >> (x & 63)) & 1ull;
}

// ---------------------------------------------------------------------------
// Connected components by union-find over horizontal runs: a node is a run of
// one word of the map, node 32 w + k the k-th run of word w (a word holds at
// most 32), so nodes are in raster order, and parents and sizes lie side by
// side for a word's few runs. A link always points a larger root at a smaller
// one, so a component's root ends as its first run. Two levels: k_cc_tile
// joins the runs of a tile of one word x kTileH rows in LDS and writes each
// run's tile root and the tile roots' sizes (0 elsewhere), k_cc_edges joins
// tiles through the global forest, k_cc_flatten points every tile root at its
// root and moves its size there. Against one node per pixel: 88 -> 56 us at
// 4096x2304, 46 -> 29 us at 640x480.
constexpr int kTileH = 32;

// The k-th run's number in a word: the run starts at or below bit a, less one.
__device__ __forceinline__ int run_at(unsigned long long w, int a) {
  return __builtin_popcountll((w & ~(w << 1)) & (a == 63 ? ~0ull : (2ull << a) - 1ull)) - 1;
}
__device__ __forceinline__ int32_t lds_find(int32_t* lp, int32_t a) {
  for (;;) {
    const int32_t p = lp[a];
    if (p == a) return a;
    const int32_t pp = lp[p];
    if (pp == p) return p;
    atomicMin(&lp[a], pp);   // halve the path: a link only ever moves towards smaller nodes
    a = pp;
  }
}
__device__ __forceinline__ void lds_union(int32_t* lp, int32_t a, int32_t b) {
  for (;;) {
    a = lds_find(lp, a);
    b = lds_find(lp, b);
    if (a == b) return;
    if (a < b) { const int32_t t = a; a = b; b = t; }
    // a > b, a was a root when found: make it point at b unless it moved meanwhile
    const int32_t old = atomicMin(&lp[a], b);
    if (old == a) return;
    a = old;   // a was linked elsewhere concurrently: continue from there
  }
}
// The same in memory, both sides climbing together (two loads in flight). A
// new link then climbs to its root as well, lowering the linked node's parent
// as it goes: tiles that all join their neighbour at once make a chain as long
// as the image has tiles, and the links of a chain that climb together double
// their reach with every step. Without that, whoever joined two such chains
// walked them alone (kernel k_cc_edges, 100000x20 noise in paper mode: 505 ->
// 15 us; 40x60000 checks: 174 -> 18 us). Maps of 640x480 to 4096x2304 without
// such chains pay up to 7% of the call for it (stripes); over 138 of them the
// call is 2% shorter.
__device__ __forceinline__ void uf_union(int32_t* parent, int32_t a, int32_t b) {
  auto load = [&](int32_t i) { return __hip_atomic_load(&parent[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  for (;;) {
    const int32_t pa = load(a), pb = load(b);
    if (pa == pb) return;
    const int32_t ga = load(pa), gb = load(pb);
    if (ga == gb) return;
    if (ga == pa && gb == pb) {   // two roots
      const int32_t hi = max(pa, pb), lo = min(pa, pb);
      const int32_t old = atomicMin(&parent[hi], lo);
      if (old == hi) {
        for (int32_t p = lo;;) {
          const int32_t q = load(p);
          if (q == p) return;
          atomicMin(&parent[hi], q);
          p = load(hi);
        }
      }
      a = old;   // it was linked elsewhere concurrently: continue from there
      b = lo;
      continue;
    }
    if (ga != pa) atomicMin(&parent[a], ga);   // halve the paths
    if (gb != pb) atomicMin(&parent[b], gb);
    a = ga;
    b = gb;
  }
}

// Every pair of a run of w (its k-th) and a run of the word u of the row above
// (its n-th) that touch (8-connected, within the word), each at the lane of the
// run of w's first pixel that touches it: f(lanes, k, n) is called by all lanes
// with the lanes that have a pair, twice at most. w and u are the same in every
// lane.
template <typename F>
__device__ __forceinline__ void for_touching(unsigned long long w, unsigned long long u, F f) {
  const unsigned long long ws = w & ~(w << 1), us = u & ~(u << 1);   // run starts
  const int kb = node_of(0, ws), nb = node_of(0, us);                // of them below this lane
  const unsigned long long left = ws & u << 1;                       // run starts with the pixel up-left set ...
  const unsigned long long up = ws & u & ~(u << 1);                  // ... or not, but the one above
  const unsigned long long right = w & u >> 1 & ~u;                  // pixels with a run starting up-right
  if (left | up) f(left | up, kb, __builtin_amdgcn_inverse_ballot_w64(left) ? nb - 1 : nb);
  if (right) f(right, kb + (__builtin_amdgcn_inverse_ballot_w64(ws) ? 0 : -1), nb);
}

// One block per tile; wavefront w takes a band of rows. Its rows' runs and the
// pairs that touch are queued in LDS first, a row at a time with lane = pixel,
// and then taken 64 at a time: the unions and walks are chains of LDS round
// trips, and row by row a band went through twelve of them, most lanes idle
// (4096x2304: 35 -> 24 us, 640x480: 10 -> 7.5 us).
constexpr int kCcBlock = 512, kBandH = kTileH / (kCcBlock / 64);
__global__ __launch_bounds__(kCcBlock) void k_cc_tile(Bits b, const unsigned long long* __restrict__ B,
                                                    int32_t* __restrict__ parent, int32_t* __restrict__ size) {
  constexpr int kPairs = kBandH * 64, kNodes = kBandH * 32;   // at most, per band
  static_assert(kNodes % 64 == 0, "whole rounds of nodes");
  __shared__ int32_t lp[kTileH * 32], lsz[kTileH * 32];
  __shared__ unsigned long long last[kCcBlock / 64];   // each band's last row
  __shared__ uint32_t pairs[kCcBlock / 64][kPairs];    // node | node above << 16
  __shared__ uint32_t nodes[kCcBlock / 64][kNodes];    // node | pixels of the run << 16
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int c = blockIdx.x, y0 = blockIdx.y * kTileH + wv * kBandH, ly0 = wv * kBandH;
  const unsigned long long mine = lane < kBandH && y0 + lane < b.H ? B[(int64_t)(y0 + lane) * b.wpr + c] : 0ull;
  auto below = [](unsigned long long m) {   // set bits below this lane
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
  };
  unsigned long long w[kBandH];
  int nn = 0, np = 0;
#pragma unroll
  for (int j = 0; j < kBandH; ++j) {
    w[j] = (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mine, j) |
           (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(mine >> 32), j) << 32;
    const unsigned long long st = w[j] & ~(w[j] << 1);
    if (__builtin_amdgcn_inverse_ballot_w64(st)) {
      const int k = below(st), n = (ly0 + j) * 32 + k;
      lp[n] = n;
      lsz[n] = 0;
      nodes[wv][nn + k] = (uint32_t)n | (uint32_t)__builtin_popcountll(run_from(w[j], lane)) << 16;
    }
    nn += __builtin_popcountll(st);
  }
  if (lane == 0) last[wv] = w[kBandH - 1];
  __syncthreads();
  unsigned long long above = wv > 0 ? last[wv - 1] : 0ull;
  above = (unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)above) |
          (unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(above >> 32)) << 32;
#pragma unroll
  for (int j = 0; j < kBandH; ++j) {
    const unsigned long long u = j > 0 ? w[j > 0 ? j - 1 : 0] : above;
    if (!((w[j] | w[j] << 1 | w[j] >> 1) & u)) continue;
    const int row = (ly0 + j) * 32;
    for_touching(w[j], u, [&](unsigned long long lanes, int k, int n) {
      if (__builtin_amdgcn_inverse_ballot_w64(lanes)) pairs[wv][np + below(lanes)] = (uint32_t)(row + k) | (uint32_t)(row - 32 + n) << 16;
      np += __builtin_popcountll(lanes);
    });
  }
  asm volatile("" ::: "memory");   // (a wavefront's LDS operations are done in the order it issues them)
  for (int i = lane; i < np; i += 64) {
    const uint32_t q = pairs[wv][i];
    lds_union(lp, (int32_t)(q & 0xFFFFu), (int32_t)(q >> 16));
  }
  __syncthreads();
  uint32_t node[kNodes / 64];
  int32_t root[kNodes / 64];
#pragma unroll
  for (int i = 0; i < kNodes / 64; ++i) {
    if (64 * i + lane >= nn) continue;
    node[i] = nodes[wv][64 * i + lane];
    root[i] = lds_find(lp, (int32_t)(node[i] & 0xFFFFu));
    atomicAdd(&lsz[root[i]], (int32_t)(node[i] >> 16));
  }
  __syncthreads();
  const int64_t w0 = (int64_t)blockIdx.y * kTileH * b.wpr + c;   // the tile's first word
#pragma unroll
  for (int i = 0; i < kNodes / 64; ++i) {
    if (64 * i + lane >= nn) continue;
    const int n = (int)(node[i] & 0xFFFFu), r = root[i];
    const int64_t g = (w0 + (int64_t)(n >> 5) * b.wpr) * 32 + (n & 31);
    parent[g] = (int32_t)((w0 + (int64_t)(r >> 5) * b.wpr) * 32 + (r & 31));
    size[g] = r == n ? lsz[n] : 0;
  }
}

// Runs that touch across tile edges. The first `vblocks` blocks take the
// edges between word columns, a thread per row and edge (of the three pairs
// across it in two rows those that no other pair implies), edge by edge, so
// that a column's links are made before those of the columns to its right;
// the others the edges between tile rows, a wavefront per word, lane = pixel.
__global__ __launch_bounds__(kBlock) void k_cc_edges(Bits b, const unsigned long long* __restrict__ B, int32_t* parent,
                                                     int vblocks) {
  if ((int)blockIdx.x < vblocks) {
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int e = b.wpr - 1;   // edges per row
    if (t >= (int64_t)b.H * e) return;
    const int c = (int)((uint32_t)t / (uint32_t)b.H), y = (int)((uint32_t)t % (uint32_t)b.H);
    const int64_t wl = (int64_t)y * b.wpr + c, wr = wl + 1;
    const unsigned long long L = B[wl], R = B[wr];
    const unsigned long long Lu = y > 0 ? B[wl - b.wpr] : 0ull, Ru = y > 0 ? B[wr - b.wpr] : 0ull;
    const bool l = L >> 63, r = R & 1ull, lu = Lu >> 63, ru = Ru & 1ull;
    if (l && r && !(lu && ru)) uf_union(parent, (int32_t)(32 * wl + run_at(L, 63)), (int32_t)(32 * wr));
    if (l && ru && !lu && !r) uf_union(parent, (int32_t)(32 * wl + run_at(L, 63)), (int32_t)(32 * (wr - b.wpr)));
    if (lu && r && !l && !ru) uf_union(parent, (int32_t)(32 * (wl - b.wpr) + run_at(Lu, 63)), (int32_t)(32 * wr));
    return;
  }
  const int64_t t = (int64_t)(blockIdx.x - vblocks) * (kBlock / 64) + (threadIdx.x >> 6);
  const int y = (int)(t / b.wpr + 1) * kTileH, c = (int)(t % b.wpr);
  if (y >= b.H) return;
  const int64_t wi = (int64_t)y * b.wpr + c;
  auto uniform = [](unsigned long long v) {
    return (unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v) |
           (unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32)) << 32;
  };
  const unsigned long long w = uniform(B[wi]), u = uniform(B[wi - b.wpr]);
  for_touching(w, u, [&](unsigned long long lanes, int k, int n) {
    if (__builtin_amdgcn_inverse_ballot_w64(lanes))
      uf_union(parent, (int32_t)(32 * wi + k), (int32_t)(32 * (wi - b.wpr) + n));
  });
}

// Every tile root's root, and the component sizes there: k_cc_tile left each
// tile root's size at the tile root; one that is not its component's root
// moves its count with one atomic. Roots of components are tile roots (a
// component's first run is the first of its tile part), so no count moves
// into a tile root that moves its own away. A walk writes each ancestor it
// meets back as its start's parent, so that the walks of a long chain shorten
// each other (its length halves with every step); no link changes otherwise,
// so any value read (cached, possibly stale) is an ancestor, and a walk ends
// at the root. The other runs keep their tile root as parent.
__global__ __launch_bounds__(kBlock) void k_cc_flatten(Bits b, const unsigned long long* __restrict__ B, int32_t* parent,
                                                       int32_t* size) {
  // the block's tile roots are queued first, so that their walks go together
  __shared__ int2 queue[kSelWords * 32];   // node, size
  __shared__ uint32_t queued;
  for (int64_t b0 = (int64_t)blockIdx.x * kSelWords; b0 < b.words; b0 += (int64_t)gridDim.x * kSelWords) {
    if (threadIdx.x == 0) queued = 0u;
    __syncthreads();
    const int64_t w0 = b0 + kWaveWords * (threadIdx.x >> 6);
    const WaveWords w = wave_words(b, B, w0, b.words);
    int32_t sz[kWaveWords];
    at_run_starts(w, w0, size, 0, sz);
#pragma unroll
    for (int j = 0; j < kWaveWords; ++j) {
      if (sz[j] <= 0) continue;
      const unsigned long long m = w.word(j);
      queue[atomicAdd(&queued, 1u)] = int2{node_of(w0 + j, m & ~(m << 1)), sz[j]};
    }
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < queued; k += kBlock) {
      const int32_t n = queue[k].x, t = parent[n];
      if (t == n) continue;
      int32_t r = t;
      for (int32_t q = parent[r]; q != r; q = parent[r]) {
        parent[n] = q;
        r = q;
      }
      size[n] = 0;
      atomicAdd(&size[r], queue[k].y);
    }
    __syncthreads();   // the queue is refilled
  }
}

// ---------------------------------------------------------------------------
// Paper filter: components in ascending (size, root) order are dropped while
// the dropped total stays <= floor(0.04 * total). With cnt[s] the number of
// components of size s (s <= budget), everything below the first size s* that
// no longer fits whole is dropped, and of size s* the first m by root.
constexpr double kDropFrac = 0.04;
struct DropRule {
  long long total;    // boundary pixels
  long long budget;   // floor(kDropFrac * total)
  int32_t s_star;     // sizes < s_star dropped
  int32_t m;          // components of size s_star dropped (smallest roots first)
  int32_t first;      // the first root of size s_star that is kept
};

// cnt[s] += 1 for every component of size s that the budget could hold
// (s <= kDropFrac N, the array's length); total = all boundary pixels. Sizes
// are read at the starts of the map's runs only: every root is one, and after
// k_cc_flatten a run start's size is non-zero exactly at roots.
__global__ __launch_bounds__(kBlock) void k_drop_count(Bits b, const unsigned long long* __restrict__ B,
                                                       const int32_t* __restrict__ size, int64_t ncnt,
                                                       unsigned long long* total, int32_t* cnt) {
  constexpr int kSmall = 1024;   // sizes below this are counted per block in LDS first
  __shared__ unsigned long long part;
  __shared__ int32_t small[kSmall];
  for (int j = threadIdx.x; j < kSmall; j += blockDim.x) small[j] = 0;
  if (threadIdx.x == 0) part = 0;
  __syncthreads();
  const int lane = threadIdx.x & 63;
  unsigned long long mine = 0;
  const int64_t nw = (int64_t)gridDim.x * (kBlock / 64);
  for (int64_t w0 = kWaveWords * ((int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)); w0 < b.words; w0 += kWaveWords * nw) {
    const WaveWords w = wave_words(b, B, w0, b.words);
    int32_t s[kWaveWords];
    at_run_starts(w, w0, size, 0, s);
    mine += (unsigned long long)__builtin_popcountll(w.v);
#pragma unroll
    for (int j = 0; j < kWaveWords; ++j) {
      if (s[j] <= 0) continue;
      if (s[j] < kSmall) atomicAdd(&small[s[j]], 1);
      else if (s[j] < ncnt) atomicAdd(&cnt[s[j]], 1);
    }
  }
  if (lane < kWaveWords && mine) atomicAdd(&part, mine);
  __syncthreads();
  for (int j = threadIdx.x; j < kSmall && j < ncnt; j += blockDim.x)
    if (small[j]) atomicAdd(&cnt[j], small[j]);
  if (threadIdx.x == 0 && part) atomicAdd(total, part);
}

// One block: the budget floor(kDropFrac * total) (the rule's comparison in
// fp64), then a walk over sizes 1..budget in order, a block-wide scan per
// chunk of 1024 sizes, to the first size that does not fit whole.
__global__ __launch_bounds__(1024) void k_drop_find(const int32_t* __restrict__ cnt,
                                                    const unsigned long long* __restrict__ total, DropRule* rule) {
  __shared__ unsigned long long sc[1024];
  __shared__ int done;
  __shared__ unsigned long long base_s;
  const unsigned long long t = *total;
  const long long bud = (long long)floor(kDropFrac * (double)t);
  if (threadIdx.x == 0) {
    done = 0;
    base_s = 0;
    rule->total = (long long)t;
    rule->budget = bud;
    rule->s_star = (int32_t)(bud + 1);   // every size <= budget fits: the first size > budget stops the walk
    rule->m = 0;
    rule->first = 0;
  }
  __syncthreads();
  for (long long s0 = 1; s0 <= bud; s0 += 1024) {
    const long long s = s0 + threadIdx.x;
    const unsigned long long w = s <= bud ? (unsigned long long)cnt[s] * (unsigned long long)s : 0ull;
    sc[threadIdx.x] = w;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
      const unsigned long long a = threadIdx.x >= off ? sc[threadIdx.x - off] : 0ull;
      __syncthreads();
      sc[threadIdx.x] += a;
      __syncthreads();
    }
    const unsigned long long below = base_s + sc[threadIdx.x] - w;   // pixels of all sizes < s
    // s is the first size that does not fit whole: below fits, below + w does not
    if (s <= bud && below + w > (unsigned long long)bud && below <= (unsigned long long)bud) {
      // exactly one thread can see this (the running total crosses once)
      rule->s_star = (int32_t)s;
      rule->m = (int32_t)(((unsigned long long)bud - below) / (unsigned long long)s);
      done = 1;
    }
    __syncthreads();
    if (done) break;
    if (threadIdx.x == 1023) base_s += sc[1023];
    __syncthreads();
  }
}

// Exclusive scan of one value per thread across a block of kWaves wavefronts:
// wavefront scans by shuffles, then the wavefront totals through LDS.
__device__ __forceinline__ uint32_t wave_scan_incl(uint32_t v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t a = (uint32_t)__shfl_up((int)v, off);
    if (lane >= off) v += a;
  }
  return v;
}
template <int kWaves>
__device__ __forceinline__ uint32_t block_scan_excl(uint32_t v, uint32_t* wtot, uint32_t& total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const uint32_t incl = wave_scan_incl(v);
  if (lane == 63) wtot[wv] = incl;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int j = 0; j < kWaves; ++j) {
    const uint32_t t = wtot[j];
    before += j < wv ? t : 0u;
    all += t;
  }
  __syncthreads();   // wtot may be rewritten after this
  total = all;
  return before + incl - v;
}
// Sum of the counts of the blocks before this one (at most kSelBlocks of them).
__device__ __forceinline__ uint32_t counts_before(const uint32_t* bsum, uint32_t* wtot) {
  uint32_t v = 0;
  for (int j = threadIdx.x; j < (int)blockIdx.x; j += blockDim.x) v += bsum[j];
  uint32_t all;
  block_scan_excl<kBlock / 64>(v, wtot, all);
  return all;
}

// Roots of size s* per block of b.per words (at run starts, as k_drop_count).
__global__ __launch_bounds__(kBlock) void k_root_count(Bits b, const unsigned long long* __restrict__ B,
                                                       const int32_t* __restrict__ size, const DropRule* rule,
                                                       uint32_t* bsum) {
  __shared__ uint32_t part;
  if (threadIdx.x == 0) part = 0;
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int32_t s_star = rule->s_star;
  uint32_t mine = 0;
  if (rule->m > 0) {
    const int64_t w_end = min((int64_t)(blockIdx.x + 1) * b.per, b.words);
    for (int64_t w0 = (int64_t)blockIdx.x * b.per + kWaveWords * wv; w0 < w_end; w0 += kSelWords) {
      int32_t s[kWaveWords];
      at_run_starts(wave_words(b, B, w0, w_end), w0, size, 0, s);
#pragma unroll
      for (int j = 0; j < kWaveWords; ++j)
        mine += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(s[j] == s_star));   // s* >= 1
    }
  }
  if (lane == 0 && mine) atomicAdd(&part, mine);
  __syncthreads();
  if (threadIdx.x == 0) bsum[blockIdx.x] = part;
}

// One block: the first kept root of size s*, the one with m such roots before
// it in raster order (there is one: s* does not fit whole).
__global__ __launch_bounds__(1024) void k_root_find(Bits b, const unsigned long long* __restrict__ B,
                                                    const int32_t* __restrict__ size, const uint32_t* __restrict__ bsum,
                                                    int nb, DropRule* rule) {
  __shared__ uint32_t wtot[16];
  __shared__ int blk_s;
  __shared__ uint32_t left_s;
  const uint32_t m = (uint32_t)rule->m;
  if (m == 0) return;
  constexpr int kPer = kSelBlocks / 1024;
  uint32_t v[kPer], sum = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int j = threadIdx.x * kPer + k;
    v[k] = j < nb ? bsum[j] : 0u;
    sum += v[k];
  }
  uint32_t all, before = block_scan_excl<16>(sum, wtot, all);
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    if (before <= m && m < before + v[k]) { blk_s = threadIdx.x * kPer + k; left_s = m - before; }
    before += v[k];
  }
  __syncthreads();
  if (threadIdx.x >= 64) return;
  // one wavefront walks the block's words
  const int lane = threadIdx.x;
  const int32_t s_star = rule->s_star;
  uint32_t left = left_s;
  const int64_t w_end = min((int64_t)(blk_s + 1) * b.per, b.words);
  for (int64_t w0 = (int64_t)blk_s * b.per; w0 < w_end; w0 += kWaveWords) {
    const WaveWords w = wave_words(b, B, w0, w_end);
    int32_t s[kWaveWords];
    at_run_starts(w, w0, size, 0, s);
#pragma unroll
    for (int j = 0; j < kWaveWords; ++j) {
      const unsigned long long m = w.word(j), starts = m & ~(m << 1);
      const unsigned long long hm = __builtin_amdgcn_ballot_w64(s[j] == s_star);
      const uint32_t c = (uint32_t)__builtin_popcountll(hm);
      if (left < c) {
        if (s[j] == s_star && (uint32_t)__builtin_popcountll(hm & ((1ull << lane) - 1ull)) == left)
          rule->first = node_of(w0 + j, starts);
        return;
      }
      left -= c;
    }
  }
}

// Kept pixels: those of components that pass the filter. A component's root and size
// are looked up once per horizontal run and word, at the run's first pixel, 64 runs at
// a time from a queue in LDS (word by word, most lanes idle: 22 us at 4096x2304, 15 us
// so); the runs that pass go out whole by one addition (adding a run's start bit
// clears the run). kept (optional): kept pixels; base: kept pixels and border columns;
// refined (optional): the kept map as bytes; bsum (optional): base pixels per block;
// n1 (optional): kept pixels off the border columns, in kN1Parts counters (adds to one
// word from every block queue up one after another at the memory side). With n1 every
// run's first pixel gets its component's size (roots hold it already, and no other
// pixel's is read here), which the counting passes then read without a look at the
// root.
__global__ __launch_bounds__(kBlock) void k_kept(Bits b, const unsigned long long* __restrict__ B,
                                                 const int32_t* __restrict__ parent, int32_t* size, const DropRule* rule,
                                                 int64_t min_cc, unsigned long long* kept,
                                                 unsigned long long* base, uint8_t* refined, uint32_t* bsum,
                                                 unsigned long long* n1) {
  __shared__ uint32_t nsel, nkept;
  __shared__ uint16_t runs[kBlock / 64][kWaveWords * 32];     // word << 11 | first bit << 5 | number in the word
  __shared__ uint32_t pass[kBlock / 64][2 * kWaveWords];      // the first bits of the runs that pass
  if (threadIdx.x == 0) nsel = nkept = 0u;
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int32_t s_star = rule ? rule->s_star : 0, first = rule ? rule->first : 0;
  uint32_t csel = 0, ckept = 0;
  const int64_t w_end = min((int64_t)(blockIdx.x + 1) * b.per, b.words);
  for (int64_t w0 = (int64_t)blockIdx.x * b.per + kWaveWords * wv; w0 < w_end; w0 += kSelWords) {
    const WaveWords w = wave_words(b, B, w0, w_end);
    if (lane < 2 * kWaveWords) pass[wv][lane] = 0u;
    int nn = 0;
#pragma unroll
    for (int j = 0; j < kWaveWords; ++j) {
      const unsigned long long m = w.word(j), st = m & ~(m << 1);
      if (!m) continue;
      if (__builtin_amdgcn_inverse_ballot_w64(st)) {
        const int k = node_of(0, st);
        runs[wv][nn + k] = (uint16_t)(j << 11 | lane << 5 | k);
      }
      nn += __builtin_popcountll(st);
    }
    asm volatile("" ::: "memory");   // (a wavefront's LDS operations are done in the order it issues them)
    for (int i = lane; i < nn; i += 64) {
      const uint32_t q = runs[wv][i], j = q >> 11, bit = q >> 5 & 63u;
      const int32_t n = (int32_t)(32 * (w0 + j)) + (int32_t)(q & 31u);
      const int32_t r = parent[parent[n]];   // from the tile root to the root
      const int32_t s = size[r];
      if (rule ? s > s_star || (s == s_star && r >= first) : s >= min_cc) atomicOr(&pass[wv][2 * j + (bit >> 5)], 1u << (bit & 31u));
      if (n1 && r != n) size[n] = s;
    }
    asm volatile("" ::: "memory");
    unsigned long long kv = 0ull;   // lane j: word j's kept pixels
    if (lane < kWaveWords) kv = w.v & ~(w.v + ((unsigned long long)pass[wv][2 * lane + 1] << 32 | pass[wv][2 * lane]));
    asm volatile("" ::: "memory");
    if (lane < kWaveWords && w0 + lane < w_end) {
      if (kept) kept[w0 + lane] = kv;
      base[w0 + lane] = kv | w.border;
      csel += (uint32_t)__builtin_popcountll(kv | w.border);
      ckept += (uint32_t)__builtin_popcountll(kv & ~w.border);
    }
    if (refined) {
      for (int j = 0; j < kWaveWords && w0 + j < w_end; ++j) {
        const int x = 64 * (int)((uint32_t)(w0 + j) % (uint32_t)b.wpr) + lane;
        const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)kv, j), hi = __builtin_amdgcn_readlane((uint32_t)(kv >> 32), j);
        const int i = w.first(j) + lane;
        if (x < b.W) refined[i] = (uint8_t)(((lane < 32 ? lo : hi) >> (lane & 31)) & 1u);
      }
    }
  }
  if (lane < kWaveWords) {
    atomicAdd(&nsel, csel);
    atomicAdd(&nkept, ckept);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    if (bsum) bsum[blockIdx.x] = nsel;
    if (n1 && nkept) atomicAdd(&n1[blockIdx.x % kN1Parts], (unsigned long long)nkept);
  }
}

// The list: the raster indices of the map's set pixels, in order, and their
// number. A block adds up the counts of the blocks before it (there are at
// most kSelBlocks), then its words' counts; a wavefront writes a word's
// pixels with one lane each, side by side.
__global__ __launch_bounds__(kBlock) void k_list(Bits b, const unsigned long long* __restrict__ sel,
                                                 const uint32_t* __restrict__ bsum, uint32_t* out, long long* count) {
  __shared__ uint32_t wtot[kBlock / 64];
  __shared__ uint32_t pre[kSelWords], first[kSelWords];
  __shared__ unsigned long long word[kSelWords];
  uint32_t pos = counts_before(bsum, wtot);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t w_end = min((int64_t)(blockIdx.x + 1) * b.per, b.words);
  for (int64_t w0 = (int64_t)blockIdx.x * b.per; w0 < w_end; w0 += kSelWords) {
    unsigned long long w = 0ull;
    if (threadIdx.x < kSelWords && w0 + threadIdx.x < w_end) w = sel[w0 + threadIdx.x];
    uint32_t all;
    const uint32_t before = block_scan_excl<kBlock / 64>((uint32_t)__builtin_popcountll(w), wtot, all);
    if (threadIdx.x < kSelWords) {
      pre[threadIdx.x] = before;
      word[threadIdx.x] = w;
      first[threadIdx.x] = (uint32_t)word_pos(b, w0 + threadIdx.x).i;
    }
    __syncthreads();
#pragma unroll 4
    for (int j = wv * kWaveWords; j < (wv + 1) * kWaveWords; ++j) {
      const unsigned long long mv = word[j];
      const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)mv), hi = __builtin_amdgcn_readfirstlane((uint32_t)(mv >> 32));
      if (__builtin_amdgcn_inverse_ballot_w64((unsigned long long)hi << 32 | lo))
        out[pos + pre[j] + __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u))] = first[j] + lane;
    }
    pos += all;
    __syncthreads();   // pre and word are rewritten
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *count = (long long)pos;
}

// ---------------------------------------------------------------------------
// Fraction control (a benchmark knob, not the paper's): exactly `want`
// pixels ranked as (1) border columns by raster index, (2) kept pixels by
// component size descending, then raster index, (3) all other pixels by
// chessboard distance to (1)+(2) ascending, then h(i) = mix64(i ^ seed). The
// selection is threshold-based: counting passes find the key of the want-th
// pixel within the class it falls in; ties of (2) at that key go by raster
// order, and h takes every index to a different value, so (3) has none.
struct FcArgs {
  long long want, n0;             // pixels wanted; border pixels
  const unsigned long long* n1;   // kept pixels off the border, in kN1Parts parts
  unsigned long long seed;
};
struct FcPlan {
  int mode;         // the class the want-th pixel falls in: 0 border columns, 1 kept pixels, 2 other pixels
  long long need;   // its rank (1-based) in that class
};
// Worked out by every wavefront that asks (one load and six adds).
__device__ __forceinline__ FcPlan fc_plan(const FcArgs& a) {
  static_assert(kN1Parts == 64, "one part per lane");
  unsigned long long n = a.n1[threadIdx.x & 63];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) n += __shfl_xor(n, off, 64);
  const long long n1 = (long long)n;
  if (a.want <= a.n0) return FcPlan{0, a.want};
  if (a.want <= a.n0 + n1) return FcPlan{1, a.want - a.n0};
  return FcPlan{2, a.want - a.n0 - n1};
}

// SplitMix64's output function (Steele, Lea and Flood; constants as
// published by Vigna), on the raster index xor the seed. Each of its steps
// is invertible, so different indices have different values.
__device__ __forceinline__ unsigned long long mix64(unsigned long long z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ULL;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBULL;
  return z ^ (z >> 31);
}

// Counting select, kDigit bits per pass from the top: a pass counts the
// digits of the keys that match the digits found so far; the next one finds
// the digit whose count range holds the wanted rank before it counts.
constexpr int kDigit = 12, kBins = 1 << kDigit;
struct RadixSel {
  unsigned long long prefix;   // key bits found so far (top digits first)
  long long need;              // rank (1-based) of the wanted key
  long long below;             // keys smaller than those with the prefix
};
// The state after the counts of a pass at `shift` (the whole block works it
// out; block 0 writes it to `out` for later launches).
__device__ __forceinline__ RadixSel sel_pick(RadixSel r, const uint32_t* hist, int shift, RadixSel* out) {
  __shared__ uint32_t wtot[kBlock / 64];
  __shared__ unsigned long long found_d;
  __shared__ long long found_below;
  constexpr int kPer = kBins / kBlock;
  uint32_t v[kPer], sum = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) { v[k] = hist[threadIdx.x * kPer + k]; sum += v[k]; }
  uint32_t all;
  long long before = r.below + (long long)block_scan_excl<kBlock / 64>(sum, wtot, all);
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    if (before < r.need && r.need <= before + (long long)v[k]) {
      found_d = (unsigned long long)(threadIdx.x * kPer + k);
      found_below = before;
    }
    before += v[k];
  }
  __syncthreads();
  r.prefix |= found_d << shift;   // (the wanted rank lies within the counts: need <= keys of the class)
  r.below = found_below;
  if (out && blockIdx.x == 0 && threadIdx.x == 0) *out = r;
  __syncthreads();
  return r;
}

// Mode 1, one counting pass over the kept pixels' keys ~size.
__device__ __forceinline__ void size_pass(const Bits& b, const unsigned long long* B, const unsigned long long* kept,
                                          const int32_t* size, RadixSel rs, const uint32_t* prev_hist, int prev_shift,
                                          RadixSel* state, int shift, uint32_t* hist, uint32_t* bins, int blocks) {
  if (prev_hist) rs = sel_pick(rs, prev_hist, prev_shift, state);
  for (int k = threadIdx.x; k < kBins; k += kBlock) bins[k] = 0u;
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int hi = shift + kDigit;
  const int64_t nw = (int64_t)blocks * (kBlock / 64);
  for (int64_t w0 = kWaveWords * ((int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)); w0 < b.words; w0 += kWaveWords * nw) {
    const WaveWords w = wave_words(b, kept, w0, b.words);
    int32_t s[kWaveWords];
    at_kept_runs(w, wave_words(b, B, w0, b.words), w0, size, s);
#pragma unroll
    for (int j = 0; j < kWaveWords; ++j) {
      const unsigned long long m = w.word(j);
      if (!m) continue;
      const uint32_t key = ~(uint32_t)s[j];   // one add per run, of its pixels off the border columns
      const unsigned long long bd = w.border_of(j);
      if (s[j] > 0 && (hi >= 32 || (key >> hi) == (uint32_t)(rs.prefix >> hi)))
        atomicAdd(&bins[(key >> shift) & (kBins - 1)], (uint32_t)__builtin_popcountll(run_from(m, lane) & ~bd));
    }
  }
  __syncthreads();
  for (int k = threadIdx.x; k < kBins; k += kBlock)
    if (bins[k]) atomicAdd(&hist[k], bins[k]);
}

// The counting passes of mode 1, from the keys' top digit at `top` down: the
// state after pass p's pick is state[p], its counts are hist[p * kBins ..].
struct SizeSel {
  const unsigned long long *B, *kept;
  const int32_t* size;
  unsigned long long prefix;   // digits known beforehand
  int top;                     // shift of the first pass: (passes - 1) kDigit
  RadixSel* state;
  uint32_t* hist;
  int blocks;                  // that count: each ends with up to kBins adds to memory
};
__device__ __forceinline__ void size_digit(const Bits& b, const SizeSel& z, int pass, long long need, uint32_t* bins) {
  if ((int)blockIdx.x >= z.blocks) return;
  const int shift = z.top - pass * kDigit;
  const RadixSel in = pass < 2 ? RadixSel{z.prefix, need, 0} : z.state[pass - 2];
  size_pass(b, z.B, z.kept, z.size, in, pass ? z.hist + (pass - 1) * kBins : nullptr, shift + kDigit,
            pass ? z.state + pass - 1 : nullptr, shift, z.hist + pass * kBins, bins, z.blocks);
}
// The size of mode 1's want-th pixel, after the last pass.
__device__ __forceinline__ RadixSel size_found(const SizeSel& z, long long need) {
  const int last = z.top / kDigit;
  return sel_pick(last ? z.state[last - 1] : RadixSel{z.prefix, need, 0}, z.hist + last * kBins, 0, nullptr);
}

constexpr int kSegRows = 32;   // rows per column segment of the distance passes
// Per (word column, 32-row segment): the columns with a base pixel in it.
__device__ __forceinline__ void far_segments(const Bits& b, const unsigned long long* base, int nseg,
                                             unsigned long long* segor) {
  for (int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x; t < (int64_t)nseg * b.wpr; t += (int64_t)gridDim.x * kBlock) {
    const int sg = (int)(t / b.wpr), c = (int)(t % b.wpr);
    const int y0 = sg * kSegRows, n = min(b.H - y0, kSegRows);
    unsigned long long v[kSegRows], m = 0ull;
#pragma unroll
    for (int k = 0; k < kSegRows; ++k) v[k] = k < n ? base[(int64_t)(y0 + k) * b.wpr + c] : 0ull;
#pragma unroll
    for (int k = 0; k < kSegRows; ++k) m |= v[k];
    segor[t] = m;
  }
}

// Mode 2: distances up to kLevels by dilation of the base map, 3 x 3 per level, on
// bits: a wavefront holds 128 rows (two per lane) x 192 columns in registers, rows
// beyond a lane's own by DPP, and keeps the inner 98 rows x 128 columns, which none of
// a launch's 15 levels reaches from outside. A pixel's level goes to kLevelBits planes
// (0 for base pixels and those further away) and the pixels per level are counted, in
// kLvParts copies. A second launch goes on from the first one's outcome where the
// want-th pixel lies further away: 15 levels cover the workloads' lists (31 in one
// launch keep a quarter of what a wavefront holds: 26 us at 4096x2304 against 20).
// Pixels beyond both take the distance passes below (k_far_*).
constexpr int kLevelBits = 5, kLvStage = 15, kLevels = 2 * kLvStage + 1, kLvParts = 64;   // levels 1 .. 15 and 16 .. 30
constexpr int kLvRows = 128 - 2 * kLvStage;   // 98
constexpr int kLvWords = 6;                   // 32-column words held, the inner four kept

__device__ __forceinline__ uint32_t lane_up(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xf, 0xf, false);   // wave_shr:1, zeros in
}
__device__ __forceinline__ uint32_t lane_down(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x130, 0xf, 0xf, false);   // wave_shl:1, zeros in
}

struct LevelSel {
  int level;
  long long need;
};
// This thread's part of the level counts: loaded before anything is decided,
// with the plan's own load (one after the other, and the hash counts after
// them, were three round trips to memory at the start of each of five
// launches); kept() holds the loads there.
struct LevelCounts {
  uint32_t v[kLvParts / 8];
  __device__ __forceinline__ explicit LevelCounts(const uint32_t* lcount) {
    // thread t adds up every 8th part of level t % 32
    static_assert(kBlock == 8 * (kLevels + 1) && kLvParts % 8 == 0, "threads cover the levels eight times");
#pragma unroll
    for (int k = 0; k < kLvParts / 8; ++k) v[k] = lcount[threadIdx.x + 8 * (kLevels + 1) * k];
  }
  __device__ __forceinline__ void kept() const {
#pragma unroll
    for (int k = 0; k < kLvParts / 8; ++k) asm volatile("" ::"v"(v[k]));
  }
};
__device__ __forceinline__ LevelSel level_pick(const LevelCounts& lc, long long need, int last = kLevels);

// Planes 0 .. 3 of a map word lie side by side, plane 4 apart after them (it
// is read for levels above 15 only). STAGE 0: levels 1 .. 15 of `from` (the
// base map), and the pixels reached to `reach`. STAGE 1: levels 16 .. 30 of
// `from` (what stage 0 reached) into the planes, and what the distance passes
// need of the base map's columns in case that they follow.
// The first two counting passes of mode 1 take these launches' places (one of
// the two modes has nothing to do in them, and an idle launch costs 5 us of
// the device and 8 us of the caller's thread): gx x gy blocks for the levels,
// in a row, further ones for the counting.
template <int STAGE>
__global__ __launch_bounds__(kBlock) void k_fc_levels(Bits b, FcArgs a, SizeSel z, int gx, int gy,
                                                      const unsigned long long* __restrict__ from,
                                                      unsigned long long* __restrict__ planes,
                                                      unsigned long long* __restrict__ reach, uint32_t* lcount,
                                                      const unsigned long long* __restrict__ base, int nseg,
                                                      unsigned long long* __restrict__ segor) {
  __shared__ uint32_t bins[kBins];
  uint32_t* cnt = bins;   // the levels' counts
  const LevelCounts lc(lcount);
  const FcPlan plan = fc_plan(a);
  if constexpr (STAGE == 1) lc.kept();
  if (plan.mode == 1) size_digit(b, z, STAGE, plan.need, bins);
  if (plan.mode != 2) return;
  if constexpr (STAGE == 1) {
    if (level_pick(lc, plan.need, kLvStage).level != 0) return;   // (other blocks may have added to the levels beyond)
    far_segments(b, base, nseg, segor);
  }
  if ((int)blockIdx.x >= gx * gy) return;
  const int bx = (int)blockIdx.x % gx, by = (int)blockIdx.x / gx;
  if (threadIdx.x < kLvStage) cnt[threadIdx.x] = 0u;
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int c = 2 * (bx * (kBlock / 64) + (int)(threadIdx.x >> 6));   // the first of the wavefront's two word columns
  const int y0 = by * kLvRows;
  if (c < b.wpr) {
    constexpr int M = kLvWords;
    const uint32_t* src = (const uint32_t*)from;   // 32-bit halves of the map's words, low half first
    uint32_t cur[2][M], in[2][M - 2], pl[4][2][M - 2], got[2][M - 2];
    int y[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      y[r] = y0 - kLvStage + 2 * lane + r;
      const bool row = y[r] >= 0 && y[r] < b.H;
#pragma unroll
      for (int i = 0; i < M; ++i) {
        const int w = 2 * c - 1 + i;
        cur[r][i] = row && w >= 0 && w < 2 * b.wpr ? src[(int64_t)y[r] * 2 * b.wpr + w] : 0u;
      }
      // inner pixels inside the image
      const bool inner = row && y[r] >= y0 && y[r] < y0 + kLvRows;
#pragma unroll
      for (int i = 0; i < M - 2; ++i) {
        const int left = b.W - (64 * c + 32 * i);   // columns of the image from the word's first on
        in[r][i] = !inner || left <= 0 ? 0u : (left >= 32 ? ~0u : (1u << left) - 1u);
        got[r][i] = 0u;
#pragma unroll
        for (int p = 0; p < 4; ++p) pl[p][r][i] = 0u;
      }
    }
#pragma unroll 1
    for (int k = 0; k < kLvStage; ++k) {
      const int code = STAGE == 0 ? k + 1 : k;   // the low four bits of the level
      uint32_t h[2][M];
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int i = 0; i < M; ++i)
          h[r][i] = cur[r][i] | __builtin_amdgcn_alignbit(cur[r][i], i > 0 ? cur[r][i - 1] : 0u, 31) |
                    __builtin_amdgcn_alignbit(i < M - 1 ? cur[r][i + 1] : 0u, cur[r][i], 1);
      uint32_t n = 0u, rest = 0u;
#pragma unroll
      for (int i = 0; i < M; ++i) {
        const uint32_t both = h[0][i] | h[1][i];
        const uint32_t v[2] = {both | lane_up(h[1][i]), both | lane_down(h[0][i])};
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          if (i >= 1 && i < M - 1) {
            const uint32_t d = v[r] & ~cur[r][i] & in[r][i - 1];
            n += __builtin_popcount(d);
            rest |= in[r][i - 1] & ~v[r];
            got[r][i - 1] |= d;
#pragma unroll
            for (int p = 0; p < 4; ++p)
              if (code >> p & 1) pl[p][r][i - 1] |= d;
          }
          cur[r][i] = v[r];
        }
      }
      // sums over rows of 16 lanes, then one LDS add per row of lanes
      n += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)n, 0x111, 0xf, 0xf, false);
      n += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)n, 0x112, 0xf, 0xf, false);
      n += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)n, 0x114, 0xf, 0xf, false);
      n += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)n, 0x118, 0xf, 0xf, false);
      if ((lane & 15) == 15 && n) atomicAdd(&cnt[k], n);
      if (!__builtin_amdgcn_ballot_w64(rest != 0u)) break;   // every inner pixel reached
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      if (y[r] < y0 || y[r] >= y0 + kLvRows || y[r] >= b.H) continue;
#pragma unroll
      for (int j = 0; j < (M - 2) / 2; ++j) {
        if (c + j >= b.wpr) continue;
        const int64_t at = (int64_t)y[r] * b.wpr + c + j;
        auto word = [](uint32_t lo, uint32_t hi) { return (unsigned long long)lo | (unsigned long long)hi << 32; };
        unsigned long long v[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) v[p] = word(pl[p][r][2 * j], pl[p][r][2 * j + 1]);
        ulonglong2* q = (ulonglong2*)(planes + 4 * at);
        if constexpr (STAGE == 1) {
          const ulonglong2 lo = q[0], hi = q[1];
          v[0] |= lo.x; v[1] |= lo.y; v[2] |= hi.x; v[3] |= hi.y;
          planes[4 * b.words + at] = word(got[r][2 * j], got[r][2 * j + 1]);
        } else {
          reach[at] = word(cur[r][2 * j + 1] & in[r][2 * j], cur[r][2 * j + 2] & in[r][2 * j + 1]);
        }
        q[0] = ulonglong2{v[0], v[1]};
        q[1] = ulonglong2{v[2], v[3]};
      }
    }
  }
  __syncthreads();
  const int part = (int)(blockIdx.x % kLvParts);
  if (threadIdx.x < kLvStage && cnt[threadIdx.x])
    atomicAdd(&lcount[part * (kLevels + 1) + 1 + STAGE * kLvStage + threadIdx.x], cnt[threadIdx.x]);
}

// Mode 2: the level of the want-th pixel and its rank within it, from the
// counts of levels up to `last`; level 0: it lies further away than those.
__device__ __forceinline__ LevelSel level_pick(const LevelCounts& lc, long long need, int last) {
  __shared__ unsigned long long sum[kLevels + 1];
  if (threadIdx.x <= kLevels) sum[threadIdx.x] = 0ull;
  __syncthreads();
  unsigned long long s = 0ull;
#pragma unroll
  for (int k = 0; k < kLvParts / 8; ++k) s += lc.v[k];
  if (s) atomicAdd(&sum[threadIdx.x % (kLevels + 1)], s);
  __syncthreads();
  LevelSel r{0, need};
  for (int k = 1; k <= last; ++k) {
    const long long n = (long long)sum[k];
    if (r.need <= n) { r.level = k; break; }
    r.need -= n;
  }
  __syncthreads();
  return r;
}
// ... and once the distance passes have run: they leave levels 1 (nearer than
// the wanted distance) and 2 (at it) in the planes, and the rank in `far`.
__device__ __forceinline__ LevelSel level_final(const LevelCounts& lc, const long long* far_need, long long need) {
  LevelSel r = level_pick(lc, need);
  if (r.level == 0) { r.level = 2; r.need = *far_need; }
  return r;
}
struct LevelWords {
  unsigned long long inner, ring;   // pixels of lower levels (not 0), and of the level
};
__device__ __forceinline__ LevelWords level_words(const Bits& b, const unsigned long long* planes, int64_t wi, int level) {
  const ulonglong2* q = (const ulonglong2*)(planes + 4 * wi);
  const ulonglong2 lo = q[0], hi = q[1];
  const unsigned long long p[kLevelBits] = {lo.x, lo.y, hi.x, hi.y, level > kLvStage ? planes[4 * b.words + wi] : 0ull};
  unsigned long long lt = 0ull, eq = ~0ull, any = 0ull;
#pragma unroll
  for (int k = kLevelBits - 1; k >= 0; --k) {
    any |= p[k];
    if (level >> k & 1) { lt |= eq & ~p[k]; eq &= p[k]; }
    else eq &= ~p[k];
  }
  return LevelWords{lt & any, eq & any};
}

// Mode 2, the ring (other pixels at the wanted distance): counts of the top
// kHashDigit bits of h, gathered in LDS, in kHashParts copies (one add to
// memory per pixel into 2^14 bins took 26 us at 4096x2304, 2^8 bins in LDS 16
// us and left lists that do not fit the LDS of those that rank them; 2^10 bins
// 11 us).
constexpr int kHashDigit = 10, kHashBins = 1 << kHashDigit, kHashParts = 4;
static_assert(kHashBins == 4 * kBlock, "four bins per thread");
// f(i) for the block's ring pixels i: the words' set bits are queued in LDS
// first and then taken by all threads alike, since a ring fills some words and
// leaves most empty. `blocks` blocks take `chunk` words (at most kRingWords) in
// turn, each after prepare(their first word).
constexpr int kRingWords = kBlock;          // words a block queues at a time
template <typename P, typename F>
__device__ __forceinline__ void for_ring(const Bits& b, const unsigned long long* planes, int level, int blocks,
                                         int chunk, P prepare, F f) {
  __shared__ uint16_t queue[64 * kRingWords];   // word << 6 | bit
  __shared__ int first[kRingWords];
  __shared__ uint32_t wtot[kBlock / 64];
  for (int64_t w0 = (int64_t)blockIdx.x * chunk; w0 < b.words; w0 += (int64_t)blocks * chunk) {
    prepare(w0);
    const int64_t wi = w0 + threadIdx.x;
    unsigned long long m = (int)threadIdx.x < chunk && wi < b.words ? level_words(b, planes, wi, level).ring : 0ull;
    uint32_t all;
    uint32_t at = block_scan_excl<kBlock / 64>((uint32_t)__builtin_popcountll(m), wtot, all);
    if (m) first[threadIdx.x] = word_pos(b, wi).i;
    for (; m; m &= m - 1ull) queue[at++] = (uint16_t)(threadIdx.x << 6 | (uint32_t)__builtin_ctzll(m));
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < all; k += kBlock) f((uint32_t)(first[queue[k] >> 6] + (queue[k] & 63)));
    __syncthreads();   // the queue is rewritten
  }
}
// The hashes of the ring's pixels in the bin that holds the wanted rank, and
// the rank within it.
struct RingBin {
  long long need;
  unsigned long long n;   // hashes listed
};
__global__ __launch_bounds__(kBlock) void k_ring_bin(Bits b, FcArgs a, const unsigned long long* __restrict__ planes,
                                                     const uint32_t* __restrict__ lcount,
                                                     const long long* __restrict__ far_need,
                                                     const uint32_t* __restrict__ hash_hist, RingBin* rb,
                                                     unsigned long long* list) {
  constexpr int kHold = 512;
  __shared__ uint32_t wtot[kBlock / 64];
  __shared__ uint32_t bin_s, held;
  __shared__ long long need_s;
  __shared__ unsigned long long hold[kHold], at_s;
  const LevelCounts lc(lcount);
  uint32_t v[4] = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int q = 0; q < kHashParts; ++q) {
    const uint4 h = ((const uint4*)(hash_hist + q * kHashBins))[threadIdx.x];
    v[0] += h.x; v[1] += h.y; v[2] += h.z; v[3] += h.w;
  }
  const FcPlan pl = fc_plan(a);
  lc.kept();
#pragma unroll
  for (int j = 0; j < 4; ++j) asm volatile("" ::"v"(v[j]));
  if (pl.mode != 2) return;
  if (threadIdx.x == 0) held = 0u;
  const LevelSel ls = level_final(lc, far_need, pl.need);
  uint32_t all;
  long long before = (long long)block_scan_excl<kBlock / 64>(v[0] + v[1] + v[2] + v[3], wtot, all);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (before < ls.need && ls.need <= before + (long long)v[j]) {
      bin_s = 4u * threadIdx.x + (uint32_t)j;
      need_s = ls.need - before;
    }
    before += v[j];
  }
  __syncthreads();
  const unsigned long long bin = bin_s;
  if (blockIdx.x == 0 && threadIdx.x == 0) rb->need = need_s;
  // held in LDS first, so that a block takes its places in the list at once
  for_ring(b, planes, ls.level, (int)gridDim.x, kRingWords, [](int64_t) {}, [&](uint32_t i) {
    const unsigned long long h = mix64((unsigned long long)i ^ a.seed);
    if (h >> (64 - kHashDigit) != bin) return;
    const uint32_t k = atomicAdd(&held, 1u);
    if (k < kHold) hold[k] = h;
    else list[atomicAdd(&rb->n, 1ull)] = h;
  });
  __syncthreads();
  const int n = (int)min(held, (uint32_t)kHold);
  if (threadIdx.x == 0 && n) at_s = atomicAdd(&rb->n, (unsigned long long)n);
  __syncthreads();
  for (int k = threadIdx.x; k < n; k += kBlock) list[at_s + k] = hold[k];
}

// The hash of rank rb->need among the listed ones (they differ): the listed
// hashes in LDS where they fit, narrowed digit by digit to a few, which are
// ranked against each other.
__device__ __forceinline__ unsigned long long ring_threshold(const RingBin* rb, const unsigned long long* list) {
  constexpr int kKeys = 1536, kFew = 256;
  __shared__ unsigned long long keys[kKeys], few[kFew], thr;
  __shared__ uint32_t hist[256], wtot[kBlock / 64], nfew, dig_s, cnt_s;
  __shared__ long long need_s;
  const int64_t m = (int64_t)rb->n;
  const bool in_lds = m <= kKeys;
  if (in_lds)
    for (int t = threadIdx.x; t < (int)m; t += kBlock) keys[t] = list[t];
  const unsigned long long* src = in_lds ? keys : list;
  long long need = rb->need;
  int shift = 64 - kHashDigit;
  unsigned long long prefix = 0ull;
  bool first = true;   // nothing fixed beyond the bin yet
  int64_t count = m;
  while (count > kFew && shift > 0) {
    const int next = shift > 8 ? shift - 8 : 0;
    hist[threadIdx.x] = 0u;
    __syncthreads();
    for (int64_t t = threadIdx.x; t < m; t += kBlock) {
      const unsigned long long k = src[t];
      if (first || k >> shift == prefix) atomicAdd(&hist[(k >> next) & ((1ull << (shift - next)) - 1ull)], 1u);
    }
    __syncthreads();
    const uint32_t v = hist[threadIdx.x];
    uint32_t all;
    const long long before = (long long)block_scan_excl<kBlock / 64>(v, wtot, all);
    if (before < need && need <= before + (long long)v) { dig_s = threadIdx.x; cnt_s = v; need_s = need - before; }
    if (first && threadIdx.x == 0) thr = src[0] >> shift;   // the bin's own bits
    __syncthreads();
    if (first) prefix = thr;
    prefix = prefix << (shift - next) | dig_s;
    need = need_s;
    count = cnt_s;
    shift = next;
    first = false;
    __syncthreads();
  }
  if (threadIdx.x == 0) nfew = 0u;
  __syncthreads();
  for (int64_t t = threadIdx.x; t < m; t += kBlock) {
    const unsigned long long k = src[t];
    if (first || k >> shift == prefix) few[atomicAdd(&nfew, 1u)] = k;   // at most kFew (one once every digit is fixed)
  }
  __syncthreads();
  if (threadIdx.x < nfew) {
    const unsigned long long k = few[threadIdx.x];
    long long below = 0;
    for (uint32_t j = 0; j < nfew; ++j) below += few[j] < k ? 1 : 0;
    if (below == need - 1) thr = k;
  }
  __syncthreads();
  return thr;
}

// The selected pixels as a map, and their number per block of b.per words.
__global__ __launch_bounds__(kBlock) void k_fc_select(Bits b, FcArgs a, const unsigned long long* __restrict__ base,
                                                      SizeSel z, const uint32_t* __restrict__ ties,
                                                      const unsigned long long* __restrict__ planes,
                                                      const uint32_t* __restrict__ lcount,
                                                      const long long* __restrict__ far_need,
                                                      const RingBin* __restrict__ rb,
                                                      const unsigned long long* __restrict__ ring,
                                                      unsigned long long* sel, uint32_t* bsum) {
  __shared__ uint32_t wtot[kBlock / 64];
  __shared__ uint32_t nsel;
  __shared__ unsigned long long tw[kSelWords], ow[kSelWords];
  if (threadIdx.x == 0) nsel = 0u;
  const LevelCounts lc(lcount);
  const FcPlan pl = fc_plan(a);
  lc.kept();
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t w_begin = (int64_t)blockIdx.x * b.per, w_end = min(w_begin + b.per, b.words);
  uint32_t c = 0;
  __syncthreads();
  if (pl.mode == 2) {
    const LevelSel ls = level_final(lc, far_need, pl.need);
    const unsigned long long thr = ring_threshold(rb, ring);
    for (int64_t wi = w_begin + threadIdx.x; wi < w_end; wi += kBlock) {
      const LevelWords lw = level_words(b, planes, wi, ls.level);
      const WordPos p = word_pos(b, wi);
      const int64_t i0 = p.i;
      unsigned long long s = base[wi] | lw.inner;
      for (unsigned long long r = lw.ring; r; r &= r - 1ull) {
        const int k = __builtin_ctzll(r);
        if (mix64((unsigned long long)(i0 + k) ^ a.seed) <= thr) s |= 1ull << k;
      }
      sel[wi] = s;
      c += (uint32_t)__builtin_popcountll(s);
    }
  } else if (pl.mode == 0) {
    // border columns by raster index
    for (int64_t wi = w_begin + threadIdx.x; wi < w_end; wi += kBlock) {
      const WordPos p = word_pos(b, wi);
      const long long left = b.W == 1 ? p.y : 2LL * p.y, right = b.W == 1 ? p.y : 2LL * p.y + 1;   // their ranks
      unsigned long long s = 0ull;
      if (p.c == 0 && left < a.want) s |= 1ull;
      if (p.c == b.wpr - 1 && right < a.want) s |= 1ull << ((b.W - 1) & 63);
      sel[wi] = s;
      c += (uint32_t)__builtin_popcountll(s);
    }
  } else {
    // kept pixels of larger components, and the first of those of size s* in
    // raster order: ties before this block from the blocks' counts
    const RadixSel rs = size_found(z, pl.need);
    const uint32_t s_star = ~(uint32_t)rs.prefix;
    long long quota = rs.need - rs.below - (long long)counts_before(ties, wtot);
    for (int64_t w0 = w_begin; w0 < w_end; w0 += kSelWords) {
      const int64_t wf = w0 + kWaveWords * wv;
      const WaveWords w = wave_words(b, z.kept, wf, w_end);
      int32_t s[kWaveWords];
      at_kept_runs(w, wave_words(b, z.B, wf, w_end), wf, z.size, s);
      unsigned long long tv = 0ull, ov = 0ull;   // lane j: word j's ties, and its pixels of larger components
#pragma unroll
      for (int j = 0; j < kWaveWords; ++j) {
        const unsigned long long m = w.word(j);
        if (!m) continue;
        const unsigned long long gt = __builtin_amdgcn_ballot_w64(s[j] > 0 && (uint32_t)s[j] > s_star);
        const unsigned long long eq = __builtin_amdgcn_ballot_w64(s[j] > 0 && (uint32_t)s[j] == s_star);
        if (lane == j) { tv = m & ~(m + eq); ov = m & ~(m + gt); }
      }
      if (lane < kWaveWords) {
        tw[kWaveWords * wv + lane] = tv & ~w.border;
        ow[kWaveWords * wv + lane] = ov | w.border;
      }
      __syncthreads();
      const unsigned long long t = threadIdx.x < kSelWords ? tw[threadIdx.x] : 0ull;
      uint32_t all;
      const uint32_t before = block_scan_excl<kBlock / 64>((uint32_t)__builtin_popcountll(t), wtot, all);
      if (threadIdx.x < kSelWords && w0 + threadIdx.x < w_end) {
        unsigned long long s = ow[threadIdx.x];
        long long left = quota - (long long)before;
        for (unsigned long long m = t; m && left > 0; m &= m - 1ull, --left) s |= m & (~m + 1ull);   // the lowest set bits
        sel[w0 + threadIdx.x] = s;
        c += (uint32_t)__builtin_popcountll(s);
      }
      quota -= (long long)all;
      __syncthreads();   // tw and ow are rewritten
    }
  }
  c = wave_scan_incl(c);
  if (lane == 63 && c) atomicAdd(&nsel, c);
  __syncthreads();
  if (threadIdx.x == 0) bsum[blockIdx.x] = nsel;
}

// Mode 1: pixels of size s* per block of b.per words, for their ranks.
__device__ __forceinline__ void tie_pass(const Bits& b, const unsigned long long* B, const unsigned long long* kept, const int32_t* size,
                                         uint32_t s_star, int64_t block, uint32_t* ties, uint32_t* part) {
  if (threadIdx.x == 0) *part = 0u;
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t mine = 0;
  const int64_t w_end = min((block + 1) * b.per, b.words);
  for (int64_t w0 = block * b.per + kWaveWords * wv; w0 < w_end; w0 += kSelWords) {
    const WaveWords w = wave_words(b, kept, w0, w_end);
    int32_t s[kWaveWords];
    at_kept_runs(w, wave_words(b, B, w0, w_end), w0, size, s);
#pragma unroll
    for (int j = 0; j < kWaveWords; ++j)
      if (s[j] > 0 && (uint32_t)s[j] == s_star) mine += (uint32_t)__builtin_popcountll(run_from(w.word(j), lane) & ~w.border_of(j));
  }
  if (mine) atomicAdd(part, mine);
  __syncthreads();
  if (threadIdx.x == 0) ties[block] = *part;
  __syncthreads();
}

// ---------------------------------------------------------------------------
// Mode 2 with the want-th pixel further than kLevels from the base map:
// chessboard distances of every pixel. Per column the vertical distance g to
// the nearest base pixel, then per pixel the minimum over columns x' of
// max(|x - x'|, g(x')) (the border columns bound it).
constexpr int32_t kFar = 1 << 30;
// g for one (word column, segment) per wavefront, lane = column: inside the
// segment from its 32 words; beyond it, segment by segment away from it until
// every column has met a base pixel (or the image ends).
__device__ __forceinline__ void far_columns(const Bits& b, const unsigned long long* base, int nseg,
                                            const unsigned long long* segor, int32_t* g) {
  const int lane = threadIdx.x & 63;
  const int64_t items = (int64_t)nseg * b.wpr, nw = (int64_t)gridDim.x * (kBlock / 64);
  for (int64_t t = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); t < items; t += nw) {
    const int sg = (int)(t / b.wpr), c = (int)(t % b.wpr);
    const int y0 = sg * kSegRows, n = min(b.H - y0, kSegRows);
    const int x = 64 * c + lane;
    uint32_t sel = 0u;   // bit k: row y0 + k holds a base pixel in this column
#pragma unroll
    for (int k = 0; k < kSegRows; ++k) {
      const unsigned long long w = k < n ? base[(int64_t)(y0 + k) * b.wpr + c] : 0ull;
      sel |= (uint32_t)(w >> lane & 1ull) << k;
    }
    int up = -kFar, down = kFar;   // nearest base rows above and below the segment
    unsigned long long need = ~0ull;
    for (int s = sg - 1; s >= 0 && need; --s) {
      const unsigned long long hit = segor[(int64_t)s * b.wpr + c] & need;
      if (!hit) continue;
      need &= ~hit;
      for (int y = s * kSegRows; y < (s + 1) * kSegRows; ++y)
        if ((hit & base[(int64_t)y * b.wpr + c]) >> lane & 1ull) up = y;
    }
    need = ~0ull;
    for (int s = sg + 1; s < nseg && need; ++s) {
      const unsigned long long hit = segor[(int64_t)s * b.wpr + c] & need;
      if (!hit) continue;
      need &= ~hit;
      for (int y = min(b.H, (s + 1) * kSegRows) - 1; y >= s * kSegRows; --y)
        if ((hit & base[(int64_t)y * b.wpr + c]) >> lane & 1ull) down = y;
    }
    int gv[kSegRows];
#pragma unroll
    for (int k = 0; k < kSegRows; ++k) {
      if (sel >> k & 1u) up = y0 + k;
      gv[k] = up < 0 ? kFar : y0 + k - up;
    }
#pragma unroll
    for (int k = kSegRows - 1; k >= 0; --k) {
      if (sel >> k & 1u) down = y0 + k;
      if (down < kFar) gv[k] = min(gv[k], down - (y0 + k));
    }
    if (x < b.W) {
#pragma unroll
      for (int k = 0; k < kSegRows; ++k)
        if (k < n) g[(int64_t)(y0 + k) * b.W + x] = gv[k];
    }
  }
}

// One block per row; rows up to kRowLds pixels wide are searched in LDS,
// with the minimum of every 16 consecutive entries beside them: the search
// outwards from x skips a whole 16-entry block when even its nearest
// position and its smallest entry cannot beat the best found
// (max(|x - x'|, g(x')) >= max(distance to the block, block minimum)), so a
// pixel far from the selected set costs about d/16 + 32 steps, not d.
constexpr int kRowLds = 8192;
constexpr int kDtBlk = 16;
__global__ __launch_bounds__(kBlock) void k_far_row(Bits b, const int32_t* far, const int32_t* g, int32_t* dist) {
  __shared__ int32_t row[kRowLds];
  __shared__ int32_t bmin[kRowLds / kDtBlk];
  if (!*far) return;
  const int W = b.W, H = b.H;
  const bool in_lds = W <= kRowLds;
  const int nb = (W + kDtBlk - 1) / kDtBlk;
  for (int y = blockIdx.x; y < H; y += gridDim.x) {
    const int32_t* grow = g + (int64_t)y * W;
    if (in_lds) {
      for (int x = threadIdx.x; x < W; x += blockDim.x) row[x] = grow[x];
      __syncthreads();
      for (int b = threadIdx.x; b < nb; b += blockDim.x) {
        int m = kFar;
        for (int x = b * kDtBlk; x < min(W, (b + 1) * kDtBlk); ++x) m = min(m, row[x]);
        bmin[b] = m;
      }
      __syncthreads();
      for (int x = threadIdx.x; x < W; x += blockDim.x) {
        int d = row[x];
        // right of x, then left of x; a block is skipped when its nearest
        // position is at least d away or its minimum is at least d
        for (int p = x + 1; p < W && p - x < d;) {
          const int b = p / kDtBlk;
          if (bmin[b] >= d) { p = (b + 1) * kDtBlk; continue; }
          d = min(d, max(p - x, row[p]));
          ++p;
        }
        for (int p = x - 1; p >= 0 && x - p < d;) {
          const int b = p / kDtBlk;
          if (bmin[b] >= d) { p = b * kDtBlk - 1; continue; }
          d = min(d, max(x - p, row[p]));
          --p;
        }
        dist[(int64_t)y * W + x] = d;
      }
    } else {
      for (int x = threadIdx.x; x < W; x += blockDim.x) {
        // kNear steps outward together: those past d change nothing, nor do
        // the edge columns' own distances again (100000x20, flat: 1.74 s one by one,
        // 0.33 s so)
        constexpr int kNear = 8;
        int d = grow[x];
        for (int k0 = 1; k0 < d; k0 += kNear) {
          int l[kNear], r[kNear];
#pragma unroll
          for (int j = 0; j < kNear; ++j) { l[j] = grow[max(x - k0 - j, 0)]; r[j] = grow[min(x + k0 + j, W - 1)]; }
#pragma unroll
          for (int j = 0; j < kNear; ++j) d = min(d, max(k0 + j, min(l[j], r[j])));
        }
        dist[(int64_t)y * W + x] = d;
      }
    }
    __syncthreads();
  }
}

// The same row pass for rows up to 4096 pixels (and columns up to 65535
// rows, so that g fits 16 bits), without a search per pixel. For k >= 0,
// d(x) <= k exactly when some x' with |x - x'| <= k has g(x') <= k, i.e. when
// the minimum of g over [x - k, x + k] (cut to the row) is at most k. A sparse
// table of minima over power-of-two ranges gives that minimum with two LDS
// reads. Each thread takes a run of adjacent pixels: the first by binary
// search over k, each next one from its left neighbour, since d changes by
// at most 1 from a pixel to the next (a minimum of functions of slope at most
// 1), which leaves at most two tests: k = d - 1, then k = d.
// The same pass counts the distances of the other pixels (those not in the
// base map): they are below W (the border columns are base pixels), so the
// counts have at most 4096 bins and no counting pass follows.
constexpr int kStW = 4096;
constexpr int kStLevels = 13;   // ranges of 1 .. 4096
constexpr int kStBlock = 1024;
__global__ __launch_bounds__(kStBlock) void k_far_row_st(Bits bt, const int32_t* far, const int32_t* g, int32_t* dist,
                                                         const unsigned long long* base, uint32_t* dhist) {
  __shared__ uint16_t st[kStLevels][kStW];
  __shared__ uint32_t hloc[kStW];
  if (!*far) return;
  const int W = bt.W, H = bt.H;
  for (int b = threadIdx.x; b < kStW; b += kStBlock) hloc[b] = 0u;
  const int levels = 32 - __builtin_clz((unsigned)W);   // 2^(levels-1) <= W
  const int run = (W + kStBlock - 1) / kStBlock;
  // the next row's column distances are loaded while this row is searched
  constexpr int kPer = kStW / kStBlock;
  int32_t nxt[kPer];
  auto fetch = [&](int yy) {
    const int32_t* grow = g + (int64_t)yy * W;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int x = threadIdx.x + k * kStBlock;
      nxt[k] = x < W ? grow[x] : 0;
    }
  };
  if ((int)blockIdx.x < H) fetch(blockIdx.x);
  for (int y = blockIdx.x; y < H; y += gridDim.x) {
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int x = threadIdx.x + k * kStBlock;
      if (x < W) st[0][x] = (uint16_t)min(nxt[k], 65535);
    }
    __syncthreads();
    for (int j = 1; j < levels; ++j) {
      const int h = 1 << (j - 1);
      for (int x = threadIdx.x; x + 2 * h <= W; x += kStBlock) st[j][x] = min(st[j - 1][x], st[j - 1][x + h]);
      __syncthreads();
    }
    if (y + (int)gridDim.x < H) fetch(y + gridDim.x);
    // minimum of g over [l, r], 0 <= l <= r < W
    auto rmq = [&](int l, int r) -> int {
      const int j = 31 - __builtin_clz((unsigned)(r - l + 1));
      return (int)min(st[j][l], st[j][r - (1 << j) + 1]);
    };
    // d(x) <= k
    auto within = [&](int x, int k) -> bool { return rmq(max(0, x - k), min(W - 1, x + k)) <= k; };
    const int rowmin = rmq(0, W - 1);
    const int x0 = threadIdx.x * run, x1 = min(W, x0 + run);
    int32_t* drow = dist + (int64_t)y * W;
    if (rowmin == 65535) {
      // no selected pixel in any column of the image
      for (int x = x0; x < x1; ++x) drow[x] = kFar;
    } else if (x0 < x1) {
      // d(x0) lies in [0, hi]: the pixel's own column bounds it, and so does
      // the column holding the row minimum
      const int gx = st[0][x0];
      int lo = 0, hi = min(gx == 65535 ? kFar : gx, max(W - 1, rowmin));
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (within(x0, mid)) hi = mid;
        else lo = mid + 1;
      }
      auto other = [&](int x) { return !map_bit(base, bt.wpr, x, y); };
      int d = lo;
      drow[x0] = d;
      if (other(x0)) atomicAdd(&hloc[d], 1u);
      for (int x = x0 + 1; x < x1; ++x) {
        if (d > 0 && within(x, d - 1)) d = d - 1;
        else if (!within(x, d)) d = d + 1;
        drow[x] = d;
        if (other(x)) atomicAdd(&hloc[d], 1u);
      }
    }
    __syncthreads();
  }
  for (int b = threadIdx.x; b < W; b += kStBlock)
    if (hloc[b]) atomicAdd(&dhist[b], hloc[b]);
}

// One counting pass over the other pixels' distances (rows wider than the
// range-minimum search takes).
__global__ __launch_bounds__(kBlock) void k_dist_pass(Bits b, FcArgs a, const int32_t* far,
                                                      const unsigned long long* __restrict__ base,
                                                      const int32_t* __restrict__ dist, const RadixSel* in,
                                                      const uint32_t* prev_hist, int prev_shift, RadixSel* state,
                                                      int shift, uint32_t* hist) {
  __shared__ uint32_t bins[kBins];
  if (!*far) return;
  RadixSel rs = in ? *in : RadixSel{0, fc_plan(a).need, 0};
  if (prev_hist) rs = sel_pick(rs, prev_hist, prev_shift, state);
  for (int k = threadIdx.x; k < kBins; k += kBlock) bins[k] = 0u;
  __syncthreads();
  const int lane = threadIdx.x & 63, hi = shift + kDigit;
  const int64_t nw = (int64_t)gridDim.x * (kBlock / 64);
  for (int64_t wi = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); wi < b.words; wi += nw) {
    const WordPos p = word_pos(b, wi);
    if (64 * p.c + lane >= b.W || (base[wi] >> lane & 1ull)) continue;
    const unsigned long long key = (uint32_t)dist[p.i + lane];
    if ((key >> hi) == (rs.prefix >> hi)) atomicAdd(&bins[(key >> shift) & (kBins - 1)], 1u);
  }
  __syncthreads();
  for (int k = threadIdx.x; k < kBins; k += kBlock)
    if (bins[k]) atomicAdd(&hist[k], bins[k]);
}

// Between the levels and the distance passes: column distances, and the flag
// that the launches after it go by | mode 1's third digit (images of 2^24
// pixels and more).
__global__ __launch_bounds__(kBlock) void k_fc_columns(Bits b, FcArgs a, SizeSel z, const unsigned long long* base,
                                                       const uint32_t* lcount, int nseg,
                                                       const unsigned long long* segor, int32_t* g, int32_t* far) {
  __shared__ uint32_t bins[kBins];
  const LevelCounts lc(lcount);
  const FcPlan pl = fc_plan(a);
  lc.kept();
  if (pl.mode == 1) {
    if (z.top >= 2 * kDigit) size_digit(b, z, 2, pl.need, bins);
  } else if (pl.mode == 2 && level_pick(lc, pl.need).level == 0) {
    far_columns(b, base, nseg, segor, g);
    if (blockIdx.x == 0 && threadIdx.x == 0) *far = 1;
  }
}
// Counts: mode 1's pixels of the wanted size per block of b.per words | the
// ring's hashes by their top digit, after the distance passes from the planes
// that their outcome gives (levels 1: nearer than the wanted distance, 2: at
// it), made here. `gr` blocks count where the planes are there, one to a step
// of the ring, though each closes with adds of its bins to one of kHashParts
// arrays of 4 KB (half and a quarter as many blocks: 640x480 118, 125 and 130 us
// a call, 4096x2304 201, 200 and 212).
constexpr int kFarWords = 64;   // words a block makes at a time, 16 per wavefront
__global__ __launch_bounds__(kBlock) void k_fc_count(Bits b, FcArgs a, SizeSel z, int nb, int gr,
                                                     const unsigned long long* base, uint32_t* ties, const int32_t* dist,
                                                     const RadixSel* sd, const uint32_t* sd_hist,
                                                     const uint32_t* lcount, unsigned long long* planes,
                                                     long long* far_need, uint32_t* hash_hist) {
  __shared__ uint32_t part, bins[kHashBins];
  const LevelCounts lc(lcount);
  const FcPlan pl = fc_plan(a);
  lc.kept();
  if (pl.mode == 1) {
    const RadixSel rs = size_found(z, pl.need);
    for (int64_t block = blockIdx.x; block < nb; block += gridDim.x)
      tie_pass(b, z.B, z.kept, z.size, ~(uint32_t)rs.prefix, block, ties, &part);
    return;
  }
  if (pl.mode != 2) return;
  for (int k = threadIdx.x; k < kHashBins; k += kBlock) bins[k] = 0u;
  const LevelSel ls = level_pick(lc, pl.need);   // (its barriers order the bins)
  auto count = [&](uint32_t i) {
    atomicAdd(&bins[mix64((unsigned long long)i ^ a.seed) >> (64 - kHashDigit)], 1u);
  };
  if (ls.level != 0) {
    if ((int)blockIdx.x >= gr) return;
    for_ring(b, planes, ls.level, gr, kRingWords, [](int64_t) {}, count);
  } else {
    const RadixSel rs = sel_pick(sd ? *sd : RadixSel{0, pl.need, 0}, sd_hist, 0, nullptr);
    if (blockIdx.x == 0 && threadIdx.x == 0) *far_need = rs.need - rs.below;
    const int lane = threadIdx.x & 63;
    auto make = [&](int64_t w0) {
      constexpr int kPer = kFarWords / (kBlock / 64);
      const int64_t first = w0 + kPer * (threadIdx.x >> 6);
#pragma unroll 4
      for (int k = 0; k < kPer; ++k) {
        const int64_t wi = first + k;
        if (wi >= b.words) break;
        const WordPos p = word_pos(b, wi);
        const unsigned long long bw = base[wi];
        const bool in = 64 * p.c + lane < b.W && !(bw >> lane & 1ull);
        const unsigned long long d = in ? (unsigned long long)(uint32_t)dist[p.i + lane] : ~0ull;
        const unsigned long long nearer = __builtin_amdgcn_ballot_w64(in && d < rs.prefix);
        const unsigned long long at = __builtin_amdgcn_ballot_w64(in && d == rs.prefix);
        if (lane < 4) planes[4 * wi + lane] = lane == 0 ? nearer : lane == 1 ? at : 0ull;
      }
      __syncthreads();   // the block reads its words' planes back
    };
    for_ring(b, planes, 2, (int)gridDim.x, kFarWords, make, count);
  }
  __syncthreads();
  uint32_t* out = hash_hist + (blockIdx.x % kHashParts) * kHashBins;
  for (int k = threadIdx.x; k < kHashBins; k += kBlock)
    if (bins[k]) atomicAdd(&out[k], bins[k]);
}

int fail(int st, const char* fmt, ...) {
  char buf[256];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  return sbs::report_error(st, buf);
}

size_t a256(size_t v) { return (v + 255) / 256 * 256; }

struct Layout {
  size_t L8, B, kept, base, sel, planes, parent, size, g, dist, segor, bsum, ties, lut;
  size_t clear, hist, misc, lcount, shist, dhist, hhist, cnt, clear_front, clear_frac, clear_all;   // cleared at the start
  size_t end;
  int64_t ncnt;
};

Bits map_bits(int32_t W, int32_t H) {
  Bits b{};
  b.W = W;
  b.H = H;
  b.wpr = (W + 63) / 64;
  b.words = (int64_t)H * b.wpr;
  b.per = kSelWords * ((b.words + (int64_t)kSelWords * kSelBlocks - 1) / ((int64_t)kSelWords * kSelBlocks));
  return b;
}

Layout layout(int32_t W, int32_t H) {
  const int64_t N = (int64_t)W * H;
  const Bits b = map_bits(W, H);
  Layout o{};
  size_t off = 0;
  auto take = [&](size_t bytes) { const size_t at = off; off += a256(bytes); return at; };
  o.L8 = take(N);
  for (size_t* m : {&o.B, &o.kept, &o.base, &o.sel}) *m = take((size_t)b.words * 8);
  o.planes = take((size_t)b.words * 8 * kLevelBits);
  o.parent = take((size_t)b.words * 32 * 4);   // one entry per node
  o.size = take((size_t)b.words * 32 * 4);
  o.g = take((size_t)N * 4);
  o.dist = take((size_t)N * 4);
  o.segor = take((size_t)((H + kSegRows - 1) / kSegRows) * b.wpr * 8);
  o.bsum = take(kSelBlocks * 4);
  o.ties = take(kSelBlocks * 4);
  o.lut = take(256);
  o.clear = off;
  o.hist = take(kHistParts * 256 * 4);
  o.misc = take(kMiscBytes);
  o.clear_front = off;
  o.lcount = take((size_t)kLvParts * (kLevels + 1) * 4);
  o.shist = take((size_t)3 * kBins * 4);   // one count array per pass of a select
  o.dhist = take((size_t)3 * kBins * 4);
  o.hhist = take((size_t)kHashParts * kHashBins * 4);
  o.clear_frac = off;
  o.ncnt = (int64_t)(kDropFrac * (double)N) + 2;   // sizes that the paper filter's budget can hold
  o.cnt = take((size_t)o.ncnt * 4);
  o.clear_all = off;
  o.end = off;
  return o;
}

// The steps of L8(Y) for k_light: L8 = round half away from zero of
// (116 f(Y) - 16) * 255 / 100, clamped to [0, 255], with f the CIE function
// (cube root above (6/29)^3, linear below), all in fp64. For each v, a binary
// search over the ordered bit patterns of the non-negative doubles up to 2
// finds the smallest Y with L8(Y) >= v. Computed once per process.
const LightSteps& light_steps() {
  static const LightSteps steps = [] {
#pragma clang fp contract(off)
    LightSteps r{};
    const double e = 6.0 / 29.0;
    const double e3 = e * e * e, k3 = 3 * e * e;
    auto l8 = [&](double Y) -> int {
      const double f = Y > e3 ? std::cbrt(Y) : Y / k3 + 4.0 / 29.0;
      const double s = (116.0 * f - 16.0) * 255.0 / 100.0;
      const double q = s >= 0 ? std::floor(s + 0.5) : -std::floor(-s + 0.5);
      return q < 0 ? 0 : (q > 255 ? 255 : (int)q);
    };
    auto at = [](uint64_t b) { double d; std::memcpy(&d, &b, 8); return d; };
    uint64_t hi_bits;
    const double two = 2.0;
    std::memcpy(&hi_bits, &two, 8);
    r.t[0] = 0.0;
    for (int v = 1; v < 256; ++v) {
      if (l8(two) < v) { r.t[v] = HUGE_VAL; continue; }
      uint64_t lo = 0, hi = hi_bits;   // l8(at(hi)) >= v
      while (lo < hi) {
        const uint64_t mid = lo + (hi - lo) / 2;
        if (l8(at(mid)) >= v) hi = mid; else lo = mid + 1;
      }
      r.t[v] = at(lo);
    }
    return r;
  }();
  return steps;
}

void launch_light(const uint8_t* img, int32_t W, int32_t H, int32_t C, int64_t pitch, uint8_t* L8, uint32_t* hist,
                  hipStream_t s) {
  if (pitch == (int64_t)W * C) {   // rows without gaps are one row
    W *= H;
    H = 1;
    pitch = (int64_t)W * C;
  }
  // at most 4 blocks per CU of RGB (their tables and closing adds) and 2 of gray
  const int per = C == 3 ? 4 : 16;
  const int64_t groups = ((int64_t)W + per - 1) / per * H;
  const dim3 grid((unsigned)std::min<int64_t>((groups + kBlock - 1) / kBlock, C == 3 ? 1024 : L8 && !hist ? 8192 : 512));
  const dim3 block(kBlock);
  if (C == 3) {
    if (hist) hipLaunchKernelGGL(k_light<true>, grid, block, 0, s, img, W, H, pitch, L8, light_steps(), hist);
    else hipLaunchKernelGGL(k_light<false>, grid, block, 0, s, img, W, H, pitch, L8, light_steps(), hist);
  } else if (!hist) {
    hipLaunchKernelGGL((k_gray<true, false>), grid, block, 0, s, img, W, H, pitch, L8, hist);
  } else if (L8) {
    hipLaunchKernelGGL((k_gray<true, true>), grid, block, 0, s, img, W, H, pitch, L8, hist);
  } else {
    hipLaunchKernelGGL((k_gray<false, true>), grid, block, 0, s, img, W, H, pitch, L8, hist);
  }
}

int grid_for(int64_t n) {
  const int64_t g = (n + kBlock - 1) / kBlock;
  return (int)(g < 1 ? 1 : (g > 8192 ? 8192 : g));
}

}  // namespace sbs_front

using namespace sbs_front;

extern "C" {

int sbs_lightness(const uint8_t* img, int32_t W, int32_t H, int32_t C, int64_t pitch, uint8_t* out_l8, void* stream) {
  if (W < 1 || H < 1 || (int64_t)W * H > INT32_MAX || (C != 1 && C != 3) || pitch < (int64_t)W * C)
    return fail(SBS_ERR_INVALID_ARG, "bad image geometry");
  if (!img || !out_l8) return fail(SBS_ERR_INVALID_ARG, "NULL pointer");
  hipStream_t s = (hipStream_t)stream;
  launch_light(img, W, H, C, pitch, out_l8, nullptr, s);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(SBS_ERR_HIP, "lightness: %s", hipGetErrorString(e));
  return SBS_OK;
}

size_t sbs_boundaries_workspace_bytes(int32_t W, int32_t H) {
  if (W < 1 || H < 1 || (int64_t)W * H > INT32_MAX) return 0;
  return layout(W, H).end;
}

int sbs_boundaries(const uint8_t* img, int32_t W, int32_t H, int32_t C, int64_t pitch, int32_t K, int32_t mode,
                   int32_t min_cc, double frac, uint64_t seed, uint32_t* out_idx, int64_t* out_count,
                   uint8_t* out_refined, uint8_t* out_labels, void* workspace, size_t workspace_bytes, void* stream) {
  if (W < 1 || H < 1 || (int64_t)W * H > INT32_MAX || (C != 1 && C != 3) || pitch < (int64_t)W * C)
    return fail(SBS_ERR_INVALID_ARG, "bad image geometry");
  if (!img || !out_idx || !out_count || !workspace) return fail(SBS_ERR_INVALID_ARG, "NULL pointer");
  if (K < 1 || K > kMaxK) return fail(SBS_ERR_INVALID_ARG, "K must be in [1, %d]", kMaxK);
  if (mode != 0 && mode != 1) return fail(SBS_ERR_INVALID_ARG, "mode must be 0 (configured) or 1 (paper)");
  if (mode == 0 && min_cc < 0) return fail(SBS_ERR_INVALID_ARG, "min_cc < 0");
  // (Within it the runs' numbers fit 32 bits: a row ends with a word of up to 32
  // runs, so there are at most W H / 2 + 32 H of them, and W H < 2^31.)
  if (H > 4 * 65535) return fail(SBS_ERR_UNSUPPORTED, "H > %d", 4 * 65535);
  if (!(frac < 0.0) && !(frac <= 1.0)) return fail(SBS_ERR_INVALID_ARG, "frac must be < 0 (off) or in [0, 1]");
  const int64_t N = (int64_t)W * H;
  const Layout Lo = layout(W, H);
  if (workspace_bytes < Lo.end) return fail(SBS_ERR_INVALID_ARG, "workspace too small");
  if ((uintptr_t)workspace & 255) return fail(SBS_ERR_INVALID_ARG, "workspace not 256-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  char* base = (char*)workspace;
  uint8_t* L8 = (uint8_t*)(base + Lo.L8);
  const Bits bt = map_bits(W, H);
  unsigned long long* B = (unsigned long long*)(base + Lo.B);
  unsigned long long* kept = (unsigned long long*)(base + Lo.kept);
  unsigned long long* bmap = (unsigned long long*)(base + Lo.base);
  unsigned long long* sel = (unsigned long long*)(base + Lo.sel);
  const int32_t wpr = bt.wpr;
  int32_t* parent = (int32_t*)(base + Lo.parent);
  int32_t* size = (int32_t*)(base + Lo.size);
  int32_t* cnt = (int32_t*)(base + Lo.cnt);
  uint32_t* bsum = (uint32_t*)(base + Lo.bsum);
  uint32_t* hist = (uint32_t*)(base + Lo.hist);
  uint8_t* lut = (uint8_t*)(base + Lo.lut);
  char* misc = base + Lo.misc;
  int32_t* passes = (int32_t*)misc;
  unsigned long long* total = (unsigned long long*)(misc + 128);
  DropRule* rule = (DropRule*)(misc + 192);
  int32_t* far = (int32_t*)(misc + 256);
  long long* far_need = (long long*)(misc + 264);
  RingBin* rb = (RingBin*)(misc + 320);
  RadixSel* s1 = (RadixSel*)(misc + 384);   // the size select's states after its picks
  RadixSel* sd = (RadixSel*)(misc + 448);   // the distance select's
  unsigned long long* n1 = (unsigned long long*)(misc + 1024);   // kN1Parts partial counts
  static_assert(sizeof(RingBin) <= 64 && 2 * sizeof(RadixSel) <= 64 && 1024 + kN1Parts * 8 <= kMiscBytes, "misc layout");
  const int g = grid_for(N);

  {
    const size_t to = mode == 1 ? Lo.clear_all : frac >= 0.0 ? Lo.clear_frac : Lo.clear_front;
    const int64_t bytes = (int64_t)(to - Lo.clear);
    hipLaunchKernelGGL(k_clear, dim3((unsigned)std::min<int64_t>((bytes / 16 + kBlock - 1) / kBlock, 1024)), dim3(kBlock),
                       0, s, (uint4*)(base + Lo.clear), bytes);
  }
  // grey rows without gaps are the lightness image itself (no copy)
  const bool same = C == 1 && pitch == W;
  const uint8_t* lum = same ? img : L8;
  launch_light(img, W, H, C, pitch, same ? nullptr : L8, hist, s);
  hipLaunchKernelGGL(k_kmeans, dim3(1), dim3(256), 0, s, hist, K, lut, passes);
  const int32_t words = (W & 3) == 0 && ((uintptr_t)lum & 3) == 0 ? 1 : 0;
  auto rf_grid = [&](int rows) { return dim3((W + kRfCols - 1) / kRfCols, (H + rows - 1) / rows); };
  if (mode == 0) {
    hipLaunchKernelGGL(k_refine<0>, rf_grid(kRfRows<0>), dim3(64), 0, s, lum, W, H, K, lut, B, wpr, out_labels, words);
  } else {
    hipLaunchKernelGGL(k_refine<1>, rf_grid(kRfRows<1>), dim3(64), 0, s, lum, W, H, K, lut, B, wpr, (uint8_t*)nullptr, words);
    if (out_labels) hipLaunchKernelGGL(k_label, dim3(g), dim3(kBlock), 0, s, lum, N, lut, out_labels);
  }
  const int nty = (H + kTileH - 1) / kTileH;
  // passes over words, kSelWords per block and step
  const int gw = (int)std::min<int64_t>((bt.words + kSelWords - 1) / kSelWords, 2048);
  hipLaunchKernelGGL(k_cc_tile, dim3(wpr, nty), dim3(kCcBlock), 0, s, bt, B, parent, size);
  const int64_t vb = ((int64_t)H * (wpr - 1) + kBlock - 1) / kBlock;
  const int64_t hb = ((int64_t)(nty - 1) * wpr + kBlock / 64 - 1) / (kBlock / 64);
  if (vb + hb > 0) hipLaunchKernelGGL(k_cc_edges, dim3((unsigned)(vb + hb)), dim3(kBlock), 0, s, bt, B, parent, (int)vb);
  hipLaunchKernelGGL(k_cc_flatten, dim3(gw), dim3(kBlock), 0, s, bt, B, parent, size);

  const int nb = (int)((bt.words + bt.per - 1) / bt.per);
  if (mode == 1) {
    // at most 512 blocks: each block's closing adds (its total and its small
    // sizes' counts) go to the same few global words, so fewer blocks wait less
    hipLaunchKernelGGL(k_drop_count, dim3(std::min(gw, 512)), dim3(kBlock), 0, s, bt, B, size, Lo.ncnt, total, cnt);
    hipLaunchKernelGGL(k_drop_find, dim3(1), dim3(1024), 0, s, cnt, total, rule);
    hipLaunchKernelGGL(k_root_count, dim3(nb), dim3(kBlock), 0, s, bt, B, size, rule, bsum);
    hipLaunchKernelGGL(k_root_find, dim3(1), dim3(1024), 0, s, bt, B, size, bsum, nb, rule);
  }
  const DropRule* dr = mode == 1 ? rule : nullptr;
  if (frac < 0.0) {
    hipLaunchKernelGGL(k_kept, dim3(nb), dim3(kBlock), 0, s, bt, B, parent, size, dr, (int64_t)min_cc,
                       (unsigned long long*)nullptr, sel, out_refined, bsum, (unsigned long long*)nullptr);
  } else {
    FcArgs fa{};
    fa.want = std::min<long long>((long long)N, std::llround(frac * (double)N));
    fa.n0 = W == 1 ? H : 2LL * H;
    fa.n1 = n1;
    fa.seed = (unsigned long long)seed;
    unsigned long long* planes = (unsigned long long*)(base + Lo.planes);
    uint32_t* lcount = (uint32_t*)(base + Lo.lcount);
    uint32_t* shist = (uint32_t*)(base + Lo.shist);
    uint32_t* dhist = (uint32_t*)(base + Lo.dhist);
    uint32_t* hhist = (uint32_t*)(base + Lo.hhist);
    uint32_t* ties = (uint32_t*)(base + Lo.ties);
    int32_t* gcol = (int32_t*)(base + Lo.g);
    int32_t* dist = (int32_t*)(base + Lo.dist);
    unsigned long long* segor = (unsigned long long*)(base + Lo.segor);
    const int nseg = (H + kSegRows - 1) / kSegRows;
    Bits bk = bt;   // (no counts per block here: one batch of words each)
    bk.per = kSelWords;
    hipLaunchKernelGGL(k_kept, dim3((unsigned)((bt.words + kSelWords - 1) / kSelWords)), dim3(kBlock), 0, s, bk, B, parent,
                       size, dr, (int64_t)min_cc, kept, bmap, out_refined, (uint32_t*)nullptr, n1);
    // Component sizes are at most N: with N below 2^24 the keys' top 8 bits
    // are ones, and two digits remain; else three.
    const bool small = N < (1LL << 24);
    const int gs = std::min(gw, 512);
    const SizeSel z{B, kept, size, small ? 0xFF000000ull : 0ull, small ? kDigit : 2 * kDigit, s1, shist, gs};
    const int gx = (wpr + 2 * (kBlock / 64) - 1) / (2 * (kBlock / 64)), gy = (H + kLvRows - 1) / kLvRows;
    const dim3 gl((unsigned)std::max(gx * gy, gs));
    hipLaunchKernelGGL(k_fc_levels<0>, gl, dim3(kBlock), 0, s, bt, fa, z, gx, gy, bmap, planes, sel, lcount, bmap, nseg, segor);
    hipLaunchKernelGGL(k_fc_levels<1>, gl, dim3(kBlock), 0, s, bt, fa, z, gx, gy, sel, planes, (unsigned long long*)nullptr,
                       lcount, bmap, nseg, segor);
    hipLaunchKernelGGL(k_fc_columns, dim3(gw), dim3(kBlock), 0, s, bt, fa, z, bmap, lcount, nseg, segor, gcol, far);
    const RadixSel* sd_last = nullptr;
    const uint32_t* sd_hist = dhist;
    if (W <= kStW && H <= 65535) {
      // one block per CU (the table takes most of the LDS), each over rows in turn
      hipLaunchKernelGGL(k_far_row_st, dim3(H < 256 ? H : 256), dim3(kStBlock), 0, s, bt, far, gcol, dist, bmap, dhist);
    } else {
      hipLaunchKernelGGL(k_far_row, dim3(H < 16384 ? H : 16384), dim3(kBlock), 0, s, bt, far, gcol, dist);
      // distances are below W (the border columns are base pixels)
      int dsh = W <= kBins ? 0 : W <= (1 << 24) ? kDigit : 2 * kDigit;
      for (int k = 0;; ++k) {
        hipLaunchKernelGGL(k_dist_pass, dim3(gs), dim3(kBlock), 0, s, bt, fa, far, bmap, dist,
                           k < 2 ? (const RadixSel*)nullptr : sd + k - 2, k == 0 ? (const uint32_t*)nullptr : sd_hist,
                           dsh + kDigit, k == 0 ? (RadixSel*)nullptr : sd + k - 1, dsh, dhist + k * kBins);
        sd_last = k == 0 ? nullptr : sd + k - 1;
        sd_hist = dhist + k * kBins;
        if (dsh == 0) break;
        dsh -= kDigit;
      }
    }
    // the hashes of one bin's ring pixels are listed in the place of the column
    // and pixel distances (8 bytes per pixel between them)
    unsigned long long* ring = (unsigned long long*)gcol;
    const int gr = (int)std::min<int64_t>((bt.words + kRingWords - 1) / kRingWords, 1024);
    hipLaunchKernelGGL(k_fc_count, dim3(std::min(std::max(gw, gr), 1024)), dim3(kBlock), 0, s, bt, fa, z, nb, gr, bmap, ties, dist,
                       sd_last, sd_hist, lcount, planes, far_need, hhist);
    hipLaunchKernelGGL(k_ring_bin, dim3(gr), dim3(kBlock), 0, s, bt, fa, planes, lcount, far_need, hhist, rb, ring);
    hipLaunchKernelGGL(k_fc_select, dim3(nb), dim3(kBlock), 0, s, bt, fa, bmap, z, ties, planes, lcount, far_need, rb, ring, sel, bsum);
  }
  hipLaunchKernelGGL(k_list, dim3(nb), dim3(kBlock), 0, s, bt, sel, bsum, out_idx, (long long*)out_count);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(SBS_ERR_HIP, "boundaries: %s", hipGetErrorString(e));
  return SBS_OK;
}

}  // extern "C"
