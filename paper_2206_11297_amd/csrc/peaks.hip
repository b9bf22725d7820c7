// peaks.hip -- peak finding on the GPU: the step before the compression path,
// producing the peak list whose windows form the ROI mask (Sec. IV-B names
// peak_finder_v3 and its parameters; non-hit rejection, Sec. IV, counts
// these peaks).
//
// k_peaks_init  zeroes each frame's peak counter.
// k_peaks_find  streams every frame once, 16 float4 loads per lane.  The
//               rare pixels at or above amax_min are taken by their whole
//               wave, a few at a time: a lane a pixel for the window maximum,
//               which most fail, then the rest of the decision (background
//               ring, peak pixels, cuts) with its sums taken from lane to
//               lane; accepted peaks are appended as (panel, row, col) keys.
// k_peaks_sort  one workgroup per frame: bitonic sort of the keys in LDS, so
//               the list comes out in raster order whatever the append order.
//
// The arithmetic of a decision follows one fixed order: fp64
// sums in raster order, a correctly rounded divide, products compared instead
// of square roots.  Compiled with -ffp-contract=off.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "rsz_internal.h"

namespace rsz {

namespace {

// A wave's candidate pixel (i, j) of a panel of H x W at xp (all uniform).
struct Candidate {
  const float *xp;
  int32_t p, i, j;
};

// This lane's pixel of the (2r + 1)^2 neighbourhood of the candidate, the
// o-th in raster order; in: it lies in the neighbourhood and the panel.
// mul = floor((2^32 - 1) / (2r + 1)) + 1 divides o < 2^16 exactly.
__device__ __forceinline__ float neighbour(const Candidate &c, int32_t H, int32_t W, int32_t r,
                                           uint32_t mul, uint32_t o, bool &in, int32_t &du,
                                           int32_t &dv) {
  const int32_t side = 2 * r + 1;
  du = (int32_t)__umulhi(o, mul);
  dv = (int32_t)o - du * side;
  du -= r;
  dv -= r;
  const int32_t u = c.i + du, v = c.j + dv;
  in = o < (uint32_t)(side * side) && u >= 0 && u < H && v >= 0 && v < W;
  return in ? *gm(c.xp + (uint32_t)u * (uint32_t)W + (uint32_t)v) : 0.0f;
}

__device__ __forceinline__ float lane_value(float x, int lane) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(x), lane));
}

// The decision for a candidate that is its window's maximum, by its wave, in
// the oracle's order: background ring mean and squared deviations, the cut,
// the 4-connected component of the maximum, its sum, the cuts.  w: lane a *
// ww + b holds the window's pixel (a, b) (in_w: the lanes inside the panel).
// The sums take the pixels one after the other from the lanes that hold them,
// each a readlane and an fp64 operation (one lane reading them from LDS,
// whatever the others, took longer than a wave's whole share of the frame).
// Frames full of candidates wait for this chain: 50 frames of 32x185x388 with
// 1% of the pixels at amax_min take 1.92 ms (3.17 with the ring loaded again
// for the deviations, 2.89 by one lane a candidate).
__device__ bool peak_decide(const rsz_peak_params &q, const Candidate &c, int32_t H, int32_t W,
                            float w, uint64_t in_w, int lane) {
  const int32_t h = (int32_t)q.rank, ww = 2 * h + 1;
  const int32_t ro = (int32_t)q.ring_out, ri = (int32_t)q.ring_in, side = 2 * ro + 1;
  const uint32_t area = (uint32_t)(side * side), mul = 0xFFFFFFFFu / (uint32_t)side + 1u;
  // background ring: mean, then the sum of squared deviations; its first 128
  // pixels (all of the default ring) are loaded once, together
  double sum = 0.0, mu = 0.0, V = 0.0;
  auto load = [&](uint32_t o0, float &x) {
    bool in;
    int32_t du, dv;
    x = neighbour(c, H, W, ro, mul, o0 + (uint32_t)lane, in, du, dv);
    return __ballot(in && max(abs(du), abs(dv)) >= ri);
  };
  auto add = [&](float x, uint64_t ring) {
#pragma unroll 1
    for (; ring; ring &= ring - 1) sum += (double)lane_value(x, __builtin_ctzll(ring));
  };
  auto deviate = [&](float x, uint64_t ring) {
#pragma unroll 1
    for (; ring; ring &= ring - 1) {
      const double e = (double)lane_value(x, __builtin_ctzll(ring)) - mu;
      V += e * e;
    }
  };
  float x0, x1;
  const uint64_t r0 = load(0, x0), r1 = load(64, x1);
  uint32_t m = (uint32_t)(__builtin_popcountll(r0) + __builtin_popcountll(r1));
  add(x0, r0);
  add(x1, r1);
#pragma unroll 1
  for (uint32_t o0 = 128; o0 < area; o0 += 64) {
    float x;
    const uint64_t ring = load(o0, x);
    m += (uint32_t)__builtin_popcountll(ring);
    add(x, ring);
  }
  if (m == 0) return false;
  mu = sum / (double)m;
  deviate(x0, r0);
  deviate(x1, r1);
#pragma unroll 1
  for (uint32_t o0 = 128; o0 < area; o0 += 64) {
    float x;
    const uint64_t ring = load(o0, x);
    deviate(x, ring);
  }
  const double k2V = q.pix_nsigma * q.pix_nsigma * V;
  // window pixels above the cut, as bits a*ww + b of the window
  const double d = (double)w - mu;
  const uint64_t above = __ballot(d > 0.0 && d * d * (double)m > k2V) & in_w;
  // the 4-connected component of the maximum: grow by one step in each of the
  // four directions until nothing changes (shifts by 1 must not wrap rows)
  uint64_t first_col = 0, last_col = 0;
  for (int32_t a = 0; a < ww; ++a) {
    first_col |= 1ull << (a * ww);
    last_col |= 1ull << (a * ww + ww - 1);
  }
  uint64_t comp = above & (1ull << (h * ww + h));
  for (;;) {
    const uint64_t grown = (comp | ((comp << 1) & ~first_col) | ((comp >> 1) & ~last_col) |
                            (comp << ww) | (comp >> ww)) & above;
    if (grown == comp) break;
    comp = grown;
  }
  double S = 0.0;
  const uint32_t n = (uint32_t)__builtin_popcountll(comp);
#pragma unroll 1
  for (uint64_t k = comp; k; k &= k - 1) S += (double)lane_value(w, __builtin_ctzll(k));
  if (n < q.npix_min || n > q.npix_max) return false;
  if (!(S > q.atot_min)) return false;
  const double num = S - (double)n * mu;
  return num > 0.0 && num * num * (double)m > q.snr_min * q.snr_min * (double)n * V;
}

__global__ __launch_bounds__(256) void k_peaks_init(PeakBatchPlan pp) {
  const uint32_t f = blockIdx.x * 256 + threadIdx.x;
  if (f < pp.nframes) *pp.frames[f].count = 0u;
}

// HBM bounds it: 1000 frames of 32x185x388 (9.19 GB) take 1.29 ms, 7.1 TB/s,
// with loads that leave the caches alone (1.44 ms without, 5.6 TB/s in a plain
// streaming read).  One lane a candidate on neighbourhoods staged in LDS,
// and a binary search for the frame, took 1.86 ms.
__global__ __launch_bounds__(256) void k_peaks_find(PeakBatchPlan pp) {
  const uint32_t blk = xcd_run();
  const uint32_t f = wave_find_frame(pp.tile_prefix, pp.nframes, blk);
  const PeakFramePlan &fp = pp.frames[f];
  if (fp.init_status != RSZ_OK) return;
  const uint64_t npix = (uint64_t)fp.P * fp.H * fp.W;
  const uint64_t base = (uint64_t)(blk - pp.tile_prefix[f]) * kPeakTile;
  const float *x = fp.frame;
  constexpr int K = (int)(kPeakTile / 1024);   // float4 loads per lane
  float v[K][4];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const uint64_t e0 = base + (uint64_t)(k * 256 + threadIdx.x) * 4;
    if (e0 + 4 <= npix) {
      // (the frame is 16-byte aligned)
      const f32x4 w = __builtin_nontemporal_load(gm((const f32x4 *)(x + e0)));
      v[k][0] = w.x;
      v[k][1] = w.y;
      v[k][2] = w.z;
      v[k][3] = w.w;
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t) v[k][t] = e0 + t < npix ? *gm(x + e0 + t) : -INFINITY;
    }
  }
  // candidates: pixels at or above amax_min (amax_f is the smallest float
  // >= amax_min, so a float compare decides exactly as the fp64 one)
  const float amax_f = pp.amax_f;
  uint64_t cand = 0;   // bit 4k + t: pixel t of load k
#pragma unroll
  for (int k = 0; k < K; ++k)
#pragma unroll
    for (int t = 0; t < 4; ++t) cand |= (uint64_t)(v[k][t] >= amax_f) << (4 * k + t);
  // The wave takes its candidates together, kBatch at a time: their windows (at
  // most 7 x 7, a pixel a lane) are loaded with all loads in flight; most
  // are not their window's maximum and end there (ties go to the first pixel
  // in raster order; NaN fails every comparison).
  uint64_t pending = __builtin_amdgcn_uicmp((uint32_t)(cand | (cand >> 32)), 0u, 33 /* ne */);
  if (!pending) return;
  constexpr int kBatch = 4;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const rsz_peak_params q = pp.q;
  // a frame has < 2^31 pixels: 32-bit index arithmetic
  const int32_t H = (int32_t)fp.H, W = (int32_t)fp.W, h = (int32_t)q.rank;
  const int32_t ww = 2 * h + 1, mid = h * ww + h;
  const uint32_t mul = 0xFFFFFFFFu / (uint32_t)ww + 1u;
  const FastDiv dW = fp.fd_W, dH = fp.fd_H;
  uint32_t *count = fp.count;
  uint64_t *keys = fp.keys;
  const uint32_t cap = fp.cap;
  uint64_t cm = 0;   // the candidates of lane L not yet taken
  int L = -1;
  for (bool more = true; more;) {
    Candidate c[kBatch];
    float w[kBatch];
    uint64_t in_w[kBatch];
    int n = 0;
#pragma unroll
    for (int t = 0; t < kBatch; ++t) {
      if (!cm && pending) {
        L = __builtin_ctzll(pending);
        pending &= pending - 1;
        cm = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(cand >> 32), L) << 32) |
             (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)cand, L);
      }
      in_w[t] = 0;
      if (!cm) {
        more = false;
        continue;
      }
      const int b = __builtin_ctzll(cm);
      cm &= cm - 1;
      const uint32_t e = (uint32_t)(base + (uint64_t)((b >> 2) * 256 + wv * 64 + L) * 4 + (b & 3));
      const uint32_t r = fdiv(dW, e), pn = fdiv(dH, r);
      c[t].p = (int32_t)pn;
      c[t].i = (int32_t)(r - pn * (uint32_t)H);
      c[t].j = (int32_t)(e - r * (uint32_t)W);
      c[t].xp = x + (uint64_t)pn * (uint32_t)H * (uint32_t)W;
      bool in;
      int32_t du, dv;
      w[t] = neighbour(c[t], H, W, h, mul, (uint32_t)lane, in, du, dv);
      in_w[t] = __ballot(in);
      n = t + 1;
    }
#pragma unroll
    for (int t = 0; t < kBatch; ++t) {
      if (t >= n) continue;
      const float v0 = lane_value(w[t], mid);
      const bool ok = lane < mid ? w[t] < v0 : w[t] <= v0;
      if (__ballot(!ok) & in_w[t] & ~(1ull << mid)) continue;
      if (!peak_decide(q, c[t], H, W, w[t], in_w[t], lane)) continue;
      if (lane == 0) {
        const uint32_t slot = atomicAdd(count, 1u);
        if (slot < cap)
          keys[slot] = ((uint64_t)c[t].p << 32) | ((uint64_t)c[t].i << 16) | (uint64_t)c[t].j;
      }
    }
  }
}

__global__ __launch_bounds__(256) void k_peaks_sort(PeakBatchPlan pp) {
  __shared__ uint64_t s_key[kPeakCapMax];
  const PeakFramePlan &fp = pp.frames[blockIdx.x];
  if (fp.init_status != RSZ_OK) {
    if (threadIdx.x == 0) {
      *fp.res_count = 0u;
      *fp.res_status = fp.init_status;
    }
    return;
  }
  const uint32_t n = *fp.count;
  if (n > fp.cap) {
    if (threadIdx.x == 0) {
      *fp.res_count = n;
      *fp.res_status = RSZ_ERR_CAPACITY;
    }
    return;
  }
  uint32_t n2 = 1;
  while (n2 < n) n2 <<= 1;
  for (uint32_t k = threadIdx.x; k < n2; k += 256) s_key[k] = k < n ? fp.keys[k] : ~0ull;
  __syncthreads();
  // ascending bitonic sort of s_key[0, n2) (keys are unique within a frame)
  for (uint32_t size = 2; size <= n2; size <<= 1)
    for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
      for (uint32_t t = threadIdx.x; t < n2 / 2; t += 256) {
        const uint32_t a = 2 * t - (t & (stride - 1)), b = a + stride;
        const bool up = (a & size) == 0;
        const uint64_t ka = s_key[a], kb = s_key[b];
        if ((ka > kb) == up) {
          s_key[a] = kb;
          s_key[b] = ka;
        }
      }
      __syncthreads();
    }
  for (uint32_t k = threadIdx.x; k < n; k += 256) {
    const uint64_t key = s_key[k];
    fp.out[k].panel = (int32_t)(key >> 32);
    fp.out[k].row = (int32_t)((key >> 16) & 0xFFFFu);
    fp.out[k].col = (int32_t)(key & 0xFFFFu);
  }
  if (threadIdx.x == 0) {
    *fp.res_count = n;
    *fp.res_status = RSZ_OK;
  }
}

}  // namespace

#define RSZ_PLAUNCH(name, kern, grid, s)                              \
  do {                                                                \
    prof_begin(name, s);                                              \
    hipLaunchKernelGGL(kern, dim3(grid), dim3(256), 0, s, pp);        \
    prof_end(s);                                                      \
    hipError_t e_ = hipGetLastError();                                \
    if (e_ != hipSuccess) return e_;                                  \
  } while (0)

hipError_t launch_find_peaks(const PeakBatchPlan &pp, hipStream_t s) {
  RSZ_PLAUNCH("k_peaks_init", k_peaks_init, (pp.nframes + 255) / 256, s);
  if (pp.total_tiles) RSZ_PLAUNCH("k_peaks_find", k_peaks_find, pp.total_tiles, s);
  RSZ_PLAUNCH("k_peaks_sort", k_peaks_sort, pp.nframes, s);
  return hipSuccess;
}

}  // namespace rsz
