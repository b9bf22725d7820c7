// On-device verification of a compressed batch: the decompress-and-check
// stage that a graph-captured pipeline appends to compression.  The batch's
// own streams are decoded by the decoder kernels (decompress.hip), whose
// plans are completed here from the totals the compression left on the
// device, and every pixel of every decoding is checked against the frame
// it came from: ROI pixels bit for bit (Sec. IV: the windows are kept
// losslessly), every other pixel within the error bound of its bin's mean
// (Sec. V-C: the bound is absolute on the binned values; Sec. IV-A: the
// bin value is restored to each of its pixels).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rsz_internal.h"

namespace rsz {

// The data-dependent fields of each frame's decoder plan, from the totals
// the compression wrote (only frames with the ROI verbatim and no run stage
// are verified); a frame whose compression failed decodes nothing.  The
// violation counts start at zero.
__global__ __launch_bounds__(256) void k_vplan(VerifyBatch vb) {
  const uint32_t f = blockIdx.x * 256 + threadIdx.x;
  if (f >= vb.n) return;
  const VerifyFrame &vf = vb.frames[f];
  *vf.bad = 0u;
  if (!vf.valid) return;
  DecodePlan *dp = vf.dplan;
  const FrameState *st = vf.cplan->st;
  const int32_t status = __hip_atomic_load(&st->status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (status != RSZ_OK) {
    dp->init_status = RSZ_ERR_ARG;
    return;
  }
  const uint64_t T = st->T;
  const uint32_t n_out = st->n_out;
  dp->T = T;
  dp->n_out = n_out;
  dp->total = st->total;
  dp->off_oidx = dp->off_bits + 4 * ((T + 31) / 32);
  dp->off_ores = dp->off_oidx + 4ull * n_out;
  dp->init_status = RSZ_OK;
}

// The mean of a bin's n included pixels.  S / n for n a power of two is S
// times its reciprocal, bit for bit.
__device__ __forceinline__ double bin_mean(double S, uint32_t n) {
  if (n == 0) return 0.0;
  if ((n & (n - 1)) == 0) return S * (1.0 / (double)n);
  return S / (double)n;
}

// Whether pixel y of a bin (x: the frame's) fails its check.
__device__ __forceinline__ bool pixel_fails(float x, float y, bool roi, double mean, double eb) {
  const double yv = (double)y;
  const double tol = eb + fabs(yv) * 0x1p-23 + fabs(mean) * 0x1p-40;
  return roi ? __float_as_uint(y) != __float_as_uint(x) : !(fabs(yv - mean) <= tol);
}

struct VerifyRows {
  const float *x, *y;        // the panel
  const uint32_t *mask;      // the block's ROI bitmap, wpr words a row from row r0, column c0
  uint32_t H, W, wpr, r0, c0, c1, mode;   // (c0 a multiple of 32 and of b)
  double eb;
};

// Bin rows [Ia, Ib) in steps of 4 of a panel whose rows are whole aligned
// 16-byte groups, b = 1, 2 or 4: a lane takes 4 columns of a bin row's b raw
// rows, so its 4 / b bins are whole, kVerifyAhead such groups' loads in
// flight together.  Failing pixels of this lane.
constexpr int kVerifyAhead = 2;
template <int B>
__device__ __forceinline__ uint32_t verify_vec(const VerifyRows &v, uint32_t Ia, uint32_t Ib,
                                               uint32_t lane) {
  const uint32_t W4 = v.W / 4, a4 = v.c0 / 4, e4 = v.c1 / 4;
  uint32_t bad = 0;
  for (uint32_t I = Ia; I < Ib; I += 4) {
    const uint32_t nrow = min((uint32_t)B, v.H - I * B);
    for (uint32_t c0 = a4; c0 < e4; c0 += 64 * kVerifyAhead) {
      f32x4 xv[kVerifyAhead][B], yv[kVerifyAhead][B];
#pragma unroll
      for (int u = 0; u < kVerifyAhead; ++u)
#pragma unroll
        for (int d = 0; d < B; ++d) {
          const size_t g = (size_t)(I * B + min((uint32_t)d, nrow - 1)) * W4 +
                           min(c0 + 64 * u + lane, e4 - 1);
          xv[u][d] = __builtin_nontemporal_load(gm((const f32x4 *)v.x) + g);
          yv[u][d] = __builtin_nontemporal_load(gm((const f32x4 *)v.y) + g);
        }
#pragma unroll
      for (int u = 0; u < kVerifyAhead; ++u) {
        const uint32_t c = c0 + 64 * u + lane;
        if (c >= e4) continue;
        uint32_t roi[B];
#pragma unroll
        for (int d = 0; d < B; ++d)
          roi[d] = v.mask[(I * B + min((uint32_t)d, nrow - 1) - v.r0) * v.wpr + ((c - a4) >> 3)] >>
                   (4 * (c & 7));
#pragma unroll
        for (int e = 0; e < 4 / B; ++e) {
          double S = 0.0;
          uint32_t n = 0;
#pragma unroll
          for (int d = 0; d < B; ++d)
#pragma unroll
            for (int k = 0; k < B; ++k) {
              const bool in = (uint32_t)d < nrow && (v.mode || !((roi[d] >> (e * B + k)) & 1u));
              const double t = S + (double)xv[u][d][e * B + k];
              S = in ? t : S;
              n += in ? 1u : 0u;
            }
          const double mean = bin_mean(S, n);
#pragma unroll
          for (int d = 0; d < B; ++d)
#pragma unroll
            for (int k = 0; k < B; ++k)
              bad += (uint32_t)d < nrow &&
                     pixel_fails(xv[u][d][e * B + k], yv[u][d][e * B + k],
                                 (roi[d] >> (e * B + k)) & 1u, mean, v.eb);
        }
      }
    }
  }
  return bad;
}

// The failing pixels of the bin whose first pixel is (ia, ja).
__device__ __forceinline__ uint32_t verify_bin(const VerifyRows &v, uint32_t b, uint32_t ia,
                                               uint32_t ja) {
  const uint32_t ie = min(ia + b, v.H), je = min(ja + b, v.W);
  double S = 0.0;
  uint32_t n = 0, bad = 0;
  for (uint32_t r = ia; r < ie; ++r)
    for (uint32_t c = ja; c < je; ++c) {
      const bool roi = (v.mask[(r - v.r0) * v.wpr + (c - v.c0) / 32] >> (c & 31)) & 1u;
      if (v.mode || !roi) {
        S += (double)*gm(v.x + (size_t)r * v.W + c);
        ++n;
      }
    }
  const double mean = bin_mean(S, n);
  for (uint32_t r = ia; r < ie; ++r)
    for (uint32_t c = ja; c < je; ++c) {
      const size_t g = (size_t)r * v.W + c;
      const bool roi = (v.mask[(r - v.r0) * v.wpr + (c - v.c0) / 32] >> (c & 31)) & 1u;
      bad += pixel_fails(*gm(v.x + g), *gm(v.y + g), roi, mean, v.eb);
    }
  return bad;
}

// The same for any b and width, a thread a bin of the block, row after row
// (300 frames of 5x127x20 at b = 6, four bins a row: 51 us, with a wave a bin
// row 189).
__device__ __forceinline__ uint32_t verify_any(const VerifyRows &v, uint32_t b, uint32_t I0,
                                               uint32_t Ib) {
  const uint32_t nb = (v.c1 - v.c0 + b - 1) / b, dI = 256 / nb, dJ = 256 - dI * nb;
  uint32_t I = I0 + threadIdx.x / nb, J = threadIdx.x - (I - I0) * nb, bad = 0;
  while (I < Ib) {
    bad += verify_bin(v, b, I * b, v.c0 + J * b);
    I += dI;
    J += dJ;
    if (J >= nb) {
      J -= nb;
      ++I;
    }
  }
  return bad;
}

// One workgroup per block of `rows` raw rows and `cols` columns of a panel:
// the block's ROI bitmap in LDS from the frame's peaks (the windows of Sec.
// IV, clipped to the panel), then its bin rows, a wave on every fourth: the
// mean of the bin's pixels that enter it (all of them, or those outside every
// window) in fp64, and each pixel's check.  A background pixel passes when
// |y - mean| <= eb + |y| 2^-23 + |mean| 2^-40: the bound, plus the float32
// rounding of the stored value and the rounding of the fp64 sums (taken here
// in another order than the compressor's).  Both frames are read once and HBM
// bounds it: 48 frames of 8x512x1024 at b = 2 take 0.28 ms, 5.7 TB/s (0.34
// with loads that fill the caches); one load a pixel in blocks of 256 rows,
// which left 12 waves a CU, took 1.10 ms.
__global__ __launch_bounds__(256) void k_verify(VerifyBatch vb) {
  extern __shared__ uint32_t s_mask[];
  const uint32_t blkx = xcd_run();
  const uint32_t f = wave_find_frame(vb.wg_prefix, vb.n, blkx);
  const VerifyFrame &vf = vb.frames[f];
  // both stages of this frame finished without an error (else k_vdone
  // reports it)
  if (!vf.valid || vf.cplan->st->status != RSZ_OK || *vf.dplan->status != RSZ_OK) return;
  const uint32_t blk = blkx - vb.wg_prefix[f];
  const uint32_t H = vf.H, W = vf.W, b = vf.b;
  uint32_t rb = blk, c0 = 0, c1 = W;
  if (vf.across > 1) {
    rb = blk / vf.across;
    c0 = (blk - rb * vf.across) * vf.cols;
    c1 = min(c0 + vf.cols, W);
  }
  const uint32_t p = rb / vf.chunks, r0 = (rb - p * vf.chunks) * vf.rows;
  const uint32_t r1 = min(r0 + vf.rows, H), nr = r1 - r0, wpr = (c1 - c0 + 31) / 32;
  for (uint32_t i = threadIdx.x; i < nr * wpr; i += 256) s_mask[i] = 0u;
  __syncthreads();
  const int32_t h = (int32_t)(vf.w / 2);
  for (uint32_t k = threadIdx.x; k < vf.npeaks; k += 256) {
    if ((uint32_t)vf.peaks[3 * k] != p) continue;
    const int32_t pr = vf.peaks[3 * k + 1] - h, pc = vf.peaks[3 * k + 2] - h;
    const int32_t ra = max(pr, (int32_t)r0), rb = min(pr + (int32_t)vf.w, (int32_t)r1);
    const int32_t ca = max(pc, (int32_t)c0), cb = min(pc + (int32_t)vf.w, (int32_t)c1);
    for (int32_t r = ra; r < rb; ++r)
      for (int32_t c = ca; c < cb;) {
        const int32_t e = min(cb, (c & ~31) + 32);
        const uint32_t bits = (e - c == 32 ? ~0u : ((1u << (e - c)) - 1u)) << (c & 31);
        atomicOr(&s_mask[(uint32_t)(r - (int32_t)r0) * wpr + ((uint32_t)c - c0) / 32], bits);
        c = e;
      }
  }
  __syncthreads();
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t I0 = r0 / b, Ia = I0 + wv, Ib = (r1 + b - 1) / b;
  VerifyRows v;
  v.x = vf.x + (size_t)p * H * W;
  v.y = vf.y + (size_t)p * H * W;
  v.mask = s_mask;
  v.H = H;
  v.W = W;
  v.wpr = wpr;
  v.r0 = r0;
  v.c0 = c0;
  v.c1 = c1;
  v.mode = vf.mode;
  v.eb = vf.eb;
  const bool vec = W % 4 == 0 && (((uintptr_t)v.x | (uintptr_t)v.y) & 15) == 0;
  uint32_t bad = 0;
  if (vec && b == 1) bad = verify_vec<1>(v, Ia, Ib, lane);
  else if (vec && b == 2) bad = verify_vec<2>(v, Ia, Ib, lane);
  else if (vec && b == 4) bad = verify_vec<4>(v, Ia, Ib, lane);
  else bad = verify_any(v, b, I0, Ib);
  if (bad) atomicAdd(vf.bad, bad);
}

// A frame whose compression or decoding failed reports 0xFFFFFFFF.
__global__ __launch_bounds__(256) void k_vdone(VerifyBatch vb) {
  const uint32_t f = blockIdx.x * 256 + threadIdx.x;
  if (f >= vb.n) return;
  const VerifyFrame &vf = vb.frames[f];
  if (!vf.valid || vf.cplan->st->status != RSZ_OK || *vf.dplan->status != RSZ_OK)
    *vf.bad = 0xFFFFFFFFu;
}

hipError_t launch_verify_plan(const VerifyBatch &vb, hipStream_t s) {
  prof_begin("k_vplan", s);
  hipLaunchKernelGGL(k_vplan, dim3((vb.n + 255) / 256), dim3(256), 0, s, vb);
  prof_end(s);
  return hipGetLastError();
}

hipError_t launch_verify_check(const VerifyBatch &vb, hipStream_t s) {
  if (vb.total_wgs) {
    prof_begin("k_verify", s);
    hipLaunchKernelGGL(k_verify, dim3(vb.total_wgs), dim3(256), 4 * vb.mask_words, s, vb);
    prof_end(s);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  prof_begin("k_vdone", s);
  hipLaunchKernelGGL(k_vdone, dim3((vb.n + 255) / 256), dim3(256), 0, s, vb);
  prof_end(s);
  return hipGetLastError();
}

}  // namespace rsz
