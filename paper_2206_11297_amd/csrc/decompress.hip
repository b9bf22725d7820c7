// decompress.hip -- HIP kernels that decode ROIBIN-SZ streams on gfx950.
//
// Each kernel is launched once for all the streams of a call: its workgroups
// are numbered across the streams (per-kernel prefixes of per-stream
// counts), and a workgroup works on one stream's plan.
//   k_dec_tables    one workgroup per stream: check code lengths (<= 32,
//                   complete prefix code), peaks and chunk offsets; build
//                   canonical decode tables (11-bit single- and multi-symbol
//                   lookup tables + per-length first codes); write the
//                   status of a stream the host rejected.
//   k_dec_runs      runs coded: one wave per chunk expands its Rice-coded
//                   zero runs back into the Huffman bits, checking
//                   parameters, offsets and that every one bit stays inside
//                   its chunk.
//   k_dec_chunks    one wave per 4096-symbol chunk, lanes on slices of its
//                   bits (self-synchronising starts): Huffman decode to code
//                   bytes; each chunk must end exactly at the next offset.
//   k_dec_outliers  scatter outlier residuals onto the code-0 positions.
//   k_dec_panels    dimension 3: prefix sum of the residuals across the
//                   panels, which leaves the panels' 2D residuals.
//   k_dec_rowsum, k_dec_carry  dimension 1: sums of the bin rows, then the
//                   carry into each row.
//   k_dec_cols      dimensions 2 and 3: the column sums above each band of
//                   kDecTH bin rows.
//   k_dec_pixels    one wave per band (in small batches several): column sums
//                   down the band, row sums across it -> q, and every pixel
//                   float(q * 2eb).  k_dec_panel: the same, a workgroup per
//                   panel, where one covers it.
//   k_dec_roi_decode  coded ROI: class tables, then per window its values
//                   and their inverse prediction (k_dec_roi_unpred for
//                   windows larger than LDS holds).
//   k_dec_roi       ROI windows restored from the payload bits, one wave
//                   per window; overlapping windows must agree on their
//                   shared pixels (with many or large windows:
//                   k_dec_roi_check).
// The inverse Lorenzo step is the prefix sum of the residuals along each
// axis the predictor spans.
#include <algorithm>

#include "rsz_internal.h"

namespace rsz {

constexpr int kLutBits = 11;
constexpr int32_t kMark = INT32_MIN;  // residual slot waiting for its outlier

// tables: first[33], count[33], offs[33], sorted[1024], then the multi-symbol
// table: per 11-bit window two words, up to 4 whole codewords' residuals (a
// signed byte each), and their start bits (bit k: one starts at bit k) | the
// bit after the last << 16 | their count << 24
constexpr int kTabFirst = 0, kTabCount = kTabFirst + 33,
              kTabOffs = kTabCount + 33, kTabSorted = kTabOffs + 33,
              kTabMulti = kTabSorted + kNumSym + 1 /* 8-byte aligned */, kTabWords = kTabMulti + 2 * (1 << kLutBits);

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ void corrupt(int32_t *status) {
  atomicCAS(status, (int32_t)RSZ_OK, (int32_t)RSZ_ERR_CORRUPT);
}

__device__ __forceinline__ bool dec_ok(const int32_t *status) {
  return __hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == RSZ_OK;
}

__device__ __forceinline__ uint32_t rd32(const uint8_t *p, uint64_t off) {
  return *(const uint32_t *)(p + off);
}

// A batch of streams: each kernel's workgroups are numbered across the
// frames, kernel K's per-frame counts in the prefix pre[K * (n + 1) ...]; a
// workgroup finds its frame (wave_find_frame) and works on that frame's plan
// with its index and count inside the frame.
#define RSZ_DEC_FRAME_AT(K, BLK)                                           \
  const uint32_t *pre_ = db.pre + (size_t)(K) * (db.n + 1);                \
  const uint32_t blk_ = (BLK);                                             \
  const uint32_t f_ = wave_find_frame(pre_, db.n, blk_);                   \
  const uint32_t bid = blk_ - pre_[f_];                                    \
  const uint32_t nblk = pre_[f_ + 1] - pre_[f_];                           \
  (void)bid;                                                               \
  (void)nblk;                                                              \
  const DecodePlan &dp = db.plans[f_]
#define RSZ_DEC_FRAME(K) RSZ_DEC_FRAME_AT(K, blockIdx.x)

// One workgroup's chain of steps, each short: a thread takes four symbols'
// lengths and all its loads go out first; the canonical first codes, the
// Kraft sum and the number of used symbols come from the counts per length;
// up to kRankSyms used symbols find their place by counting (a symbol a
// thread, LDS broadcasts); a window's codeword is found against the first
// codes in scalar registers, and the eight windows of a thread go through
// the multi-symbol lookups together. One CSPAD stream: 12.2 us
// (17.6 with LDS searches one after the other and one thread's loops).
constexpr uint32_t kRankSyms = 256;
__global__ __launch_bounds__(256) void k_dec_tables(DecBatch db) {
  RSZ_DEC_FRAME(0);
  __shared__ uint8_t s_len[kNumSym];
  __shared__ uint32_t s_count[kMaxLen + 1], s_first[kMaxLen + 1], s_offs[kMaxLen + 1],
      s_fill[kMaxLen + 1];
  __shared__ uint16_t s_sorted[kNumSym], s_csym[kRankSyms];
  __shared__ uint8_t s_clen[kRankSyms];
  __shared__ uint32_t s_lut[1 << kLutBits], s_tmp[4];
  __shared__ uint64_t s_kraft;
  __shared__ uint32_t s_used;
  __shared__ int s_bad;
  // a stream the host already rejected gets its status and no other work
  if (dp.init_status != RSZ_OK) {
    if (threadIdx.x == 0) *dp.status = dp.init_status;
    return;
  }
  const uint32_t t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const uint32_t l4 = *gm((const uint32_t *)(dp.in + dp.off_lens) + t);   // 4 lengths
  bool bad = false;
  const RSZ_G uint16_t *pk = gm((const uint16_t *)(dp.in + dp.off_peaks));
  for (uint32_t k = t; k < dp.npeaks; k += 256)
    bad |= pk[3 * k] >= dp.P || pk[3 * k + 1] >= dp.H || pk[3 * k + 2] >= dp.W;
  const RSZ_G uint32_t *co = gm((const uint32_t *)(dp.in + dp.off_chunks));
  for (uint32_t c = t; c < dp.nchunks; c += 256) {
    const uint32_t o = co[c], before = co[max(c, 1u) - 1];
    if (o > dp.T || (c == 0 && o != 0) || (c > 0 && o < before)) bad = true;
    // the words that two chunks share, cleared for k_dec_runs
    else if (dp.run_coding) *gm(dp.hbits + (o >> 5)) = 0u;
  }
  if (t == 0) {
    if (dp.run_coding) *gm(dp.hbits + (dp.T >> 5)) = 0u;
    s_bad = 0;
    *dp.status = RSZ_OK;
  }
  if (t <= kMaxLen) {
    s_count[t] = 0;
    s_fill[t] = 0;
  }
  for (int i = t; i < kNumSym; i += 256) s_sorted[i] = 0;
  ((uint32_t *)s_len)[t] = l4;
  __syncthreads();
  uint32_t used = 0;   // of this thread's symbols
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t L = (l4 >> (8 * e)) & 0xFFu;
    if (L > kMaxLen) {
      bad = true;
    } else if (L) {
      atomicAdd(&s_count[L], 1u);
      ++used;
    }
  }
  if (bad) s_bad = 1;
  const uint32_t incl = wave_inclusive_sum(used);
  if (lane == 63) s_tmp[wv] = incl;
  __syncthreads();
  if (t <= kMaxLen) {
    // the codes and symbols of the shorter lengths; thread 0: of all
    uint32_t code = 0, start = 0, n = 0;
    uint64_t kraft = 0;
#pragma unroll
    for (uint32_t k = 1; k <= (uint32_t)kMaxLen; ++k) {
      const uint32_t x = s_count[k];
      kraft += (uint64_t)x << (kMaxLen - k);
      n += x;
      if (k < t) {
        code += x << (t - k);
        start += x;
      }
    }
    s_first[t] = code;
    s_offs[t] = start;
    if (t == 0) {
      s_kraft = kraft;
      s_used = n;
    }
  }
  uint32_t at = incl - used;   // this thread's first used symbol
  for (uint32_t i = 0; i < wv; ++i) at += s_tmp[i];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t L = (l4 >> (8 * e)) & 0xFFu;
    if (L && L <= kMaxLen) {
      if (at < kRankSyms) {
        s_csym[at] = (uint16_t)(4 * t + e);
        s_clen[at] = (uint8_t)L;
      }
      ++at;
    }
  }
  __syncthreads();
  const uint32_t nused = s_used;
  const bool complete = s_kraft == (1ull << kMaxLen);
  const bool single = nused == 1 && s_kraft == (1ull << (kMaxLen - 1));
  if (s_bad || !(complete || single)) {
    if (t == 0) *dp.status = RSZ_ERR_CORRUPT;
    return;
  }
  uint32_t *tab = dp.tables;
  if (t <= kMaxLen && t > 0) {
    *gm(tab + kTabFirst + t) = s_first[t];
    *gm(tab + kTabCount + t) = s_count[t];
    *gm(tab + kTabOffs + t) = s_offs[t];
  }
  // symbols in (length, symbol) order
  if (nused <= kRankSyms) {
    if (t < nused) {
      const uint32_t L = s_clen[t];
      uint32_t r = 0;
#pragma unroll 8
      for (uint32_t j = 0; j < nused; ++j) r += s_clen[j] == L && j < t;
      s_sorted[s_offs[L] + r] = s_csym[t];
    }
  } else if (t < 64) {
    // wave 0 walks the symbols 64 at a time; a symbol's rank among its
    // length is the count of earlier ones
    for (int i = 0; i < kNumSym / 64; ++i) {
      const uint32_t sym = i * 64 + lane, L = s_len[sym];
      uint64_t pending = __builtin_amdgcn_uicmp(L, 0u, 33 /* ne */);
      while (pending) {
        const int leader = __builtin_ctzll(pending);
        const uint32_t Lc = __builtin_amdgcn_readlane(L, leader);
        const uint64_t same = __builtin_amdgcn_uicmp(L, Lc, 32 /* eq */) & pending;
        if ((same >> lane) & 1ull)
          s_sorted[s_offs[Lc] + s_fill[Lc] + __builtin_popcountll(same & ((1ull << lane) - 1))] =
              (uint16_t)sym;
        wave_sync();
        if ((int)lane == leader) s_fill[Lc] += (uint32_t)__builtin_popcountll(same);
        wave_sync();
        pending &= ~same;
      }
    }
  }
  __syncthreads();
  for (int i = t; i < kNumSym; i += 256) *gm(tab + kTabSorted + i) = s_sorted[i];
  // lookup entry of an 11-bit window: the codeword (at most 11 bits) that is
  // its prefix, if any (the code is prefix-free: at most one)
  constexpr int kWin = (1 << kLutBits) / 256;   // windows a thread
  uint32_t slot[kWin], len[kWin];
#pragma unroll
  for (int w = 0; w < kWin; ++w) slot[w] = len[w] = 0;
#pragma unroll
  for (uint32_t L = 1; L <= (uint32_t)kLutBits; ++L) {
    const uint32_t n = __builtin_amdgcn_readfirstlane(s_count[L]);
    const uint32_t f = __builtin_amdgcn_readfirstlane(s_first[L]);
    const uint32_t o = __builtin_amdgcn_readfirstlane(s_offs[L]);
#pragma unroll
    for (int w = 0; w < kWin; ++w) {
      const uint32_t cd = ((t + 256 * w) >> (kLutBits - L)) - f;
      const bool hit = cd < n && len[w] == 0;
      slot[w] = hit ? o + cd : slot[w];
      len[w] = hit ? L : len[w];
    }
  }
#pragma unroll
  for (int w = 0; w < kWin; ++w)
    s_lut[t + 256 * w] = len[w] ? (uint32_t)s_sorted[slot[w]] | len[w] << 16 : 0u;
  __syncthreads();
  // multi-symbol entry: the whole codewords (at most 4) that the window
  // holds one after the other, while their residuals fit a byte
  uint32_t bytes[kWin], n[kWin], pos[kWin], starts[kWin];
#pragma unroll
  for (int w = 0; w < kWin; ++w) bytes[w] = n[w] = pos[w] = starts[w] = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    uint32_t e[kWin];
#pragma unroll
    for (int w = 0; w < kWin; ++w)
      e[w] = s_lut[((t + 256 * w) << pos[w]) & ((1u << kLutBits) - 1)];
#pragma unroll
    for (int w = 0; w < kWin; ++w) {
      const uint32_t L = e[w] >> 16;
      const int32_t r = (int32_t)(e[w] & 0x3FFu) - kRadius;
      const bool take = n[w] == (uint32_t)k && e[w] && pos[w] + L <= (uint32_t)kLutBits &&
                        r >= -127 && r <= 127;
      if (take) {
        bytes[w] |= (uint32_t)(uint8_t)r << (8 * k);
        starts[w] |= 1u << pos[w];
        pos[w] += L;
        ++n[w];
      }
    }
  }
#pragma unroll
  for (int w = 0; w < kWin; ++w)
    *(RSZ_G u32x2 *)gm(tab + kTabMulti + 2 * (t + 256 * w)) =
        u32x2{bytes[w], starts[w] | pos[w] << 16 | n[w] << 24};
}

// Exclusive prefix sum of v over the lanes of a wave; total of all lanes.
__device__ __forceinline__ uint64_t wave_exclusive_scan_u64(uint64_t v, uint64_t &total) {
  const int lane = threadIdx.x & 63;
  uint64_t x = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint64_t y = __shfl_up(x, d);
    if (lane >= d) x += y;
  }
  total = __shfl(x, 63);
  return x - v;
}

// The 32 bits of words (n of them, zero beyond) from bit pos, MSB-first.
__device__ __forceinline__ uint32_t peek_bits(const uint32_t *w, uint32_t n, uint32_t pos) {
  const uint32_t i = pos >> 5, s = pos & 31;
  const uint32_t hi = i < n ? *gm(w + i) : 0u, lo = i + 1 < n ? *gm(w + i + 1) : 0u;
  return (uint32_t)((((uint64_t)hi << 32 | lo) << s) >> 32);
}

// A wave's stretch of a bit section: staged (words from w0 in LDS, zero words
// after them) or in the stream.
struct BitSrc {
  const uint32_t *lds, *words;
  uint32_t w0, n;
  bool staged;
  __device__ __forceinline__ uint32_t peek(uint32_t pos) const {
    if (!staged) return peek_bits(words, n, pos);
    const uint32_t i = (pos >> 5) - w0;
    return (uint32_t)((((uint64_t)lds[i] << 32 | lds[i + 1]) << (pos & 31)) >> 32);
  }
};

// ------------------------------------------------------------ run stage

constexpr uint32_t kRunKMax = 20;

// A wave's words of run bits and of expanded Huffman bits in LDS; a chunk
// with more works in global memory.
constexpr uint32_t kRunIn = 512, kRunOut = 1024;

// Run codes from pos while pos < lim: each is a unary quotient q (ones closed
// by a zero) and k low bits, the zero run before the next one bit.  Leaves
// pos at the first boundary >= lim and returns the Huffman bits they stand
// for; inval when a code runs past rend.  Calls f(run) for each.
template <class F>
__device__ __forceinline__ uint64_t rice_codes(const BitSrc &src, uint32_t &pos, uint32_t lim,
                                               uint32_t rend, uint32_t k, bool &inval, F f) {
  uint64_t adv = 0;
  while (pos < lim) {
    uint64_t q = 0;
    uint32_t x = src.peek(pos), n = ~x ? (uint32_t)__builtin_clz(~x) : 32u;
    while (n == 32 && rend - pos > 32) {   // 32 ones and more to come
      q += 32;
      pos += 32;
      x = src.peek(pos);
      n = ~x ? (uint32_t)__builtin_clz(~x) : 32u;
    }
    // no closing zero, or no room for the low bits, before the chunk's end
    if (n + 1 + k > rend - pos || n == 32) {
      inval = true;
      break;
    }
    q += n;
    uint32_t low = 0;
    if (k) low = n + 1 + k <= 32 ? (x << (n + 1)) >> (32 - k) : src.peek(pos + n + 1) >> (32 - k);
    pos += n + 1 + k;
    const uint64_t run = (q << k) | low;
    f(run);
    adv += run + 1;
  }
  return adv;
}

// Fewest bits of a slice (but for a chunk's only one), a few codes of parameter
// k: a start is found by the lane before only once a slice holds some, and
// where each held less than one, as in chunks of few and long runs, the lanes
// found theirs one after the other (10 frames of 16x512x1024 at b = 2, eb 5: 21
// us, 40 in 64 slices whatever the length; 32 bits for every k are too many for
// short codes: 300 frames of 2x34x91 at b = 8, eb 0.5: 13 us against 25).
__device__ __forceinline__ uint32_t run_slice(uint32_t k) { return 4 * (k + 2); }

// One wave per chunk.  Chunk c's codes occupy run bits [runoffs[c],
// runoffs[c + 1]), cut into up to 64 slices and decoded as k_dec_chunks decodes
// its own (self-synchronising starts); a scan of the Huffman bits that the lanes'
// codes stand for places their one bits, which are ORed into the chunk's
// words in LDS and leave as whole words (the two that the chunks beside may
// share by atomics, on words that k_dec_tables cleared).  One thread a chunk,
// as before, waited for its own loads bit by bit: 0.55 against 0.09 ms on
// 250 CSPAD frames.  A valid section has parameters <= 20 (zero padding),
// offsets from 0 that never decrease, a last offset whose words end the
// stream exactly, codes that end exactly at the next offset, and every one
// bit inside its chunk [chunk_off[c], chunk_off[c + 1]).  Reads stay inside
// the section once its size is checked; every loop ends after at most one
// step per run bit.
__global__ __launch_bounds__(256) void k_dec_runs(DecBatch db) {
  RSZ_DEC_FRAME(1);
  __shared__ uint32_t s_in[4][kRunIn + 2], s_out[4][kRunOut];
  const int lane = threadIdx.x & 63;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t c = bid * 4 + wv;
  if (c >= dp.nchunks || !dec_ok(dp.status)) return;
  const RSZ_G uint8_t *kpar = gm(dp.in + dp.off_run);
  const RSZ_G uint32_t *ro = gm((const uint32_t *)(dp.in + dp.off_runoffs));
  const RSZ_G uint32_t *co = gm((const uint32_t *)(dp.in + dp.off_chunks));
  const uint32_t Trun = ro[dp.nchunks], r0 = ro[0];
  const uint32_t k = kpar[c], rs = ro[c], rend = ro[c + 1];
  const uint32_t start = co[c];
  const uint32_t end = c + 1 < dp.nchunks ? co[c + 1] : (uint32_t)dp.T;   // T < 2^32
  const uint64_t nrw = ((uint64_t)Trun + 31) / 32;
  bool bad = dp.off_runbits + 4 * nrw != dp.total || r0 != 0 || k > kRunKMax;
  if (c + 1 == dp.nchunks)   // padding of the parameters
    for (uint64_t t = dp.nchunks; t < align_up(dp.nchunks, 4); ++t) bad |= kpar[t] != 0;
  bad |= start > end || end > dp.T || rend < rs || rend > Trun;
  if (bad) {
    if (lane == 0) corrupt(dp.status);
    return;
  }
  BitSrc src;
  src.words = (const uint32_t *)(dp.in + dp.off_runbits);
  src.n = (uint32_t)nrw;
  src.lds = s_in[wv];
  src.w0 = rs >> 5;
  const uint32_t nin = (uint32_t)(((uint64_t)rend + 31) / 32) - src.w0;
  src.staged = nin <= kRunIn;
  if (src.staged)
    for (uint32_t i = lane; i < nin + 2; i += 64)
      s_in[wv][i] = i < nin ? *gm(src.words + src.w0 + i) : 0u;
  const uint32_t ow0 = start >> 5;
  const uint32_t nout = (uint32_t)(((uint64_t)end + 31) / 32) - ow0;
  const bool sout = nout <= kRunOut;
  if (sout)
    for (uint32_t i = lane; i < nout; i += 64) s_out[wv][i] = 0u;
  wave_sync();
  const uint64_t len = rend - rs;
  const uint32_t slices = min(64u, max(1u, (rend - rs) / run_slice(k)));
  auto cut = [&](uint32_t i) {
    if (slices == 64) return i == 64 ? rend : rs + (uint32_t)(len * i / 64);
    return i >= slices ? rend : rs + (uint32_t)len * i / slices;   // (a short chunk)
  };
  const uint32_t lim = cut((uint32_t)lane + 1);
  uint32_t from = cut((uint32_t)lane), pos = from;
  uint64_t adv = 0;
  bool converged = false, inv = false, last_ok = false;
  for (int round = 0; round <= 64 && !converged; ++round) {
    pos = from;
    inv = false;
    adv = rice_codes(src, pos, lim, rend, k, inv, [](uint64_t) {});
    // a lane stuck on no code hands on no boundary (its next lane's slice)
    const uint32_t stop = inv ? lim : pos;
    const uint32_t prev = __shfl_up(stop, 1);
    const bool changed = lane > 0 && prev != from;
    converged = __ballot(changed) == 0;
    if (!converged && lane > 0) from = prev;
  }
  last_ok = __shfl((int)(pos == rend), 63) != 0;
  uint64_t tot;
  const uint64_t ex = wave_exclusive_scan_u64(adv, tot);
  bad = !converged || __ballot(inv) != 0 || !last_ok || tot > (uint64_t)(end - start);
  if (bad) {
    if (lane == 0) corrupt(dp.status);
    return;
  }
  if (!sout) {   // the chunk's own words, cleared before any bit is set
    for (uint32_t i = lane; i < nout; i += 64)
      if ((i > 0 || !(start & 31)) && (i + 1 < nout || !(end & 31))) *gm(dp.hbits + ow0 + i) = 0u;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  }
  uint32_t b = start + (uint32_t)ex;   // next Huffman bit
  uint32_t cw = b >> 5, acc = 0;       // the one bits of word cw so far
  auto flush = [&]() {
    if (!acc) return;
    if (sout) atomicOr(&s_out[wv][cw - ow0], acc);
    else atomicOr(dp.hbits + cw, acc);
  };
  pos = from;
  rice_codes(src, pos, lim, rend, k, inv, [&](uint64_t run) {
    b += (uint32_t)run;
    if ((b >> 5) != cw) {
      flush();
      cw = b >> 5;
      acc = 0;
    }
    acc |= 0x80000000u >> (b & 31);
    ++b;
  });
  flush();
  if (!sout) return;
  wave_sync();
  for (uint32_t i = lane; i < nout; i += 64) {
    const uint32_t v = s_out[wv][i];
    if ((i > 0 || !(start & 31)) && (i + 1 < nout || !(end & 31))) *gm(dp.hbits + ow0 + i) = v;
    else if (v) atomicOr(dp.hbits + ow0 + i, v);
  }
}

// The chunk decoder's tables in LDS.
struct CodeTables {
  uint2 multi[1 << kLutBits];
  uint32_t first[kMaxLen + 1], count[kMaxLen + 1], offs[kMaxLen + 1];
  uint16_t sorted[kNumSym];
};

// The codeword at the top of v by its length class, for those that have no
// multi-symbol entry: its symbol, L its length (0: no codeword).
__device__ __forceinline__ uint32_t long_codeword(const CodeTables &t, uint32_t v, uint32_t &L) {
#pragma unroll 1
  for (L = 1; L <= (uint32_t)kMaxLen; ++L) {
    const uint32_t n = t.count[L], cd = (v >> (32 - L)) - t.first[L];
    if (n && cd < n) return t.sorted[t.offs[L] + cd];
  }
  L = 0;
  return 0;
}

// One step of the decoder at pos (< lim): up to n symbols that start before
// lim.  n: how many (0: no codeword), adv: their bits, starts: the start bits
// of the first 32 of them, bytes: their residuals (signed bytes; run: a run of
// residuals 0, whose bytes are 0).  esc: the one symbol's byte is kEscByte and
// sym its symbol.  With `zrun` (residual 0's codeword is the single bit 0) a
// window of zero bits is a run of residuals 0, taken at once up to lim.
constexpr uint32_t kEscByte = 0x80u;
struct Step {
  uint32_t n, adv, starts, bytes, sym;
  bool esc;
};
__device__ __forceinline__ Step code_step(const CodeTables &t, uint32_t v, uint32_t room,
                                          bool zrun) {
  Step s;
  s.esc = false;
  if (zrun && !(v >> (32 - kLutBits))) {
    s.n = s.adv = min(v ? (uint32_t)__builtin_clz(v) : 32u, room);
    s.starts = s.n == 32 ? ~0u : (1u << s.n) - 1u;
    s.bytes = 0;
    return s;
  }
  const uint2 e = t.multi[v >> (32 - kLutBits)];
  s.n = e.y >> 24;
  if (s.n) {
    const uint32_t all = e.y & 0xFFFFu, in = all & ((1u << min(room, 16u)) - 1u);
    s.adv = (e.y >> 16) & 0xFFu;
    s.starts = in;
    s.bytes = e.x;
    if (in != all) {   // the first start at or past the limit ends the step
      s.n = __builtin_popcount(in);
      s.adv = (uint32_t)__builtin_ctz(all & ~in);
      s.bytes &= (1u << (8 * s.n)) - 1u;   // n < 4 here
    }
    return s;
  }
  uint32_t L;
  s.sym = long_codeword(t, v, L);
  s.n = L ? 1u : 0u;
  s.adv = L;
  s.starts = 1;
  const int32_t r = (int32_t)s.sym - kRadius;
  s.esc = r < -127 || r > 127;
  s.bytes = s.esc ? kEscByte : (uint32_t)(uint8_t)r;
  return s;
}

// One wave per chunk.  The chunk's bits split into 64 equal slices; lane i
// decodes from a start s_i until the first codeword boundary at or past the
// next slice.  Lane 0 starts at the chunk offset, a true boundary; every
// other lane starts at its slice's first bit, and keeps where in the slice's
// first 64 bits its codewords started.  Then it starts again at the boundary
// the lane before it stopped at, until no start changes: then every start is
// a true boundary (by induction from lane 0).  Huffman decoding
// resynchronises within a few codewords: once the second decode meets a start
// of the first, the rest is the first's, so a restart takes a few symbols and
// not the slice.  A scan of the lanes' symbol counts places their outputs,
// and a last pass ORs their bytes into the chunk's in LDS, which leave as
// whole 16-byte stores.  A valid chunk decodes to exactly its symbol count
// and ends exactly at the next chunk offset.
//
// The LDS lookups of a lane follow one another and bound it (the bits come
// from LDS too, when the chunk has at most kChunkIn words of them), at 16
// waves a CU: 8 share the tables' 18 KB (4 a workgroup 0.39 ms, 16 0.35, 8
// 0.34 on 1000 CSPAD streams), and the next chunk's words arrive while one is
// decoded (0.32 ms; 0.25 on 128 dense streams of 8x512x1024, 0.28 without).
// With the bits by global loads, three whole decodes a slice and byte stores
// straight to HBM it took 0.40 and 0.48 ms. kChunkIn is what two workgroups a
// CU leave of the 160 KB: 7.25 bits a symbol (512 frames of 16x512x1024 at
// eb 1, about 5.5 bits: 7.2 ms, with 640 words 8.3; at eb 10 1.8 with both).
constexpr uint32_t kChunkIn = 928;
constexpr uint32_t kChunkWaves = 8;
__global__ __launch_bounds__(64 * kChunkWaves) void k_dec_chunks(DecBatch db) {
  RSZ_DEC_FRAME(2);
  __shared__ CodeTables s_t;
  __shared__ uint32_t s_in[kChunkWaves][kChunkIn + 2];
  __shared__ __align__(16) uint32_t s_out[kChunkWaves][kChunk / 4];
  for (int i = threadIdx.x; i < (1 << kLutBits); i += 64 * kChunkWaves)
    s_t.multi[i] = make_uint2(dp.tables[kTabMulti + 2 * i], dp.tables[kTabMulti + 2 * i + 1]);
  for (int i = threadIdx.x; i < kNumSym; i += 64 * kChunkWaves)
    s_t.sorted[i] = (uint16_t)dp.tables[kTabSorted + i];
  if (threadIdx.x <= kMaxLen) {
    s_t.first[threadIdx.x] = dp.tables[kTabFirst + threadIdx.x];
    s_t.count[threadIdx.x] = dp.tables[kTabCount + threadIdx.x];
    s_t.offs[threadIdx.x] = dp.tables[kTabOffs + threadIdx.x];
  }
  const int lane = threadIdx.x & 63;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool ok = dec_ok(dp.status);
  const RSZ_G uint32_t *co = gm((const uint32_t *)(dp.in + dp.off_chunks));
  const uint32_t T = (uint32_t)dp.T;   // <= 32 nbins < 2^32
  const uint32_t nchunks = dp.nchunks, nbins = dp.nbins;
  int32_t *status = dp.status, *res = dp.res;
  uint8_t *res8 = dp.res8;
  BitSrc src;
  src.words = dp.bits;   // the stream's bitstream, or the expanded runs
  src.n = (uint32_t)((dp.T + 31) / 32);
  src.lds = s_in[wv];
  __syncthreads();   // tables loaded
  if (!ok) return;
  // residual 0 (symbol 512) coded as the single bit 0: the only length-1
  // code, canonical code 0
  const bool zrun = s_t.count[1] == 1 && s_t.first[1] == 0 && s_t.sorted[s_t.offs[1]] == kRadius;
  // the chunk's words and the two after them (a window reaches past its end),
  // fetched while the chunk before is decoded
  constexpr int kFetch = (int)((kChunkIn + 2 + 63) / 64);
  uint32_t next[kFetch], S = 0, E = 0, nin = 0;
  const uint32_t c0 = bid * db.chunk_reps * kChunkWaves + wv;
  const uint32_t cend = min(c0 + db.chunk_reps * kChunkWaves, nchunks);
  auto bounds = [&](uint32_t c, uint32_t &lo, uint32_t &hi) {
    lo = co[c];
    hi = max(lo, c + 1 < nchunks ? co[c + 1] : T);
  };
  auto fetch = [&](uint32_t lo, uint32_t hi) {
    nin = (uint32_t)(((uint64_t)hi + 31) / 32) - (lo >> 5) + 2;
#pragma unroll
    for (int i = 0; i < kFetch; ++i) {
      const uint32_t k = 64 * i + (uint32_t)lane, w = (lo >> 5) + k;
      next[i] = nin <= kChunkIn + 2 && k < nin && w < src.n ? *gm(src.words + w) : 0u;
    }
  };
  if (c0 < cend) {
    bounds(c0, S, E);
    fetch(S, E);
  }
  for (uint32_t c = c0; c < cend; c += kChunkWaves) {
    src.w0 = S >> 5;
    src.staged = nin <= kChunkIn + 2;
    if (src.staged) {
#pragma unroll
      for (int i = 0; i < kFetch; ++i)
        if (64 * i + (uint32_t)lane < nin) s_in[wv][64 * i + lane] = next[i];
    }
    uint32_t nS = 0, nE = 0;
    if (c + kChunkWaves < cend) bounds(c + kChunkWaves, nS, nE);
    for (uint32_t i = lane; i < kChunk / 16; i += 64)
      *(uint4 *)(s_out[wv] + 4 * i) = make_uint4(0u, 0u, 0u, 0u);
    wave_sync();
    const uint32_t g0 = c * kChunk;
    const uint32_t nsym = min(kChunk, nbins - g0);
    const uint64_t len = E - S;
    const uint32_t lim = lane == 63 ? E : S + (uint32_t)(len * (uint64_t)(lane + 1) / 64);
    const uint32_t s0 = S + (uint32_t)(len * (uint64_t)lane / 64);   // the slice's first bit
    constexpr uint32_t kStuck = ~0u;   // (no position: T < 2^32 - 1)
    // the first decode: its codeword starts within 64 bits of s0, its symbols,
    // where it stopped (kStuck: at a bit pattern that is no codeword)
    uint64_t seen = 0;
    uint32_t m0 = 0, stop0;
    {
      uint32_t pos = s0;
      bool inv = false;
      while (pos < lim) {
        const Step st = code_step(s_t, src.peek(pos), lim - pos, zrun);
        if (!st.n) {
          inv = true;
          break;
        }
        const uint32_t off = pos - s0;
        if (off < 64) seen |= (uint64_t)st.starts << off;
        pos += st.adv;
        m0 += st.n;
      }
      stop0 = inv ? kStuck : pos;
    }
    if (c + kChunkWaves < cend) fetch(nS, nE);
    uint32_t start = s0, stop = stop0, m = m0;
    bool converged = false;
    for (int round = 0; round <= 64 && !converged; ++round) {
      // the boundary the lane before stopped at is this lane's start (a stuck
      // lane hands on none)
      const uint32_t prev = __shfl_up(stop, 1);
      const uint32_t next = lane == 0 ? S : (prev == kStuck ? lim : prev);
      const bool changed = next != start;
      converged = __ballot(changed) == 0;
      if (!changed) continue;
      start = next;
      uint32_t pos = start, n = 0;
      bool inv = false, met = false;
      while (pos < lim) {
        const uint32_t off = pos - s0;
        if (off < 64 && ((seen >> off) & 1u)) {
          met = true;
          n += m0 - (uint32_t)__builtin_popcountll(seen & ((1ull << off) - 1ull));
          break;
        }
        // one symbol at a time while the first decode's starts are known
        Step st = code_step(s_t, src.peek(pos), lim - pos, zrun);
        if (!st.n) {
          inv = true;
          break;
        }
        if (off < 64 && st.n > 1) {
          const uint32_t second = st.starts & (st.starts - 1);
          st.adv = (uint32_t)__builtin_ctz(second);
          st.n = 1;
        }
        pos += st.adv;
        n += st.n;
      }
      m = n;
      stop = met ? stop0 : (inv ? kStuck : pos);
    }
    uint64_t tot;
    const uint32_t off = (uint32_t)wave_exclusive_scan_u64(m, tot);
    const uint32_t last = __shfl(stop, 63);
    // a valid chunk converges (64 rounds at most) with no non-codeword on its path
    if (!converged || __ballot(stop == kStuck) != 0 || tot != nsym || last != E) {
      if (lane == 0) corrupt(status);
      return;
    }
    // the output pass, from the true starts
    uint32_t pos = start, k = off;
    while (pos < lim) {
      const Step st = code_step(s_t, src.peek(pos), lim - pos, zrun);
      if (!st.n) break;   // (not reached: the same steps succeeded above)
      if (st.bytes) {
        const uint64_t w = (uint64_t)st.bytes << (8 * (k & 3));
        if ((uint32_t)w) atomicOr(&s_out[wv][k >> 2], (uint32_t)w);
        if ((uint32_t)(w >> 32)) atomicOr(&s_out[wv][(k >> 2) + 1], (uint32_t)(w >> 32));
        if (st.esc) *gm(res + g0 + k) = st.sym ? (int32_t)st.sym - kRadius : kMark;
      }
      pos += st.adv;
      k += st.n;
    }
    wave_sync();
    // whole 16-byte groups (the region holds 64 bytes past the last chunk)
    uint8_t *rc = res8 + g0;
    for (uint32_t i = 16 * lane; i < nsym; i += 1024) {
      const u32x4 x = *(const u32x4 *)((const uint8_t *)s_out[wv] + i);
      *gm((u32x4 *)(rc + i)) = x ^ 0x80808080u;
    }
    wave_sync();
    S = nS;
    E = nE;
  }
}

// The outliers into their bins' residual slots; the frame's workgroups take
// every nblk-th block of 256 (a verification plan launches a fixed number
// per frame, the outlier count being known only on the device).
__global__ __launch_bounds__(256) void k_dec_outliers(DecBatch db) {
  RSZ_DEC_FRAME(3);
  if (!dec_ok(dp.status)) return;
  const uint32_t *oi = (const uint32_t *)(dp.in + dp.off_oidx);
  const int32_t *orr = (const int32_t *)(dp.in + dp.off_ores);
  // |q| < 2^28 bounds a residual of dimension d below 2^(28+d) in magnitude
  const int64_t lim = (int64_t)1 << (28 + dp.dim);
  for (uint32_t k = bid * 256 + threadIdx.x; k < dp.n_out; k += nblk * 256) {
    const uint32_t g = oi[k];
    const int32_t r = orr[k];
    // the bin must have decoded as code 0 (its code byte 0 and the mark in res)
    if (g >= dp.nbins || (k > 0 && g <= oi[k - 1]) || (r > -kRadius && r < kRadius) ||
        (int64_t)r <= -lim || (int64_t)r >= lim || dp.res8[g] != 0 ||
        dp.res[g] != kMark) {
      corrupt(dp.status);
      return;
    }
    dp.res[g] = r;
  }
}

// ------------------------------------------------- inverse Lorenzo, pixels

// The residuals travel as one byte a bin (res8), and every pass below reads
// them as such: r + 128, or 0 with the residual in res (an escape).  A panel
// is cut into bands of kDecTH bin rows.  q of a bin is the sum of every
// residual above and left of it, so a band needs the column sums of the rows
// above it (k_dec_cols reads the bytes once more for them, 1 byte a bin
// against the 4 b^2 its pixels take) and nothing of its neighbours beside:
// one wave walks it from left to right with the rows' carries in scalar
// registers, takes all its rows' bytes of a strip at once and writes whole
// lines of pixels.  Panels that one workgroup covers (k_dec_panel) take the
// column sums through LDS instead and read the bytes once.  Any panel size
// and dimension takes these passes; int32 residuals in HBM with a pass per
// axis took 0.86 ms where this takes 0.43 on 128 frames of 8x512x1024 at b =
// 2, and 1.95 ms against 0.56 on 250 frames of 32x185x388 in 3D.  What bounds
// them is the pixels' stores: 5.0 TB/s on 8x512x1024, 4.9 on 32x185x388,
// where a kernel that only stores reaches 5.3 to 5.7 in this order.

// 0x80 in each byte of x that is zero, 0 elsewhere.
__device__ __forceinline__ uint32_t zero_bytes(uint32_t x) {
  return ~(((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x | 0x7F7F7F7Fu);
}

// Words at any address (global accesses take any alignment).
typedef uint32_t u32_any __attribute__((aligned(1)));
typedef uint16_t u16_any __attribute__((aligned(1)));
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(1)));
__device__ __forceinline__ uint32_t ld_any32(const uint8_t *p) {
  return *(const RSZ_G u32_any *)p;
}
__device__ __forceinline__ uint32_t ld_any16(const uint8_t *p) {
  return *(const RSZ_G u16_any *)p;
}

// Dimension 3: the residuals' inclusive prefix sum across the panels, in
// place, after which each panel holds its 2D residuals.  A thread takes 4
// consecutive bins of the panel plane through its panels, kPanelsAhead
// panels' bytes loaded before any is stored: through all of them, or, where
// the planes are small and the panels many, through one of dp.panel_segs
// segments, whose sums are taken first.
constexpr uint32_t kPanelsAhead = 8;

// Panels [p0, p1) of the n (<= 4) bins at src: run advances past them; WRITE:
// they become their prefix sums.  Returns whether an outlier's mark is left.
template <bool WRITE>
__device__ __forceinline__ bool panels_sum(uint8_t *src, int32_t *res, uint32_t plane, uint32_t p0,
                                           uint32_t p1, uint32_t n, uint32_t (&run)[4]) {
  bool bad = false;
  for (; p0 < p1; p0 += kPanelsAhead) {
    uint32_t w[kPanelsAhead];
#pragma unroll
    for (uint32_t k = 0; k < kPanelsAhead; ++k)
      w[k] = ld_any32(src + (size_t)min(p0 + k, p1 - 1) * plane);
#pragma unroll
    for (uint32_t k = 0; k < kPanelsAhead; ++k) {
      if (p0 + k >= p1) break;
      const size_t o = (size_t)(p0 + k) * plane;
      uint32_t y = 0;
#pragma unroll
      for (uint32_t t = 0; t < 4; ++t) {
        const uint32_t by = (w[k] >> (8 * t)) & 0xFFu;
        int32_t r = (int32_t)by - 128;
        if (by == 0 && t < n) {
          r = *gm(res + o + t);
          bad |= r == kMark;
        }
        run[t] += (uint32_t)r;
        if (WRITE) {
          const bool small = run[t] + 127u < 255u;
          y |= (small ? run[t] + 128u : 0u) << (8 * t);
          if (!small && t < n) *gm(res + o + t) = (int32_t)run[t];
        }
      }
      if (WRITE && n == 4) {
        *(RSZ_G u32_any *)(src + o) = y;
      } else if (WRITE) {   // the plane's last bins: the bytes after them are another's
        for (uint32_t t = 0; t < n; ++t) *gm(src + o + t) = (uint8_t)(y >> (8 * t));
      }
    }
  }
  return bad;
}

__global__ __launch_bounds__(256) void k_dec_panels(DecBatch db) {
  RSZ_DEC_FRAME(4);
  const uint32_t plane = dp.Hb * dp.Wb, P = dp.P, segs = dp.panel_segs;
  if (segs == 1) {
    const uint32_t c = (bid * 256 + threadIdx.x) * 4;
    if (c >= plane || !dec_ok(dp.status)) return;
    uint32_t run[4] = {0u, 0u, 0u, 0u};
    if (panels_sum<true>(dp.res8 + c, dp.res + c, plane, 0, P, min(4u, plane - c), run))
      corrupt(dp.status);
    return;
  }
  __shared__ uint32_t s_sum[256][4];
  __shared__ int s_ok;
  if (threadIdx.x == 0) s_ok = dec_ok(dp.status);
  __syncthreads();
  if (!s_ok) return;
  const uint32_t cols = 256 / segs, seg = threadIdx.x / cols, col = threadIdx.x - seg * cols;
  const uint32_t c = (bid * cols + col) * 4, n = c < plane ? min(4u, plane - c) : 0u;
  const uint32_t len = (P + segs - 1) / segs, p0 = min(seg * len, P), p1 = min(p0 + len, P);
  uint32_t run[4] = {0u, 0u, 0u, 0u};
  if (n) (void)panels_sum<false>(dp.res8 + c, dp.res + c, plane, p0, p1, n, run);
#pragma unroll
  for (uint32_t t = 0; t < 4; ++t) {
    s_sum[threadIdx.x][t] = run[t];
    run[t] = 0;
  }
  __syncthreads();   // (every segment of these bins is read before any is written)
  for (uint32_t i = col; i < threadIdx.x; i += cols)
#pragma unroll
    for (uint32_t t = 0; t < 4; ++t) run[t] += s_sum[i][t];
  if (n && panels_sum<true>(dp.res8 + c, dp.res + c, plane, p0, p1, n, run)) corrupt(dp.status);
}

// Dimension 1: the sum of each bin row (kDecRowsPerWave rows a wave).
constexpr uint32_t kDecRowsPerWave = 4;
__global__ __launch_bounds__(256) void k_dec_rowsum(DecBatch db) {
  RSZ_DEC_FRAME(5);
  const uint32_t row0 = (bid * 4 + (threadIdx.x >> 6)) * kDecRowsPerWave;
  const int lane = threadIdx.x & 63;
  const uint32_t nrows = dp.P * dp.Hb, Wb = dp.Wb;
  if (row0 >= nrows || !dec_ok(dp.status)) return;
  uint32_t sum[kDecRowsPerWave];
#pragma unroll
  for (uint32_t k = 0; k < kDecRowsPerWave; ++k) sum[k] = 0;
  for (uint32_t j0 = 0; j0 < Wb; j0 += 256) {
    const uint32_t j = j0 + 4 * lane, jc = min(j, Wb - 1);
    const uint32_t n = j < Wb ? min(4u, Wb - j) : 0u;   // this lane's bins of the row
    const uint32_t keep = n == 4 ? ~0u : (1u << (8 * n)) - 1u;
    uint32_t w[kDecRowsPerWave];
#pragma unroll
    for (uint32_t k = 0; k < kDecRowsPerWave; ++k)
      w[k] = ld_any32(dp.res8 + (size_t)min(row0 + k, nrows - 1) * Wb + jc);
#pragma unroll
    for (uint32_t k = 0; k < kDecRowsPerWave; ++k) {
      const uint32_t x = w[k] & keep;
      sum[k] = __builtin_amdgcn_sad_u8(x, 0u, sum[k]) - 128u * n;
      for (uint32_t z = zero_bytes(x) & keep; z; z &= z - 1) {   // escapes
        const uint32_t t = (uint32_t)__builtin_ctz(z) >> 3;
        sum[k] += 128u + (uint32_t)*gm(dp.res + (size_t)min(row0 + k, nrows - 1) * Wb + j + t);
      }
    }
  }
#pragma unroll
  for (uint32_t k = 0; k < kDecRowsPerWave; ++k) {
    const uint32_t tot = wave_inclusive_sum(sum[k]);
    if (lane == 63 && row0 + k < nrows) *gm(dp.carry + row0 + k) = tot;
  }
}

// Dimension 1: the raster sequence continues across rows, so each row adds
// the sum of every row before it.  One workgroup scans the row sums into
// exclusive carries.
__global__ __launch_bounds__(256) void k_dec_carry(DecBatch db) {
  RSZ_DEC_FRAME(6);
  __shared__ uint32_t s_w[4];
  __shared__ int s_ok;
  if (threadIdx.x == 0) s_ok = dec_ok(dp.status);
  __syncthreads();
  if (!s_ok) return;
  const uint32_t rows = dp.P * dp.Hb;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t run = 0;
  for (uint32_t r0 = 0; r0 < rows; r0 += 1024) {
    const uint32_t row = r0 + 4 * threadIdx.x;
    uint32_t v[4], sum = 0;
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) v[k] = row + k < rows ? *gm(dp.carry + row + k) : 0u;
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) sum += v[k];
    const uint32_t x = wave_inclusive_sum(sum);
    if (lane == 63) s_w[wv] = x;
    __syncthreads();
    uint32_t before = run + x - sum;
    for (int i = 0; i < wv; ++i) before += s_w[i];
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
      if (row + k < rows) *gm(dp.carry + row + k) = before;
      before += v[k];
    }
    run += s_w[0] + s_w[1] + s_w[2] + s_w[3];
    __syncthreads();
  }
}

// The column sums above each band, within its segment of bands, and the sums
// of whole segments: one thread per segment and 4 bin columns, walking the
// segment's rows a band at a time (its kDecTH loads in flight together).
__global__ __launch_bounds__(256) void k_dec_cols(DecBatch db) {
  RSZ_DEC_FRAME(7);
  const uint32_t Wb = dp.Wb, Hb = dp.Hb, nq = (Wb + 3) / 4;
  const uint32_t t = bid * 256 + threadIdx.x;
  if (t >= dp.P * dp.nsegs * nq || !dec_ok(dp.status)) return;
  const uint32_t ps = t / nq, J = (t - ps * nq) * 4;
  const uint32_t p = ps / dp.nsegs, seg = ps - p * dp.nsegs;
  const uint32_t n = min(4u, Wb - J), keep = n == 4 ? ~0u : (1u << (8 * n)) - 1u;
  const uint32_t b0 = seg * dp.seg_bands, b1 = min(b0 + dp.seg_bands, dp.nbands);
  const size_t row0 = (size_t)p * Hb;
  const uint8_t *src = dp.res8 + row0 * Wb + J;
  const int32_t *res = dp.res + row0 * Wb + J;
  uint32_t run[4] = {0u, 0u, 0u, 0u};
  auto put = [&](uint32_t *to) {
    if (n == 4) *(RSZ_G u32x4a *)to = u32x4a{run[0], run[1], run[2], run[3]};
    else
      for (uint32_t k = 0; k < n; ++k) *gm(to + k) = run[k];
  };
  for (uint32_t band = b0; band < b1; ++band) {
    if (band > b0) put(dp.colbase + ((size_t)p * dp.nbands + band) * Wb + J);
    if (band + 1 == dp.nbands) return;   // nothing lies below the last band
    uint32_t w[kDecTH], lo = 0, hi = 0, z = 0;
#pragma unroll
    for (uint32_t i = 0; i < kDecTH; ++i)
      w[i] = ld_any32(src + (size_t)(band * kDecTH + i) * Wb);
#pragma unroll
    for (uint32_t i = 0; i < kDecTH; ++i) {   // bytes 0, 2 and 1, 3 in 16-bit fields
      lo += w[i] & 0x00FF00FFu;
      hi += (w[i] >> 8) & 0x00FF00FFu;
      z |= zero_bytes(w[i]);
    }
    run[0] += (lo & 0xFFFFu) - 128u * kDecTH;
    run[1] += (hi & 0xFFFFu) - 128u * kDecTH;
    run[2] += (lo >> 16) - 128u * kDecTH;
    run[3] += (hi >> 16) - 128u * kDecTH;
    if (z & keep) {   // escapes, counted as -128 above
#pragma unroll
      for (uint32_t i = 0; i < kDecTH; ++i)
        for (uint32_t k = 0; k < n; ++k)
          if (((w[i] >> (8 * k)) & 0xFFu) == 0) {
            const uint32_t x = 128u + (uint32_t)*gm(res + (size_t)(band * kDecTH + i) * Wb + k);
            run[0] += k == 0 ? x : 0u;
            run[1] += k == 1 ? x : 0u;
            run[2] += k == 2 ? x : 0u;
            run[3] += k == 3 ? x : 0u;
          }
    }
  }
  put(dp.segtot + ((size_t)p * dp.nsegs + seg) * Wb + J);
}

// n pixels of value v from a pixel row's address.
__device__ __forceinline__ void fill_px(RSZ_G float *o, uint32_t n, float v) {
  uint32_t k = 0;
  for (; k + 4 <= n; k += 4) *(RSZ_G f32x4a *)(o + k) = f32x4a{v, v, v, v};
  if (n & 2) {
    *(RSZ_G f32x2a *)(o + k) = f32x2a{v, v};
    k += 2;
  }
  if (n & 1) o[k] = v;
}

// A wave's band, in registers: the bytes of kDecTH rows of S strips.  A lane
// takes V consecutive bins of a strip of 64 V, so that its pixels of a row
// are 16 bytes for b = 1, 2 and 4.  B: the bin factor, 0 for any other.
template <int B>
struct Band {
  static constexpr int V = B == 1 ? 4 : (B == 2 ? 2 : 1);
  static constexpr int S = B == 1 ? 2 : 4;
  static constexpr int R = (int)kDecTH;
  static constexpr int C = 4 / V;                 // rows packed in a word
  static constexpr uint32_t kCols = 64 * V * S;   // bin columns of the strips
  // signed bytes: the residuals, kEsc (code byte 0) an escape
  uint32_t w[S][R / C];
  bool esc;   // some byte of the wave is an escape (wave-uniform)
  static constexpr int kEsc = -128;
  // rows [0, nr) of the code bytes from src (row stride Wb), columns from j0,
  // NS strips (0: ns); rows past nr and columns past the row hold residual 0
  template <int NS>
  __device__ __forceinline__ void load(const uint8_t *src, uint32_t Wb, uint32_t j0, int ns,
                                       uint32_t nr, int lane) {
    uint32_t z = 0;
    // a strip's loads, of all the rows, go out together
#pragma unroll
    for (int s = 0; s < (NS ? NS : S); ++s) {
      if (!NS && s >= ns) continue;
      const uint32_t J = j0 + (uint32_t)((64 * s + lane) * V), Jc = min(J, Wb - 1);
      uint32_t keep = 0;   // the lane's bytes inside the row
#pragma unroll
      for (int v = 0; v < V; ++v) keep |= J + v < Wb ? 0xFFu << (8 * v) : 0u;
      if constexpr (V == 1) keep |= keep << 8;
      if constexpr (V <= 2) keep |= keep << 16;
      uint32_t x[R];
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const uint8_t *a = src + min((uint32_t)i, nr - 1) * Wb;
        if constexpr (V == 4) x[i] = ld_any32(a + Jc);
        else if constexpr (V == 2) x[i] = ld_any16(a + Jc);
        else x[i] = *gm(a + Jc);
      }
#pragma unroll
      for (int k = 0; k < R / C; ++k) {
        uint32_t y = 0;
#pragma unroll
        for (int t = 0; t < C; ++t)
          y |= ((uint32_t)(k * C + t) < nr ? x[k * C + t] : 0x80808080u >> (32 - 8 * V)) << (8 * V * t);
        w[s][k] = (y ^ 0x80808080u) & keep;
        z |= zero_bytes(w[s][k] ^ 0x80808080u);
      }
    }
    esc = __ballot(z != 0) != 0;
  }
  // Rows [0, lo) leave and row lo becomes row 0.
  __device__ __forceinline__ void drop(uint32_t lo) {
    auto words = [&](int d) {
#pragma unroll
      for (int s = 0; s < S; ++s)
#pragma unroll
        for (int k = 0; k < R / C; ++k) w[s][k] = k + d < R / C ? w[s][k + d] : 0u;
    };
    auto bits = [&](int d) {
#pragma unroll
      for (int s = 0; s < S; ++s)
#pragma unroll
        for (int k = 0; k < R / C; ++k)
          w[s][k] = __builtin_amdgcn_alignbit(k + 1 < R / C ? w[s][k + 1] : 0u, w[s][k], d);
    };
    if (lo & 8) words(8 / C);
    if (lo & 4) words(4 / C);
    if (lo & 2) {
      if constexpr (C <= 2) words(2 / C);
      else bits(16);
    }
    if (lo & 1) {
      if constexpr (C == 1) words(1);
      else bits(8 * V);
    }
  }
  __device__ __forceinline__ int32_t residual(int s, int i, int v) const {
    return (int8_t)(w[s][i / C] >> (8 * ((i % C) * V + v)));
  }
};

// Column sums of the band's strips into sum.
template <int B, int NS>
__device__ __forceinline__ void band_sums(const Band<B> &bd, const int32_t *res, uint32_t Wb,
                                          int ns, int lane,
                                          uint32_t (&sum)[Band<B>::S][Band<B>::V]) {
  using D = Band<B>;
#pragma unroll
  for (int s = 0; s < (NS ? NS : D::S); ++s) {
#pragma unroll
    for (int v = 0; v < D::V; ++v) sum[s][v] = 0u;
    if (!NS && s >= ns) continue;
#pragma unroll
    for (int i = 0; i < D::R; ++i)
#pragma unroll
      for (int v = 0; v < D::V; ++v) sum[s][v] += (uint32_t)bd.residual(s, i, v);
    if (bd.esc) {   // escapes, counted as -128 above
      const uint32_t J = (uint32_t)((64 * s + lane) * D::V);
#pragma unroll
      for (int i = 0; i < D::R; ++i)
#pragma unroll
        for (int v = 0; v < D::V; ++v)
          if (bd.residual(s, i, v) == D::kEsc)
            sum[s][v] += 128u + (uint32_t)*gm(res + (size_t)i * Wb + J + v);
    }
  }
}

// The column sums of the band's rows [0, lo), added to acc.
template <int B, int NS>
__device__ __forceinline__ void add_rows(const Band<B> &bd, const int32_t *res, uint32_t Wb,
                                         int ns, uint32_t lo, int lane,
                                         uint32_t (&acc)[Band<B>::S][Band<B>::V]) {
  using D = Band<B>;
#pragma unroll
  for (int s = 0; s < (NS ? NS : D::S); ++s) {
    if (!NS && s >= ns) continue;
#pragma unroll
    for (int i = 0; i < D::R; ++i)
#pragma unroll
      for (int v = 0; v < D::V; ++v)
        acc[s][v] += (uint32_t)i < lo ? (uint32_t)bd.residual(s, i, v) : 0u;
    if (bd.esc) {   // escapes, counted as -128 above
      const uint32_t J = (uint32_t)((64 * s + lane) * D::V);
#pragma unroll
      for (int i = 0; i < D::R; ++i)
#pragma unroll
        for (int v = 0; v < D::V; ++v)
          if ((uint32_t)i < lo && bd.residual(s, i, v) == D::kEsc)
            acc[s][v] += 128u + (uint32_t)*gm(res + (size_t)i * Wb + J + v);
    }
  }
}

// What the row loop needs of the plan, in registers before it starts.
struct EmitPlan {
  uint32_t b, Wb, H, W;
  double step;
  const uint8_t *src;   // the band's first bin
  const int32_t *res;
  float *out;           // and its first pixel
  uint32_t I0, nr;
  // rows [lo, lo + n) of the band alone
  __device__ __forceinline__ EmitPlan rows(uint32_t lo, uint32_t n) const {
    EmitPlan e = *this;
    e.src += (size_t)lo * Wb;
    e.res += (size_t)lo * Wb;
    e.out += (size_t)lo * b * W;
    e.I0 += lo;
    e.nr = n;
    return e;
  }
};

// One row's q of the band's strips: r the residuals, acc the column sums
// above (advanced past the row), carry the row's q left of the strips
// (advanced past them).
template <int B, int NS, bool D1>
__device__ __forceinline__ void row_q(double step, int ns,
                                      const int32_t (&r)[NS ? NS : Band<B>::S][Band<B>::V],
                                      uint32_t (&acc)[Band<B>::S][Band<B>::V], uint32_t &carry,
                                      float (&q)[NS ? NS : Band<B>::S][Band<B>::V]) {
  using D = Band<B>;
#pragma unroll
  for (int s = 0; s < (NS ? NS : D::S); ++s) {
    if (!NS && s >= ns) continue;
    uint32_t x[D::V], sum = 0;
#pragma unroll
    for (int v = 0; v < D::V; ++v) {
      acc[s][v] = D1 ? (uint32_t)r[s][v] : acc[s][v] + (uint32_t)r[s][v];
      sum += acc[s][v];
      x[v] = sum;
    }
    const uint32_t incl = wave_inclusive_sum(sum);
    const uint32_t before = incl - sum + carry;
    carry += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
#pragma unroll
    for (int v = 0; v < D::V; ++v) q[s][v] = (float)((double)(int32_t)(before + x[v]) * step);
  }
}

// The pixels of bin row I (the panel's) from prow.  They leave in consecutive
// stores, which complete each other's lines (a panel row is seldom whole
// lines; strip by strip over a band, the pieces of a line left the L2 one by
// one).
template <int B, int NS>
__device__ __forceinline__ void row_pixels(const EmitPlan &ep, uint32_t I, float *prow,
                                           uint32_t j0, int ns, int lane,
                                           const float (&q)[NS ? NS : Band<B>::S][Band<B>::V]) {
  using D = Band<B>;
  const uint32_t b = B ? (uint32_t)B : ep.b;
  const uint32_t Wb = ep.Wb, W = ep.W;
  const bool ragged = Wb % D::V != 0 || W % b != 0;   // some lane's pixels are cut by the edge
  const uint32_t nrow = min(b, ep.H - I * b);
  for (uint32_t d = 0; d < nrow; ++d, prow += W) {
#pragma unroll
    for (int s = 0; s < (NS ? NS : D::S); ++s) {
      if (!NS && s >= ns) continue;
      const uint32_t J = j0 + (uint32_t)((64 * s + lane) * D::V);
      const float *e = q[s];
      RSZ_G float *o = gm(prow) + J * b;
      if ((J + D::V) * b <= W) {   // all of its bins' pixels lie in the panel
        if constexpr (B == 1) *(RSZ_G f32x4a *)o = f32x4a{e[0], e[1], e[2], e[3]};
        else if constexpr (B == 2) *(RSZ_G f32x4a *)o = f32x4a{e[0], e[0], e[1], e[1]};
        else if constexpr (B == 3) *(RSZ_G f32x3a *)o = f32x3a{e[0], e[0], e[0]};
        else if constexpr (B == 4) *(RSZ_G f32x4a *)o = f32x4a{e[0], e[0], e[0], e[0]};
        else fill_px(o, b, e[0]);
      }
      if (ragged && s + 1 == (NS ? NS : ns) && (J + D::V) * b > W) {
#pragma unroll
        for (int v = 0; v < D::V; ++v)
          if (J + v < Wb) fill_px(o + v * b, min(b, W - (J + v) * b), e[v]);
      }
    }
  }
}

// The q and the pixels of a band without escapes.  carry: lane i holds row
// i's.  The loop loads nothing: loads and stores share one wait counter, so
// a load's wait would wait for every store before it too, and the pixels of
// a row would leave only when the row before had reached memory.
template <int B, int NS, bool D1>
__device__ __forceinline__ void band_emit(const EmitPlan &ep, const Band<B> &bd, uint32_t j0,
                                          int ns, int lane,
                                          uint32_t (&acc)[Band<B>::S][Band<B>::V],
                                          uint32_t &carry) {
  using D = Band<B>;
  constexpr int N = NS ? NS : D::S;
  const uint32_t b = B ? (uint32_t)B : ep.b;
#pragma unroll
  for (int i = 0; i < D::R; ++i) {
    if ((uint32_t)i >= ep.nr) continue;
    int32_t r[N][D::V];
    float q[N][D::V];
#pragma unroll
    for (int s = 0; s < N; ++s)
#pragma unroll
      for (int v = 0; v < D::V; ++v) r[s][v] = bd.residual(s, i, v);
    uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)carry, i);
    row_q<B, NS, D1>(ep.step, ns, r, acc, c, q);
    carry = lane == i ? c : carry;
    row_pixels<B, NS>(ep, ep.I0 + i, ep.out + (size_t)i * b * ep.W, j0, ns, lane, q);
  }
}

// The same for a band with escapes (rare): row by row, the bytes read again
// (one row ahead) and the residuals of the bytes 0 from res.  Returns
// whether an outlier's mark is left.
template <int B, bool D1>
__device__ __forceinline__ bool band_emit_esc(const EmitPlan &ep, uint32_t j0, int ns, int lane,
                                              uint32_t (&acc)[Band<B>::S][Band<B>::V],
                                              uint32_t &carry) {
  using D = Band<B>;
  const uint32_t b = B ? (uint32_t)B : ep.b, Wb = ep.Wb;
  uint32_t next[D::S];
  auto load = [&](uint32_t i) {
#pragma unroll
    for (int s = 0; s < D::S; ++s)
      if (s < ns) {
        const uint32_t J = j0 + (uint32_t)((64 * s + lane) * D::V);
        const uint8_t *a = ep.src + (size_t)min(i, ep.nr - 1) * Wb + min(J, Wb - 1);
        if constexpr (D::V == 4) next[s] = ld_any32(a);
        else if constexpr (D::V == 2) next[s] = ld_any16(a);
        else next[s] = *gm(a);
      }
  };
  bool bad = false;
  load(0);
#pragma unroll 1
  for (uint32_t i = 0; i < ep.nr; ++i) {
    int32_t r[D::S][D::V];
    float q[D::S][D::V];
#pragma unroll
    for (int s = 0; s < D::S; ++s)
      if (s < ns)
#pragma unroll
        for (int v = 0; v < D::V; ++v) {
          const uint32_t J = j0 + (uint32_t)((64 * s + lane) * D::V) + v;
          r[s][v] = J < Wb ? (int32_t)((next[s] >> (8 * v)) & 0xFFu) - 128 : 0;
          if (r[s][v] == D::kEsc) r[s][v] = *gm(ep.res + (size_t)i * Wb + J);
        }
    load(i + 1);
#pragma unroll
    for (int s = 0; s < D::S; ++s)
      if (s < ns)
#pragma unroll
        for (int v = 0; v < D::V; ++v) bad |= r[s][v] == kMark;
    uint32_t c = (uint32_t)__builtin_amdgcn_readlane((int)carry, (int)i);
    row_q<B, 0, D1>(ep.step, ns, r, acc, c, q);
    carry = (uint32_t)lane == i ? c : carry;
    row_pixels<B, 0>(ep, ep.I0 + i, ep.out + (size_t)i * b * ep.W, j0, ns, lane, q);
  }
  return bad;
}

__device__ __forceinline__ EmitPlan emit_plan(const DecodePlan &dp, uint32_t p, uint32_t I0,
                                              uint32_t nr) {
  EmitPlan ep;
  ep.b = dp.b;
  ep.Wb = dp.Wb;
  ep.H = dp.H;
  ep.W = dp.W;
  ep.step = dp.step;
  ep.src = dp.res8 + ((size_t)p * dp.Hb + I0) * dp.Wb;
  ep.res = dp.res + ((size_t)p * dp.Hb + I0) * dp.Wb;
  ep.out = dp.frame + ((size_t)p * dp.H + (size_t)I0 * dp.b) * dp.W;
  ep.I0 = I0;
  ep.nr = nr;
  return ep;
}

// The parts of a band's rows, of kDecTH / split rows each.  A panel of one band
// has as many as its rows fill, as evenly as they go: workgroups without a row
// leave CUs idle (66 frames of 6x56x714 at b = 7, half of whose parts were
// empty, 37 us; 24 without them).
__host__ __device__ inline uint32_t band_parts(const DecodePlan &dp, uint32_t split) {
  const uint32_t rows = kDecTH / split;
  return dp.nbands > 1 ? split : (dp.Hb + rows - 1) / rows;
}
__device__ __forceinline__ uint32_t part_rows(const DecodePlan &dp, uint32_t split) {
  const uint32_t parts = band_parts(dp, split);
  return dp.nbands > 1 ? kDecTH / split : (dp.Hb + parts - 1) / parts;
}

// One of the waves that share a row's groups of strips.
struct ColPart {
  uint32_t part, split;
};

// A lane's part of the sum of n rows of residuals over their first cols
// columns (a multiple of 256): 16 columns of 8 rows at a time.
__device__ __forceinline__ uint32_t left_sum(const uint8_t *src, const int32_t *res, uint32_t Wb,
                                             uint32_t n, uint32_t cols, int lane) {
  constexpr uint32_t R = 8;
  uint32_t sum = 0;
  for (uint32_t i0 = 0; i0 < n; i0 += R)
    for (uint32_t j = 16 * (uint32_t)lane; j < cols; j += 1024) {
      u32x4 w[R];
#pragma unroll
      for (uint32_t i = 0; i < R; ++i)
        w[i] = *(const RSZ_G u32x4_any *)(src + (size_t)min(i0 + i, n - 1) * Wb + j);
#pragma unroll
      for (uint32_t i = 0; i < R; ++i) {
        if (i0 + i >= n) continue;
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
          sum = __builtin_amdgcn_sad_u8(w[i][k], 0u, sum) - 128u * 4u;
          for (uint32_t z = zero_bytes(w[i][k]); z; z &= z - 1)   // escapes
            sum += 128u + (uint32_t)*gm(res + (size_t)(i0 + i) * Wb + j + 4 * k +
                                        ((uint32_t)__builtin_ctz(z) >> 3));
        }
      }
    }
  return sum;
}

// One wave's band of a panel of any size: strips group by group from left to
// right, the column sums above from k_dec_cols.  D1: Lorenzo dimension 1
// (each row continues the one before: only row sums, from the row's carry).
template <int B, bool D1, bool SPLIT>
__device__ __forceinline__ void dec_band(const DecodePlan &dp, uint32_t p, uint32_t band,
                                         uint32_t part, uint32_t split, ColPart cols, int lane) {
  using D = Band<B>;
  const uint32_t Hb = dp.Hb, Wb = dp.Wb;
  // the part's rows, from row lo of the band (dimension 1 needs nothing of the
  // rows above: its part is a band of its own)
  const uint32_t rows = SPLIT ? part_rows(dp, split) : kDecTH;
  const uint32_t B0 = band * kDecTH, lo = part * rows;
  if (SPLIT && B0 + lo >= Hb) return;   // (a last band of few rows)
  const uint32_t nr = min(rows, Hb - B0 - lo);
  const EmitPlan ep = emit_plan(dp, p, B0 + lo, nr);
  const uint32_t up = SPLIT && !D1 ? lo : 0u;   // rows of the band above the part's
  const uint32_t seg = band / dp.seg_bands, nsegs = dp.nsegs;
  const uint32_t *cb = D1 || band == seg * dp.seg_bands
                           ? nullptr : dp.colbase + ((size_t)p * dp.nbands + band) * Wb;
  const uint32_t *st = D1 ? nullptr : dp.segtot + (size_t)p * nsegs * Wb;
  const bool marks = dp.dim != 3;   // (dimension 3: k_dec_panels looked)
  int32_t *status = dp.status;
  uint32_t carry = D1 ? *gm(dp.carry + (size_t)p * Hb + ep.I0 + min((uint32_t)lane, nr - 1)) : 0u;
  bool bad = false;
  uint32_t ja = 0, jb = Wb;   // the columns of its group of strips
  if (SPLIT && cols.split > 1) {
    const uint32_t groups = (Wb + D::kCols - 1) / D::kCols;
    ja = D::kCols * (groups * cols.part / cols.split);
    jb = min(Wb, D::kCols * (groups * (cols.part + 1) / cols.split));
    if (ja >= jb) return;
    // and its one row's q left of them
    uint32_t left = left_sum(ep.src - (size_t)up * Wb, ep.res - (size_t)up * Wb, Wb, up + 1, ja,
                             lane);
    auto add = [&](const uint32_t *sums) {
      for (uint32_t j = 4 * (uint32_t)lane; j < ja; j += 256) {
        const u32x4 x = *(const RSZ_G u32x4a *)(sums + j);
        left += x[0] + x[1] + x[2] + x[3];
      }
    };
    if (!D1)
      for (uint32_t g = 0; g < seg; ++g) add(st + (size_t)g * Wb);
    if (!D1 && cb) add(cb);
    carry += (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_sum(left), 63);
  }
  for (uint32_t j0 = ja; j0 < jb; j0 += D::kCols) {
    const int ns = (int)min((uint32_t)D::S, (Wb - j0 + 64 * D::V - 1) / (64 * D::V));
    D bd;
    bd.template load<0>(ep.src - (size_t)up * Wb, Wb, j0, ns, up + nr, lane);
    uint32_t acc[D::S][D::V];
#pragma unroll
    for (int s = 0; s < D::S; ++s) {
#pragma unroll
      for (int v = 0; v < D::V; ++v) acc[s][v] = 0;
      if (D1 || s >= ns) continue;
      const uint32_t J = j0 + (uint32_t)((64 * s + lane) * D::V);
      for (uint32_t g = 0; g < seg; ++g)
#pragma unroll
        for (int v = 0; v < D::V; ++v)
          if (J + v < Wb) acc[s][v] += *gm(st + (size_t)g * Wb + J + v);
      if (cb) {
#pragma unroll
        for (int v = 0; v < D::V; ++v)
          if (J + v < Wb) acc[s][v] += *gm(cb + J + v);
      }
    }
    if (SPLIT && up) {
      add_rows<B, 0>(bd, ep.res - (size_t)up * Wb + j0, Wb, ns, up, lane, acc);
      bd.drop(up);
    }
    if (bd.esc) bad |= band_emit_esc<B, D1>(ep, j0, ns, lane, acc, carry);
    else if (!D1 && ns == D::S) band_emit<B, D::S, D1>(ep, bd, j0, ns, lane, acc, carry);
    else band_emit<B, 0, D1>(ep, bd, j0, ns, lane, acc, carry);
  }
  if (bad && marks) corrupt(status);
}

// SPLIT: db.row_split waves share a band's rows and db.col_split a row's
// columns.  Each reads the bytes of the band's rows up to its own (1 byte a
// bin, from the L2, against the 4 b^2 its pixels take) and those left of its
// columns.  A kernel of its own: the bounds on every row cost the other a
// third of its occupancy.
template <bool SPLIT>
__global__ __launch_bounds__(256) void k_dec_pixels(DecBatch db) {
  RSZ_DEC_FRAME_AT(8, xcd_run());
  const uint32_t it = bid * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t split = SPLIT ? db.row_split : 1u;
  ColPart cols = {0u, SPLIT ? db.col_split : 1u};
  const uint32_t parts = SPLIT ? band_parts(dp, split) : 1u;
  const uint32_t row = it / cols.split, pb = row / parts, part = row - pb * parts;
  cols.part = it - row * cols.split;
  if (pb >= dp.P * dp.nbands || !dec_ok(dp.status)) return;
  const int lane = threadIdx.x & 63;
  const uint32_t p = pb / dp.nbands, band = pb - p * dp.nbands;
  if (dp.dim == 1) {
    switch (dp.b) {
      case 1: dec_band<1, true, SPLIT>(dp, p, band, part, split, cols, lane); break;
      case 2: dec_band<2, true, SPLIT>(dp, p, band, part, split, cols, lane); break;
      case 3: dec_band<3, true, SPLIT>(dp, p, band, part, split, cols, lane); break;
      case 4: dec_band<4, true, SPLIT>(dp, p, band, part, split, cols, lane); break;
      default: dec_band<0, true, SPLIT>(dp, p, band, part, split, cols, lane); break;
    }
  } else {
    switch (dp.b) {
      case 1: dec_band<1, false, SPLIT>(dp, p, band, part, split, cols, lane); break;
      case 2: dec_band<2, false, SPLIT>(dp, p, band, part, split, cols, lane); break;
      case 3: dec_band<3, false, SPLIT>(dp, p, band, part, split, cols, lane); break;
      case 4: dec_band<4, false, SPLIT>(dp, p, band, part, split, cols, lane); break;
      default: dec_band<0, false, SPLIT>(dp, p, band, part, split, cols, lane); break;
    }
  }
}

// Panels whose bands are at most the waves of a workgroup and whose rows one
// group of strips holds (panel_fits): one workgroup per panel and a wave per
// band, so the column sums above a band come through LDS and the bytes are
// read once.
__host__ __device__ inline bool panel_fits(const DecodePlan &dp) {
  const uint32_t cols = dp.b == 1 ? Band<1>::kCols : (dp.b == 2 ? Band<2>::kCols : Band<0>::kCols);
  return dp.dim != 1 && dp.nbands <= kDecPanelWaves && dp.Wb <= cols;
}

// Wave wv's band of panel p; every wave of the workgroup calls it (mine: the
// panel has the band).  own: its rows to emit, from row lo of the band.
// Returns whether the band holds escapes, its pixels then left to the caller
// (acc: the column sums above).
template <int B, int NS, bool SPLIT>
__device__ __forceinline__ bool dec_panel_ns(const EmitPlan &ep, const EmitPlan &own, uint32_t lo,
                                             bool mine, uint32_t wv, uint32_t *s_col, int lane,
                                             uint32_t (&acc)[Band<B>::S][Band<B>::V]) {
  using D = Band<B>;
  const uint32_t Wb = ep.Wb;
  D bd;
  if (mine) {
    bd.template load<NS>(ep.src, Wb, 0, NS, ep.nr, lane);
    band_sums<B, NS>(bd, ep.res, Wb, NS, lane, acc);
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int v = 0; v < D::V; ++v) {
        const uint32_t J = (uint32_t)((64 * s + lane) * D::V + v);
        if (J < Wb) s_col[wv * Wb + J] = acc[s][v];
      }
  }
  __syncthreads();
  if (!mine || (SPLIT && own.nr == 0)) return false;
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int v = 0; v < D::V; ++v) acc[s][v] = 0;
  for (uint32_t k = 0; k < wv; ++k)
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int v = 0; v < D::V; ++v)
        acc[s][v] += s_col[k * Wb + min((uint32_t)((64 * s + lane) * D::V + v), Wb - 1)];
  if (SPLIT && lo) {
    add_rows<B, NS>(bd, ep.res, Wb, NS, lo, lane, acc);
    bd.drop(lo);
  }
  // lanes past the row add nothing to its sums
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int v = 0; v < D::V; ++v)
      if ((uint32_t)((64 * s + lane) * D::V + v) >= Wb) acc[s][v] = 0;
  if (bd.esc) return true;
  uint32_t carry = 0;
  band_emit<B, NS, false>(own, bd, 0, NS, lane, acc, carry);
  return false;
}

template <int B, bool SPLIT>
__device__ __forceinline__ void dec_panel(const DecodePlan &dp, uint32_t p, uint32_t part,
                                          uint32_t split, uint32_t wv, uint32_t *s_col,
                                          int lane) {
  using D = Band<B>;
  const bool mine = wv < dp.nbands;
  const uint32_t I0 = mine ? wv * kDecTH : 0u;
  const EmitPlan ep = emit_plan(dp, p, I0, min(kDecTH, dp.Hb - I0));
  const uint32_t rows = SPLIT ? part_rows(dp, split) : kDecTH, lo = min(part * rows, ep.nr);
  const EmitPlan own = ep.rows(lo, min(rows, ep.nr - lo));
  const bool marks = dp.dim != 3;   // (dimension 3: k_dec_panels looked)
  int32_t *status = dp.status;
  const int ns = (int)((ep.Wb + 64 * D::V - 1) / (64 * D::V));
  uint32_t acc[D::S][D::V];
  bool esc = false;
  switch (ns) {
    case 1: esc = dec_panel_ns<B, 1, SPLIT>(ep, own, lo, mine, wv, s_col, lane, acc); break;
    case 2: esc = dec_panel_ns<B, 2, SPLIT>(ep, own, lo, mine, wv, s_col, lane, acc); break;
    case 3: if constexpr (D::S >= 3) esc = dec_panel_ns<B, 3, SPLIT>(ep, own, lo, mine, wv, s_col, lane, acc); break;
    default: if constexpr (D::S >= 4) esc = dec_panel_ns<B, 4, SPLIT>(ep, own, lo, mine, wv, s_col, lane, acc); break;
  }
  if (esc) {
    uint32_t carry = 0;
    if (band_emit_esc<B, false>(own, 0, ns, lane, acc, carry) && marks) corrupt(status);
  }
}

// LDS: the bands' column sums.  SPLIT: as many workgroups a panel, each with
// all the column sums and a part of every band's rows.
template <bool SPLIT>
__global__ __launch_bounds__(1024) void k_dec_panel(DecBatch db) {
  RSZ_DEC_FRAME_AT(9, xcd_run());
  extern __shared__ __align__(16) uint32_t s_col[];
  __shared__ int s_ok;
  // one read of the status for the whole workgroup (another panel may
  // change it meanwhile), so every thread takes the same branch
  if (threadIdx.x == 0) s_ok = dec_ok(dp.status);
  __syncthreads();
  if (!s_ok) return;
  const int lane = threadIdx.x & 63;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t split = SPLIT ? db.row_split : 1u;
  const uint32_t parts = SPLIT ? band_parts(dp, split) : 1u, p = bid / parts, part = bid - p * parts;
  switch (dp.b) {
    case 1: dec_panel<1, SPLIT>(dp, p, part, split, wv, s_col, lane); break;
    case 2: dec_panel<2, SPLIT>(dp, p, part, split, wv, s_col, lane); break;
    case 3: dec_panel<3, SPLIT>(dp, p, part, split, wv, s_col, lane); break;
    case 4: dec_panel<4, SPLIT>(dp, p, part, split, wv, s_col, lane); break;
    default: dec_panel<0, SPLIT>(dp, p, part, split, wv, s_col, lane); break;
  }
}

// ------------------------------------------------------- coded ROI windows

// Tables of the ROI class code: per length L the first canonical code, the
// number of classes and where they start in the (length, class) order, then
// that order.
constexpr int kRoiTabFirst = 0, kRoiTabCount = 33, kRoiTabBase = 66, kRoiTabSym = 99;
constexpr int kRoiTabWords = 132;
constexpr int kRoiLutBits = 10;   // k_dec_roi_decode: codes this short by one lookup

// Builds the tables in LDS by one wave (lane c holds class c's length).  The
// lengths must be a complete prefix code (or one class of length 1), padding
// zero; no class at all when there is no window.  Returns whether they are.
__device__ __forceinline__ bool roi_tables(const DecodePlan &dp, uint32_t *t, int lane) {
  const uint32_t L = lane < (int)kRoiLens ? *gm(dp.in + dp.off_rsec + lane) : 0u;
  const bool cls = lane < kRoiClasses;
  const bool wrong = cls ? L > (uint32_t)kMaxLen : L != 0;
  if (__ballot(wrong)) return false;
  uint32_t code = 0, n = 0, prev = 0;
  uint64_t kraft = 0;
#pragma unroll 1
  for (uint32_t l = 1; l <= (uint32_t)kMaxLen; ++l) {
    const uint64_t m = __ballot(cls && L == l);
    const uint32_t cnt = (uint32_t)__builtin_popcountll(m);
    code = (code + prev) << 1;
    if (lane == 0) {
      t[kRoiTabFirst + l - 1] = code;
      t[kRoiTabCount + l - 1] = cnt;
      t[kRoiTabBase + l - 1] = n;
    }
    if ((m >> lane) & 1u)
      t[kRoiTabSym + n + (uint32_t)__builtin_popcountll(m & ((1ull << lane) - 1))] = (uint32_t)lane;
    kraft += (uint64_t)cnt << (kMaxLen - l);
    n += cnt;
    prev = cnt;
  }
  if (dp.npeaks == 0) return n == 0;
  return kraft == (1ull << kMaxLen) || (n == 1 && kraft == (1ull << (kMaxLen - 1)));
}

// Windows decoded by one wave, a lane each, into its LDS slice (w <= 48), or
// into roi_payload, its prediction left to k_dec_roi_unpred.  Few lanes a
// wave on purpose: a lane's values follow one another, so the windows want
// waves of their own, and the more lanes share one the more often all wait
// for one lane's next words.
constexpr uint32_t kRoiWins = 8, kRoiSlice = 2368;
constexpr uint32_t kRoiIn = 2368;   // words of a wave's windows' bits in LDS
__host__ __device__ inline uint32_t roi_wins(uint32_t w) {
  const uint32_t ww = w * w;
  return ww <= kRoiSlice ? (kRoiSlice / ww < kRoiWins ? kRoiSlice / ww : kRoiWins) : kRoiWins;
}
__host__ __device__ inline bool roi_in_lds(uint32_t w) { return w * w <= kRoiSlice; }

// The windows of a frame: classes and raw bits into the zigzag residuals r
// (mod 2^32), then the prediction undone.  A window must start at its offset
// (the first at 0) and end exactly at the next offset, the last at Troi.
// With D = M - 2^31 (zero outside the window), D(u, v) = r + D(u-1, v) +
// D(u, v-1) - D(u-1, v-1), so D is the 2D prefix sum of r: a wave scan along
// each row plus the column sums kept per lane; M = D + 2^31 maps back to the
// float bits.  The residuals stay in LDS on the way: stored to HBM value by
// value, the loop's loads waited for its stores (0.32 ms + 0.03 for the
// prediction + 0.09 for tables by one thread on 250 CSPAD frames, against
// 0.12 together here).
__global__ __launch_bounds__(256) void k_dec_roi_decode(DecBatch db) {
  RSZ_DEC_FRAME(10);
  // the frame's class tables, and a lookup of every code of at most
  // kRoiLutBits bits by the stream's next kRoiLutBits bits: class | L << 8
  // (0: a longer code, or none)
  __shared__ uint32_t s_t[kRoiTabWords];
  __shared__ uint16_t s_lut[1 << kRoiLutBits];
  __shared__ uint32_t s_r[4][kRoiSlice], s_in[4][kRoiIn + 2];
  __shared__ int s_ok;
  const int lane = threadIdx.x & 63;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // one read of the status for the workgroup (a window may set it
  // meanwhile), so that every thread takes the same branch
  if (wv == 0) {
    bool ok = dec_ok(dp.status);
    if (ok && !roi_tables(dp, s_t, lane)) {
      if (lane == 0) corrupt(dp.status);
      ok = false;
    }
    if (lane == 0) s_ok = ok;
  }
  __syncthreads();
  if (!s_ok) return;
  for (uint32_t x = threadIdx.x; x < (1u << kRoiLutBits); x += 256) {
    uint16_t e = 0;
    for (int L = 1; L <= kRoiLutBits; ++L) {
      const uint32_t code = x >> (kRoiLutBits - L);
      const uint32_t cnt = s_t[kRoiTabCount + L - 1], first = s_t[kRoiTabFirst + L - 1];
      if (cnt && code - first < cnt) {
        e = (uint16_t)(s_t[kRoiTabSym + s_t[kRoiTabBase + L - 1] + (code - first)] | (L << 8));
        break;
      }
    }
    s_lut[x] = e;
  }
  __syncthreads();
  const uint32_t w = dp.w, ww = w * w, wins = roi_wins(w);
  const bool lds = roi_in_lds(w);
  const uint32_t k0 = (bid * 4 + wv) * wins;
  const uint32_t k = k0 + (uint32_t)lane, kn = min(k0 + wins, dp.npeaks);
  if (k0 >= kn) return;
  // the wave's windows' bits lie one after the other: [first, last)
  const RSZ_G uint32_t *offs = gm((const uint32_t *)(dp.in + dp.off_roffs));
  const uint32_t Troi = (uint32_t)dp.Troi;   // <= 63 * 2^26
  const uint32_t first = offs[k0], last = kn < dp.npeaks ? offs[kn] : Troi;
  const bool sane = first <= last && last <= Troi;
  BitSrc src;
  src.words = (const uint32_t *)(dp.in + dp.off_rbits);
  src.n = (uint32_t)(((uint64_t)Troi + 31) / 32);
  src.lds = s_in[wv];
  src.w0 = first >> 5;
  const uint32_t nin = sane ? (uint32_t)(((uint64_t)last + 31) / 32) - src.w0 : 0u;
  src.staged = nin <= kRoiIn;
  if (src.staged)
    for (uint32_t i = lane; i < nin + 2; i += 64)
      s_in[wv][i] = i < nin ? *gm(src.words + src.w0 + i) : 0u;
  wave_sync();
  if (k < kn) {
    const uint32_t start = offs[k], end = k + 1 < dp.npeaks ? offs[k + 1] : Troi;
    bool bad = !sane || (k == 0 && start != 0) || start < first || end < start || end > last;
    uint32_t *out = dp.roi_payload + (uint64_t)k * ww;
    uint32_t *sl = s_r[wv] + (uint32_t)lane * ww;
    // the class code at the top of the bits: class | length << 8, 0 for none
    auto long_code = [&](uint32_t peek) {
      for (uint32_t L = kRoiLutBits + 1; L <= (uint32_t)kMaxLen; ++L) {
        const uint32_t code = peek >> (32 - L);
        const uint32_t cnt = s_t[kRoiTabCount + L - 1], first_code = s_t[kRoiTabFirst + L - 1];
        if (cnt && code - first_code < cnt)
          return s_t[kRoiTabSym + s_t[kRoiTabBase + L - 1] + (code - first_code)] | L << 8;
      }
      return 0u;
    };
    if (!bad && src.staged && lds) {
      // every value's step is straight code: the word index is clamped to the
      // staged words, and a window whose values overrun its end ends past it
      // (no value takes 0 bits), so one comparison after the loop finds it
      uint32_t pos = start;
      const uint32_t *in = s_in[wv];
      for (uint32_t e = 0; e < ww; ++e) {
        const uint32_t i = min((pos >> 5) - src.w0, nin);
        const uint64_t x = ((uint64_t)in[i] << 32 | in[i + 1]) << (pos & 31);
        uint32_t hit = s_lut[(uint32_t)(x >> (64 - kRoiLutBits))];
        if (!hit) {
          hit = long_code((uint32_t)(x >> 32));
          bad |= !hit;
          hit = max(hit, 1u << 8);
        }
        const uint32_t cls = hit & 0xFFu, L = hit >> 8, extra = max(cls, 1u) - 1u;
        uint32_t raw = (uint32_t)((x << L) >> 32);   // the 32 bits after the code,
        if (L + extra > 33) {                        // some past the two words (at least 33 hold)
          const uint32_t q = pos + L, j = min((q >> 5) - src.w0, nin);
          raw = (uint32_t)((((uint64_t)in[j] << 32 | in[j + 1]) << (q & 31)) >> 32);
        }
        const uint32_t z = cls ? (uint32_t)(((1ull << 32) | raw) >> (32 - extra)) : 0u;
        sl[e] = (z >> 1) ^ (0u - (z & 1u));
        pos += L + extra;
      }
      bad |= pos != end;
    } else if (!bad) {
      uint32_t pos = start;
      for (uint32_t e = 0; e < ww; ++e) {
        if (pos >= end) {   // every value takes a bit at least
          bad = true;
          break;
        }
        const uint32_t peek = src.peek(pos);
        uint32_t hit = s_lut[peek >> (32 - kRoiLutBits)];
        if (!hit) hit = long_code(peek);
        const uint32_t cls = hit & 0xFFu, L = hit >> 8, extra = max(cls, 1u) - 1u;
        if (!hit || L + extra > end - pos) {
          bad = true;
          break;
        }
        uint32_t z = cls ? 1u : 0u;
        if (extra) z = (1u << extra) | (src.peek(pos + L) >> (32 - extra));
        pos += L + extra;
        const uint32_t r = (z >> 1) ^ (0u - (z & 1u));
        if (lds) sl[e] = r;
        else *gm(out + e) = r;
      }
      bad |= pos != end;
    }
    if (bad) corrupt(dp.status);
  }
  if (!lds) return;
  wave_sync();
  for (uint32_t i = 0; k0 + i < kn; ++i) {
    uint32_t *out = dp.roi_payload + (uint64_t)(k0 + i) * ww;
    const uint32_t *sl = s_r[wv] + i * ww;
    uint32_t col = 0;
    for (uint32_t u = 0; u < w; ++u) {
      const uint32_t x = (uint32_t)lane < w ? sl[u * w + lane] : 0u;
      col += wave_inclusive_sum(x);   // D(u, v) = row prefix of row u + D(u - 1, v)
      const uint32_t m = col + 0x80000000u;
      if ((uint32_t)lane < w)
        *gm(out + u * w + lane) = (m & 0x80000000u) ? (m & 0x7FFFFFFFu) : ~m;
    }
  }
}

// The same for windows too large for LDS, whose residuals k_dec_roi_decode
// left in roi_payload: one wave per window.
constexpr int kRoiMaxChunks = 16;   // w <= 1023: 16 chunks of 64 columns
__global__ __launch_bounds__(256) void k_dec_roi_unpred(DecBatch db) {
  RSZ_DEC_FRAME(11);
  const uint32_t k = bid * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (k >= dp.npeaks || !dec_ok(dp.status)) return;
  const uint32_t w = dp.w;
  uint32_t *win = dp.roi_payload + (uint64_t)k * w * w;
  uint32_t col[kRoiMaxChunks];
#pragma unroll
  for (int c = 0; c < kRoiMaxChunks; ++c) col[c] = 0u;
  for (uint32_t u = 0; u < w; ++u) {
    uint32_t carry = 0;
#pragma unroll
    for (int c = 0; c < kRoiMaxChunks; ++c) {
      if (c * 64 < (int)w) {   // uniform
        const uint32_t v = c * 64 + lane;
        uint32_t x = v < w ? win[u * w + v] : 0u;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
          const uint32_t y = __shfl_up(x, d);
          if (lane >= d) x += y;
        }
        x += carry;
        carry = __shfl(x, 63);
        col[c] += x;   // D(u, v) = row prefix of row u + D(u - 1, v)
        if (v < w) {
          const uint32_t m = col[c] + 0x80000000u;
          win[u * w + v] = (m & 0x80000000u) ? (m & 0x7FFFFFFFu) : ~m;
        }
      }
    }
  }
}

// Window k of a frame, one wave: lane l starts at window element l and steps
// 64 elements at a time, its (row, column) in the window advanced without a
// division.  Pixels outside the frame are not part of the window.  CHECK
// compares the frame with the payload instead of writing it.
template <bool CHECK>
__device__ __forceinline__ bool roi_window(const DecodePlan &dp, uint32_t k, uint32_t lane) {
  const uint32_t w = dp.w, ww = w * w;
  const uint16_t *pk = (const uint16_t *)(dp.in + dp.off_peaks);
  const RSZ_G uint32_t *pay = gm(
      (dp.roi_coding ? dp.roi_payload : (const uint32_t *)(dp.in + dp.off_roi)) + (size_t)k * ww);
  const uint32_t pa = pk[3 * k];
  if (pa >= dp.P) return false;
  const int32_t h = (int32_t)(w / 2), H = (int32_t)dp.H, W = (int32_t)dp.W;
  const int32_t i0 = (int32_t)pk[3 * k + 1] - h, j0 = (int32_t)pk[3 * k + 2] - h;
  RSZ_G uint32_t *fr = gm((uint32_t *)dp.frame + (size_t)pa * dp.H * dp.W);
  const uint32_t du = 64 / w, dv = 64 % w;
  uint32_t u = lane / w, v = lane - u * w;
  bool bad = false;
  constexpr uint32_t kSlots = 8;   // elements a lane loads before it stores any
  for (uint32_t e0 = lane; e0 < ww; e0 += 64 * kSlots) {
    uint32_t x[kSlots];
#pragma unroll
    for (uint32_t t = 0; t < kSlots; ++t)
      x[t] = e0 + 64 * t < ww ? pay[e0 + 64 * t] : 0u;
#pragma unroll
    for (uint32_t t = 0; t < kSlots; ++t) {
      const int32_t i = i0 + (int32_t)u, j = j0 + (int32_t)v;
      if (e0 + 64 * t < ww && i >= 0 && i < H && j >= 0 && j < W) {
        RSZ_G uint32_t *px = fr + (size_t)i * dp.W + j;
        if (CHECK) bad |= *px != x[t];
        else *px = x[t];
      }
      u += du;
      v += dv;
      if (v >= w) {
        v -= w;
        ++u;
      }
    }
  }
  return bad;
}

// Windows that overlap must carry the same bits for the pixels they share.
// With few windows (roi_pairs) the wave of window k lists the earlier windows
// that meet it, 64 a step.  Where these cover little of it, it compares the
// rectangle shared with each.  Where they crowd, it compares each of its
// pixels with one of them that covers it, the nearest in the list: by
// induction along the windows over a pixel all of them then agree, so a pixel
// is compared once however many windows lie over it.  More windows are
// compared with the frame that all of them were written to, by
// k_dec_roi_check: the listing grows with the square of their number, and
// where they crowd a wave steps through its list for every 64 pixels.  So the
// line lies at kRoiListed windows and kRoiSteps such steps of the last wave
// (256 windows of 17, 128 of 25, 60 of 36), both known from the header.
// k_dec_roi (and k_dec_roi_check) in us on 1 and on 50 frames with 60 windows
// of 17: spread out 7 and 10 (the pass: 13 and 18), on one spot 10 and 13,
// crowded in 51 x 51 pixels 18 and 24; 256 on one spot 11 and 30 (12 and 24);
// 8 of 60 on 7 frames, in pairs, 18 (pixel by pixel 44).  Every element
// against every window met, with the line at 512 windows of any size: 60 on
// one spot 103 and 116, 256 427 and 1311, 512 windows of 101 there 35 and 112
// ms against 0.10 and 0.45 of the pass.
constexpr uint32_t kRoiListed = 512, kRoiSteps = 1280;
__host__ __device__ inline bool roi_pairs(const DecodePlan &dp) {
  return dp.npeaks <= kRoiListed && dp.npeaks * ((dp.w * dp.w + 63) / 64) <= kRoiSteps;
}

// An earlier window in a wave's list: its number (9 bits), and where its
// corner lies from this one's, row and column + 1023 (11 bits each).
__device__ __forceinline__ uint32_t roi_entry(uint32_t o, int32_t dr, int32_t dc) {
  return o << 22 | (uint32_t)(dr + 1023) << 11 | (uint32_t)(dc + 1023);
}

// Whether the rectangle that window k (its corner at row r, column c of the
// panel) shares with the listed window x differs inside the panel.
__device__ __forceinline__ bool roi_rect_differs(const RSZ_G uint32_t *pay, uint32_t k, uint32_t x,
                                                 int32_t w, int32_t r, int32_t c, int32_t H,
                                                 int32_t W, uint32_t lane) {
  const int32_t dr = (int32_t)((x >> 11) & 2047u) - 1023, dc = (int32_t)(x & 2047u) - 1023;
  const int32_t u0 = max(max(0, dr), -r), u1 = min(min(w, w + dr), H - r);
  const int32_t v0 = max(max(0, dc), -c), v1 = min(min(w, w + dc), W - c);
  if (u0 >= u1 || v0 >= v1) return false;
  const uint32_t rw = (uint32_t)(v1 - v0), rh = (uint32_t)(u1 - u0);
  const uint32_t ww = (uint32_t)(w * w);
  const RSZ_G uint32_t *mine = pay + (size_t)k * ww + u0 * w + v0;
  const RSZ_G uint32_t *other = pay + (size_t)(x >> 22) * ww + (u0 - dr) * w + (v0 - dc);
  const uint32_t da = 64 / rw, db = 64 - da * rw;
  uint32_t a = lane / rw, b = lane - a * rw;   // row and column of the rectangle
  constexpr int kAhead = 4;   // elements a lane loads before it compares any
  bool bad = false;
  for (uint32_t e0 = lane; e0 < rw * rh; e0 += 64 * kAhead) {
    uint32_t m[kAhead], o[kAhead];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) {
      const bool in = e0 + 64 * q < rw * rh;
      const uint32_t at = a * (uint32_t)w + b;
      m[q] = in ? mine[at] : 0u;
      o[q] = in ? other[at] : 0u;
      a += da;
      b += db;
      if (b >= rw) {
        b -= rw;
        ++a;
      }
    }
#pragma unroll
    for (int q = 0; q < kAhead; ++q) bad |= m[q] != o[q];
  }
  return bad;
}

// list: this wave's kRoiListed words.
__device__ __forceinline__ bool roi_overlaps(const DecodePlan &dp, uint32_t k, uint32_t *list,
                                             uint32_t lane) {
  const uint32_t w = dp.w, ww = w * w;
  const RSZ_G uint16_t *pk = gm((const uint16_t *)(dp.in + dp.off_peaks));
  const int32_t h = (int32_t)(w / 2), H = (int32_t)dp.H, W = (int32_t)dp.W, iw = (int32_t)w;
  const int32_t pa = pk[3 * k], r = (int32_t)pk[3 * k + 1] - h, c = (int32_t)pk[3 * k + 2] - h;
  uint32_t n = 0, area = 0;   // the earlier windows that meet this one; of the shared rectangles
  for (uint32_t b = 0; b < k; b += 64) {
    const uint32_t o = min(b + lane, k - 1);
    const int32_t opa = pk[3 * o];
    const int32_t dr = (int32_t)pk[3 * o + 1] - h - r, dc = (int32_t)pk[3 * o + 2] - h - c;
    const bool meet = b + lane < k && opa == pa && dr > -iw && dr < iw && dc > -iw && dc < iw;
    const uint64_t m = __ballot(meet);
    if (meet) {
      list[n + (uint32_t)__builtin_popcountll(m & ((1ull << lane) - 1ull))] = roi_entry(o, dr, dc);
      area += (uint32_t)((iw - abs(dr)) * (iw - abs(dc)));
    }
    n += (uint32_t)__builtin_popcountll(m);
  }
  if (n == 0) return false;
  wave_sync();
  const RSZ_G uint32_t *pay =
      gm(dp.roi_coding ? dp.roi_payload : (const uint32_t *)(dp.in + dp.off_roi));
  area = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_sum(area), 63);
  bool bad = false;
  uint32_t t0 = (n - 1) & ~63u, x64 = list[min(t0 + lane, n - 1)];   // the list's last 64
  if (area <= 2 * ww && t0 == 0) {
    for (uint32_t t = 0; t < n; ++t)
      bad |= roi_rect_differs(pay, k, (uint32_t)__builtin_amdgcn_readlane((int)x64, (int)t), iw, r,
                              c, H, W, lane);
    return bad;
  }
  const RSZ_G uint32_t *mine = pay + (size_t)k * ww;
  const int32_t du = (int32_t)(64 / w), dv = (int32_t)(64 % w);
  int32_t u = (int32_t)(lane / w), v = (int32_t)lane - u * iw;   // element e of window k
  for (uint32_t e0 = 0; e0 < ww; e0 += 64) {
    const int32_t i = r + u, j = c + v;
    bool open = u < iw && i >= 0 && i < H && j >= 0 && j < W;   // in the panel, not yet compared
    uint32_t at = 0;
    bool found = false;
    for (uint32_t t = n; t > 0 && __ballot(open) != 0;) {
      if (((t - 1) & ~63u) != t0) {
        t0 = (t - 1) & ~63u;
        x64 = list[min(t0 + lane, n - 1)];
      }
      for (; t > t0 && __ballot(open) != 0; --t) {
        const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)x64, (int)((t - 1) & 63));
        const int32_t ou = u - ((int32_t)((x >> 11) & 2047u) - 1023);
        const int32_t ov = v - ((int32_t)(x & 2047u) - 1023);
        if (open && (uint32_t)ou < w && (uint32_t)ov < w) {
          at = (x >> 22) * ww + (uint32_t)ou * w + (uint32_t)ov;
          found = true;
          open = false;
        }
      }
    }
    if (found) bad |= mine[e0 + lane] != pay[at];
    u += du;
    v += dv;
    if (v >= iw) {
      v -= iw;
      ++u;
    }
  }
  return bad;
}

__global__ __launch_bounds__(256) void k_dec_roi(DecBatch db) {
  RSZ_DEC_FRAME(12);
  __shared__ uint32_t s_list[4][kRoiListed];
  const uint32_t wv = threadIdx.x >> 6, k = bid * 4 + wv;
  if (k >= dp.npeaks || !dec_ok(dp.status)) return;
  roi_window<false>(dp, k, threadIdx.x & 63);
  if (roi_pairs(dp) && roi_overlaps(dp, k, s_list[wv], threadIdx.x & 63)) corrupt(dp.status);
}
__global__ __launch_bounds__(256) void k_dec_roi_check(DecBatch db) {
  RSZ_DEC_FRAME(13);
  const uint32_t k = bid * 4 + (threadIdx.x >> 6);
  if (k >= dp.npeaks || !dec_ok(dp.status)) return;
  if (roi_window<true>(dp, k, threadIdx.x & 63)) corrupt(dp.status);
}

void decode_blocks(const DecodePlan &dp, uint32_t reps, BandSplit split, uint32_t *nb) {
  for (int k = 0; k < kDecKernels; ++k) nb[k] = 0;
  nb[0] = 1;   // k_dec_tables writes every frame's status
  if (dp.init_status != RSZ_OK) return;
  if (dp.run_coding) nb[1] = (dp.nchunks + 3) / 4;
  nb[2] = (dp.nchunks + kChunkWaves * reps - 1) / (kChunkWaves * reps);
  nb[kDecOutliers] = (dp.n_out + 255) / 256;
  // inverse Lorenzo: prefix sums along each axis the predictor spans
  if (dp.dim == 3) {
    const uint32_t cols = 4 * (256 / dp.panel_segs);
    nb[4] = (dp.Hb * dp.Wb + cols - 1) / cols;
  }
  if (panel_fits(dp)) {
    nb[9] = dp.P * band_parts(dp, split.rows);
  } else {
    if (dp.dim == 1) {
      nb[5] = (dp.P * dp.Hb + 4 * kDecRowsPerWave - 1) / (4 * kDecRowsPerWave);
      nb[6] = 1;
    } else if (dp.nbands > 1) {
      nb[7] = (uint32_t)(((uint64_t)dp.P * dp.nsegs * ((dp.Wb + 3) / 4) + 255) / 256);
    }
    nb[8] = (uint32_t)(
        ((uint64_t)dp.P * dp.nbands * band_parts(dp, split.rows) * split.cols + 3) / 4);
  }
  if (dp.roi_coding) {
    const uint32_t wins = 4 * roi_wins(dp.w);
    nb[10] = std::max(1u, (dp.npeaks + wins - 1) / wins);   // (no window: the lengths' check)
    if (!roi_in_lds(dp.w)) nb[11] = (dp.npeaks + 3) / 4;
  }
  nb[12] = (dp.npeaks + 3) / 4;   // a wave per window
  if (!roi_pairs(dp)) nb[13] = nb[12];
}

#define RSZ_DLAUNCH_S(k, name, kern, block, lds)                       \
  do {                                                                 \
    if (total[k]) {                                                    \
      prof_begin(name, s);                                             \
      hipLaunchKernelGGL(kern, dim3(total[k]), dim3(block), lds, s, db); \
      prof_end(s);                                                     \
      hipError_t e_ = hipGetLastError();                               \
      if (e_ != hipSuccess) return e_;                                 \
    }                                                                  \
  } while (0)
#define RSZ_DLAUNCH(k, name, kern, block) RSZ_DLAUNCH_S(k, name, kern, block, 0)

hipError_t launch_decompress(const DecBatch &db, const uint32_t *total, hipStream_t s) {
  RSZ_DLAUNCH(0, "k_dec_tables", k_dec_tables, 256);
  RSZ_DLAUNCH(1, "k_dec_runs", k_dec_runs, 256);
  RSZ_DLAUNCH(2, "k_dec_chunks", k_dec_chunks, 64 * kChunkWaves);
  RSZ_DLAUNCH(kDecOutliers, "k_dec_outliers", k_dec_outliers, 256);
  RSZ_DLAUNCH(4, "k_dec_panels", k_dec_panels, 256);
  RSZ_DLAUNCH(5, "k_dec_rowsum", k_dec_rowsum, 256);
  RSZ_DLAUNCH(6, "k_dec_carry", k_dec_carry, 256);
  RSZ_DLAUNCH(7, "k_dec_cols", k_dec_cols, 256);
  if (db.row_split > 1) {
    RSZ_DLAUNCH(8, "k_dec_pixels", k_dec_pixels<true>, 256);
    RSZ_DLAUNCH_S(9, "k_dec_panel", k_dec_panel<true>, 64 * db.panel_waves, 4 * db.panel_lds);
  } else {
    RSZ_DLAUNCH(8, "k_dec_pixels", k_dec_pixels<false>, 256);
    RSZ_DLAUNCH_S(9, "k_dec_panel", k_dec_panel<false>, 64 * db.panel_waves, 4 * db.panel_lds);
  }
  RSZ_DLAUNCH(10, "k_dec_roi_decode", k_dec_roi_decode, 256);
  RSZ_DLAUNCH(11, "k_dec_roi_unpred", k_dec_roi_unpred, 256);
  RSZ_DLAUNCH(12, "k_dec_roi", k_dec_roi, 256);
  RSZ_DLAUNCH(13, "k_dec_roi_check", k_dec_roi_check, 256);
  return hipSuccess;
}

// The bands of kDecTH bin rows and the segments of bands that k_dec_cols
// walks.  Every segment of a panel is summed by threads of its own and a band
// adds the segments above it, so a tall panel is split (8 bands, 128 rows, a
// segment) but into at most 16, which bounds what a band adds.
//
// And the segments of panels of k_dec_panels: a thread's panels follow one
// another, 0.33 us each, so a frame with few bins a panel leaves the GPU to a
// few long chains.  Up to 64 segments of 16 panels or more, while the threads
// are few (a segment's panels are read twice).  k_dec_panels on one frame of
// 300x48x60 at b = 1 105 -> 47 us, of 4000x48x8 1290 -> 72, of 60000x3x5 23.6
// -> 0.64 ms.
void decode_geometry(DecodePlan &dp) {
  dp.nbands = (dp.Hb + kDecTH - 1) / kDecTH;
  dp.seg_bands = std::max(8u, (dp.nbands + 15) / 16);
  dp.nsegs = (dp.nbands + dp.seg_bands - 1) / dp.seg_bands;
  const uint32_t cols = (dp.Hb * dp.Wb + 3) / 4;
  dp.panel_segs = 1;
  while (dp.panel_segs < 64 && cols * dp.panel_segs < 2048 && dp.P >= 32 * dp.panel_segs)
    dp.panel_segs *= 2;
}

// A workgroup of k_dec_chunks copies its stream's tables (18 KB) to LDS first,
// so in a large batch its waves take several chunks each; a small one wants
// every chunk on a wave of its own.
uint32_t decode_chunk_reps(uint64_t all_chunks) {
  return (uint32_t)std::min<uint64_t>(4, std::max<uint64_t>(1, all_chunks / (kChunkWaves * 1024)));
}

// How many waves share a band: with one wave each, a batch of few bands leaves
// the GPU idle while its waves walk their rows, so the bands are split, by
// rows down to one and then by columns, until there are kDecWaves (with two
// and four times as many, waves read the bytes above them too often: 8 frames
// of 32x185x388 at b = 2 take 18 us, 27 and 38).  The pixel kernel on one
// frame of 1x2048x2048 at b = 5 79 -> 18 us, at b = 2 49 -> 34, of 32x185x388
// 15 -> 10, of 1x40x30000 at b = 5 390 -> 25.
constexpr uint64_t kDecWaves = 1024;
BandSplit decode_split(uint64_t all_bands) {
  BandSplit split = {1, 1};
  while (split.rows < kDecTH && all_bands * split.rows < kDecWaves) split.rows *= 2;
  if (split.rows == kDecTH)
    while (split.cols < 16 && all_bands * kDecTH * split.cols < kDecWaves) split.cols *= 2;
  return split;
}

// k_dec_panel's waves and LDS words: the most that a panel of the batch takes.
void decode_panel_shape(DecBatch &db, const DecodePlan &dp) {
  if (dp.init_status != RSZ_OK || !panel_fits(dp)) return;
  db.panel_waves = std::max(db.panel_waves, dp.nbands);
  db.panel_cols = std::max(db.panel_cols, dp.Wb);
  db.panel_lds = db.panel_waves * db.panel_cols;
}

// A stream's workspace region from w (its buffers one after the other, each
// on a 256-byte boundary; dp's pointers into it are set); returns its end.
uint8_t *decode_region(DecodePlan &dp, uint8_t *w) {
  auto take = [&](uint64_t bytes) {
    uint8_t *at = w;
    w += align_up(bytes, 256);
    return at;
  };
  dp.res = (int32_t *)take(4ull * dp.nbins);
  dp.res8 = take(dp.nbins + 64ull);
  dp.status = (int32_t *)take(4);
  dp.tables = (uint32_t *)take(4ull * kTabWords);
  if (dp.dim == 1) {
    dp.carry = (uint32_t *)take(4ull * dp.P * dp.Hb);
  } else if (dp.nbands > 1 && !panel_fits(dp)) {
    dp.colbase = (uint32_t *)take(4ull * dp.P * dp.nbands * dp.Wb);
    dp.segtot = (uint32_t *)take(4ull * dp.P * dp.nsegs * dp.Wb);
  }
  if (dp.roi_coding) dp.roi_payload = (uint32_t *)take(4ull * dp.npeaks * dp.w * dp.w);
  // the Huffman words: in the stream, or expanded from the run section
  dp.bits = (const uint32_t *)(dp.in + dp.off_bits);
  if (dp.run_coding) {
    dp.hbits = (uint32_t *)take(4 * ((dp.T + 31) / 32 + 2));
    dp.bits = dp.hbits;
  }
  return w;
}

}  // namespace rsz
