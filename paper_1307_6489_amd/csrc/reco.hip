// HIP kernels of the low-level reconstruction for gfx950 (CDNA4).
//
// Calibration / signal extraction, two-level tailcut cleaning, islands and
// Hillas moments of camera events (the calibration and image-parameter stage
// of the real-time reconstruction, Sections 4.1-4.2 of the paper), plus the
// per-array-event stereo direction.  The operations are defined in rta.h.
//
// Data flow of one camera event inside a workgroup:
//   1. extraction   each lane owns PPL consecutive pixels and streams their
//                   samples slice by slice (one PPL*2-byte load per slice, a
//                   wavefront reads 64*PPL*2 contiguous bytes).  A running
//                   w-sample window sum lives in registers; the argmax is a
//                   single unsigned max of (W << 8 | 255 - s).  Dual-gain
//                   cameras track the raw high-gain maximum with packed
//                   16-bit max and re-stream the low gain only for lanes that
//                   own a switched pixel.  D and the threshold flags go to LDS.
//   2. mask         only pixels at or above a threshold can be mask pixels;
//                   each wavefront keeps a run of its flagged ones and decides
//                   them by their neighbours' flags in LDS.
//   3. slots        popcount prefix over the mask words gives every cleaned
//                   pixel a slot (pixel order); the peak time comes from a
//                   re-read of its window samples.
//   4. islands      images of up to 64 mask pixels: flood fill over slot
//                   masks by one wavefront; larger ones: lock-free union-find
//                   over the slots in LDS.
//   5. Hillas       three reductions (cog, centred second moments,
//                   longitudinal moments + time sums), each a fixed-order
//                   wavefront butterfly + wave-ordered sum, so results are
//                   deterministic.
//
// Where the trace read is short (the fixed window: 16 KB of a 2048-pixel
// event) a telescope is one serial chain of some ten microseconds, bound by
// the latencies of steps 2 to 5, and the rate is the telescopes in flight
// over that chain.  Both were worked on together: the chain after the
// extraction went from 11 to 5 us, the LDS of a telescope from 32.3 to 16.8
// KB and the fixed window's registers from 72 to 60 (eight workgroups per
// compute unit, five before).  8000 camera events of the 1:3:6 mix: fixed
// window 134 -> 61 us.
#include <cfloat>
#include <cmath>

#include "descriptors.h"
#include "mlp_device.h"
#include "nbr_rule.h"
#include "pixel_runs.h"
#include "rta_internal.h"

namespace rta {
namespace {

constexpr int kWave = 64;
constexpr float kNaN = __builtin_nanf("");

__device__ __forceinline__ uint32_t lo16(uint32_t d) { return d & 0xffffu; }
__device__ __forceinline__ uint32_t hi16(uint32_t d) { return d >> 16; }

typedef unsigned short us2 __attribute__((ext_vector_type(2)));

// Per-halfword unsigned maximum of two packed pairs of uint16.
__device__ __forceinline__ uint32_t pkmax16(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t,
                            __builtin_elementwise_max(__builtin_bit_cast(us2, a), __builtin_bit_cast(us2, b)));
}

// Trace loads go through a buffer resource spanning one camera event: the
// per-lane byte offset (its pixel group) stays in one VGPR and the per-slice
// offset is wave-uniform, so it rides in the scalar soffset operand.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// Cache-policy bits of the trace loads (bit 1 = non-temporal: every trace
// byte is read once, so the L2 should not keep it).
#ifndef RTA_TRACE_CPOL
#define RTA_TRACE_CPOL 2
#endif

__device__ __forceinline__ __amdgpu_buffer_rsrc_t event_rsrc(const uint16_t* base, int64_t elems) {
  // word 3 = 0x00020000: raw 32-bit data format, bounds-checked against num_records
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(base), 0, (int)(elems * 2), 0x00020000);
}

template <int ND>
__device__ __forceinline__ void load_slice(uint32_t (&d)[ND], __amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  if constexpr (ND == 4) {
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, RTA_TRACE_CPOL);
    d[0] = v[0]; d[1] = v[1]; d[2] = v[2]; d[3] = v[3];
  } else if constexpr (ND == 2) {
    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, (int)soff, RTA_TRACE_CPOL);
    d[0] = v[0]; d[1] = v[1];
  } else {
    d[0] = __builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, (int)soff, RTA_TRACE_CPOL);
  }
}

template <int PPL>
__device__ __forceinline__ void load_i32(int32_t (&v)[PPL], const int32_t* p) {
  if constexpr (PPL == 8) {
    const int4 a = *reinterpret_cast<const int4*>(p);
    const int4 b = *reinterpret_cast<const int4*>(p + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  } else if constexpr (PPL == 4) {
    const int4 a = *reinterpret_cast<const int4*>(p);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  } else {
    const int2 a = *reinterpret_cast<const int2*>(p);
    v[0] = a.x; v[1] = a.y;
  }
}

__device__ __forceinline__ int uniform_i32(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ long long uniform_i64(long long v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)(unsigned long long)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((unsigned long long)v >> 32));
  return (long long)(((unsigned long long)hi << 32) | lo);
}
template <typename T>
__device__ __forceinline__ T* uniform_ptr(T* p) {
  return reinterpret_cast<T*>(uniform_i64(reinterpret_cast<long long>(p)));
}

// A wave-uniform copy of a camera's tables: every field forced into scalar
// registers, so loops over samples / pixels and buffer descriptors built from
// them stay scalar (no per-lane waterfall around buffer loads).
__device__ __forceinline__ DevCam uniform_cam(const DevCam& c) {
  DevCam u;
  u.n_pix = uniform_i32(c.n_pix);
  u.n_pix_pad = uniform_i32(c.n_pix_pad);
  u.n_samp = uniform_i32(c.n_samp);
  u.n_gain = uniform_i32(c.n_gain);
  u.window = uniform_i32(c.window);
  u.hg_switch = uniform_i32(c.hg_switch);
  u.event_elems = uniform_i64(c.event_elems);
  u.focal = __int_as_float(uniform_i32(__float_as_int(c.focal)));
  u.fixed_start = uniform_i32(c.fixed_start);
  u.P256 = uniform_ptr(c.P256);
  u.thr_pic = uniform_ptr(c.thr_pic);
  u.thr_bnd = uniform_ptr(c.thr_bnd);
  u.a = uniform_ptr(c.a);
  u.x = uniform_ptr(c.x);
  u.y = uniform_ptr(c.y);
  u.nbr = uniform_ptr(c.nbr);
  u.border = uniform_ptr(c.border);
  u.crc_tab = uniform_ptr(c.crc_tab);
  return u;
}

// ---------------------------------------------------------------------------
// Sliding-window argmax over one pixel group.
// p0 points at sample 0 of the group's first pixel; sample k of the group is
// the PPL*2 bytes at p0 + k*np.  On return key[p] = max over starts s of
// (W(s) << 8) | (255 - s): the largest window sum, ties to the smallest s.
// With TRACK_MAX, rmax holds the packed per-pixel raw maximum over all T.
//
// Samples stream in chunks of CH slices, double buffered: the loads of chunk
// c+1 are in flight while chunk c is reduced, so a wavefront keeps up to 2*CH
// slice loads outstanding.  Slices past the end of the trace (the tail of the
// last chunk) read whatever follows in the event, or 0 beyond the buffer's
// bounds, and are ignored by the uniform k < T guard.
// ---------------------------------------------------------------------------
template <int PPL, int CH>
__device__ __forceinline__ void load_chunk(uint32_t (&buf)[CH][PPL / 2], __amdgpu_buffer_rsrc_t r, uint32_t voff,
                                           uint32_t sbase, uint32_t stride, int k0) {
  uint32_t soff = sbase + (uint32_t)k0 * stride;
#pragma unroll
  for (int j = 0; j < CH; ++j) {
    load_slice<PPL / 2>(buf[j], r, voff, soff);
    soff += stride;
  }
}

// Slice j of the chunk starting at k0 enters the window whose start is
// k0 + j - W + 1; the sample leaving it is slice j - W of the same chunk, or
// slice CH + j - W of the previous chunk (still intact: the next prefetch into
// that buffer is issued only after the first W slices are reduced).
//
// Within a chunk the candidates are ranked by a chunk-local key
// (W << 4) | (15 - j): the largest sum, then the earliest slice, with an
// inline-constant low part.  merge_chunk folds the chunk's best into the
// global key (W << 8) | (255 - s).
template <int PPL, int W, int CH, bool TRACK_MAX, bool GUARD, bool FIRST, int J0, int J1>
__device__ __forceinline__ void reduce_slices(const uint32_t (&cur)[CH][PPL / 2], const uint32_t (&prev)[CH][PPL / 2],
                                              int k0, int T, uint32_t (&ws)[PPL], uint32_t (&loc)[PPL],
                                              uint32_t (&rmax)[PPL / 2]) {
  constexpr int ND = PPL / 2;
#pragma unroll
  for (int j = J0; j < J1; ++j) {
    if (GUARD && k0 + j >= T) continue;
#pragma unroll
    for (int h = 0; h < ND; ++h) {
      const uint32_t nw = cur[j][h];
      if constexpr (TRACK_MAX) rmax[h] = pkmax16(rmax[h], nw);
      if (FIRST && j < W) {
        ws[2 * h] += lo16(nw);
        ws[2 * h + 1] += hi16(nw);
        if (j == W - 1) {
          loc[2 * h] = max(loc[2 * h], (ws[2 * h] << 4) | (uint32_t)(15 - j));
          loc[2 * h + 1] = max(loc[2 * h + 1], (ws[2 * h + 1] << 4) | (uint32_t)(15 - j));
        }
      } else {
        const uint32_t od = (j >= W) ? cur[j - W][h] : prev[CH + j - W][h];
        ws[2 * h] += lo16(nw) - lo16(od);
        ws[2 * h + 1] += hi16(nw) - hi16(od);
        loc[2 * h] = max(loc[2 * h], (ws[2 * h] << 4) | (uint32_t)(15 - j));
        loc[2 * h + 1] = max(loc[2 * h + 1], (ws[2 * h + 1] << 4) | (uint32_t)(15 - j));
      }
    }
  }
}

// Global key from the chunk-local best: start s = k0 + j - W + 1, so
// 255 - s = (254 - k0 + W - 15) + (15 - j).
template <int PPL, int W>
__device__ __forceinline__ void merge_chunk(int k0, uint32_t (&loc)[PPL], uint32_t (&key)[PPL]) {
  const uint32_t c = (uint32_t)(254 - k0 + W - 15);
#pragma unroll
  for (int p = 0; p < PPL; ++p) {
    const uint32_t cand = ((loc[p] >> 4) << 8) | (c + (loc[p] & 15u));
    key[p] = max(key[p], cand);
    loc[p] = 0;
  }
}

template <int PPL, int W, int CH, bool TRACK_MAX, bool GUARD, bool FIRST>
__device__ __forceinline__ void reduce_chunk(const uint32_t (&cur)[CH][PPL / 2], const uint32_t (&prev)[CH][PPL / 2],
                                             int k0, int T, uint32_t (&ws)[PPL], uint32_t (&loc)[PPL],
                                             uint32_t (&key)[PPL], uint32_t (&rmax)[PPL / 2]) {
  reduce_slices<PPL, W, CH, TRACK_MAX, GUARD, FIRST, 0, CH>(cur, prev, k0, T, ws, loc, rmax);
  merge_chunk<PPL, W>(k0, loc, key);
}

// stop(key) is asked after the first chunk, whose windows key then holds, with
// the second one's loads in flight: true ends the pass, and false is returned.
template <int PPL, int W, int CH, bool TRACK_MAX, class Stop>
__device__ __forceinline__ bool window_argmax(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t sbase, uint32_t stride,
                                              int T, uint32_t (&key)[PPL], uint32_t (&rmax)[PPL / 2], Stop&& stop) {
  static_assert(CH % W == 0 && CH >= W && CH <= 16, "chunk must be a multiple of the window, at most 16");
  constexpr int ND = PPL / 2;
  uint32_t ws[PPL], loc[PPL];
  uint32_t A[CH][ND], B[CH][ND];
#pragma unroll
  for (int p = 0; p < PPL; ++p) { ws[p] = 0; loc[p] = 0; key[p] = 0; }
  const int nchunk = (T + CH - 1) / CH;
  const int nfull = T / CH;  // chunks with all CH slices inside the trace
  load_chunk<PPL, CH>(A, r, voff, sbase, stride, 0);
  if (nchunk > 1) load_chunk<PPL, CH>(B, r, voff, sbase, stride, CH);
  if (nfull >= 1)
    reduce_chunk<PPL, W, CH, TRACK_MAX, false, true>(A, A, 0, T, ws, loc, key, rmax);
  else
    reduce_chunk<PPL, W, CH, TRACK_MAX, true, true>(A, A, 0, T, ws, loc, key, rmax);
  if (stop(key)) return false;
  // Chunk c lives in B (odd c) or A (even c); the other buffer holds c - 1.
  for (int c = 1; c < nchunk; c += 2) {
    const int k0 = c * CH;
    if (c < nfull) {
      reduce_slices<PPL, W, CH, TRACK_MAX, false, false, 0, W>(B, A, k0, T, ws, loc, rmax);
      if (c + 1 < nchunk) load_chunk<PPL, CH>(A, r, voff, sbase, stride, k0 + CH);
      reduce_slices<PPL, W, CH, TRACK_MAX, false, false, W, CH>(B, A, k0, T, ws, loc, rmax);
    } else {
      reduce_slices<PPL, W, CH, TRACK_MAX, true, false, 0, CH>(B, A, k0, T, ws, loc, rmax);
    }
    merge_chunk<PPL, W>(k0, loc, key);
    if (c + 1 >= nchunk) break;
    const int k1 = k0 + CH;
    if (c + 1 < nfull) {
      reduce_slices<PPL, W, CH, TRACK_MAX, false, false, 0, W>(A, B, k1, T, ws, loc, rmax);
      if (c + 2 < nchunk) load_chunk<PPL, CH>(B, r, voff, sbase, stride, k1 + CH);
      reduce_slices<PPL, W, CH, TRACK_MAX, false, false, W, CH>(A, B, k1, T, ws, loc, rmax);
    } else {
      reduce_slices<PPL, W, CH, TRACK_MAX, true, false, 0, CH>(A, B, k1, T, ws, loc, rmax);
    }
    merge_chunk<PPL, W>(k1, loc, key);
  }
  return true;
}

template <int PPL, int W, int CH, bool TRACK_MAX>
__device__ __forceinline__ void window_argmax(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t sbase, uint32_t stride,
                                              int T, uint32_t (&key)[PPL], uint32_t (&rmax)[PPL / 2]) {
  window_argmax<PPL, W, CH, TRACK_MAX>(r, voff, sbase, stride, T, key, rmax,
                                       [](const uint32_t (&)[PPL]) { return false; });
}

// The two partners of a lane in one step of a butterfly over the wavefront
// (see butterfly below), as register moves.
template <int STEP>
__device__ __forceinline__ void partner_u32(uint32_t v, uint32_t* a, uint32_t* b) {
  if constexpr (STEP == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    *a = r[0];
    *b = r[1];
  } else if constexpr (STEP == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    *a = r[0];
    *b = r[1];
  } else {
    constexpr int ctrl = STEP == 8 ? 0x128 : STEP == 4 ? 0x124 : STEP == 2 ? 0x4E : 0xB1;
    *a = v;
    *b = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, 0xF, 0xF, false);
  }
}

// Maximum over the wavefront, in every lane.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  uint32_t a, b;
  partner_u32<32>(v, &a, &b); v = max(a, b);
  partner_u32<16>(v, &a, &b); v = max(a, b);
  partner_u32<8>(v, &a, &b); v = max(a, b);
  partner_u32<4>(v, &a, &b); v = max(a, b);
  partner_u32<2>(v, &a, &b); v = max(a, b);
  partner_u32<1>(v, &a, &b); v = max(a, b);
  return v;
}

// Best window of a trace spread over the wavefront, lane l holding samples
// l, l + 64, ... in x (any value past the trace): the largest
// (sum << 8) | (255 - start), in every lane.
template <int W, int NR>
__device__ __forceinline__ uint32_t wave_window(const uint32_t (&x)[NR], int T) {
  const int lane = threadIdx.x & (kWave - 1);
  uint32_t best = 0;
  uint32_t nxt[W - 1];  // the current 64 samples shifted down by 1 .. W-1 lanes
#pragma unroll
  for (int u = 1; u < W; ++u) nxt[u - 1] = (uint32_t)__shfl((int)x[0], (lane + u) & (kWave - 1), kWave);
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    if (k * kWave >= T) continue;
    const bool more = (k + 1) * kWave < T;
    uint32_t sum = x[k];
#pragma unroll
    for (int u = 1; u < W; ++u) {
      uint32_t nx = 0;
      if (k + 1 < NR && more) nx = (uint32_t)__shfl((int)x[k + 1 < NR ? k + 1 : k], (lane + u) & (kWave - 1), kWave);
      sum += lane + u < kWave ? nxt[u - 1] : nx;
      nxt[u - 1] = nx;
    }
    const int s = lane + k * kWave;
    if (s + W <= T) best = max(best, (sum << 8) | (uint32_t)(255 - s));
  }
  return wave_max_u32(best);
}

// Keys of a few pixels of the wavefront's groups by the whole wavefront: lane
// l takes the samples l, l + 64, ... of a pixel (one 2-byte load each, all in
// flight together), gets the next W - 1 from its neighbour lanes and ranks
// the windows that start at its own samples.  want: the pixels of this lane's
// group, bit p; their keys are replaced.  A round takes one pixel of each p,
// up to PPL at once.
template <int PPL, int W>
__device__ __forceinline__ void pixel_keys(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t sbase, uint32_t stride,
                                           int T, uint32_t want, uint32_t (&key)[PPL]) {
  constexpr int NR = (RTA_MAX_SAMP + kWave - 1) / kWave;
  const int lane = threadIdx.x & (kWave - 1);
  uint64_t m[PPL], any = 0;
#pragma unroll
  for (int p = 0; p < PPL; ++p) {
    m[p] = __ballot((want >> p) & 1u);
    any |= m[p];
  }
  while (any) {
    uint32_t x[PPL][NR];
#pragma unroll
    for (int p = 0; p < PPL; ++p) {
      if (!m[p]) continue;
      const uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)voff, __builtin_ctzll(m[p])) + 2u * p;
#pragma unroll
      for (int k = 0; k < NR; ++k)  // past the trace: its last sample, never ranked
        if (k * kWave < T)
          x[p][k] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(
              r, (int)(at + (uint32_t)min(lane + k * kWave, T - 1) * stride), (int)sbase, 0);
    }
    any = 0;
#pragma unroll
    for (int p = 0; p < PPL; ++p) {
      if (!m[p]) continue;
      const uint32_t best = wave_window<W>(x[p], T);
      if (lane == __builtin_ctzll(m[p])) key[p] = best;
      m[p] &= m[p] - 1ull;
      any |= m[p];
    }
  }
}

// Extraction of one pixel group on its selected gain.  Returns the bit mask
// of pixels that switched to low gain.  Their low-gain windows: a wavefront
// with at most 2 PPL switched pixels gathers those pixels' samples alone (a
// pixel's T samples cost T memory sectors of 64 bytes, a re-stream of the
// wavefront's groups 2 PPL sectors a slice); with more it streams its groups
// again.  A switched pixel held its telescope for 10.5 us of re-stream at
// 2048 x 128, against 2-3 us of gather.
template <int PPL, int W, int CH>
__device__ __forceinline__ uint32_t extract_group(const DevCam& c, __amdgpu_buffer_rsrc_t r, int pix0, int np, int T,
                                                  bool dual, uint32_t (&key)[PPL]) {
  uint32_t rmax[PPL / 2];
#pragma unroll
  for (int h = 0; h < PPL / 2; ++h) rmax[h] = 0;
  const uint32_t voff = (uint32_t)pix0 * 2u, stride = (uint32_t)np * 2u;
  uint32_t sw = 0;
  if (dual) {
    window_argmax<PPL, W, CH, true>(r, voff, 0u, stride, T, key, rmax);
    int n_sw = 0;
#pragma unroll
    for (int p = 0; p < PPL; ++p) {
      const uint32_t m = (p & 1) ? hi16(rmax[p >> 1]) : lo16(rmax[p >> 1]);
      const bool low = (int)m >= c.hg_switch && pix0 + p < c.n_pix;
      if (low) sw |= 1u << p;
      n_sw += __popcll(__ballot(low));
    }
    // wave-uniform branches (the buffer operands stay scalar)
    if (n_sw > 2 * PPL) {
      uint32_t kl[PPL], unused[PPL / 2];
      window_argmax<PPL, W, CH, false>(r, voff, (uint32_t)T * stride, stride, T, kl, unused);
#pragma unroll
      for (int p = 0; p < PPL; ++p)
        if ((sw >> p) & 1u) key[p] = kl[p];
    } else if (n_sw > 0) {
      pixel_keys<PPL, W>(r, voff, (uint32_t)T * stride, stride, T, sw, key);
    }
  } else {
    window_argmax<PPL, W, CH, false>(r, voff, 0u, stride, T, key, rmax);
  }
  return sw;
}

// ---------------------------------------------------------------------------
// Sliding-window argmax that also keeps each pixel's best window (the
// unfused calibration call reports Nt and the peak of every pixel, not only of
// the cleaned ones, so re-reading the window samples afterwards would fetch
// scattered rows of the whole trace a second time).  While the samples
// stream past, the window ending at slice k replaces the best one when its
// sum is strictly larger (ties keep the earliest start, as the packed key
// does), and then the window's four samples, already in registers, are kept
// packed two per register.  W = 4 only.
// ---------------------------------------------------------------------------
template <int PPL>
struct KeepState {
  uint32_t ws[PPL];   // running window sum
  uint32_t key[PPL];  // best (sum << 8) | (255 - start) so far (0 before the first window)
  uint32_t sv0[PPL];  // samples s*, s*+1 of the best window (low, high half)
  uint32_t sv1[PPL];  // samples s*+2, s*+3
};

// (half of word a, the same half of word b) packed low / high: the samples
// of one pixel at two consecutive slices.
template <int HALF>
__device__ __forceinline__ uint32_t pair16(uint32_t a, uint32_t b) {
  return __builtin_amdgcn_perm(b, a, HALF ? 0x07060302u : 0x05040100u);
}

template <int PPL, int CH, bool TRACK_MAX, bool GUARD, bool FIRST, int J0, int J1>
__device__ __forceinline__ void keep_slices(const uint32_t (&cur)[CH][PPL / 2], const uint32_t (&prev)[CH][PPL / 2],
                                            int k0, int T, KeepState<PPL>& st, uint32_t (&rmax)[PPL / 2]) {
  constexpr int ND = PPL / 2, W = 4;
#pragma unroll
  for (int j = J0; j < J1; ++j) {
    if (GUARD && k0 + j >= T) continue;
#pragma unroll
    for (int h = 0; h < ND; ++h) {
      const uint32_t nw = cur[j][h];
      if constexpr (TRACK_MAX) rmax[h] = pkmax16(rmax[h], nw);
      // words of slices k-1, k-2, k-3 (from the previous chunk near its start;
      // only read once the first window is complete)
      const uint32_t w1 = j >= 1 ? cur[j - 1][h] : prev[CH - 1][h];
      const uint32_t w2 = j >= 2 ? cur[j - 2][h] : prev[CH + j - 2][h];
      const uint32_t w3 = j >= 3 ? cur[j - 3][h] : prev[CH + j - 3][h];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int p = 2 * h + u;
        const uint32_t x = u ? hi16(nw) : lo16(nw);
        if (FIRST && j < W) {
          st.ws[p] += x;
        } else {
          const uint32_t od = j >= W ? cur[j - W][h] : prev[CH + j - W][h];
          st.ws[p] += x - (u ? hi16(od) : lo16(od));
        }
        if (!FIRST || j >= W - 1) {
          // the window starting at k - 3 wins on a larger sum; on an equal
          // sum the earlier start, already held, has the larger key
          const uint32_t nk = (st.ws[p] << 8) | (uint32_t)(255 - (k0 + j - (W - 1)));
          const bool better = nk > st.key[p];
          st.key[p] = better ? nk : st.key[p];
          st.sv0[p] = better ? (u ? pair16<1>(w3, w2) : pair16<0>(w3, w2)) : st.sv0[p];
          st.sv1[p] = better ? (u ? pair16<1>(w1, nw) : pair16<0>(w1, nw)) : st.sv1[p];
        }
      }
    }
  }
}

template <int PPL, int CH, bool TRACK_MAX>
__device__ __forceinline__ void window_keep(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t sbase, uint32_t stride,
                                            int T, KeepState<PPL>& st, uint32_t (&rmax)[PPL / 2]) {
  constexpr int W = 4;
  static_assert(CH % W == 0 && CH >= W && CH <= 16, "chunk must be a multiple of the window, at most 16");
  constexpr int ND = PPL / 2;
  uint32_t A[CH][ND], B[CH][ND];
#pragma unroll
  for (int p = 0; p < PPL; ++p) {
    st.ws[p] = 0; st.key[p] = 0; st.sv0[p] = 0; st.sv1[p] = 0;
  }
  const int nchunk = (T + CH - 1) / CH;
  const int nfull = T / CH;
  load_chunk<PPL, CH>(A, r, voff, sbase, stride, 0);
  if (nchunk > 1) load_chunk<PPL, CH>(B, r, voff, sbase, stride, CH);
  if (nfull >= 1)
    keep_slices<PPL, CH, TRACK_MAX, false, true, 0, CH>(A, A, 0, T, st, rmax);
  else
    keep_slices<PPL, CH, TRACK_MAX, true, true, 0, CH>(A, A, 0, T, st, rmax);
  for (int c = 1; c < nchunk; c += 2) {
    const int k0 = c * CH;
    if (c < nfull) {
      keep_slices<PPL, CH, TRACK_MAX, false, false, 0, W>(B, A, k0, T, st, rmax);
      if (c + 1 < nchunk) load_chunk<PPL, CH>(A, r, voff, sbase, stride, k0 + CH);
      keep_slices<PPL, CH, TRACK_MAX, false, false, W, CH>(B, A, k0, T, st, rmax);
    } else {
      keep_slices<PPL, CH, TRACK_MAX, true, false, 0, CH>(B, A, k0, T, st, rmax);
    }
    if (c + 1 >= nchunk) break;
    const int k1 = k0 + CH;
    if (c + 1 < nfull) {
      keep_slices<PPL, CH, TRACK_MAX, false, false, 0, W>(A, B, k1, T, st, rmax);
      if (c + 2 < nchunk) load_chunk<PPL, CH>(B, r, voff, sbase, stride, k1 + CH);
      keep_slices<PPL, CH, TRACK_MAX, false, false, W, CH>(A, B, k1, T, st, rmax);
    } else {
      keep_slices<PPL, CH, TRACK_MAX, true, false, 0, CH>(A, B, k1, T, st, rmax);
    }
  }
}

// Extraction of one pixel group with its best windows kept: the high gain,
// then, when any lane of the wave owns a switched pixel, the low gain, whose
// window replaces the high-gain one for the switched pixels.  Returns the
// switch mask; st holds the selected gain's windows.
template <int PPL, int CH>
__device__ __forceinline__ uint32_t keep_group(const DevCam& c, __amdgpu_buffer_rsrc_t r, int pix0, int np, int T,
                                               bool dual, KeepState<PPL>& st) {
  uint32_t rmax[PPL / 2];
#pragma unroll
  for (int h = 0; h < PPL / 2; ++h) rmax[h] = 0;
  const uint32_t voff = (uint32_t)pix0 * 2u, stride = (uint32_t)np * 2u;
  uint32_t sw = 0;
  if (dual) {
    window_keep<PPL, CH, true>(r, voff, 0u, stride, T, st, rmax);
#pragma unroll
    for (int p = 0; p < PPL; ++p) {
      const uint32_t m = (p & 1) ? hi16(rmax[p >> 1]) : lo16(rmax[p >> 1]);
      if ((int)m >= c.hg_switch) sw |= 1u << p;
    }
    if (__ballot(sw != 0u)) {
      KeepState<PPL> lg;
      uint32_t unused[PPL / 2];
      window_keep<PPL, CH, false>(r, voff, (uint32_t)T * stride, stride, T, lg, unused);
#pragma unroll
      for (int p = 0; p < PPL; ++p)
        if ((sw >> p) & 1u) {
          st.key[p] = lg.key[p];
          st.sv0[p] = lg.sv0[p];
          st.sv1[p] = lg.sv1[p];
        }
    }
  } else {
    window_keep<PPL, CH, false>(r, voff, 0u, stride, T, st, rmax);
  }
  return sw;
}

// Nt = sum_k k*(256*x[s*+k] - P) and the earliest in-window peak from a kept
// window (samples x0..x3 = low / high halves of sv0, sv1).
__device__ __forceinline__ int32_t kept_nt(uint32_t sv0, uint32_t sv1, int32_t P, int s, int* peak) {
  const uint32_t x[4] = {lo16(sv0), hi16(sv0), lo16(sv1), hi16(sv1)};
  int32_t nt = 0;
  uint32_t pmax = x[0];
  int pk = s;
#pragma unroll
  for (int k = 1; k < 4; ++k) {
    nt += k * (256 * (int32_t)x[k] - P);
    if (x[k] > pmax) { pmax = x[k]; pk = s + k; }
  }
  *peak = pk;
  return nt;
}

// ---------------------------------------------------------------------------
// Window placement by the other extractors.  They produce the same packed key
// (S << 8) | (255 - s*) as the sliding window, so every later step is shared.
// ---------------------------------------------------------------------------
enum : int {
  kExSliding = RTA_EXTRACT_SLIDING,
  kExFixed = RTA_EXTRACT_FIXED,
  kExGlobal = RTA_EXTRACT_GLOBAL_PEAK,
  kExNeighbour = RTA_EXTRACT_NEIGHBOUR_PEAK
};

// Neighbour peak: high-gain slices staged in LDS this many at a time.
constexpr int kNbrRows = 4;
// Most pixels whose neighbour windows are formed apart, and most staged
// traces (with those, eight slices fit at once).
constexpr int kNbrAsk = 512, kNbrStage = 600;

// Sums of the W samples from slice s on of every pixel of the group (one
// load per slice) and, with TRACK_MAX, their packed per-pixel maximum.
template <int PPL, int W, bool TRACK_MAX>
__device__ __forceinline__ void window_at(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t sbase, uint32_t stride,
                                          int s, uint32_t (&S)[PPL], uint32_t (&mx)[PPL / 2]) {
  constexpr int ND = PPL / 2;
  uint32_t d[W][ND];
  uint32_t soff = sbase + (uint32_t)s * stride;
#pragma unroll
  for (int k = 0; k < W; ++k) {
    load_slice<ND>(d[k], r, voff, soff);
    soff += stride;
  }
#pragma unroll
  for (int p = 0; p < PPL; ++p) S[p] = 0;
#pragma unroll
  for (int h = 0; h < ND; ++h) mx[h] = 0;
#pragma unroll
  for (int k = 0; k < W; ++k) {
#pragma unroll
    for (int h = 0; h < ND; ++h) {
      S[2 * h] += lo16(d[k][h]);
      S[2 * h + 1] += hi16(d[k][h]);
      if constexpr (TRACK_MAX) mx[h] = pkmax16(mx[h], d[k][h]);
    }
  }
}

// Keys of a group whose window start s is known; sw: pixels on low gain.
template <int PPL, int W>
__device__ __forceinline__ void keys_at(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t stride, int T, int s,
                                        const uint32_t (&S_hg)[PPL], uint32_t sw, uint32_t (&key)[PPL]) {
  uint32_t S[PPL];
#pragma unroll
  for (int p = 0; p < PPL; ++p) S[p] = S_hg[p];
  if (__ballot(sw != 0u)) {
    uint32_t SL[PPL], unused[PPL / 2];
    window_at<PPL, W, false>(r, voff, (uint32_t)T * stride, stride, s, SL, unused);
#pragma unroll
    for (int p = 0; p < PPL; ++p)
      if ((sw >> p) & 1u) S[p] = SL[p];
  }
  const uint32_t low = 255u - (uint32_t)s;
#pragma unroll
  for (int p = 0; p < PPL; ++p) key[p] = (S[p] << 8) | low;
}

// Fixed window: samples s0 .. s0+W-1 of every pixel, the gain decided on the
// high-gain samples of that window; nothing else of the trace is read.
template <int PPL, int W>
__device__ __forceinline__ uint32_t fixed_group(const DevCam& c, __amdgpu_buffer_rsrc_t r, int pix0, int np, int T,
                                                bool dual, uint32_t (&key)[PPL]) {
  const uint32_t voff = (uint32_t)pix0 * 2u, stride = (uint32_t)np * 2u;
  const int s0 = c.fixed_start;
  uint32_t S[PPL], mx[PPL / 2];
  window_at<PPL, W, true>(r, voff, 0u, stride, s0, S, mx);
  uint32_t sw = 0;
  if (dual) {
#pragma unroll
    for (int p = 0; p < PPL; ++p) {
      const uint32_t m = (p & 1) ? hi16(mx[p >> 1]) : lo16(mx[p >> 1]);
      if ((int)m >= c.hg_switch) sw |= 1u << p;
    }
  }
  keys_at<PPL, W>(r, voff, stride, T, s0, S, sw, key);
  return sw;
}

// Sum of v over the wavefront, valid in lane 63, with DPP lane moves only
// (no LDS traffic): pairs and quads by quad permutes, eights and sixteens by
// the half-row and row mirrors, then rows by the row-15 and row-31
// broadcasts (rows outside the row mask add 0).
__device__ __forceinline__ uint32_t wave_sum_u32_last(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);   // quad_perm [2,3,0,1]
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false);  // row_half_mirror
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false);  // row_mirror
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);  // row_bcast:15
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);  // row_bcast:31
  return v;
}

// Sums over the wavefront of eight values at once.  On return lane 16 r
// holds the totals of v[2 r] and v[2 r + 1] (r = 0..3): two lane swaps fold
// the halves and then the rows together while they halve the number of
// registers (a swap of two registers leaves one value's partners in the
// lower lanes and the other's in the upper ones), and the rows of 16 end
// with rotations.  About 20 instructions, against 48 for eight separate
// sums.
__device__ __forceinline__ u32x2 wave_sum8(const uint32_t (&v)[8]) {
  uint32_t u[4], w[2];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const auto r = __builtin_amdgcn_permlane32_swap(v[k], v[k + 4], false, false);
    u[k] = r[0] + r[1];
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const auto r = __builtin_amdgcn_permlane16_swap(u[k], u[k + 2], false, false);
    w[k] = r[0] + r[1];
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    w[k] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w[k], 0x128, 0xF, 0xF, false);  // row_ror:8
    w[k] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w[k], 0x124, 0xF, 0xF, false);  // row_ror:4
    w[k] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w[k], 0x122, 0xF, 0xF, false);  // row_ror:2
    w[k] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w[k], 0x121, 0xF, 0xF, false);  // row_ror:1
  }
  return u32x2{w[0], w[1]};
}

// Global peak, first stage for one group: the wave's sum of the raw
// high-gain samples of pixels below N, slice by slice, added into rows[k]
// (stored on the first pass); returns the group's low-gain bits (full-trace
// raw high-gain maximum >= switch).  Slices stream in chunks, whose sums are
// reduced eight at a time; AHEAD: the next chunk's loads are in flight
// meanwhile (twice the registers).
template <int PPL, int CH, bool AHEAD>
__device__ __forceinline__ uint32_t global_rows_group(const DevCam& c, __amdgpu_buffer_rsrc_t r, int pix0, int np,
                                                      int T, bool dual, uint32_t* rows, bool first) {
  static_assert(CH % 8 == 0, "slices are summed eight at a time");
  constexpr int ND = PPL / 2;
  const uint32_t voff = (uint32_t)pix0 * 2u, stride = (uint32_t)np * 2u;
  const int nv = min(max(c.n_pix - pix0, 0), PPL);
  uint32_t msk[ND], rmax[ND];
#pragma unroll
  for (int h = 0; h < ND; ++h) {
    msk[h] = (2 * h + 1 < nv) ? 0xffffffffu : (2 * h < nv ? 0x0000ffffu : 0u);
    rmax[h] = 0;
  }
  const int lane = threadIdx.x & (kWave - 1);
  const us2 ones = {1, 1};
  auto reduce = [&](const uint32_t (&A)[CH][ND], int k0) {
#pragma unroll
    for (int j0 = 0; j0 < CH; j0 += 8) {
      if (k0 + j0 >= T) continue;
      uint32_t v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        // slices past the trace are summed too (their totals are never
        // read) but must not enter the maximum
        const uint32_t keep = k0 + j0 + j < T ? 0xffffffffu : 0u;
        v[j] = 0;
#pragma unroll
        for (int h = 0; h < ND; ++h) {
          const uint32_t x = A[j0 + j][h] & msk[h];
          v[j] = __builtin_amdgcn_udot2(__builtin_bit_cast(us2, x), ones, v[j], false);
          rmax[h] = pkmax16(rmax[h], x & keep);
        }
      }
      const u32x2 t = wave_sum8(v);
      if ((lane & 15) == 0) {
        uint32_t* dst = rows + k0 + j0 + (lane >> 3);
        dst[0] = first ? t[0] : dst[0] + t[0];
        dst[1] = first ? t[1] : dst[1] + t[1];
      }
    }
  };
  // a wavefront without pixels (8 pixels per lane, 8 wavefronts: half of them)
  // leaves the loads and reductions to the others: 8000 events of the 1:3:6
  // mix 823 -> 469 us in chunks of 8, 967 -> 659 of 16
  if (!__ballot(nv > 0)) {
    for (int k = lane; first && k < T; k += kWave) rows[k] = 0u;
    return 0u;
  }
  uint32_t A[CH][ND], B[CH][ND];
  if constexpr (AHEAD) {
    load_chunk<PPL, CH>(A, r, voff, 0u, stride, 0);
    for (int k0 = 0; k0 < T; k0 += 2 * CH) {
      if (k0 + CH < T) load_chunk<PPL, CH>(B, r, voff, 0u, stride, k0 + CH);
      reduce(A, k0);
      if (k0 + CH >= T) break;
      if (k0 + 2 * CH < T) load_chunk<PPL, CH>(A, r, voff, 0u, stride, k0 + 2 * CH);
      reduce(B, k0 + CH);
    }
  } else {
    for (int k0 = 0; k0 < T; k0 += CH) {
      load_chunk<PPL, CH>(A, r, voff, 0u, stride, k0);
      reduce(A, k0);
    }
  }
  uint32_t sw = 0;
  if (dual) {
#pragma unroll
    for (int p = 0; p < PPL; ++p) {
      const uint32_t m = (p & 1) ? hi16(rmax[p >> 1]) : lo16(rmax[p >> 1]);
      if ((int)m >= c.hg_switch) sw |= 1u << p;
    }
  }
  return sw;
}

// Global peak start: the earliest maximiser of C(s) = sum_{k<W} of the
// camera-summed slices, from the per-wave partial sums rows[w * 256 + k].
// Called by every thread of the block (contains a barrier).
template <int NT, int W>
__device__ __forceinline__ int global_start(const uint32_t* rows, int T, int32_t* start) {
  constexpr int NW = NT / kWave;
  if (threadIdx.x < kWave) {
    uint64_t best = 0;
    for (int s = threadIdx.x; s + W <= T; s += kWave) {
      uint64_t C = 0;
#pragma unroll
      for (int k = 0; k < W; ++k)
#pragma unroll
        for (int w = 0; w < NW; ++w) C += rows[w * 256 + s + k];
      const uint64_t cand = (C << 8) | (uint64_t)(255 - s);
      best = cand > best ? cand : best;
    }
#pragma unroll
    for (int off = kWave / 2; off >= 1; off >>= 1) {
      const uint64_t o = __shfl_xor(best, off, kWave);
      best = o > best ? o : best;
    }
    if (threadIdx.x == 0) *start = 255 - (int)(best & 255u);
  }
  __syncthreads();
  return *start;
}

// Neighbour peak for every pixel of the event: the earliest maximiser of
// C_i(s) = sum over the neighbours j of i of the raw high-gain window sum
// W_j(s).  Four high-gain slices at a time are staged in LDS transposed,
// one 64-bit word of four halfwords per pixel (slices k0..k0+3; word Npad = 0
// stands in for a missing neighbour), so a pixel's neighbours cost one 8-byte
// read each per four slices.  The next four slices are loaded while the
// current ones are used.  Words sit at the pixels' lattice-row positions, and
// in this stage lane t takes positions t, t + NT, ...: the lanes of one read
// are neighbours along a row, so each direction's neighbour words are (nearly)
// consecutive; the pixels' best keys then go through LDS to the lanes'
// PPL-pixel groups.  The raw high-gain maximum (gain decision on the whole
// trace, as for the sliding window) is kept where the slices are staged.
//
// nbr_scan makes the pass over the slices.  Sums stay in saturating packed
// 16-bit halves, two slices to a register, while they fit: the neighbour sums,
// the window sums C(k) = p(k) + p(k - 2) with p(k) = y(k) + y(k - 1) (one
// funnel shift per two slices gives the pairs), and a key is one byte permute
// of the halfword with the slice's index byte: 24 vector instructions per
// pixel and four slices where the 32-bit form takes about 50 (the mix 1123 ->
// 1042 us: the scan waits more for LDS and barriers than for them).  Every
// neighbour sum of four slices is part of a window sum that is ranked with
// them, so a best sum below 65535 says that all of them fitted.  Otherwise (an
// image has to put some 8500 p.e. into six pixels, or the pedestals do) the
// wavefront forms these four slices again in 32 bits, from the state before
// them, and stays there until the trace ends.  (An event that was repeated
// from the start in 32 bits took 129 us by itself, 65 so, 61 where all sums
// fit; 200 bright events 160 us and 93; 2048 x 128.)
template <int W, int NT>
__device__ __forceinline__ void nbr_scan(const DevCam& c, __amdgpu_buffer_rsrc_t r, uint64_t* xs, uint32_t* keys,
                                         uint8_t* low) {
  static_assert(kNbrRows == 4 && W == 4, "four slices per staged pixel word pair, windows of four");
  constexpr int MAXK = (kMaxPix + NT - 1) / NT;  // pixels per lane: t, t + NT, ...
  static_assert(MAXK % 2 == 0, "positions go in pairs");
  const int N = c.n_pix, np = c.n_pix_pad, T = c.n_samp;
  // position p = 8 g + m lives in word 8 g + (m ^ (g & 7)): consecutive
  // lanes reading consecutive positions touch distinct banks
  auto slot = [](uint32_t j) { return (j & ~7u) | ((j ^ (j >> 3)) & 7u); };
  uint32_t nb[MAXK][3];  // six neighbour words per position: LDS byte offsets, 16 bits each (word Npad if missing)
  uint32_t best[MAXK];
  // in halves, (y(k0-2), y(k0-1)) and (p(k0-2), p(k0-1)); in 32 bits, y(k0-1),
  // y(k0-2) and y(k0-3), 19 bits each (six samples)
  uint32_t st[MAXK][2];
  bool wide = false;  // in 32 bits, uniform over the wavefront
#pragma unroll
  for (int k = 0; k < MAXK; ++k) {
    const int p = (int)threadIdx.x + k * NT;
    nb[k][0] = nb[k][1] = nb[k][2] = (uint32_t)np * 8u * 0x10001u;
    if (p < N) {
      const int4 v = *reinterpret_cast<const int4*>(c.lat + (size_t)p * kNbrCols);
      const uint32_t w3[3] = {(uint32_t)v.x, (uint32_t)v.y, (uint32_t)v.z};
#pragma unroll
      for (int h = 0; h < 3; ++h) {
        const uint32_t lo = (w3[h] & 0x8000u) ? (uint32_t)np : slot(w3[h] & 0xffffu);
        const uint32_t hi = (w3[h] & 0x80000000u) ? (uint32_t)np : slot(w3[h] >> 16);
        nb[k][h] = (lo << 3) | (hi << 19);  // (Npad + 1) * 8 bytes < 2^16
      }
    }
    st[k][0] = st[k][1] = 0;
    best[k] = 0;
  }
  if (threadIdx.x == 0) xs[np] = 0ull;
  // thread q stages 16-byte pixel group q (np / 8 <= kMaxPix / 8 <= NT
  // groups), the next four slices loaded while the current ones are used
  static_assert(kMaxPix / 8 <= NT, "one staged pixel group per thread");
  const int q = threadIdx.x;
  const bool stager = q < np / 8;
  const us2 row_lo = {1, 0}, row_hi = {0, 1};
  // the words of this thread's eight pixels, at their positions
  uint32_t dst[8];
  if (stager) {
    const int4 lp = *reinterpret_cast<const int4*>(c.lpos + (size_t)q * 8);
    const uint32_t w4[4] = {(uint32_t)lp.x, (uint32_t)lp.y, (uint32_t)lp.z, (uint32_t)lp.w};
#pragma unroll
    for (int m = 0; m < 8; ++m) dst[m] = slot((w4[m >> 1] >> ((m & 1) * 16)) & 0xffffu);
  }
  u32x4 d[kNbrRows], hmax = {0, 0, 0, 0};
  auto load4 = [&](int k0) {
#pragma unroll
    for (int k = 0; k < kNbrRows; ++k)
      d[k] = __builtin_amdgcn_raw_buffer_load_b128(r, q * 16, (k0 + k) * np * 2, RTA_TRACE_CPOL);
  };
  if (stager) load4(0);
  for (int k0 = 0; k0 < T; k0 += kNbrRows) {
    // keep the neighbour offsets packed: unpacked out of the loop they
    // would take six registers per position instead of three
#pragma unroll
    for (int k = 0; k < MAXK; ++k)
#pragma unroll
      for (int h = 0; h < 3; ++h) asm volatile("" : "+v"(nb[k][h]));
    __syncthreads();  // the previous slices are consumed
    if (stager) {
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const uint32_t sel = (m & 1) ? 0x07060302u : 0x05040100u;  // high / low halfwords
        xs[dst[m]] = (uint64_t)__builtin_amdgcn_perm(d[1][m >> 1], d[0][m >> 1], sel) |
                     ((uint64_t)__builtin_amdgcn_perm(d[3][m >> 1], d[2][m >> 1], sel) << 32);
      }
#pragma unroll
      for (int k = 0; k < kNbrRows; ++k)
        if (k0 + k < T) {
#pragma unroll
          for (int h = 0; h < 4; ++h) hmax[h] = pkmax16(hmax[h], d[k][h]);
        }
    }
    __syncthreads();
    if (stager && k0 + kNbrRows < T) load4(k0 + kNbrRows);
    // uniform: every slice of this step has a full window inside the trace
    const bool full = k0 >= W - 1 && k0 + kNbrRows <= T;
    const uint32_t key0 = (uint32_t)(255 - (k0 - (W - 1)));  // 255 - window start of slice k0
    // the four slices' index bytes (slices without a window are not ranked)
    const uint32_t idx = (key0 & 255u) | (((key0 - 1u) & 255u) << 8) | (((key0 - 2u) & 255u) << 16) |
                         (((key0 - 3u) & 255u) << 24);
    // positions past the camera read the zero word; their keys are not used
    auto load = [&](int k, uint64_t (&v)[6]) {
#pragma unroll
      for (int m = 0; m < 6; ++m) {
        const uint32_t off = (nb[k][m >> 1] >> ((m & 1) * 16)) & 0xffffu;
        v[m] = *reinterpret_cast<const uint64_t*>(reinterpret_cast<const char*>(xs) + off);
      }
    };
    // in halves: the state after these slices in s, the best key returned
    auto halves = [&](int k, uint32_t (&s)[2], bool whole) {
      uint64_t v[6];
      load(k, v);
      us2 s01 = __builtin_bit_cast(us2, (uint32_t)v[0]), s23 = __builtin_bit_cast(us2, (uint32_t)(v[0] >> 32));
#pragma unroll
      for (int m = 1; m < 6; ++m) {
        s01 = __builtin_elementwise_add_sat(s01, __builtin_bit_cast(us2, (uint32_t)v[m]));
        s23 = __builtin_elementwise_add_sat(s23, __builtin_bit_cast(us2, (uint32_t)(v[m] >> 32)));
      }
      // (y(k0-1), y(k0)) and (y(k0+1), y(k0+2))
      const us2 m10 =
          __builtin_bit_cast(us2, __builtin_amdgcn_alignbit(__builtin_bit_cast(uint32_t, s01), st[k][0], 16));
      const us2 s12 = __builtin_bit_cast(us2, __builtin_amdgcn_alignbit(__builtin_bit_cast(uint32_t, s23),
                                                                        __builtin_bit_cast(uint32_t, s01), 16));
      const us2 p01 = __builtin_elementwise_add_sat(s01, m10), p23 = __builtin_elementwise_add_sat(s23, s12);
      const uint32_t C01 = __builtin_bit_cast(
          uint32_t, __builtin_elementwise_add_sat(p01, __builtin_bit_cast(us2, st[k][1])));
      const uint32_t C23 = __builtin_bit_cast(uint32_t, __builtin_elementwise_add_sat(p23, p01));
      s[0] = __builtin_bit_cast(uint32_t, s23);
      s[1] = __builtin_bit_cast(uint32_t, p23);
      // (C << 8) | index byte: bytes 4..7 of the permute are C's, 0..3 the indices'
      const uint32_t kk[kNbrRows] = {
          __builtin_amdgcn_perm(C01, idx, 0x0c050400u), __builtin_amdgcn_perm(C01, idx, 0x0c070601u),
          __builtin_amdgcn_perm(C23, idx, 0x0c050402u), __builtin_amdgcn_perm(C23, idx, 0x0c070603u)};
      if (whole) {
        best[k] = max(max(best[k], kk[0]), kk[1]);
        best[k] = max(max(best[k], kk[2]), kk[3]);
      } else {
#pragma unroll
        for (int u = 0; u < kNbrRows; ++u)
          if (k0 + u >= W - 1 && k0 + u < T) best[k] = max(best[k], kk[u]);
      }
    };
    auto exact = [&](int k) {
      uint64_t v[6];
      load(k, v);
      uint32_t y[W - 1 + kNbrRows] = {st[k][1] >> 6, st[k][0] >> 19 | (st[k][1] & 63u) << 13, st[k][0] & 0x7ffffu};
#pragma unroll
      for (int m = 0; m < 6; ++m) {
        const uint32_t v01 = (uint32_t)v[m], v23 = (uint32_t)(v[m] >> 32);
        y[3] = __builtin_amdgcn_udot2(__builtin_bit_cast(us2, v01), row_lo, y[3], false);
        y[4] = __builtin_amdgcn_udot2(__builtin_bit_cast(us2, v01), row_hi, y[4], false);
        y[5] = __builtin_amdgcn_udot2(__builtin_bit_cast(us2, v23), row_lo, y[5], false);
        y[6] = __builtin_amdgcn_udot2(__builtin_bit_cast(us2, v23), row_hi, y[6], false);
      }
#pragma unroll
      for (int u = 0; u < kNbrRows; ++u)
        if (k0 + u >= W - 1 && k0 + u < T)
          best[k] = max(best[k], ((y[u] + y[u + 1] + y[u + 2] + y[u + 3]) << 8) | (uint32_t)(255 - (k0 + u - (W - 1))));
      st[k][0] = y[6] | y[5] << 19;
      st[k][1] = y[5] >> 13 | y[4] << 6;
    };
    if (!wide) {
      // two positions at a time without a branch between them, so that the
      // second's reads are in flight during the first's sums
      uint32_t s[MAXK][2], top = 0;
#pragma unroll
      for (int k = 0; k < MAXK; k += 2) {
        if (k * NT >= N) continue;
        if (full) {
          halves(k, s[k], true);
          halves(k + 1, s[k + 1], true);
        } else {
          halves(k, s[k], false);
          halves(k + 1, s[k + 1], false);
        }
        top = max(max(top, best[k]), best[k + 1]);
      }
      wide = __ballot(top >= 0xffff00u) != 0ull;
#pragma unroll
      for (int k = 0; k < MAXK; ++k) {
        if (wide) {
          const uint32_t y1 = hi16(st[k][0]), y2 = lo16(st[k][0]), y3 = lo16(st[k][1]) - y2;
          st[k][0] = y1 | y2 << 19;
          st[k][1] = y2 >> 13 | y3 << 6;
        } else {
          st[k][0] = s[k][0];
          st[k][1] = s[k][1];
        }
      }
    }
    if (wide) {
#pragma unroll
      for (int k = 0; k < MAXK; ++k)
        if (k * NT < N) exact(k);
    }
  }
  // hand the keys over to the lanes' pixel groups, the low-gain decisions by
  // their own bytes
#pragma unroll
  for (int k = 0; k < MAXK; ++k) {
    const int p = (int)threadIdx.x + k * NT;
    if (p < N) {
      keys[(uint32_t)c.lat[(size_t)p * kNbrCols + 6] & 0xffffu] = best[k];  // the pixel at position p
    }
  }
  if (stager) {
    uint64_t b = 0;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const uint32_t x = (m & 1) ? hi16(hmax[m >> 1]) : lo16(hmax[m >> 1]);
      b |= (uint64_t)(c.n_gain == 2 && (int)x >= c.hg_switch && q * 8 + m < N) << (8 * m);
    }
    *reinterpret_cast<uint64_t*>(low + q * 8) = b;
  }
  __syncthreads();
}

// The neighbour peak's keys of every pixel group: the scan, then the pixel's
// own W samples at its start on its selected gain give S.  Called by every
// thread of the block (contains barriers).
template <int PPL, int W, int NT, class Fn>
__device__ __forceinline__ void neighbour_event(const DevCam& c, __amdgpu_buffer_rsrc_t r,
                                                const uint16_t* __restrict__ ev, uint16_t* xrow, uint32_t* keys,
                                                uint8_t* low, Fn&& fn) {
  constexpr int MAXP = (kMaxPix + NT * PPL - 1) / (NT * PPL);
  const int N = c.n_pix, np = c.n_pix_pad, T = c.n_samp;
  const int npass = (N + NT * PPL - 1) / (NT * PPL);
  // staged words: slices k0, k0+1 in the low dword, k0+2, k0+3 in the high one
  nbr_scan<W, NT>(c, r, reinterpret_cast<uint64_t*>(xrow), keys, low);
#pragma unroll
  for (int ps = 0; ps < MAXP; ++ps) {
    if (ps >= npass) continue;
    const int pix0 = (ps * NT + (int)threadIdx.x) * PPL;
    uint32_t sw = 0, key[PPL];
#pragma unroll
    for (int p = 0; p < PPL; ++p) {
      const int i = pix0 + p;
      key[p] = 0;
      if (i >= N) continue;
      const int g = low[i], s = 255 - (int)(keys[i] & 255u);
      sw |= (uint32_t)g << p;
      const uint16_t* col = ev + ((size_t)g * T + s) * np + i;
      uint32_t S = 0;
#pragma unroll
      for (int u = 0; u < W; ++u) S += col[(size_t)u * np];
      key[p] = (S << 8) | (uint32_t)(255 - s);
    }
    fn(pix0, key, sw);
  }
}

// D = 256*S - w*P from the packed key.
template <int W>
__device__ __forceinline__ int32_t key_to_d(uint32_t key, int32_t P) {
  return (int32_t)(key & 0xFFFFFF00u) - W * P;
}

// Upper bounds for the neighbour peak: the sliding window's key on the high
// gain of every pixel group, and its low-gain bits.  With 8 pixels per lane in
// chunks of 8: chunks of 16 need 190 registers, or 316 bytes of scratch (8000
// events of the 1:3:6 mix 1172 us, 596 with chunks of 8).
//
// Where the night sky brings many pixels to the boundary level, the windows would
// cost more than a scan of every pixel, and the bounds would have read the trace
// for nothing.  Two pixels per lane of the first pass tell so after one chunk
// (the share of them with a window at the boundary level against c.nbr_noise), if
// LOOK: false is returned, with fn not called for any group.
template <int PPL, int W, int CH, int NT, bool LOOK, class Fn>
__device__ __forceinline__ bool bound_event(const DevCam& c, __amdgpu_buffer_rsrc_t r, uint32_t* seen, Fn&& fn) {
  constexpr int MAXP = (kMaxPix + NT * PPL - 1) / (NT * PPL), BCH = PPL == 8 ? 8 : CH;
  const int N = c.n_pix, np = c.n_pix_pad, T = c.n_samp;
  auto pass = [&](int ps, auto&& stop) {
    const int pix0 = (ps * NT + (int)threadIdx.x) * PPL;
    uint32_t key[PPL], rmax[PPL / 2];
#pragma unroll
    for (int h = 0; h < PPL / 2; ++h) rmax[h] = 0;
    if (!window_argmax<PPL, W, BCH, true>(r, (uint32_t)pix0 * 2u, 0u, (uint32_t)np * 2u, T, key, rmax, stop))
      return false;
    uint32_t sw = 0;
#pragma unroll
    for (int p = 0; p < PPL; ++p) {
      const uint32_t m = (p & 1) ? hi16(rmax[p >> 1]) : lo16(rmax[p >> 1]);
      if (c.n_gain == 2 && (int)m >= c.hg_switch) sw |= 1u << p;
    }
    fn(pix0, key, sw);
    return true;
  };
  const bool all = pass(0, [&](const uint32_t (&k)[PPL]) {
    if constexpr (!LOOK) return false;
    const int pix0 = (int)threadIdx.x * PPL, q0 = pix0 < N ? pix0 : 0;
    const int2 P = *reinterpret_cast<const int2*>(c.P256 + q0);
    const int2 Tb = *reinterpret_cast<const int2*>(c.thr_bnd + q0);
    const uint64_t in0 = __ballot(pix0 < N), in1 = __ballot(pix0 + 1 < N);
    const uint64_t at0 = __ballot(key_to_d<W>(k[0], P.x) >= Tb.x), at1 = __ballot(key_to_d<W>(k[1], P.y) >= Tb.y);
    if ((threadIdx.x & (kWave - 1)) == 0)
      seen[threadIdx.x / kWave] =
          (uint32_t)(__popcll(in0 & at0) + __popcll(in1 & at1)) | (uint32_t)(__popcll(in0) + __popcll(in1)) << 16;
    __syncthreads();
    uint32_t n = 0;
#pragma unroll
    for (int w = 0; w < NT / kWave; ++w) n += seen[w];
    return (float)(n & 0xffffu) > nbr_share(c.nbr_noise, BCH) * (float)(n >> 16);
  });
  if (!all) return false;
  if constexpr (MAXP > 1) {
    const int npass = (N + NT * PPL - 1) / (NT * PPL);
    for (int ps = 1; ps < npass; ++ps) pass(ps, [](const uint32_t (&)[PPL]) { return false; });
  }
  return true;
}

// Keys of every pixel of one event, group by group: fn(pix0, key, sw) for
// each of this thread's groups.  rows / start: LDS scratch of the global
// peak (NT/64 * 256 words, one word); xrow, low: LDS slices of the neighbour
// peak (kNbrRows * (kMaxPix + 8) halfwords) and a byte per pixel.  AHEAD: of
// the global peak's first stage.
template <int EX, int PPL, int W, int CH, int NT, bool AHEAD, class Fn>
__device__ __forceinline__ void extract_event(const DevCam& c, __amdgpu_buffer_rsrc_t r, const uint16_t* ev,
                                              uint32_t* rows, int32_t* start, uint16_t* xrow, uint8_t* low, Fn&& fn) {
  const int N = c.n_pix, np = c.n_pix_pad, T = c.n_samp;
  const bool dual = c.n_gain == 2;
  // Uniform pass loop: every lane streams (loads past the event read 0 from
  // the bounds-checked buffer); the callback guards its stores.
  const int npass = (N + NT * PPL - 1) / (NT * PPL);
  if constexpr (EX == kExSliding || EX == kExFixed) {
    for (int ps = 0; ps < npass; ++ps) {
      const int pix0 = (ps * NT + (int)threadIdx.x) * PPL;
      uint32_t key[PPL];
      uint32_t sw;
      if constexpr (EX == kExSliding)
        sw = extract_group<PPL, W, CH>(c, r, pix0, np, T, dual, key);
      else
        sw = fixed_group<PPL, W>(c, r, pix0, np, T, dual, key);
      fn(pix0, key, sw);
    }
  } else if constexpr (EX == kExNeighbour) {
    neighbour_event<PPL, W, NT>(c, r, ev, xrow, rows, low, fn);
  } else {
    constexpr int MAXP = (kMaxPix + NT * PPL - 1) / (NT * PPL);
    uint32_t* my_rows = rows + (threadIdx.x / kWave) * 256;
    uint32_t swp[MAXP];
#pragma unroll
    for (int ps = 0; ps < MAXP; ++ps) {
      swp[ps] = 0;
      if (ps < npass)
        swp[ps] = global_rows_group<PPL, CH, AHEAD>(c, r, (ps * NT + (int)threadIdx.x) * PPL, np, T, dual, my_rows,
                                             ps == 0);
    }
    __syncthreads();
    const int s = global_start<NT, W>(rows, T, start);
    const uint32_t stride = (uint32_t)np * 2u;
#pragma unroll
    for (int ps = 0; ps < MAXP; ++ps) {
      if (ps < npass) {
        const int pix0 = (ps * NT + (int)threadIdx.x) * PPL;
        const uint32_t voff = (uint32_t)pix0 * 2u;
        uint32_t S[PPL], unused[PPL / 2], key[PPL];
        window_at<PPL, W, false>(r, voff, 0u, stride, s, S, unused);
        keys_at<PPL, W>(r, voff, stride, T, s, S, swp[ps], key);
        fn(pix0, key, swp[ps]);
      }
    }
  }
}

// Time numerator Nt = sum_k k*(256*x[s+k] - P) and the in-window peak index
// from the window samples (re-read from the trace).
template <int W>
__device__ __forceinline__ int32_t window_nt(const uint16_t* __restrict__ col, int np, int s, int32_t P, int* peak) {
  int32_t nt = 0;
  uint32_t pmax = col[(size_t)s * np];
  int pk = s;
#pragma unroll
  for (int k = 1; k < W; ++k) {
    const uint32_t x = col[(size_t)(s + k) * np];
    nt += k * (256 * (int32_t)x - P);
    if (x > pmax) { pmax = x; pk = s + k; }
  }
  if (peak) *peak = pk;
  return nt;
}

// Peak time t = s* + Nt/D (window centre when D <= 0), evaluated in FP64.
template <int W>
__device__ __forceinline__ double peak_time(int s, int32_t nt, int32_t d) {
  return d > 0 ? (double)s + (double)nt / (double)d : (double)s + 0.5 * (double)(W - 1);
}

__device__ __forceinline__ uint32_t pixel_flag(const DevCam& c, int g, int i, int32_t d) {
  const int o = g * c.n_pix_pad + i;
  return (uint32_t)(d >= c.thr_bnd[o]) | ((uint32_t)(d >= c.thr_pic[o]) << 1);
}

// The same with given levels (p.e.): the thresholds ceil(256 a T) formed in
// FP64 in the order the camera creation forms its tables (256 a is exact,
// then one rounded product), so the levels the camera was made with give
// its tables' values.  The host bounds them to |.| <= 2e9.
__device__ __forceinline__ uint32_t pixel_flag_at(const DevCam& c, int g, int i, int32_t d, float t_pic,
                                                  float t_bnd) {
  const double a256 = 256.0 * (double)c.a[g * c.n_pix_pad + i];
  const int32_t tp = (int32_t)ceil(a256 * (double)t_pic), tb = (int32_t)ceil(a256 * (double)t_bnd);
  return (uint32_t)(d >= tb) | ((uint32_t)(d >= tp) << 1);
}

// ---------------------------------------------------------------------------
// Workgroup-shared state of one camera event: 16.5 KB, so that LDS has room for
// nine 256-thread workgroups on a compute unit, one more than its wavefronts
// allow (it was 32.3 KB, five, while every mask pixel had its packed charge and
// time here; the fixed window, bound by how many telescopes are in flight, runs
// by it).
// ---------------------------------------------------------------------------
// One mask pixel of a small image, as the lane that found it leaves it for
// wavefront 0.
struct SmallSlot {
  int32_t d, nt;   // D and Nt of its window
  float a, x, y;   // ADC per p.e., position
  uint32_t s;      // window start | border << 8
};

struct TelSmem {
  union {
    uint32_t key[kMaxPix];   // (S << 8) | (255 - s*) per pixel; reused as union-find parents
    uint32_t rows[kMaxPix];  // global peak: per-wave slice sums; neighbour peak: key hand-over (extraction only)
  };
  uint8_t flag[kMaxPix];     // bit 0: D >= Tb, bit 1: D >= Tp, bit 2: low gain
  uint64_t mbits[kMaxWords]; // cleaning mask, one word per 64 pixels
  int32_t wbase[kMaxWords];  // slot of each word's first mask pixel
  int32_t nlow_w[16];        // per-wave counts of low-gain pixels
  int32_t start;             // global peak window start
  alignas(16) uint16_t list[kMaxPix];  // flagged pixels, a run per wavefront; then slot -> pixel (large images)
  union {
    struct {
      SmallSlot slot[kWave];
      unsigned long long adj[kWave];  // slots adjacent to each slot
    } small;
    double red[16 * 8];      // cross-wave reduction scratch (large images)
    uint16_t ask[kNbrAsk];   // neighbour peak: pixels whose windows are wanted
  };
};

static_assert(sizeof(uint16_t) * kNbrAsk <= sizeof(SmallSlot) * kWave + 8 * kWave, "the list overlays the small slots");
// The neighbour peak's workgroup: its staged slices or traces and their
// pixels beside the rest.
constexpr int kXrow = kNbrRows * (kMaxPix + 8);
static_assert(kXrow / (kNbrStage + 1) >= 12, "eight slices of every staged trace fit");
struct NbrSmem {
  TelSmem tel;
  alignas(16) uint16_t xrow[kXrow];
  uint16_t px[kMaxPix];  // pixels whose traces are staged
  uint32_t seen[16];     // per wavefront: probed pixels << 16 | those at the boundary level
};
template <int EX>
constexpr size_t smem_bytes() {
  return EX == kExNeighbour ? sizeof(NbrSmem) : sizeof(TelSmem);
}

// Butterfly sum of a 32-bit or 64-bit value over the wavefront: every lane
// gets the sum over the pairing tree (i, i ^ 32), (i, i ^ 16), ... (i, i ^ 1).
// The exchanges are register moves, none through LDS: the halves and rows
// by the lane swaps (a swap of a register with its copy leaves the two
// partners of every lane in the two results), then within a row of 16 a
// rotation by 8, a rotation by 4 (the values already agree under i ^ 8, so
// lane i + 4 holds what lane i ^ 4 does) and quad permutes.  A dependent
// step costs a few cycles where an LDS permute costs over a hundred; the
// three reductions of an image went from 1.4 us to 0.3 us.
template <int STEP, typename T>
__device__ __forceinline__ T butterfly_step(T v) {
  if constexpr (sizeof(T) == 4) {
    uint32_t a, b;
    partner_u32<STEP>(__builtin_bit_cast(uint32_t, v), &a, &b);
    return __builtin_bit_cast(T, a) + __builtin_bit_cast(T, b);
  } else {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    uint32_t al, bl, ah, bh;
    partner_u32<STEP>((uint32_t)u, &al, &bl);
    partner_u32<STEP>((uint32_t)(u >> 32), &ah, &bh);
    return __builtin_bit_cast(T, ((uint64_t)ah << 32) | al) + __builtin_bit_cast(T, ((uint64_t)bh << 32) | bl);
  }
}

template <typename T, int NV>
__device__ __forceinline__ void butterfly(T (&v)[NV]) {
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = butterfly_step<32>(v[k]);
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = butterfly_step<16>(v[k]);
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = butterfly_step<8>(v[k]);
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = butterfly_step<4>(v[k]);
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = butterfly_step<2>(v[k]);
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = butterfly_step<1>(v[k]);
}

template <typename T, int NV, int NT>
__device__ __forceinline__ void block_sum(T (&v)[NV], double* red_raw) {
  T* red = reinterpret_cast<T*>(red_raw);
  constexpr int NW = NT / kWave;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  butterfly(v);
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < NV; ++k) red[wave * NV + k] = v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    T s = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) s += red[w * NV + k];
    v[k] = s;
  }
  __syncthreads();
}

// The same sums over one wavefront (the other wavefronts hold nothing): the
// butterfly of block_sum, then its cross-wave sum, here 0 + the wave's sum.
template <typename T, int NV>
__device__ __forceinline__ void wave_sum(T (&v)[NV]) {
  butterfly(v);
#pragma unroll
  for (int k = 0; k < NV; ++k) v[k] = T(0) + v[k];
}

// Workgroup total of the wavefronts' low-gain counts (sm.nlow_w, behind a barrier).
template <int NT>
__device__ __forceinline__ int total_count(const TelSmem& sm) {
  int s = 0;
#pragma unroll
  for (int w = 0; w < NT / kWave; ++w) s += sm.nlow_w[w];
  return s;
}

__device__ __forceinline__ bool mask_bit(const TelSmem& sm, int i) { return (sm.mbits[i >> 6] >> (i & 63)) & 1ull; }

// Slot of mask pixel i (after scan_phase).
__device__ __forceinline__ int mask_slot(const TelSmem& sm, int i) {
  const uint64_t w = sm.mbits[i >> 6];
  return sm.wbase[i >> 6] + __popcll(w & ((1ull << (i & 63)) - 1ull));
}

template <int PPL>
__device__ __forceinline__ void store_keys(uint32_t* dst, const uint32_t (&key)[PPL]) {
  if constexpr (PPL == 2) {
    *reinterpret_cast<u32x2*>(dst) = u32x2{key[0], key[1]};
  } else {
#pragma unroll
    for (int p = 0; p < PPL; p += 4)
      *reinterpret_cast<u32x4*>(dst + p) = u32x4{key[p], key[p + 1], key[p + 2], key[p + 3]};
  }
}

template <int PPL>
__device__ __forceinline__ void store_flags(uint8_t* dst, uint64_t fl) {
  if constexpr (PPL == 8)
    *reinterpret_cast<uint64_t*>(dst) = fl;
  else if constexpr (PPL == 4)
    *reinterpret_cast<uint32_t*>(dst) = (uint32_t)fl;
  else
    *reinterpret_cast<uint16_t*>(dst) = (uint16_t)fl;
}

// Phase 1 (fused): extraction of all pixels into LDS: keys, flags, and each
// wavefront's run of flagged pixels (D >= the boundary or the picture
// threshold: the only pixels that can enter the mask) with their number
// returned.  A group's keys and flags are stored whole: the padding pixels
// of the last group get flags 0 (their thresholds are the largest int32).
// BOUND: the windows are upper bounds of the pixels' sums, and a low-gain
// pixel, whose sum they do not bound, counts as at both thresholds; -1 in every
// wavefront if they are given up.
template <int EX, int PPL, int W, int CH, int NT, bool BOUND, bool LOOK = false>
__device__ __forceinline__ int extract_phase(const DevCam& c, const uint16_t* __restrict__ ev, TelSmem& sm,
                                             uint16_t* xrow, uint32_t* seen = nullptr) {
  static_assert(kRunWave == kWave && kMaxPix % run_length(kMaxPix, NT, PPL) == 0, "whole runs fill the list");
  const int N = c.n_pix, np = c.n_pix_pad;
  const int wave = threadIdx.x / kWave;
  const __amdgpu_buffer_rsrc_t r = event_rsrc(ev, c.event_elems);
  uint16_t* cand = sm.list + run_begin(kMaxPix, NT, PPL, wave);
  int ncand = 0, nlow = 0;
  if (threadIdx.x < kMaxWords) sm.mbits[threadIdx.x] = 0ull;
  auto take = [&](int pix0, const uint32_t (&key)[PPL], uint32_t sw) {
    const bool mine = pix0 < N;
    const int q0 = mine ? pix0 : 0;
    int32_t P[PPL], Tb[PPL], Tp[PPL];
    load_i32<PPL>(P, c.P256 + q0);
    load_i32<PPL>(Tb, c.thr_bnd + q0);
    load_i32<PPL>(Tp, c.thr_pic + q0);
    uint64_t fl = 0;  // one flag byte per pixel
#pragma unroll
    for (int p = 0; p < PPL; ++p) {
      const int g = mine ? (int)((sw >> p) & 1u) : 0;
      int32_t Pv = P[p], tb = Tb[p], tp = Tp[p];
      if (g) { Pv = c.P256[np + q0 + p]; tb = c.thr_bnd[np + q0 + p]; tp = c.thr_pic[np + q0 + p]; }
      const int32_t d = key_to_d<W>(key[p], Pv);
      const uint32_t f = BOUND && g ? 3u : (uint32_t)(d >= tb) | ((uint32_t)(d >= tp) << 1);
      fl |= (uint64_t)(f | ((uint32_t)g << 2)) << (8 * p);
      const uint64_t has = __ballot(mine && f != 0u);
      if (mine && f != 0u)
        cand[ncand + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(has >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)has, 0u))] =
            (uint16_t)(q0 + p);
      ncand += __popcll(has);
      if (__ballot(g != 0)) nlow += __popcll(__ballot(g != 0 && q0 + p < N));
    }
    if (mine) {
      store_keys<PPL>(sm.key + pix0, key);
      store_flags<PPL>(sm.flag + pix0, fl);
    }
  };
  if constexpr (BOUND) {
    if (!bound_event<PPL, W, CH, NT, LOOK>(c, r, seen, take)) return -1;
  } else
    extract_event<EX, PPL, W, CH, NT, true>(c, r, ev, sm.rows, &sm.start, xrow, sm.flag, take);
  if ((threadIdx.x & (kWave - 1)) == 0) sm.nlow_w[wave] = nlow;
  return ncand;
}

// Whether a pixel with own flags f and neighbour row nv enters the mask.
__device__ __forceinline__ bool passes(const TelSmem& sm, uint32_t f, const int4& nv) {
  const int32_t nb2[3] = {nv.x, nv.y, nv.z};
  uint32_t any = 0;
#pragma unroll
  for (int h = 0; h < 3; ++h) {
    const int j0 = (int16_t)nb2[h], j1 = nb2[h] >> 16;
    if (j0 >= 0) any |= sm.flag[j0];
    if (j1 >= 0) any |= sm.flag[j1];
  }
  return ((f & 1u) && (any & 2u)) || ((f & 2u) && (any & 1u));
}

__device__ __forceinline__ int4 neighbour_row(const DevCam& c, int i) {
  return *reinterpret_cast<const int4*>(c.nbr + (size_t)i * kNbrCols);
}

// Mask words from given flags of all pixels (unfused cleaning).
template <int NT>
__device__ __forceinline__ void mask_phase(const DevCam& c, TelSmem& sm) {
  const int N = c.n_pix, nw = (N + 63) >> 6;
  const int lane = threadIdx.x & (kWave - 1);
  for (int base = threadIdx.x & ~(kWave - 1); base < nw * kWave; base += NT) {
    const int i = base + lane;
    const uint32_t f = i < N ? sm.flag[i] & 3u : 0u;
    bool m = false;
    if (f) m = passes(sm, f, neighbour_row(c, i));
    const uint64_t b = __ballot(m);
    if (lane == 0) sm.mbits[base >> 6] = b;
  }
}

// Exclusive prefix of the mask-word popcounts, by every wavefront for itself
// (no barrier): lane w returns the base slot of word w, total the number of
// mask pixels.  Every wavefront also writes the same bases to sm.wbase, for
// its own lookups at any word.
__device__ __forceinline__ int scan_phase(int N, TelSmem& sm, int* total) {
  const int nw = (N + 63) >> 6;
  const int lane = threadIdx.x & (kWave - 1);
  const int cnt = lane < nw ? __popcll(sm.mbits[lane]) : 0;
  int inc = cnt;  // inclusive prefix by lane moves: within rows of 16, then across them
  inc += __builtin_amdgcn_update_dpp(0, inc, 0x111, 0xF, 0xF, false);  // row_shr:1
  inc += __builtin_amdgcn_update_dpp(0, inc, 0x112, 0xF, 0xF, false);  // row_shr:2
  inc += __builtin_amdgcn_update_dpp(0, inc, 0x114, 0xF, 0xF, false);  // row_shr:4
  inc += __builtin_amdgcn_update_dpp(0, inc, 0x118, 0xF, 0xF, false);  // row_shr:8
  inc += __builtin_amdgcn_update_dpp(0, inc, 0x142, 0xA, 0xF, false);  // row_bcast:15
  inc += __builtin_amdgcn_update_dpp(0, inc, 0x143, 0xC, 0xF, false);  // row_bcast:31
  static_assert(kMaxWords <= kWave, "one mask word per lane");
  if (lane < nw) sm.wbase[lane] = inc - cnt;
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  *total = __builtin_amdgcn_readlane(inc, kWave - 1);
  return inc - cnt;
}

// What the Hillas passes take of one mask pixel.
struct Slot {
  float q, x, y;
  double t;
  bool border;
};

// Charge and peak time of a mask pixel from its window key and a re-read of
// its window samples.  load asks for everything, finish forms the values, so
// that other work can stand between them.
template <int W>
struct FusedSource {
  const uint16_t* __restrict__ ev;
  struct Raw {
    uint32_t key;
    int32_t P;
    float a;
    uint32_t x[W];
  };
  __device__ __forceinline__ Raw load(const DevCam& c, const TelSmem& sm, int i) const {
    const int np = c.n_pix_pad;
    Raw r;
    r.key = sm.key[i];
    const int g = (int)(sm.flag[i] >> 2), s0 = 255 - (int)(r.key & 255u);
    r.P = c.P256[g * np + i];
    r.a = c.a[g * np + i];
    const uint16_t* col = ev + ((size_t)g * c.n_samp + s0) * np + i;
#pragma unroll
    for (int u = 0; u < W; ++u) r.x[u] = col[(size_t)u * np];
    return r;
  }
  static __device__ __forceinline__ void finish(const Raw& r, Slot& s) {
    const int32_t d = key_to_d<W>(r.key, r.P);
    int32_t nt = 0;
#pragma unroll
    for (int u = 1; u < W; ++u) nt += u * (256 * (int32_t)r.x[u] - r.P);
    s.q = (float)d / (256.0f * r.a);
    s.t = peak_time<W>(255 - (int)(r.key & 255u), nt, d);
  }
};

// The same from given charges (or D and gain: D / (256 a) formed as the
// calibration forms q) and times of this event.
struct GivenSource {
  const float* __restrict__ q;
  const int32_t* __restrict__ D;
  const uint8_t* __restrict__ gain;
  const float* __restrict__ t;
  struct Raw {
    float q, t;
  };
  __device__ __forceinline__ Raw load(const DevCam& c, const TelSmem&, int i) const {
    Raw r;
    r.q = q ? q[i] : (float)D[i] / (256.0f * c.a[(gain ? (int)gain[i] : 0) * c.n_pix_pad + i]);
    r.t = t[i];
    return r;
  }
  static __device__ __forceinline__ void finish(const Raw& r, Slot& s) {
    s.q = r.q;
    s.t = (double)r.t;
  }
};

__device__ __forceinline__ void load_place(const DevCam& c, int i, Slot& s) {
  s.x = c.x[i];
  s.y = c.y[i];
  s.border = c.border[i] != 0;
}

template <class Src>
__device__ __forceinline__ Slot load_slot(const DevCam& c, const TelSmem& sm, int i, const Src& src) {
  Slot s;
  load_place(c, i, s);
  Src::finish(src.load(c, sm, i), s);
  return s;
}

// Islands of an image of at most 64 mask pixels by one wavefront: adj holds
// the slots adjacent to the lane's slot, symmetric over the lanes.  The
// islands one after another by flood fill on the wave-uniform slot set: a
// lane joins when its mask meets the set.  One step is a handful of
// instructions without a memory access; the steps are at most the slots
// plus the islands.  (A union-find over LDS took 2.3-7 us of a telescope's
// chain of 13 us after the extraction, its finds and compare-and-swaps each
// an LDS round trip; this takes 0.2-0.6 us.)
__device__ __forceinline__ int wave_islands(int n, uint64_t adj) {
  uint64_t todo = n == kWave ? ~0ull : (1ull << n) - 1ull;
  int roots = 0;
  while (todo) {
    uint64_t comp = todo & (0ull - todo);
    for (;;) {
      const uint64_t next = comp | __ballot((adj & comp) != 0ull);
      if (next == comp) break;
      comp = next;
    }
    todo &= ~comp;
    ++roots;
  }
  return roots;
}

// Enters the edges of slot j (pixel i, neighbour row nv) into sm.small.adj
// (cleared before): each edge is taken from the row of its smaller pixel, as
// in islands_phase, and entered at both ends.
__device__ __forceinline__ void enter_edges(TelSmem& sm, int j, int i, const int4& nv) {
  const int32_t nb2[3] = {nv.x, nv.y, nv.z};
  unsigned long long own = 0;
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const int m = (k & 1) ? nb2[k >> 1] >> 16 : (int)(int16_t)nb2[k >> 1];
    if (m > i && mask_bit(sm, m)) {
      const int s = mask_slot(sm, m);
      own |= 1ull << s;
      atomicOr(&sm.small.adj[s], 1ull << j);
    }
  }
  if (own) atomicOr(&sm.small.adj[j], own);
}

__device__ __forceinline__ int uf_find(volatile int32_t* par, int x) {
  int p = par[x];
  while (p != x) {
    x = p;
    p = par[x];
  }
  return x;
}

// Hooks the larger root under the smaller; a root changes only by a CAS from
// itself to a smaller index, so parents strictly decrease and find ends.
__device__ __forceinline__ void uf_union(int32_t* par, int a, int b) {
  volatile int32_t* vp = par;
  for (;;) {
    a = uf_find(vp, a);
    b = uf_find(vp, b);
    if (a == b) return;
    if (a < b) { const int t = a; a = b; b = t; }
    if (atomicCAS(&par[a], a, b) == a) return;
  }
}

// Islands of an image of more than 64 mask pixels: roots of the union-find
// forest over mask slots.  Returns this thread's root count.  The per-pixel
// keys (no longer needed: a barrier lies behind their last use) hold the
// parents.  A first pass hooks every slot under the smallest slot with an
// edge to it (an edge is taken from the row of its smaller pixel) by atomic
// minima, without finds, and two jumps shorten the chains, so that few edges
// are left to the finds and compare-and-swaps of the unions.
template <int NT>
__device__ __forceinline__ int islands_phase(const DevCam& c, TelSmem& sm, int n) {
  int32_t* par = reinterpret_cast<int32_t*>(sm.key);
  auto each_edge = [&](int j, auto&& fn) {  // fn(slot of the larger pixel)
    const int i = sm.list[j];
    const int4 nv = neighbour_row(c, i);
    const int32_t nb2[3] = {nv.x, nv.y, nv.z};
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      const int m = (k & 1) ? nb2[k >> 1] >> 16 : (int)(int16_t)nb2[k >> 1];
      if (m > i && mask_bit(sm, m)) fn(mask_slot(sm, m));
    }
  };
  for (int j = threadIdx.x; j < n; j += NT) par[j] = j;
  __syncthreads();
  for (int j = threadIdx.x; j < n; j += NT) each_edge(j, [&](int m) { atomicMin(&par[m], j); });
  __syncthreads();
  volatile int32_t* vp = par;
#pragma unroll
  for (int k = 0; k < 2; ++k)  // an ancestor is replaced by an ancestor of it: any interleaving is valid
    for (int j = threadIdx.x; j < n; j += NT) vp[j] = vp[vp[j]];
  __syncthreads();
  for (int j = threadIdx.x; j < n; j += NT)
    each_edge(j, [&](int m) {
      if (vp[j] != vp[m]) uf_union(par, j, m);
    });
  __syncthreads();
  int roots = 0;
  for (int j = threadIdx.x; j < n; j += NT) roots += (vp[j] == j);
  return roots;
}

// Hillas reductions and the record (its island count is filled in by the
// caller).  each(fn) calls fn(slot) for every mask pixel of this thread, in
// the same order each time; l0_of(fn) returns fn(x, y) of slot 0.  WAVE:
// wavefront 0 alone holds pixels.
// Centre of gravity and second moments are FP32 sums of centred terms.  The
// third pass takes the longitudinal and transverse coordinates l, w in the
// rotated frame: skewness and kurtosis from q l^3, q l^4, the width from the
// minor-axis moment q w^2 (exact for collinear pixels, unlike
// sqrt(det / l+), which keeps only half the digits when the width is small),
// and the time regression from the FP64 sums of l, l^2, t and l t (times are
// absolute sample numbers, so FP32 would cancel most digits of small time
// gradients; in FP64 the centring cancels about t / spread(t) x mean(l) /
// spread(l) digits, harmless).
template <int NT, bool WAVE, class Each, class L0>
__device__ __forceinline__ rta_hillas_rec hillas_phase(TelSmem& sm, int n, int nlow, Each&& each, L0&& l0_of) {
  float v1[4] = {0.f, 0.f, 0.f, 0.f};
  each([&](const Slot& s) {
    v1[0] += s.q;
    v1[1] += s.q * s.x;
    v1[2] += s.q * s.y;
    if (s.border) v1[3] += s.q;
  });
  if constexpr (WAVE)
    wave_sum(v1);
  else
    block_sum<float, 4, NT>(v1, sm.red);
  const float S = v1[0];
  rta_hillas_rec r;
  r.size = S;
  r.n_pix = n;
  r.n_islands = 0;
  r.n_lowgain = nlow;
  r.flags = r.n_lowgain > 0 ? RTA_FLAG_LOW_GAIN : 0u;
  if (n < 2 || !(S > 0.f)) {
    r.cog_x = r.cog_y = r.length = r.width = r.psi = r.skewness = r.kurtosis = kNaN;
    r.time_gradient = r.time_intercept = r.leakage = r.cog_dist = kNaN;
    r.flags |= RTA_FLAG_HILLAS_INVALID | RTA_FLAG_TIME_INVALID;
    return r;
  }
  const float xm = v1[1] / S, ym = v1[2] / S;
  float v2[3] = {0.f, 0.f, 0.f};
  each([&](const Slot& s) {
    const float q = s.q, dx = s.x - xm, dy = s.y - ym;
    v2[0] += q * dx * dx;
    v2[1] += q * dy * dy;
    v2[2] += q * dx * dy;
  });
  if constexpr (WAVE)
    wave_sum(v2);
  else
    block_sum<float, 3, NT>(v2, sm.red);
  const float sxx = v2[0] / S, syy = v2[1] / S, sxy = v2[2] / S;
  const float hd = 0.5f * (sxx - syy);
  const float lp = 0.5f * (sxx + syy) + sqrtf(hd * hd + sxy * sxy);
  float psi = 0.5f * atan2f(2.0f * sxy, sxx - syy);
  if (psi <= -0.5f * (float)M_PI) psi += (float)M_PI;
  const float len = sqrtf(lp);
  const float cs = cosf(psi), sn = sinf(psi);
  // l of slot 0: every l equal to it (fewer than two distinct l) leaves the
  // time gradient undefined
  const float l0 = l0_of([&](float x, float y) { return (x - xm) * cs + (y - ym) * sn; });
  // q l^3, q l^4, q w^2, l, l^2, t, l t, |l - l0|
  double v3[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  each([&](const Slot& s) {
    const float q = s.q, dx = s.x - xm, dy = s.y - ym;
    const float l = dx * cs + dy * sn;
    const float w = dy * cs - dx * sn;
    const float l2 = l * l;
    v3[0] += (double)(q * l2 * l);
    v3[1] += (double)(q * l2 * l2);
    v3[2] += (double)(q * w * w);
    const double ld = (double)l, td = s.t;
    v3[3] += ld;
    v3[4] += ld * ld;
    v3[5] += td;
    v3[6] += ld * td;
    v3[7] += fabs(ld - (double)l0);
  });
  if constexpr (WAVE)
    wave_sum(v3);
  else
    block_sum<double, 8, NT>(v3, sm.red);
  const double nd = (double)n, lbar = v3[3] / nd, tbar = v3[5] / nd;
  const double sll = v3[4] - v3[3] * lbar, slt = v3[6] - v3[3] * tbar;
  r.cog_x = xm;
  r.cog_y = ym;
  r.length = len;
  r.width = sqrtf(fmaxf((float)v3[2] / S, 0.f));
  r.psi = psi;
  const float len3 = len * len * len;
  r.skewness = (float)v3[0] / (S * len3);
  r.kurtosis = (float)v3[1] / (S * len3 * len);
  r.leakage = v1[3] / S;
  r.cog_dist = sqrtf(xm * xm + ym * ym);
  if (v3[7] > 0.0 && sll > 0.0) {
    const double g = slt / sll;
    r.time_gradient = (float)g;
    r.time_intercept = (float)(tbar - g * lbar);
  } else {
    r.time_gradient = r.time_intercept = kNaN;
    r.flags |= RTA_FLAG_TIME_INVALID;
  }
  return r;
}

// Islands and Hillas of an image of 1 to 64 mask pixels by wavefront 0, slot
// j in lane j: the slot stays in registers through the three Hillas passes.
// The sums are the block's bit for bit, where the other wavefronts would
// contribute exact zeros.
template <int NT>
__device__ __forceinline__ rta_hillas_rec small_image(TelSmem& sm, int n, int nlow, const Slot& s, uint64_t adj) {
  const int lane = threadIdx.x & (kWave - 1);
  const int roots = wave_islands(n, adj);
  rta_hillas_rec r = hillas_phase<NT, true>(
      sm, n, nlow,
      [&](auto&& fn) {
        if (lane < n) fn(s);
      },
      [&](auto&& fn) {
        return fn(__int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(s.x))),
                  __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(s.y))));
      });
  r.n_islands = roots;
  return r;
}

__device__ __forceinline__ rta_hillas_rec empty_image(int nlow) {
  rta_hillas_rec r;
  r.size = 0.f;
  r.cog_x = r.cog_y = r.length = r.width = r.psi = r.skewness = r.kurtosis = kNaN;
  r.time_gradient = r.time_intercept = r.leakage = r.cog_dist = kNaN;
  r.n_pix = 0;
  r.n_islands = 0;
  r.n_lowgain = nlow;
  r.flags = (nlow > 0 ? RTA_FLAG_LOW_GAIN : 0u) | RTA_FLAG_HILLAS_INVALID | RTA_FLAG_TIME_INVALID;
  return r;
}

// Hillas and islands of an image of more than 64 mask pixels by all threads:
// the slot list from the mask words, the first slot of every thread kept in
// registers through the passes (further ones, in images of more than NT mask
// pixels, formed again in each).  With one slot per thread the islands are
// found while the slots' loads are in flight; otherwise after the passes,
// whose slots need the keys that the union-find overwrites.  Such images are
// the last to end in a small batch: one array event 33.1 -> 30.5 us with
// both, 8000 fixed-window events of the mix 59.2 -> 56.4.
template <int NT, class Src>
__device__ __forceinline__ rta_hillas_rec large_image(const DevCam& c, TelSmem& sm, int wbase, int n, int nlow,
                                                      const Src& src) {
  const int nw = (c.n_pix + 63) >> 6;
  const int lane = threadIdx.x & (kWave - 1);
  for (int w = threadIdx.x / kWave; w < nw; w += NT / kWave) {
    const uint64_t bits = sm.mbits[w];
    const int first = __builtin_amdgcn_readlane(wbase, __builtin_amdgcn_readfirstlane(w));
    if ((bits >> lane) & 1ull) sm.list[first + __popcll(bits & ((1ull << lane) - 1ull))] = (uint16_t)((w << 6) | lane);
  }
  __syncthreads();
  const bool mine = (int)threadIdx.x < n;
  const int i0 = sm.list[mine ? (int)threadIdx.x : 0];
  Slot own;
  load_place(c, i0, own);
  const typename Src::Raw raw = src.load(c, sm, i0);
  int32_t roots[1] = {0};
  if (n <= NT) {
    __syncthreads();  // every thread has its key
    roots[0] = islands_phase<NT>(c, sm, n);
  }
  Src::finish(raw, own);
  rta_hillas_rec r = hillas_phase<NT, false>(
      sm, n, nlow,
      [&](auto&& fn) {
        if (mine) fn(own);
        for (int j = (int)threadIdx.x + NT; j < n; j += NT) fn(load_slot(c, sm, sm.list[j], src));
      },
      [&](auto&& fn) {
        const int i = sm.list[0];
        return fn(c.x[i], c.y[i]);
      });
  if (n > NT) roots[0] = islands_phase<NT>(c, sm, n);
  block_sum<int32_t, 1, NT>(roots, sm.red);
  r.n_islands = roots[0];
  return r;
}

// Mask, image list, islands and Hillas of an extracted event.  Only flagged
// pixels can be mask pixels, and they are few, so each wavefront works on its
// run of them, one per lane (a wavefront with more than 64 takes further
// rounds): neighbour rows loaded while other wavefronts still extract, the
// mask decided by the neighbours' flags and entered in the mask words; the
// loads that a mask pixel needs later (position, gain, window samples)
// issued at once, in flight across the barrier and the prefix sum over the
// mask words.  In an image of at most 64 mask pixels (95 % of the throughput
// mix) every pixel's lane then writes its slot and edges, and wavefront 0
// ends alone; the other wavefronts return an unused record.
template <int PPL, int NT, int W>
__device__ __forceinline__ rta_hillas_rec fused_image(const DevCam& c, TelSmem& sm, int ncand,
                                                      const uint16_t* __restrict__ ev) {
  const int np = c.n_pix_pad, lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const uint16_t* cand = sm.list + run_begin(kMaxPix, NT, PPL, wave);
  uint32_t* m32 = reinterpret_cast<uint32_t*>(sm.mbits);
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  const bool has = lane < ncand;
  const int i = has ? cand[lane] : 0;
  const uint32_t f = has ? sm.flag[i] : 0u;
  int4 nv = make_int4(-1, -1, -1, -1);
  if (has) nv = neighbour_row(c, i);
  __syncthreads();
  if (threadIdx.x < kWave) sm.small.adj[lane] = 0ull;
  bool in = false;
  if (has) in = passes(sm, f, nv);
  SmallSlot s;
  int32_t P = 0;
  uint32_t key = 0, x[W];
  if (in) {
    atomicOr(&m32[i >> 5], 1u << (i & 31));
    const int g = (int)(f >> 2);
    key = sm.key[i];
    P = c.P256[g * np + i];
    s.a = c.a[g * np + i];
    s.x = c.x[i];
    s.y = c.y[i];
    s.s = (255u - (key & 255u)) | ((uint32_t)c.border[i] << 8);
    const uint16_t* col = ev + ((size_t)g * c.n_samp + (255u - (key & 255u))) * np + i;
#pragma unroll
    for (int u = 0; u < W; ++u) x[u] = col[(size_t)u * np];
  }
  for (int b = kWave; b < ncand; b += kWave) {
    const int j = b + lane;
    if (j < ncand) {
      const int i2 = cand[j];
      if (passes(sm, sm.flag[i2], neighbour_row(c, i2))) atomicOr(&m32[i2 >> 5], 1u << (i2 & 31));
    }
  }
  __syncthreads();
  const int nlow = total_count<NT>(sm);
  int n;
  const int wbase = scan_phase(c.n_pix, sm, &n);
  if (n > kWave) return large_image<NT>(c, sm, wbase, n, nlow, FusedSource<W>{ev});
  if (n == 0) return empty_image(nlow);
  if (in) {
    const int j = mask_slot(sm, i);
    s.d = key_to_d<W>(key, P);
    s.nt = 0;
#pragma unroll
    for (int u = 1; u < W; ++u) s.nt += u * (256 * (int32_t)x[u] - P);
    sm.small.slot[j] = s;
    enter_edges(sm, j, i, nv);
  }
  for (int b = kWave; b < ncand; b += kWave) {
    const int j2 = b + lane;
    const int i2 = j2 < ncand ? cand[j2] : 0;
    const bool in2 = j2 < ncand && mask_bit(sm, i2);
    if (in2) {
      const int g = (int)(sm.flag[i2] >> 2), j = mask_slot(sm, i2);
      const uint32_t k2 = sm.key[i2];
      const int s0 = 255 - (int)(k2 & 255u);
      const int32_t P2 = c.P256[g * np + i2];
      SmallSlot t;
      t.d = key_to_d<W>(k2, P2);
      t.nt = window_nt<W>(ev + (size_t)g * c.n_samp * np + i2, np, s0, P2, nullptr);
      t.a = c.a[g * np + i2];
      t.x = c.x[i2];
      t.y = c.y[i2];
      t.s = (uint32_t)s0 | ((uint32_t)c.border[i2] << 8);
      sm.small.slot[j] = t;
      enter_edges(sm, j, i2, neighbour_row(c, i2));
    }
  }
  __syncthreads();
  if (threadIdx.x >= kWave) return rta_hillas_rec{};
  const SmallSlot t = sm.small.slot[min(lane, n - 1)];
  Slot h;
  h.q = (float)t.d / (256.0f * t.a);
  h.x = t.x;
  h.y = t.y;
  h.t = peak_time<W>((int)(t.s & 255u), t.nt, t.d);
  h.border = (t.s >> 8) != 0u;
  return small_image<NT>(sm, n, nlow, h, sm.small.adj[lane]);
}

// The same from given mask words (behind a barrier), charges and times.
template <int NT>
__device__ __forceinline__ rta_hillas_rec given_image(const DevCam& c, TelSmem& sm, int nlow, const GivenSource& src) {
  const int lane = threadIdx.x & (kWave - 1);
  int n;
  const int wbase = scan_phase(c.n_pix, sm, &n);
  if (n > kWave) return large_image<NT>(c, sm, wbase, n, nlow, src);
  if (threadIdx.x >= kWave) return rta_hillas_rec{};
  if (n == 0) return empty_image(nlow);
  sm.small.adj[lane] = 0ull;
  uint64_t words = __ballot(lane < ((c.n_pix + 63) >> 6) && sm.mbits[lane & (kMaxWords - 1)] != 0ull);
  while (words) {
    const int w = __builtin_ctzll(words);
    words &= words - 1ull;
    const uint64_t bits = sm.mbits[w];
    if ((bits >> lane) & 1ull)
      sm.list[__builtin_amdgcn_readlane(wbase, w) + __popcll(bits & ((1ull << lane) - 1ull))] =
          (uint16_t)((w << 6) | lane);
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  const int i = sm.list[min(lane, n - 1)];
  const int4 nv = neighbour_row(c, i);
  const Slot s = load_slot(c, sm, i, src);
  if (lane < n) enter_edges(sm, lane, i, nv);
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  return small_image<NT>(sm, n, nlow, s, ((volatile unsigned long long*)sm.small.adj)[lane]);
}

// Neighbour peak windows of the pixels that can matter, after the bounds
// (sm.key, sm.flag and the wavefronts' runs of flagged pixels hold those).
// The mask of the bounds' flags contains the image's mask, and the image's
// mask looks only at the flags of its pixels and of the neighbours they
// list; those pixels, usually few more than the image, are asked, and all
// other flags are cleared.  The traces of the asked pixels and of their
// neighbours are staged in LDS, as many slices at once as fit (the whole
// trace of 128 slices for 60 pixels): lanes on pixels, which share cache
// lines within a slice.  (A wavefront per asked pixel with lanes on slices
// took a line per lane and load, 130 us for an image of 33 pixels.)  Then a
// lane has an asked pixel, each wavefront a part of the windows.  8000
// events of the 1:3:6 mix: 1123 us with the full scan of every pixel (six
// 8-byte LDS reads and some 50 vector instructions per pixel and four
// slices), 592 us so, at 6.5 TB/s for the trace once and the asked pixels'
// cache lines a second time (3.84 GB fetched for 2.85 GB of trace).  Returns false if
// more than c.nbr_most traces are needed, or more than fit: every pixel is then
// scanned, from the start.  none: set when no pixel is asked.
template <int PPL, int NT, int W>
__device__ __forceinline__ bool nbr_windows(const DevCam& c, NbrSmem& nm, int ncand, const uint16_t* __restrict__ ev,
                                            bool* none) {
  TelSmem& sm = nm.tel;
  constexpr int NW = NT / kWave;
  const int np = c.n_pix_pad, T = c.n_samp, nw = (c.n_pix + 63) >> 6;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const uint16_t* cand = sm.list + run_begin(kMaxPix, NT, PPL, wave);
  uint32_t* m32 = reinterpret_cast<uint32_t*>(sm.mbits);
  auto each_neighbour = [](const int4& nv, auto&& fn) {
    const int32_t nb2[3] = {nv.x, nv.y, nv.z};
#pragma unroll
    for (int k = 0; k < 6; ++k) fn(k, (k & 1) ? nb2[k >> 1] >> 16 : (int)(int16_t)nb2[k >> 1]);
  };
  auto list_mask = [&](int wbase, uint16_t* list) {  // mask pixels in order
    for (int w = wave; w < nw; w += NW) {
      const uint64_t bits = sm.mbits[w];
      const int first = __builtin_amdgcn_readlane(wbase, __builtin_amdgcn_readfirstlane(w));
      if ((bits >> lane) & 1ull) list[first + __popcll(bits & ((1ull << lane) - 1ull))] = (uint16_t)((w << 6) | lane);
    }
  };
  __syncthreads();
  for (int b = lane; b < ncand; b += kWave) {
    const int i = cand[b];
    const int4 nv = neighbour_row(c, i);
    if (!passes(sm, sm.flag[i], nv)) continue;
    atomicOr(&m32[i >> 5], 1u << (i & 31));
    each_neighbour(nv, [&](int, int j) {
      if (j >= 0 && (sm.flag[j] & 3u)) atomicOr(&m32[j >> 5], 1u << (j & 31));
    });
  }
  __syncthreads();
  int n;
  const int abase = scan_phase(c.n_pix, sm, &n);
  *none = n == 0;
  if (n == 0) return true;
  if (n > min(c.nbr_most, kNbrAsk)) return false;
  list_mask(abase, sm.ask);
  for (int b = lane; b < ncand; b += kWave) {
    const int i = cand[b];
    if (!mask_bit(sm, i)) sm.flag[i] &= 4u;
  }
  __syncthreads();
  for (int j = threadIdx.x; j < n; j += NT) {
    const int i = sm.ask[j];
    sm.key[i] = 0u;
    each_neighbour(neighbour_row(c, i), [&](int, int k) {
      if (k >= 0) atomicOr(&m32[k >> 5], 1u << (k & 31));
    });
  }
  __syncthreads();
  int nu;
  const int ubase = scan_phase(c.n_pix, sm, &nu);
  if (nu > min(c.nbr_most, kNbrStage)) return false;
  list_mask(ubase, nm.px);
  // Tc slices at once, rows of rw dwords (2 mod 4, so that the lanes of a
  // store spread over the banks), row nu all zero for missing neighbours
  int Tc = ((kXrow / (nu + 1)) & ~3) - 4;
  Tc = min(Tc, (T + 3) & ~3);
  const int rw = Tc / 2 + ((Tc & 4) ? 0 : 2);
  uint32_t* xw = reinterpret_cast<uint32_t*>(nm.xrow);
  for (int z = threadIdx.x; z < rw; z += NT) xw[nu * rw + z] = 0u;
  const int starts = Tc - (W - 1);  // windows of a stage
  for (int s0 = 0; s0 + W <= T; s0 += starts) {
    __syncthreads();
    const int slices = min(Tc, T - s0);
    // 64 pixels of one slice per load; a wavefront's loads go in runs of 32
    // that are in flight together
    const int blocks = (nu + kWave - 1) / kWave;
    constexpr int U = 24;
    int u0 = 0, t = wave;
    while (t >= slices) {  // fewer slices than wavefronts
      t -= slices;
      u0 += kWave;
    }
    while (u0 < blocks * kWave) {
      uint16_t x[U];
      int at[U];  // store position, -1: none
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const int u = u0 + lane;
        at[k] = u < nu ? u * rw * 2 + t : -1;
        x[k] = ev[(size_t)(s0 + t) * np + nm.px[min(u, nu - 1)]];
        t += NW;
        while (t >= slices) {
          t -= slices;
          u0 += kWave;
        }
      }
#pragma unroll
      for (int k = 0; k < U; ++k)
        if (at[k] >= 0) nm.xrow[at[k]] = x[k];
    }
    __syncthreads();
    // this wavefront's windows: starts [a, b) of the stage
    const int nwin = slices - (W - 1), part = ((nwin + NW - 1) / NW + 3) & ~3;
    const int a = wave * part, b = min(a + part, nwin);
    if (a < b)
      for (int j = lane; j < n; j += kWave) {
        const int i = sm.ask[j];
        int off[6];
        each_neighbour(neighbour_row(c, i),
                       [&](int k, int m) { off[k] = (m >= 0 ? mask_slot(sm, m) : nu) * rw + (a >> 1); });
        const us2 row_lo = {1, 0}, row_hi = {0, 1};
        uint32_t y[7] = {0, 0, 0, 0, 0, 0, 0}, best = 0;  // y(t-3) .. y(t+3)
        for (int t = a; t < b + W - 1; t += 4) {
          y[0] = y[4]; y[1] = y[5]; y[2] = y[6];
          y[3] = y[4] = y[5] = y[6] = 0;
#pragma unroll
          for (int k = 0; k < 6; ++k) {
            // a 64-bit word, not a two-element vector: the packed dot of such
            // a vector's second element has been seen compiled onto its first
            const uint64_t v = *reinterpret_cast<const uint64_t*>(xw + off[k]);
            const uint32_t v01 = (uint32_t)v, v23 = (uint32_t)(v >> 32);
            off[k] += 2;
            y[3] = __builtin_amdgcn_udot2(__builtin_bit_cast(us2, v01), row_lo, y[3], false);
            y[4] = __builtin_amdgcn_udot2(__builtin_bit_cast(us2, v01), row_hi, y[4], false);
            y[5] = __builtin_amdgcn_udot2(__builtin_bit_cast(us2, v23), row_lo, y[5], false);
            y[6] = __builtin_amdgcn_udot2(__builtin_bit_cast(us2, v23), row_hi, y[6], false);
          }
#pragma unroll
          for (int z = 0; z < 4; ++z) {
            const int s = t + z - (W - 1);  // the window that ends with slice t + z
            const uint32_t C = y[z] + y[z + 1] + y[z + 2] + y[z + 3];
            if (s >= a && s < b) best = max(best, (C << 8) | (uint32_t)(255 - (s0 + s)));
          }
        }
        atomicMax(&sm.key[i], best);
      }
  }
  __syncthreads();
  if (threadIdx.x < kMaxWords) sm.mbits[threadIdx.x] = 0ull;  // for the image's own mask
  // four lanes per asked pixel take its window's samples on its gain
  static_assert(W == 4, "one sample per lane of a quad");
  for (int j0 = 0; j0 < n; j0 += NT / 4) {
    const int j = j0 + ((int)threadIdx.x >> 2);
    const int i = sm.ask[min(j, n - 1)];
    const int g = (int)(sm.flag[i] >> 2), o = g * np + i, s = 255 - (int)(sm.key[i] & 255u);
    const int32_t P = c.P256[o], tb = c.thr_bnd[o], tp = c.thr_pic[o];
    uint32_t S = ev[((size_t)g * T + s + (threadIdx.x & 3)) * np + i];
    S += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)S, 0xB1, 0xF, 0xF, false);
    S += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)S, 0x4E, 0xF, 0xF, false);
    if (j < n && (threadIdx.x & 3) == 0) {
      const uint32_t key = (S << 8) | (uint32_t)(255 - s);
      const int32_t d = key_to_d<W>(key, P);
      sm.key[i] = key;
      sm.flag[i] = (uint8_t)((uint32_t)(d >= tb) | ((uint32_t)(d >= tp) << 1) | ((uint32_t)g << 2));
    }
  }
  __syncthreads();
  return true;
}

// Calibration -> cleaning -> Hillas of one camera event; the threads of
// wavefront 0 return the record.
template <int EX, int PPL, int W, int CH, int NT>
__device__ __forceinline__ rta_hillas_rec process_telescope(const DevCam& c, const uint16_t* __restrict__ ev, bool look,
                                                            uint8_t* raw) {
  TelSmem& sm = *reinterpret_cast<TelSmem*>(raw);
  uint16_t* xrow = nullptr;
  if constexpr (EX == kExNeighbour) {
    NbrSmem& nm = *reinterpret_cast<NbrSmem*>(raw);
    xrow = nm.xrow;
    if (c.nbr_most > 0) {
      int ncand;
      if (look && c.nbr_noise < 1.f)
        ncand = extract_phase<EX, PPL, W, CH, NT, true, true>(c, ev, sm, xrow, nm.seen);
      else
        ncand = extract_phase<EX, PPL, W, CH, NT, true>(c, ev, sm, xrow);
      bool none;
      if (ncand >= 0 && nbr_windows<PPL, NT, W>(c, nm, ncand, ev, &none)) {
        if (none) return empty_image(total_count<NT>(sm));
        return fused_image<PPL, NT, W>(c, sm, ncand, ev);
      }
      __syncthreads();  // the wavefronts' runs and the mask words have been read
    }
  }
  const int ncand = extract_phase<EX, PPL, W, CH, NT, false>(c, ev, sm, xrow);
  return fused_image<PPL, NT, W>(c, sm, ncand, ev);
}

__device__ __forceinline__ void bad_record(rta_hillas_rec* out) {
  rta_hillas_rec r;
  r.size = r.cog_x = r.cog_y = r.length = r.width = r.psi = r.skewness = r.kurtosis = kNaN;
  r.time_gradient = r.time_intercept = r.leakage = r.cog_dist = kNaN;
  r.n_pix = r.n_islands = r.n_lowgain = 0;
  r.flags = RTA_FLAG_BAD_DESCRIPTOR | RTA_FLAG_HILLAS_INVALID | RTA_FLAG_TIME_INVALID;
  *out = r;
}

// Waves per SIMD the register allocation must leave room for: the neighbour
// peak's 256-thread workgroups fit four to a compute unit by their LDS (37
// KB), if the registers allow it (512-thread ones two); its full scan, bound by
// latency, loses 8 % with three.  The sliding window keeps two: with 8 pixels per lane, chunks
// of 16 and 4 wavefronts the compiler's own choice is 260 registers, one wave
// (8000 events of the 1:3:6 mix 600 us, 457 with two).  Elsewhere that choice
// stands.
template <int EX>
constexpr int min_waves() {
  return EX == kExNeighbour ? 4 : EX == kExSliding ? 2 : 1;
}

// ---------------------------------------------------------------------------
// Kernels
// ---------------------------------------------------------------------------

// Stores a lane's first n of K consecutive values, in one piece if all are
// there (an event's outputs begin at any multiple of the value's size).
// Two pixels' seven outputs in seven stores instead of fourteen: 1000 events of
// 1855 x 30 samples 35.4 to 33.1 us, of which 31 are the bytes; four pixels per
// lane 34.3 (twice the registers, half the wavefronts).
template <int K, typename V>
__device__ __forceinline__ void store_run(V* dst, const V (&v)[K], int n) {
  typedef V vec __attribute__((ext_vector_type(K)));
  typedef vec loose __attribute__((aligned(sizeof(V))));
  if (n >= K) {
    vec x;
#pragma unroll
    for (int p = 0; p < K; ++p) x[p] = v[p];
    *reinterpret_cast<loose*>(dst) = x;
  } else {
#pragma unroll
    for (int p = 0; p < K; ++p)
      if (p < n) dst[p] = v[p];
  }
}

// Unfused calibration: one workgroup per camera event, per-pixel results to HBM.
template <int EX, int PPL, int W, int NT, bool AHEAD = true>
__global__ __launch_bounds__(NT) void k_calibrate(DevCam c, const uint16_t* __restrict__ traces, int32_t* S,
                                                  int32_t* D, uint8_t* sstar, uint8_t* peak, uint8_t* gain,
                                                  float* q, float* t) {
  __shared__ uint32_t rows[EX == kExGlobal ? NT / kWave * 256 : (EX == kExNeighbour ? kMaxPix : 1)];
  __shared__ __attribute__((aligned(16))) uint16_t xrow[EX == kExNeighbour ? kNbrRows * (kMaxPix + 8) : 8];
  __shared__ __attribute__((aligned(8))) uint8_t low[EX == kExNeighbour ? kMaxPix : 8];
  __shared__ int32_t start;
  const int64_t e = blockIdx.x;
  const int N = c.n_pix, np = c.n_pix_pad, T = c.n_samp;
  const uint16_t* ev = traces + e * c.event_elems;
  const size_t ob = (size_t)e * N;
  const __amdgpu_buffer_rsrc_t r = event_rsrc(ev, c.event_elems);
  if constexpr (EX == kExSliding && W == 4) {
    // the trace is read once: every pixel's window kept while it streams.
    // Pixels are independent here, so the pixel passes of an event are
    // spread over blockIdx.y: many more, shorter workgroups than events,
    // which evens out the last round of workgroups on a small batch
    const int npass = (N + NT * PPL - 1) / (NT * PPL);
    for (int ps = (int)blockIdx.y; ps < npass; ps += (int)gridDim.y) {
      const int pix0 = (ps * NT + (int)threadIdx.x) * PPL;
      KeepState<PPL> st;
      const uint32_t sw = keep_group<PPL, 2 * W>(c, r, pix0, np, T, c.n_gain == 2, st);
      if (pix0 >= N) continue;
      int32_t sum[PPL], d[PPL];
      uint8_t s[PPL], pk[PPL], g[PPL];
      float qv[PPL], tv[PPL];
#pragma unroll
      for (int p = 0; p < PPL; ++p) {
        g[p] = (uint8_t)((sw >> p) & 1);
        const int o = g[p] * np + pix0 + p;  // padding pixels have table entries
        s[p] = (uint8_t)(255 - (int)(st.key[p] & 255u));
        const int32_t P = c.P256[o];
        sum[p] = (int32_t)(st.key[p] >> 8);
        d[p] = key_to_d<W>(st.key[p], P);
        int peak_at;
        const int32_t nt = kept_nt(st.sv0[p], st.sv1[p], P, s[p], &peak_at);
        pk[p] = (uint8_t)peak_at;
        qv[p] = (float)d[p] / (256.0f * c.a[o]);
        tv[p] = (float)peak_time<W>(s[p], nt, d[p]);
      }
      const size_t at = ob + pix0;
      const int n = N - pix0;
      if (S) store_run(S + at, sum, n);
      if (D) store_run(D + at, d, n);
      if (sstar) store_run(sstar + at, s, n);
      if (peak) store_run(peak + at, pk, n);
      if (gain) store_run(gain + at, g, n);
      if (q) store_run(q + at, qv, n);
      if (t) store_run(t + at, tv, n);
    }
    return;
  }
  extract_event<EX, PPL, W, 2 * W, NT, AHEAD>(c, r, ev, rows, &start, xrow, low, [&](int pix0,
                                                                                const uint32_t (&key)[PPL],
                                                                                uint32_t sw) {
#pragma unroll
    for (int p = 0; p < PPL; ++p) {
      const int i = pix0 + p;
      if (i >= N) break;
      const int g = (sw >> p) & 1u;
      const int s = 255 - (int)(key[p] & 255u);
      const int32_t P = c.P256[g * np + i];
      const int32_t d = key_to_d<W>(key[p], P);
      int pk;
      const int32_t nt = window_nt<W>(ev + (size_t)g * T * np + i, np, s, P, &pk);
      const float tv = (float)peak_time<W>(s, nt, d);
      if (S) S[ob + i] = (int32_t)(key[p] >> 8);
      if (D) D[ob + i] = d;
      if (sstar) sstar[ob + i] = (uint8_t)s;
      if (peak) peak[ob + i] = (uint8_t)pk;
      if (gain) gain[ob + i] = (uint8_t)g;
      if (q) q[ob + i] = (float)d / (256.0f * c.a[g * np + i]);
      if (t) t[ob + i] = tv;
    }
  });
}

template <int NT>
__global__ __launch_bounds__(NT) void k_clean(DevCam c, const int32_t* __restrict__ D, const uint8_t* __restrict__ gain,
                                              uint8_t* __restrict__ mask, int have_levels, float t_pic, float t_bnd) {
  __shared__ TelSmem sm;
  const int64_t e = blockIdx.x;
  const int N = c.n_pix;
  const size_t ob = (size_t)e * N;
  // pixels per thread, their loads all in flight (1000 events of 1855 pixels:
  // 9.4 us, 10.1 with one pixel after the other)
  constexpr int K = kMaxPix / NT;
  int32_t d[K];
  int g[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int i = min(k * NT + (int)threadIdx.x, N - 1);
    g[k] = gain ? (int)gain[ob + i] : 0;
    d[k] = D[ob + i];
  }
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int i = k * NT + (int)threadIdx.x, at = min(i, N - 1);
    const uint32_t fl = have_levels ? pixel_flag_at(c, g[k], at, d[k], t_pic, t_bnd) : pixel_flag(c, g[k], at, d[k]);
    if (i < N) sm.flag[i] = (uint8_t)fl;
  }
  __syncthreads();
  mask_phase<NT>(c, sm);
  __syncthreads();
  for (int i = threadIdx.x; i < N; i += NT) mask[ob + i] = (uint8_t)mask_bit(sm, i);
}

template <int W, int NT>
__global__ __launch_bounds__(NT) void k_hillas(DevCam c, const float* __restrict__ q, const int32_t* __restrict__ D,
                                               const float* __restrict__ t, const uint8_t* __restrict__ mask,
                                               const uint8_t* __restrict__ gain, rta_hillas_rec* out) {
  __shared__ TelSmem sm;
  const int64_t e = blockIdx.x;
  const int N = c.n_pix, nw = (N + 63) >> 6;
  const size_t ob = (size_t)e * N;
  const int lane = threadIdx.x & (kWave - 1);
  int nlow = 0;
  constexpr int K = kMaxPix / NT;  // pixels per thread, their loads all in flight
  uint8_t mk[K], gn[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int i = k * NT + (int)threadIdx.x;
    mk[k] = i < N ? mask[ob + i] : (uint8_t)0;
    gn[k] = gain && i < N ? gain[ob + i] : (uint8_t)0;
  }
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const uint64_t b = __ballot(mk[k] != 0);
    nlow += gn[k] == 1;
    const int word = (k * NT + (int)threadIdx.x) >> 6;
    if (lane == 0 && word < nw) sm.mbits[word] = b;
  }
  const uint32_t nl = wave_sum_u32_last((uint32_t)nlow);
  if (lane == kWave - 1) sm.nlow_w[threadIdx.x / kWave] = (int32_t)nl;
  __syncthreads();
  const rta_hillas_rec r =
      given_image<NT>(c, sm, total_count<NT>(sm),
                      GivenSource{q ? q + ob : nullptr, D ? D + ob : nullptr, gain ? gain + ob : nullptr, t + ob});
  if (threadIdx.x == 0) out[e] = r;
}

__global__ void k_queue_reset(unsigned long long* q) {
  if (threadIdx.x == 0) *q = 0ull;
}

// Classification of one telescope right after its Hillas parameters, by the
// first wavefront: the record is row 0 of a 16-row network tile (the other
// rows zero; a tile's rows do not affect each other, so the outputs equal
// those of the same record in any other tile), then the network-or-box-cut
// decision.  Lane 0 writes the score and log10 E and marks the fallback in
// the record; records without a valid image get NaN.  (Spreading the four
// tiles of each layer over four wavefronts, with the activations exchanged
// through LDS, was no faster: the layers wait on their weight loads.)
__device__ __forceinline__ void classify_telescope(const FusedArgs& a, long long tel, rta_hillas_rec& r) {
  const int lane = threadIdx.x & (kWave - 1), col = lane & 15, grp = lane >> 4;
  const bool valid = !(r.flags & RTA_FLAG_HILLAS_INVALID);
  float logit = 0.f, me = 0.f;
  if (valid && a.have_mlp) {  // uniform over the wavefront
    float x[4], mean[4], stdv[4];
    mlpdev::load_scale(a.mlp, grp, mean, stdv);
    mlpdev::record_features4(r, grp, x);
    mlpdev::bf16x4 xin = mlpdev::record_inputs(x, mean, stdv);
    if (col != 0) xin = mlpdev::pack4(0.f, 0.f, 0.f, 0.f);
    mlpdev::bf16x4 h1[4], h2[4], h3[4];
    const mlpdev::f32x4 o = mlpdev::mlp_forward_tile(a.mlp, xin, h1, h2, h3);
    logit = o[0];
    me = o[1];
  }
  if (lane == 0) {
    float score = kNaN, log10e = kNaN;
    if (valid) {
      const mlpdev::ClassOut co = mlpdev::classify_record(r, a.bc, a.have_mlp != 0, logit, me);
      if (co.fallback) r.flags |= RTA_FLAG_MLP_FALLBACK;
      score = co.score;
      log10e = co.log10e;
    }
    a.tel_class[2 * tel] = score;
    a.tel_class[2 * tel + 1] = log10e;
  }
}

// Per-telescope body of the fused kernel: descriptor checks, then
// calibration -> cleaning -> Hillas with all intermediates in LDS.
template <int EX, int PPL, int W, int CH, int NT>
__device__ __forceinline__ void fused_telescope(const FusedArgs& a, long long tel, uint8_t* raw) {
  const int ty = uniform_i32(a.tel_type[tel]);
  const long long off = uniform_i64(a.tel_trace_off[tel]);
  const uint32_t bad = tel_descriptor_status(ty, off, a.n_types, a.traces_len,
                                             [&](int t) { return (int64_t)a.cams[t].event_elems; });
  if (bad) {
    if (threadIdx.x == 0) {
      bad_record(a.out + tel);
      if (a.classify) {
        a.tel_class[2 * tel] = kNaN;
        a.tel_class[2 * tel + 1] = kNaN;
      }
      atomicOr(a.status, bad);
    }
    return;
  }
  rta_hillas_rec r = process_telescope<EX, PPL, W, CH, NT>(a.cams[ty], uniform_ptr(a.traces + off), a.nbr_look != 0,
                                                           raw);
  if (a.classify && threadIdx.x < kWave) classify_telescope(a, tel, r);
  if (threadIdx.x == 0) a.out[tel] = r;
}

// Persistent form: a fixed grid of workgroups pulls telescopes from a global
// counter until the batch is drained.
// At least two wavefronts per SIMD: values hoisted out of the telescope loop
// would otherwise push some shapes just past half the register file.
template <int EX, int PPL, int W, int CH, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2))) void k_fused(FusedArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t raw[smem_bytes<EX>()];
  __shared__ long long s_tel;
  for (;;) {
    if (threadIdx.x == 0) s_tel = (long long)atomicAdd(a.queue, 1ull);
    __syncthreads();
    const long long tel = uniform_i64(s_tel);
    __syncthreads();
    if (tel >= a.n_tel) return;
    fused_telescope<EX, PPL, W, CH, NT>(a, tel, raw);
    __syncthreads();
  }
}

// Grid form: one workgroup per telescope, dispatched by the hardware's
// workgroup scheduler (no loop-carried state, so no register pressure from
// values hoisted across telescopes).
template <int EX, int PPL, int W, int CH, int NT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(min_waves<EX>()))) void k_fused_grid(
    FusedArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t raw[smem_bytes<EX>()];
  fused_telescope<EX, PPL, W, CH, NT>(a, (long long)blockIdx.x, raw);
}

// Array events: stereo direction from the telescope records and, when
// enabled, per-telescope classification aggregated into size-weighted event
// values, in telescope order.
//
// NET: the network runs here, on 16-telescope MFMA tiles (box-cut fallback
// per telescope).  SPLIT: an array event has a workgroup, whose wavefronts
// take its tiles side by side (wavefront 0, which forms the stereo sums,
// every fourth); the scores meet in LDS and are added in tile order.
// Otherwise an event has a wavefront.
constexpr int kEvtNT = 256;
template <bool NET, bool SPLIT>
__device__ __forceinline__ void event_record(const EventArgs& a, int64_t e, const mlpdev::MlpFrag& net,
                                             float (&tile_sum)[kEvtNT / kWave][3][16]) {
  constexpr int NW = kEvtNT / kWave;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int64_t lo = a.evt_tel_off[e], hi = a.evt_tel_off[e + 1];
  rta_event_rec r;
  r.gammaness = kNaN;
  r.log10_energy = kNaN;
  if (!event_range_ok(lo, hi, a.n_tel)) {
    if (lane == 0 && (!SPLIT || wave == 0)) {
      r.dir_x = r.dir_y = r.cond = kNaN;
      r.n_tel = 0;
      r.n_used = 0;
      r.flags = RTA_EVT_STEREO_INVALID | RTA_EVT_NO_MLP;
      a.out[e] = r;
      if (a.done_clock) a.done_clock[e] = wall_clock64();
      atomicOr(a.status, RTA_STATUS_BAD_EVENT);
    }
    return;
  }
  float v[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};  // A00, A01, A11, b0, b1, used
  if (!SPLIT || wave == 0) {
    for (int64_t k = lo + lane; k < hi; k += kWave) {
      const int ty = a.tel_type[k];
      if (ty < 0 || ty >= a.n_types) continue;
      const rta_hillas_rec h = a.tel[k];
      if (h.flags & (RTA_FLAG_HILLAS_INVALID | RTA_FLAG_BAD_DESCRIPTOR)) continue;
      if (!(h.length > 0.f) || !(h.width >= 0.f) || !isfinite(h.psi) || !isfinite(h.size)) continue;
      const float ratio = h.width / h.length;
      if (ratio > a.max_width_ratio) continue;
      const float w = h.size * (1.0f - ratio);
      const float f = a.focal[ty];
      const float nx = -sinf(h.psi), ny = cosf(h.psi);
      const float cx = h.cog_x / f, cy = h.cog_y / f;
      const float nc = nx * cx + ny * cy;
      v[0] += w * nx * nx;
      v[1] += w * nx * ny;
      v[2] += w * ny * ny;
      v[3] += w * nc * nx;
      v[4] += w * nc * ny;
      v[5] += 1.f;
    }
    butterfly(v);
  }
  // classification: rows = telescopes of this event, 16 per MFMA tile
  float c[3] = {0.f, 0.f, 0.f};  // sum size*score, sum size*log10E, sum size
  if (NET || a.have_box) {
    const int col = lane & 15, grp = lane >> 4;
    // row of a tile: size, score and log10 E, or size 0 where it has none
    auto row = [&](int64_t k, float logit, float me, float (&o)[3]) {
      o[0] = o[1] = o[2] = 0.f;
      if (k >= hi) return;
      rta_hillas_rec h = a.tel[k];
      const int ty = a.tel_type[k];
      if (ty < 0 || ty >= a.n_types || (h.flags & (RTA_FLAG_HILLAS_INVALID | RTA_FLAG_BAD_DESCRIPTOR))) return;
      float score, log10e;
      if (!NET && a.tel_class) {  // classified in the reconstruction kernel
        score = a.tel_class[2 * k];
        log10e = a.tel_class[2 * k + 1];
      } else {
        const mlpdev::ClassOut co = mlpdev::classify_record(h, a.bc, NET, logit, me);
        if (co.fallback) a.tel[k].flags = h.flags | RTA_FLAG_MLP_FALLBACK;
        score = co.score;
        log10e = co.log10e;
      }
      if (isfinite(log10e) && h.size > 0.f) {
        o[0] = h.size;
        o[1] = score;
        o[2] = log10e;
      }
    };
    auto add = [&](const float (&o)[3]) {
      if (o[0] > 0.f) {
        c[0] += o[0] * o[1];
        c[1] += o[0] * o[2];
        c[2] += o[0];
      }
    };
    float o[3];
    auto tile = [&](int64_t t0) {
      mlpdev::bf16x4 h1[4], h2[4], h3[4];
      const mlpdev::f32x4 z = mlpdev::mlp_forward(net, mlpdev::mlp_record_tile(a.mlp, a.tel, hi, t0), h1, h2, h3);
      if (grp == 0) row(t0 + col, z[0], z[1], o);
    };
    if constexpr (SPLIT) {
      for (int64_t r0 = lo; r0 < hi; r0 += 16 * NW) {
        const int mine = (wave + NW - 1) & (NW - 1);  // wavefront 0 takes the last of four tiles
        const int64_t t0 = r0 + 16 * mine;
        if (t0 < hi) {
          tile(t0);
          if (grp == 0) {
#pragma unroll
            for (int q = 0; q < 3; ++q) tile_sum[mine][q][col] = o[q];
          }
        }
        __syncthreads();
        if (wave == 0 && grp == 0) {
#pragma unroll
          for (int t = 0; t < NW; ++t)
            if (r0 + 16 * t < hi) {
#pragma unroll
              for (int q = 0; q < 3; ++q) o[q] = tile_sum[t][q][col];
              add(o);
            }
        }
        __syncthreads();
      }
    } else {
      for (int64_t r0 = lo; r0 < hi; r0 += 16) {
        if constexpr (NET)
          tile(r0);
        else if (grp == 0)
          row(r0 + col, 0.f, 0.f, o);
        if (grp == 0) add(o);
      }
    }
    if (!SPLIT || wave == 0) butterfly(c);
  }
  if (lane == 0 && (!SPLIT || wave == 0)) {
    const float A00 = v[0], A01 = v[1], A11 = v[2], b0 = v[3], b1 = v[4];
    const float tr = A00 + A11, det = A00 * A11 - A01 * A01;
    const float hd = 0.5f * (A00 - A11);
    const float lmax = 0.5f * tr + sqrtf(hd * hd + A01 * A01);
    const float lmin = lmax > 0.f ? det / lmax : 0.f;
    const float cond = lmin > 0.f ? lmax / lmin : INFINITY;
    r.cond = cond;
    r.n_tel = (int32_t)(hi - lo);
    r.n_used = (int32_t)v[5];
    r.flags = a.have_mlp ? 0u : RTA_EVT_NO_MLP;
    if (r.n_used < 2 || !(cond < a.max_cond)) {
      r.dir_x = r.dir_y = kNaN;
      r.flags |= RTA_EVT_STEREO_INVALID;
    } else {
      r.dir_x = (A11 * b0 - A01 * b1) / det;
      r.dir_y = (A00 * b1 - A01 * b0) / det;
    }
    if (a.have_box && c[2] > 0.f) {
      r.gammaness = c[0] / c[2];
      r.log10_energy = c[1] / c[2];
    }
    a.out[e] = r;
    if (a.done_clock) a.done_clock[e] = wall_clock64();
  }
}

// No network: little work, bound by the launch and two dependent loads.
__global__ __launch_bounds__(kEvtNT) void k_event(EventArgs a) {
  float unused[kEvtNT / kWave][3][16];
  const mlpdev::MlpFrag none = {};
  const int64_t e = (int64_t)blockIdx.x * (kEvtNT / kWave) + threadIdx.x / kWave;
  if (e < a.n_evt) event_record<false, false>(a, e, none, unused);
}

// Few events: a workgroup each.  Two tiles in turn behind the stereo sums,
// each layer waiting for its weights, held 100 events of 21 telescopes for
// 24.6 us; side by side with the weights loaded at once, 10.6 us.
__global__ __launch_bounds__(kEvtNT) void k_event_split(EventArgs a) {
  __shared__ float tile_sum[kEvtNT / kWave][3][16];  // size (0: not counted), score, log10 E per row of a tile
  mlpdev::MlpFrag net;
  mlpdev::mlp_load(a.mlp, net);
  event_record<true, true>(a, (int64_t)blockIdx.x, net, tile_sum);
}

// Many events: persistent wavefronts that keep the network's weights in
// registers from event to event (18 KB from L2 per event otherwise bounds it):
// 200000 events of 2 to 40 telescopes 1873 -> 898 us.
__global__ __launch_bounds__(kEvtNT) void k_event_stream(EventArgs a) {
  float unused[kEvtNT / kWave][3][16];
  mlpdev::MlpFrag net;
  mlpdev::mlp_load(a.mlp, net);
  const int64_t step = (int64_t)gridDim.x * (kEvtNT / kWave);
  for (int64_t e = (int64_t)blockIdx.x * (kEvtNT / kWave) + threadIdx.x / kWave; e < a.n_evt; e += step)
    event_record<true, false>(a, e, net, unused);
}

__global__ void k_stamp(uint64_t* slot) {
  if (threadIdx.x == 0) *slot = wall_clock64();
}

// Network inputs of records, one thread per record.
__global__ __launch_bounds__(256) void k_features(const rta_hillas_rec* __restrict__ rec, int64_t n,
                                                  float* __restrict__ x) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const rta_hillas_rec r = rec[i];
#pragma unroll
  for (int f = 0; f < mlpdev::kIn; ++f) x[i * mlpdev::kIn + f] = mlpdev::record_feature(r, f);
}

struct BoxTables {
  float w_mean[RTA_BOXCUT_MAX_BINS], w_std[RTA_BOXCUT_MAX_BINS], l_mean[RTA_BOXCUT_MAX_BINS],
      l_std[RTA_BOXCUT_MAX_BINS];
};

__device__ __forceinline__ void load_tables(const rta_boxcut_desc& bc, BoxTables& tab) {
  static_assert(RTA_BOXCUT_MAX_BINS <= kWave, "a bin per lane");
  const int k = threadIdx.x;
  if (k < RTA_BOXCUT_MAX_BINS) {
    tab.w_mean[k] = bc.w_mean[k];
    tab.w_std[k] = bc.w_std[k];
    tab.l_mean[k] = bc.l_mean[k];
    tab.l_std[k] = bc.l_std[k];
  }
}

__device__ __forceinline__ void store_class(float* dst, const mlpdev::ClassOut& co) {
  dst[0] = co.score;
  dst[1] = co.log10e;
  dst[2] = (float)co.gamma;
  dst[3] = (float)co.fallback;
}

// Without a network: a record per thread, as many wavefronts as there are
// (the persistent tiles of the network, 16 records per wavefront and round on
// two wavefronts per SIMD, took 70.7 us for 2000000 records; 23.6 so).
__global__ __launch_bounds__(256) void k_classify_box(rta_boxcut_desc bc, const rta_hillas_rec* __restrict__ rec,
                                                      int64_t n, float* __restrict__ out) {
  __shared__ BoxTables tab;
  load_tables(bc, tab);
  __syncthreads();
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n)
    store_class(out + i * 4, mlpdev::classify_decide(rec[i], bc, tab.w_mean, tab.w_std, tab.l_mean, tab.l_std, false,
                                                     0.f, 0.f));
}

// Per-record classification, 16 records per wavefront and round.  The network
// is 18 kFLOP a record against 80 bytes of memory, but with its 18 KB of
// weights read from L2 for every tile, layer by layer, 200000 records took
// 70 us.  Persistent single-wavefront workgroups, two per SIMD, keep the
// weights in registers and load the next tile's records during a tile; the
// features are picked by selects, not a switch that every lane steps
// through, and the range checks are spread over a row's four lanes.  68.8 ->
// 23.2 us per call; bound by the chain of a tile (about 3 us: logarithm,
// divisions, four dependent layers) with few wavefronts to cover it.  Three
// wavefronts per SIMD with the biases in LDS (147 registers), 25.5, and one
// per SIMD, 27.3, were slower: each wavefront loads the weights once.
__global__ __launch_bounds__(kWave) void k_classify(MlpDev w, rta_boxcut_desc bc,
                                                    const rta_hillas_rec* __restrict__ rec, int64_t n,
                                                    float* __restrict__ out) {
  __shared__ BoxTables tab;
  const int lane = threadIdx.x, col = lane & 15, grp = lane >> 4;
  load_tables(bc, tab);
  // a lane has features 4 grp .. 4 grp + 3 of row col: their standardisation
  // and trained range
  mlpdev::MlpFrag net;
  float mean[4], stdv[4], lo[4], hi[4];
  mlpdev::mlp_load(w, net);
  mlpdev::load_scale(w, grp, mean, stdv);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int f = min(4 * grp + j, mlpdev::kIn - 1);
    lo[j] = bc.feat_lo[f];
    hi[j] = bc.feat_hi[f];
  }
  __syncthreads();
  const int64_t step = (int64_t)gridDim.x * 16;
  int64_t r0 = (int64_t)blockIdx.x * 16;
  rta_hillas_rec next = rec[min(r0 + col, n - 1)];
  for (; r0 < n; r0 += step) {
    const rta_hillas_rec r = next;
    if (r0 + step < n) next = rec[min(r0 + step + col, n - 1)];
    float x[4];
    mlpdev::record_features4(r, grp, x);
    bool ok = true;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      ok = ok && (4 * grp + j >= mlpdev::kIn || (isfinite(x[j]) && x[j] >= lo[j] && x[j] <= hi[j]));
    const uint64_t m = __ballot(ok);  // row col is in range when its four lanes' features are
    const bool in_range = (m >> col & m >> (col + 16) & m >> (col + 32) & m >> (col + 48)) & 1ull;
    mlpdev::bf16x4 h1[4], h2[4], h3[4];
    const mlpdev::f32x4 o = mlpdev::mlp_forward(net, mlpdev::record_inputs(x, mean, stdv), h1, h2, h3);
    if (grp == 0 && r0 + col < n)
      store_class(out + (r0 + col) * 4, mlpdev::classify_decide(r, bc, tab.w_mean, tab.w_std, tab.l_mean, tab.l_std,
                                                                in_range, o[0], o[1]));
  }
}

// ---------------------------------------------------------------------------
// Dispatch tables
// ---------------------------------------------------------------------------
constexpr int kUnfusedNT = 256;
constexpr int kUnfusedPPL = 4;
constexpr int kKeepPPL = 2;  // sliding-window calibrate: the kept windows take registers

template <int W>
hipError_t launch_calibrate_w(const DevCam& c, int ex, const uint16_t* tr, int64_t n, int n_cu, int32_t* S,
                              int32_t* D, uint8_t* ss, uint8_t* pk, uint8_t* g, float* q, float* t, hipStream_t st) {
  switch (ex) {
    case kExSliding: {
      const unsigned npass = (unsigned)((c.n_pix + kUnfusedNT * kKeepPPL - 1) / (kUnfusedNT * kKeepPPL));
      hipLaunchKernelGGL((k_calibrate<kExSliding, kKeepPPL, W, kUnfusedNT>), dim3((unsigned)n, npass),
                         dim3(kUnfusedNT), 0, st, c, tr, S, D, ss, pk, g, q, t);
      break;
    }
    case kExFixed:
      hipLaunchKernelGGL((k_calibrate<kExFixed, kUnfusedPPL, W, kUnfusedNT>), dim3((unsigned)n), dim3(kUnfusedNT), 0,
                         st, c, tr, S, D, ss, pk, g, q, t);
      break;
    case kExGlobal:
      // Up to two events per compute unit the next chunk's loads are asked for
      // ahead (2048 x 128: 256 events 39.3 us, 46.4 without; 512 73 either
      // way); with more there are streams enough, and the registers of one
      // chunk alone keep eight workgroups resident (600 events 90.0 -> 86.9,
      // 1000 129.6 -> 123.7, 3000 372 -> 366).
      if (n <= 2 * (int64_t)n_cu)
        hipLaunchKernelGGL((k_calibrate<kExGlobal, kUnfusedPPL, W, kUnfusedNT, true>), dim3((unsigned)n),
                           dim3(kUnfusedNT), 0, st, c, tr, S, D, ss, pk, g, q, t);
      else
        hipLaunchKernelGGL((k_calibrate<kExGlobal, kUnfusedPPL, W, kUnfusedNT, false>), dim3((unsigned)n),
                           dim3(kUnfusedNT), 0, st, c, tr, S, D, ss, pk, g, q, t);
      break;
    case kExNeighbour:
      hipLaunchKernelGGL((k_calibrate<kExNeighbour, kUnfusedPPL, W, kUnfusedNT>), dim3((unsigned)n),
                         dim3(kUnfusedNT), 0, st, c, tr, S, D, ss, pk, g, q, t);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int W>
hipError_t launch_hillas_w(const DevCam& c, const float* q, const int32_t* D, const float* t, const uint8_t* m,
                           const uint8_t* g, int64_t n, rta_hillas_rec* out, hipStream_t st) {
  hipLaunchKernelGGL((k_hillas<W, kUnfusedNT>), dim3((unsigned)n), dim3(kUnfusedNT), 0, st, c, q, D, t, m, g, out);
  return hipGetLastError();
}

// grid == 0: one workgroup per telescope; otherwise the persistent form
// (sliding window only: the other extractors always use the grid form).
template <int PPL, int W, int CH, int NT>
hipError_t launch_fused_t(const FusedArgs& a, int grid, hipStream_t st) {
  const dim3 g1((unsigned)a.n_tel);
  switch (a.extractor) {
    case kExSliding:
      if (grid == 0)
        hipLaunchKernelGGL((k_fused_grid<kExSliding, PPL, W, CH, NT>), g1, dim3(NT), 0, st, a);
      else
        hipLaunchKernelGGL((k_fused<kExSliding, PPL, W, CH, NT>), dim3(grid), dim3(NT), 0, st, a);
      break;
    case kExFixed: hipLaunchKernelGGL((k_fused_grid<kExFixed, PPL, W, CH, NT>), g1, dim3(NT), 0, st, a); break;
    case kExGlobal: hipLaunchKernelGGL((k_fused_grid<kExGlobal, PPL, W, CH, NT>), g1, dim3(NT), 0, st, a); break;
    case kExNeighbour:
      hipLaunchKernelGGL((k_fused_grid<kExNeighbour, PPL, W, CH, NT>), g1, dim3(NT), 0, st, a);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int W>
hipError_t launch_fused_w(const FusedArgs& a, const rta_schedule& s, int grid, hipStream_t st) {
  const int key = s.pix_per_lane * 1000 + s.waves_per_wg * 100 + s.chunk;
  switch (key) {
    case 2408: return launch_fused_t<2, W, 8, 256>(a, grid, st);
    case 2416: return launch_fused_t<2, W, 16, 256>(a, grid, st);
    case 2808: return launch_fused_t<2, W, 8, 512>(a, grid, st);
    case 2816: return launch_fused_t<2, W, 16, 512>(a, grid, st);
    case 4408: return launch_fused_t<4, W, 8, 256>(a, grid, st);
    case 4416: return launch_fused_t<4, W, 16, 256>(a, grid, st);
    case 4808: return launch_fused_t<4, W, 8, 512>(a, grid, st);
    case 4816: return launch_fused_t<4, W, 16, 512>(a, grid, st);
    case 8408: return launch_fused_t<8, W, 8, 256>(a, grid, st);
    case 8416: return launch_fused_t<8, W, 16, 256>(a, grid, st);
    case 8808: return launch_fused_t<8, W, 8, 512>(a, grid, st);
    case 8816: return launch_fused_t<8, W, 16, 512>(a, grid, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

bool window_supported(int w) { return w == 4; }

bool extractor_supported(int ex) {
  return ex == kExSliding || ex == kExFixed || ex == kExGlobal || ex == kExNeighbour;
}

bool schedule_supported(const rta_schedule& s) {
  const bool ppl = s.pix_per_lane == 2 || s.pix_per_lane == 4 || s.pix_per_lane == 8;
  const bool wv = s.waves_per_wg == 4 || s.waves_per_wg == 8;
  const bool ch = s.chunk == 8 || s.chunk == 16;
  return ppl && wv && ch && s.wg_per_cu >= 0 && s.wg_per_cu <= 4;
}

int list_schedules(rta_schedule* out, int cap) {
  int n = 0;
  const int ppls[3] = {2, 4, 8}, waves[2] = {4, 8}, chunks[2] = {8, 16};
  for (int p : ppls)
    for (int w : waves)
      for (int ch : chunks)
        for (int g = 0; g <= 4; ++g) {
          if (out && n < cap) out[n] = rta_schedule{p, w, g, ch};
          ++n;
        }
  return n;
}

hipError_t launch_calibrate(const DevCam& c, int extractor, const uint16_t* traces, int64_t n_evt, int n_cu,
                            int32_t* S, int32_t* D, uint8_t* sstar, uint8_t* peak, uint8_t* gain, float* q, float* t,
                            hipStream_t st) {
  switch (c.window) {
    case 4: return launch_calibrate_w<4>(c, extractor, traces, n_evt, n_cu, S, D, sstar, peak, gain, q, t, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_clean(const DevCam& c, const rta_clean_params* levels, const int32_t* D, const uint8_t* gain,
                        int64_t n_evt, uint8_t* mask, hipStream_t st) {
  hipLaunchKernelGGL((k_clean<kUnfusedNT>), dim3((unsigned)n_evt), dim3(kUnfusedNT), 0, st, c, D, gain, mask,
                     levels ? 1 : 0, levels ? levels->t_pic : 0.f, levels ? levels->t_bnd : 0.f);
  return hipGetLastError();
}

hipError_t launch_hillas(const DevCam& c, const float* q, const int32_t* D, const float* t, const uint8_t* mask,
                         const uint8_t* gain, int64_t n_evt, rta_hillas_rec* out, hipStream_t st) {
  switch (c.window) {
    case 4: return launch_hillas_w<4>(c, q, D, t, mask, gain, n_evt, out, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_queue_reset(unsigned long long* queue, hipStream_t st) {
  hipLaunchKernelGGL(k_queue_reset, dim3(1), dim3(64), 0, st, queue);
  return hipGetLastError();
}

bool fused_uses_queue(int extractor, const rta_schedule& s) { return s.wg_per_cu != 0 && extractor == kExSliding; }

hipError_t launch_fused(const FusedArgs& a, const rta_schedule& s, int n_cu, hipStream_t st) {
  long long grid = (long long)n_cu * s.wg_per_cu;
  if (grid > a.n_tel) grid = a.n_tel;
  if (grid < 1) grid = 1;
  if (!fused_uses_queue(a.extractor, s)) grid = 0;
  switch (a.window) {
    case 4: return launch_fused_w<4>(a, s, (int)grid, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_features(const rta_hillas_rec* rec, int64_t n, float* x, hipStream_t st) {
  hipLaunchKernelGGL(k_features, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, rec, n, x);
  return hipGetLastError();
}

hipError_t launch_classify(const MlpDev* w, int n_cu, const rta_boxcut_desc& bc, const rta_hillas_rec* rec, int64_t n,
                           float* out, hipStream_t st) {
  const int64_t tiles = (n + 15) / 16, most = 8 * (int64_t)n_cu;  // two wavefronts per SIMD
  if (w)
    hipLaunchKernelGGL(k_classify, dim3((unsigned)(tiles < most ? tiles : most)), dim3(kWave), 0, st, *w, bc, rec, n,
                       out);
  else
    hipLaunchKernelGGL(k_classify_box, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, bc, rec, n, out);
  return hipGetLastError();
}

hipError_t launch_stamp(uint64_t* slot, hipStream_t st) {
  hipLaunchKernelGGL(k_stamp, dim3(1), dim3(64), 0, st, slot);
  return hipGetLastError();
}

hipError_t launch_event(const EventArgs& a, int n_cu, hipStream_t st) {
  const int64_t per = kEvtNT / kWave;
  const unsigned grid = (unsigned)((a.n_evt + per - 1) / per);
  if (!(a.have_box && a.have_mlp && !a.tel_class))
    hipLaunchKernelGGL(k_event, dim3(grid), dim3(kEvtNT), 0, st, a);
  else if (a.n_evt <= 2 * (int64_t)n_cu)  // resident at once: two workgroups of 184 registers fit a compute unit
    hipLaunchKernelGGL(k_event_split, dim3((unsigned)a.n_evt), dim3(kEvtNT), 0, st, a);
  else
    hipLaunchKernelGGL(k_event_stream, dim3(grid < 2u * n_cu ? grid : 2u * n_cu), dim3(kEvtNT), 0, st, a);
  return hipGetLastError();
}

}  // namespace rta
