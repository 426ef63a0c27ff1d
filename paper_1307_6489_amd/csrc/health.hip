// HIP kernels of the real-time health monitor for gfx950 (CDNA4).
//
// A basic quality check of the acquired data (paper, Section 4.2): per pixel
// and gain, the sample count, sum, sum of squares and saturated samples over
// a batch of camera events of one type, then mean / rms, the camera's median
// rms and the bad-pixel flags (definitions in rta.h).
//   accumulate  workgroups of four slots take groups of 8 samples in turn;
//               each lane of a slot owns 8 consecutive pixels and streams
//               their 16-byte slices (non-temporal loads: the traces are
//               read once), the slots add up in LDS and a workgroup stores
//               one partial block;
//   reduce      per pixel, the sum of the partial blocks (16 slices of
//               blocks per output, combined in LDS), so the totals are exact
//               integers independent of the schedule; FP64 mean / rms
//               without contraction, the record, its flags but the noisy one;
//   verdict     one workgroup: the lower median of the rms of each gain, the
//               noisy flags, pixels flagged in any gain, the verdict.
#include <cmath>

#include "rta_internal.h"

namespace rta {
namespace {

constexpr int kSlotNT = 256, kSlots = 4, kHealthNT = kSlotNT * kSlots;
constexpr int kHealthPPL = 8;
constexpr int kGroup = 8;
constexpr int kWave = 64;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
static_assert(kSlotNT * kHealthPPL == kMaxPix, "a slot's lanes cover the largest camera");

// A pixel's running sums over bytes of its samples x = 256 h + l: of l, h,
// l l, h h and l h.
struct ByteSums {
  uint32_t l, h, ll, hh, lh;
};

// Four samples of two pixels, the words a..d.
__device__ __forceinline__ void take4(uint32_t a, uint32_t b, uint32_t c, uint32_t d, ByteSums& p, ByteSums& q) {
  // bytes of (a, b): low of both, high of both, per pixel; then of all four
  const uint32_t ab0 = __builtin_amdgcn_perm(b, a, 0x05010400u), ab1 = __builtin_amdgcn_perm(b, a, 0x07030602u);
  const uint32_t cd0 = __builtin_amdgcn_perm(d, c, 0x05010400u), cd1 = __builtin_amdgcn_perm(d, c, 0x07030602u);
  const uint32_t l0 = __builtin_amdgcn_perm(cd0, ab0, 0x05040100u), h0 = __builtin_amdgcn_perm(cd0, ab0, 0x07060302u);
  const uint32_t l1 = __builtin_amdgcn_perm(cd1, ab1, 0x05040100u), h1 = __builtin_amdgcn_perm(cd1, ab1, 0x07060302u);
  p.l = __builtin_amdgcn_udot4(l0, 0x01010101u, p.l, false);
  p.h = __builtin_amdgcn_udot4(h0, 0x01010101u, p.h, false);
  p.ll = __builtin_amdgcn_udot4(l0, l0, p.ll, false);
  p.hh = __builtin_amdgcn_udot4(h0, h0, p.hh, false);
  p.lh = __builtin_amdgcn_udot4(l0, h0, p.lh, false);
  q.l = __builtin_amdgcn_udot4(l1, 0x01010101u, q.l, false);
  q.h = __builtin_amdgcn_udot4(h1, 0x01010101u, q.h, false);
  q.ll = __builtin_amdgcn_udot4(l1, l1, q.ll, false);
  q.hh = __builtin_amdgcn_udot4(h1, h1, q.hh, false);
  q.lh = __builtin_amdgcn_udot4(l1, h1, q.lh, false);
}

__device__ __forceinline__ void hold(ByteSums& s) {
  asm volatile("" : "+v"(s.l), "+v"(s.h), "+v"(s.ll), "+v"(s.hh), "+v"(s.lh));
}

__device__ __forceinline__ uint32_t max_u16x2(uint32_t a, uint32_t b) {
  typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a),
                                                                __builtin_bit_cast(u16x2, b)));
}

// part: [gridDim.x][3][G][Npad] = s1, s2, n_sat of this workgroup's groups,
// pixel 8 k + p at p Npad/8 + k.
//
// Bound by the HBM stream: 500 events of 2 gains x 2048 pixels x 128 samples
// (524 MB) take 83.7 us, 6.3 TB/s.  One unit of work is 8 samples of one gain of one event,
// so a batch divides evenly among the slots whatever its events and trace
// length; one gain per workgroup halves the sums a lane holds.  The sums of
// bytes by 4-way dot products take 2.25 instructions a sample (7 with 64-bit
// sums of each sample), they hold kFlush groups before a 32-bit one can
// overflow, and samples at the saturation level are counted only in groups
// that have one.  Whole events per workgroup, both gains and a partial block
// each (49 MB written and read again) took 108 us.
__global__ __launch_bounds__(kHealthNT) void k_health_accum(DevCam c, const uint16_t* __restrict__ traces,
                                                            int64_t n_evt, int per_event,
                                                            uint64_t* __restrict__ part) {
  // a group adds at most 8 * 255 * 255 to a 32-bit sum
  constexpr int kFlush = 8192;
  static_assert((uint64_t)kFlush * kGroup * 255 * 255 < (1ull << 32), "byte sums overflow");
  __shared__ uint64_t sum[3][kMaxPix];
  const int N = c.n_pix, np = c.n_pix_pad, T = c.n_samp, G = c.n_gain, g = blockIdx.y;
  const int k = (int)threadIdx.x % kSlotNT, lanes = np / kHealthPPL;
  const bool act = k < lanes;
  const uint32_t lvl = G == 2 && g == 0 ? (uint32_t)c.hg_switch : 65535u;
  for (int i = threadIdx.x; i < 3 * kMaxPix; i += kHealthNT) (&sum[0][0])[i] = 0;
  __syncthreads();
  const int slot = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kSlotNT);
  const int u = (int)blockIdx.x * kSlots + slot, step = (int)gridDim.x * kSlots;
  if (act && u / per_event < n_evt) {
    ByteSums s[kHealthPPL];
    const uint16_t* base = traces + (size_t)g * T * np + k * kHealthPPL;
    // four slices from sample k0 of the event at col; past the trace, the
    // last one again
    auto load4 = [&](u32x4 (&d)[4], const uint16_t* col, int k0) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        d[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(col + (size_t)min(k0 + j, T - 1) * np));
    };
    auto sums4 = [&](u32x4 (&d)[4], int k0) {
      if (k0 + 4 > T) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (k0 + j >= T) d[j] = u32x4{0, 0, 0, 0};
      }
      uint32_t top = 0;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        take4(d[0][w], d[1][w], d[2][w], d[3][w], s[2 * w], s[2 * w + 1]);
        // the sums are taken here: left to itself, the compiler moves them
        // below the branch and the loads, and spills
        hold(s[2 * w]);
        hold(s[2 * w + 1]);
        top = max_u16x2(top, max_u16x2(max_u16x2(d[0][w], d[1][w]), max_u16x2(d[2][w], d[3][w])));
      }
      if (__ballot(max(top & 0xFFFFu, top >> 16) >= lvl)) {
#pragma unroll
        for (int p = 0; p < kHealthPPL; ++p) {
          uint32_t ns = 0;
#pragma unroll
          for (int j = 0; j < 4; ++j)
            ns += k0 + j < T && ((d[j][p >> 1] >> ((p & 1) * 16)) & 0xFFFFu) >= lvl ? 1u : 0u;
          if (ns) atomicAdd((unsigned long long*)&sum[2][p * lanes + k], (uint64_t)ns);
        }
      }
    };
    u32x4 A[4], B[4];
    int64_t e = u / per_event;
    int k0 = (u - (int)e * per_event) * kGroup;
    const int64_t step_e = step / per_event;
    const int step_k = (step - (int)step_e * per_event) * kGroup;
    const uint16_t* col = base + e * c.event_elems;
    load4(A, col, k0);
    load4(B, col, k0 + 4);
    for (bool more = true; more;) {
#pragma unroll
      for (int p = 0; p < kHealthPPL; ++p) s[p] = {0, 0, 0, 0, 0};
      for (int held = 0; more && held < kFlush; ++held) {
        // the next group: its loads follow the use of their registers
        e += step_e;
        int k1 = k0 + step_k;
        if (k1 >= per_event * kGroup) {
          k1 -= per_event * kGroup;
          ++e;
        }
        more = e < n_evt;
        col = base + e * c.event_elems;
        sums4(A, k0);
        if (more) load4(A, col, k1);
        sums4(B, k0 + 4);
        if (more) load4(B, col, k1 + 4);
        k0 = k1;
      }
#pragma unroll
      for (int p = 0; p < kHealthPPL; ++p) {
        const int o = p * lanes + k;
        atomicAdd((unsigned long long*)&sum[0][o], ((uint64_t)s[p].h << 8) + s[p].l);
        atomicAdd((unsigned long long*)&sum[1][o], ((uint64_t)s[p].hh << 16) + ((uint64_t)s[p].lh << 9) + s[p].ll);
      }
    }
  }
  __syncthreads();
  // padding pixels (i >= N) store zeros
  const int64_t plane = (int64_t)G * np;
  uint64_t* __restrict__ dst = part + (int64_t)blockIdx.x * 3 * plane + (int64_t)g * np;
  for (int o = threadIdx.x; o < np; o += kHealthNT) {
    const int p = o / lanes, i = (o - p * lanes) * kHealthPPL + p;
#pragma unroll
    for (int q = 0; q < 3; ++q) dst[q * plane + o] = i < N ? sum[q][o] : 0ull;
  }
}

__device__ __forceinline__ void pixel_stats(uint64_t s1, uint64_t s2, uint64_t n, double& mean, double& rms) {
#pragma clang fp contract(off)
  const double dn = (double)n;
  mean = (double)s1 / dn;
  const double var = (double)s2 / dn - mean * mean;
  rms = sqrt(var > 0.0 ? var : 0.0);
}

// Sums of the n_part partial blocks, the pixel records and, packed for the
// verdict, acc = [rms][G][Npad], [flags][G][Npad].  A workgroup owns 16
// outputs of a gain; its 16 lane groups sum every 16th block, then LDS adds
// the 16 group sums: 5.1 us for the 12.6 MB of 256 blocks (10.4 for 49 MB of
// 500, with the totals alone as output).
constexpr int kRedOut = 16, kRedSlices = 16;

__global__ __launch_bounds__(kRedOut * kRedSlices) void k_health_reduce(DevCam c, const uint64_t* __restrict__ part,
                                                                        int n_part, int64_t n_evt,
                                                                        rta_health_params prm,
                                                                        uint64_t* __restrict__ acc,
                                                                        rta_pixel_health* __restrict__ pix) {
  __shared__ uint64_t red[3][kRedSlices][kRedOut];
  __shared__ uint64_t tot[3][kRedOut];
  const int N = c.n_pix, np = c.n_pix_pad, G = c.n_gain, g = blockIdx.y;
  const int64_t plane = (int64_t)G * np;
  const int ol = threadIdx.x % kRedOut, sl = threadIdx.x / kRedOut;
  const int o = (int)blockIdx.x * kRedOut + ol;
  uint64_t s[3] = {0, 0, 0};
  if (o < np) {
    constexpr int U = 8;
    const uint64_t* src = part + (int64_t)g * np + o;
    for (int w = sl; w < n_part; w += kRedSlices * U) {
      uint64_t v[3][U];
#pragma unroll
      for (int r = 0; r < U; ++r) {
        const int x = w + kRedSlices * r;
#pragma unroll
        for (int q = 0; q < 3; ++q) v[q][r] = x < n_part ? src[(3 * (int64_t)x + q) * plane] : 0ull;
      }
#pragma unroll
      for (int r = 0; r < U; ++r)
#pragma unroll
        for (int q = 0; q < 3; ++q) s[q] += v[q][r];
    }
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) red[q][sl][ol] = s[q];
  __syncthreads();
  if (sl < 3) {
    uint64_t t = 0;
#pragma unroll
    for (int r = 0; r < kRedSlices; ++r) t += red[sl][r][ol];
    tot[sl][ol] = t;
  }
  __syncthreads();
  const int lanes = np / kHealthPPL, p = o / lanes, i = (o - p * lanes) * kHealthPPL + p;
  if (sl || o >= np || i >= N) return;
  const uint64_t n = (uint64_t)n_evt * (uint64_t)c.n_samp;
  rta_pixel_health h;
  h.n = n;
  h.s1 = tot[0][ol];
  h.s2 = tot[1][ol];
  h.n_sat = tot[2][ol];
  pixel_stats(h.s1, h.s2, n, h.mean, h.rms);
  uint32_t f = 0;
  if (h.rms < (double)prm.rms_dead) f |= RTA_HEALTH_DEAD;
  const double ped = (double)c.P256[g * np + i] / 256.0;
  if (fabs(h.mean - ped) > (double)prm.ped_tol) f |= RTA_HEALTH_PED_SHIFT;
  if ((double)h.n_sat > (double)prm.sat_frac * (double)n) f |= RTA_HEALTH_SATURATING;
  h.flags = f;
  h.pad_ = 0;
  h.reserved_ = 0;
  pix[(int64_t)g * N + i] = h;
  acc[(int64_t)g * np + i] = __builtin_bit_cast(uint64_t, h.rms);
  acc[plane + (int64_t)g * np + i] = f;
}

// Median and verdict in one workgroup, half of it per gain.  A rms is finite
// and not negative, so its bits order as the value does: the lower median's
// bits are narrowed 11 at a time from the top by a histogram of the values
// still in the range, until at most a wavefront's worth is left, which is
// ranked by comparing each with each (two passes on ordinary data, six at
// most).  One workgroup per gain sorting all its values and another launch
// for the verdict took 23.3 us, 8.5 us so.
constexpr int kVerdictNT = 1024, kHalf = kVerdictNT / 2, kMine = kMaxPix / kHalf, kBits = 11;
static_assert(kHalf * (1 << kBits) / kHalf == kMaxPix, "four histogram bins per thread");

__global__ __launch_bounds__(kVerdictNT) void k_health_verdict(DevCam c, const uint64_t* __restrict__ acc,
                                                               rta_health_params prm,
                                                               rta_pixel_health* __restrict__ pix,
                                                               rta_camera_health* __restrict__ out) {
  __shared__ uint32_t hist[2][1 << kBits];
  __shared__ uint64_t cand[2][kWave];
  __shared__ uint64_t prefix[2], median[2];
  __shared__ int32_t wsum[2][kHalf / kWave], rank[2], left[2], n_cand[2];
  __shared__ uint32_t any[kMaxPix / 32];
  const int N = c.n_pix, np = c.n_pix_pad, G = c.n_gain;
  const int g = (int)threadIdx.x / kHalf, t = (int)threadIdx.x % kHalf, lane = t % kWave, wave = t / kWave;
  const int64_t plane = (int64_t)G * np;
  uint64_t v[kMine];
  uint32_t f[kMine];
  bool in[kMine];
#pragma unroll
  for (int e = 0; e < kMine; ++e) {
    const int i = t + kHalf * e;
    in[e] = g < G && i < N;
    v[e] = in[e] ? acc[(int64_t)g * np + i] : 0;
    f[e] = in[e] ? (uint32_t)acc[plane + (int64_t)g * np + i] : 0;
  }
  if (t == 0) {
    prefix[g] = 0;
    median[g] = 0;
    rank[g] = (N - 1) / 2;
    left[g] = g < G ? N : 0;
    n_cand[g] = 0;
  }
  if (threadIdx.x < kMaxPix / 32) any[threadIdx.x] = 0;
  bool cur[kMine];
#pragma unroll
  for (int e = 0; e < kMine; ++e) cur[e] = in[e];
  int shift = 64;
  for (;;) {
    __syncthreads();
    // a gain's range is down to a wavefront's worth, or to one value
    if (shift == 0 || (left[0] <= kWave && left[1] <= kWave)) break;
    const int width = min(shift, kBits);
    shift -= width;
    const uint32_t mask = (1u << width) - 1u;
    for (int b = t; b < (1 << kBits); b += kHalf) hist[g][b] = 0;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kMine; ++e) {
      const uint32_t b = (uint32_t)(v[e] >> shift) & mask;
      // the values of a wavefront that share the first one's bin count as
      // one: most do in the pass over the exponents
      const uint64_t live = __ballot(cur[e]);
      if (!live) continue;
      const int first = __ffsll((unsigned long long)live) - 1;
      const uint32_t b0 = (uint32_t)__builtin_amdgcn_readlane((int)b, first);
      const uint64_t same = __ballot(cur[e] && b == b0);
      if (lane == first) atomicAdd(&hist[g][b0], (uint32_t)__popcll(same));
      else if (cur[e] && b != b0) atomicAdd(&hist[g][b], 1u);
    }
    __syncthreads();
    // four bins per thread: exclusive sums over the wavefront, the half
    int32_t n[4], mine = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) mine += n[b] = (int32_t)hist[g][4 * t + b];
    int32_t inc = mine;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const int32_t up = __shfl_up(inc, d, kWave);
      if (lane >= d) inc += up;
    }
    if (lane == kWave - 1) wsum[g][wave] = inc;
    const int32_t r = rank[g];
    const uint64_t pre = prefix[g];
    __syncthreads();
    int32_t below = inc - mine;
    for (int w = 0; w < wave; ++w) below += wsum[g][w];
    if (r >= below && r < below + mine) {
      int b = 0;
      while (r >= below + n[b]) below += n[b++];
      rank[g] = r - below;
      left[g] = n[b];
      prefix[g] = (pre << width) | (uint64_t)(4 * t + b);
    }
    __syncthreads();
    const uint64_t now = prefix[g];
#pragma unroll
    for (int e = 0; e < kMine; ++e) cur[e] = cur[e] && (v[e] >> shift) == now;
  }
  if (left[g] > kWave) {
    if (t == 0) median[g] = prefix[g];
  } else {
#pragma unroll
    for (int e = 0; e < kMine; ++e)
      if (cur[e]) cand[g][atomicAdd(&n_cand[g], 1)] = v[e];
  }
  __syncthreads();
  if (wave == 0 && lane < n_cand[g]) {
    const uint64_t x = cand[g][lane];
    int less = 0;
    for (int j = 0; j < n_cand[g]; ++j) less += cand[g][j] < x || (cand[g][j] == x && j < lane) ? 1 : 0;
    if (less == rank[g]) median[g] = x;
  }
  __syncthreads();
  const double med = __builtin_bit_cast(double, median[g]);
#pragma unroll
  for (int e = 0; e < kMine; ++e) {
    const int i = t + kHalf * e;
    if (!in[e]) continue;
    if (__builtin_bit_cast(double, v[e]) > (double)prm.noisy_factor * med) {
      f[e] |= RTA_HEALTH_NOISY;
      pix[(int64_t)g * N + i].flags = f[e];
    }
    if (f[e]) atomicOr(&any[i / 32], 1u << (i % 32));
  }
  __syncthreads();
  if (t == 0) out->median_rms[g] = g < G ? med : 0.0;
  if (threadIdx.x < kWave) {
    static_assert(kMaxPix / 32 == kWave, "a word of pixels per lane");
    int bad = __popc(any[threadIdx.x]);
#pragma unroll
    for (int d = kWave / 2; d; d >>= 1) bad += __shfl_xor(bad, d, kWave);
    if (threadIdx.x == 0) {
      out->n_bad = bad;
      out->verdict = (double)bad > (double)prm.bad_frac_max * (double)N ? 1 : 0;
    }
  }
}

}  // namespace

hipError_t launch_health(const DevCam& c, const uint16_t* traces, int64_t n_evt, const rta_health_params& p,
                         uint64_t* part, uint64_t* acc, rta_pixel_health* pix, rta_camera_health* out,
                         hipStream_t st) {
  // one workgroup of 16 wavefronts per compute unit over both gains
  const int per_event = (c.n_samp + kGroup - 1) / kGroup;
  const int64_t n_groups = n_evt * per_event, want = (n_groups + kSlots - 1) / kSlots;
  const int grid = (int)(want < kHealthParts / c.n_gain ? want : kHealthParts / c.n_gain);
  hipLaunchKernelGGL(k_health_accum, dim3((unsigned)grid, (unsigned)c.n_gain), dim3(kHealthNT), 0, st, c, traces,
                     n_evt, per_event, part);
  hipLaunchKernelGGL(k_health_reduce, dim3((unsigned)((c.n_pix_pad + kRedOut - 1) / kRedOut), (unsigned)c.n_gain),
                     dim3(kRedOut * kRedSlices), 0, st, c, (const uint64_t*)part, grid, n_evt, p, acc, pix);
  hipLaunchKernelGGL(k_health_verdict, dim3(1), dim3(kVerdictNT), 0, st, c, (const uint64_t*)acc, p, pix, out);
  return hipGetLastError();
}

}  // namespace rta
