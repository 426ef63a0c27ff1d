// HIP kernels of the science alert monitor for gfx950 (CDNA4).
//
// The real-time analysis searches its event list for transients on several
// integration timescales, in a source region and anywhere in the field of
// view (paper, Section 2 requirement (ii); Section 4.2).  The definitions are
// in rta.h.  Three small data-parallel steps:
//   fill     one thread per event: selection, FP64 time bin and sky cell,
//            an integer atomic increment of the counts cube (exact and
//            independent of the order of events);
//   window   one thread per (timescale, 64-bin chunk of the window, cell):
//            the chunk's sum (16 loads in flight, consecutive threads on
//            consecutive cells of a bin) added to the window sum with an
//            integer atomic, so every bin of the longest window is read by
//            its own thread rather than in one long chain;
//   search   one thread per (timescale, cell): on-disc and background-ring
//            sums over a host-built offset list from a tile of the window
//            sums in LDS, alpha from the cells counted inside the grid when
//            the monitor is made, the Li & Ma significance in FP64 with the
//            zero excess decided in integers, alerts appended through an
//            atomic counter.
#include <algorithm>
#include <cmath>

#include "rta_internal.h"

namespace rta {
namespace {

// n zeros from p (16-byte aligned): 16-byte stores, 59 MB in 10 us (4-byte
// ones took 16.4).
__global__ __launch_bounds__(256) void k_sam_clear(int32_t* p, int64_t n) {
  const int64_t i0 = (int64_t)blockIdx.x * 256 + threadIdx.x, step = (int64_t)gridDim.x * 256;
  int4* q = reinterpret_cast<int4*>(p);
  for (int64_t i = i0; i < n / 4; i += step) q[i] = make_int4(0, 0, 0, 0);
  if (i0 < n % 4) p[n / 4 * 4 + i0] = 0;
}

// The same over the window sums, and the alert counter: one launch of 2.0 us for
// two of 3.2 us together.
__global__ __launch_bounds__(256) void k_sam_reset(int32_t* win, int64_t n, int32_t* n_alerts) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) win[i] = 0;
  if (i == 0) *n_alerts = 0;
}

__global__ void k_sam_fill(SamDev d, const rta_event_rec* __restrict__ evt, const double* __restrict__ t,
                           int64_t n) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const rta_event_rec e = evt[k];
  if (e.flags & RTA_EVT_STEREO_INVALID) return;
  if (!(e.gammaness >= d.gamma_cut)) return;
  const double fb = floor((t[k] - d.t0) / d.bin_s);
  const double half = 0.5 * (double)d.grid;
  const double fx = floor((double)e.dir_x / (double)d.cell + half);
  const double fy = floor((double)e.dir_y / (double)d.cell + half);
  if (!(fb >= 0.0 && fb < (double)d.n_bins && fx >= 0.0 && fx < (double)d.grid && fy >= 0.0 &&
        fy < (double)d.grid))
    return;
  const int64_t G = d.grid;
  atomicAdd(&d.counts[((int64_t)fb * G + (int64_t)fy) * G + (int64_t)fx], 1);
}

// Window jobs of one search: the chunks of timescale s are jobs
// [job0[s], job0[s + 1]), chunk j of it covers bins lo[s] + 64 j .. up to
// end_bin.
constexpr int kSamChunk = 64;
struct SamJobs {
  int32_t job0[RTA_SAM_MAX_SCALES + 1];
  int32_t lo[RTA_SAM_MAX_SCALES];
};

__global__ void k_sam_window(SamDev d, int end_bin, SamJobs jb) {
  const int64_t G2 = (int64_t)d.grid * d.grid;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t job = i / G2;
  if (job >= jb.job0[d.n_scales]) return;
  const int64_t cell = i - job * G2;
  int s = 0;
  while (job >= jb.job0[s + 1]) ++s;
  const int b0 = jb.lo[s] + (int)(job - jb.job0[s]) * kSamChunk;
  const int b1 = min(b0 + kSamChunk, end_bin + 1);
  const int32_t* __restrict__ src = d.counts + cell;
  int32_t acc = 0;
  int b = b0;
  for (; b + 16 <= b1; b += 16) {
    int32_t v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = src[(int64_t)(b + u) * G2];
#pragma unroll
    for (int u = 0; u < 16; ++u) acc += v[u];
  }
  for (; b < b1; ++b) acc += src[(int64_t)b * G2];
  if (acc) atomicAdd(&d.win[s * G2 + cell], acc);
}

__device__ double li_ma(int64_t n_on, int64_t n_off, int64_t c_on, int64_t c_off) {
  if (c_off <= 0 || n_on * c_off == c_on * n_off) return 0.0;
  const double on = (double)n_on, off = (double)n_off, alpha = (double)c_on / (double)c_off;
  const double tot = on + off;
  const double t1 = n_on > 0 ? on * log((1.0 + alpha) / alpha * on / tot) : 0.0;
  const double t2 = n_off > 0 ? off * log((1.0 + alpha) * off / tot) : 0.0;
  const double v = fmax(2.0 * (t1 + t2), 0.0);
  return copysign(sqrt(v), on - alpha * off);
}

// Cells of the disc and of the ring that lie inside the grid, per cell: they
// depend on the geometry alone and are counted when the monitor is made.
__global__ __launch_bounds__(256) void k_sam_cells(SamDev d) {
  const int G = d.grid, i = (int)(blockIdx.x * 256 + threadIdx.x);
  if (i >= G * G) return;
  const int y = i / G, x = i - y * G;
  int32_t c[2] = {0, 0};
  for (int k = 0; k < d.n_offs; ++k) {
    const int32_t o = d.offs[k];
    const int xx = x + (o & 0xFF) - 128, yy = y + ((o >> 8) & 0xFF) - 128;
    c[k < d.n_disc ? 0 : 1] += xx >= 0 && xx < G && yy >= 0 && yy < G ? 1 : 0;
  }
  d.cells[2 * i] = c[0];
  d.cells[2 * i + 1] = c[1];
}

// A workgroup takes up to 256 cells of one timescale, whole rows of the grid,
// with the rows and columns within reach around them in LDS (zero outside the
// grid), so the sums over the disc and then the ring read LDS at wave-uniform
// offsets that scalar loads bring 16 at a time.  With every thread reading the
// window sums from L2 behind bounds checks and counting its cells again, 5
// timescales of 64 x 64 cells and 141 offsets took 16.4 us; 9.8 us so, a chain
// of latencies on 80 of the 256 CUs.  With the offsets unsorted and a branch on
// the kind of each one, the same tiles take 27.9 us.
constexpr int kSearchNT = 256;
constexpr int kTileInts = (1 + 2 * RTA_SAM_MAX_REACH) * (RTA_SAM_MAX_GRID + 2 * RTA_SAM_MAX_REACH);

// Rows of cells per workgroup.
__host__ __device__ inline int search_rows(int grid) {
  const int r = kSearchNT / grid;
  return r < grid ? (r > 1 ? r : 1) : grid;
}

__global__ __launch_bounds__(kSearchNT) void k_sam_search(SamDev d, double* __restrict__ sig,
                                                          int32_t* __restrict__ non_out,
                                                          int32_t* __restrict__ noff_out,
                                                          rta_sam_alert* __restrict__ alerts, int max_alerts,
                                                          int32_t* n_alerts) {
  __shared__ int32_t tile[kTileInts];
  const int G = d.grid, R = d.reach, rows = search_rows(G), ld = G + 2 * R;
  const int s = (int)blockIdx.y, y0 = (int)blockIdx.x * rows;
  const int64_t G2 = (int64_t)G * G;
  const int32_t* W = d.win + s * G2;
  const int r = (int)threadIdx.x / G, x = (int)threadIdx.x - r * G, y = y0 + r;
  const bool mine = r < rows && y < G;
  int2 cells = make_int2(0, 0);
  if (mine) cells = *reinterpret_cast<const int2*>(d.cells + 2 * ((int64_t)y * G + x));
  const int n_tile = (rows + 2 * R) * ld;
  int ty = (int)threadIdx.x / ld, tx = (int)threadIdx.x - ty * ld;
  for (int i = threadIdx.x; i < n_tile;) {
    constexpr int U = 8;
    int32_t v[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int yy = y0 + ty - R, xx = tx - R;
      v[k] = 0;
      if (i + k * kSearchNT < n_tile && yy >= 0 && yy < G && xx >= 0 && xx < G) v[k] = W[(int64_t)yy * G + xx];
      for (tx += kSearchNT; tx >= ld; tx -= ld) ++ty;
    }
#pragma unroll
    for (int k = 0; k < U; ++k)
      if (i + k * kSearchNT < n_tile) tile[i + k * kSearchNT] = v[k];
    i += U * kSearchNT;
  }
  __syncthreads();
  if (!mine) return;
  const int32_t* at = tile + (r + R) * ld + x + R;
  int64_t n_on = 0, n_off = 0;
#pragma unroll 16
  for (int k = 0; k < d.n_disc; ++k) n_on += at[d.deltas[k]];
#pragma unroll 16
  for (int k = d.n_disc; k < d.n_offs; ++k) n_off += at[d.deltas[k]];
  const int64_t i = s * G2 + (int64_t)y * G + x;
  const double S = li_ma(n_on, n_off, cells.x, cells.y);
  if (sig) sig[i] = S;
  if (non_out) non_out[i] = (int32_t)n_on;
  if (noff_out) noff_out[i] = (int32_t)n_off;
  if (S >= (double)d.sigma_alert) {
    const int slot = atomicAdd(n_alerts, 1);
    if (slot < max_alerts) {
      rta_sam_alert a;
      a.scale = s;
      a.ix = x;
      a.iy = y;
      a.n_on = (int32_t)n_on;
      a.significance = S;
      a.n_off = (int32_t)n_off;
      a.pad_ = 0;
      alerts[slot] = a;
    }
  }
}

unsigned blocks_for(int64_t n, int nt) { return (unsigned)((n + nt - 1) / nt); }

}  // namespace

hipError_t launch_sam_clear(const SamDev& d, hipStream_t st) {
  const int64_t n = (int64_t)d.n_bins * d.grid * d.grid;
  const int64_t blocks = std::min<int64_t>((n / 4 + 256) / 256, 65536);
  hipLaunchKernelGGL(k_sam_clear, dim3((unsigned)blocks), dim3(256), 0, st, d.counts, n);
  return hipGetLastError();
}

hipError_t launch_sam_cells(const SamDev& d, hipStream_t st) {
  hipLaunchKernelGGL(k_sam_cells, dim3(blocks_for((int64_t)d.grid * d.grid, 256)), dim3(256), 0, st, d);
  return hipGetLastError();
}

hipError_t launch_sam_fill(const SamDev& d, const rta_event_rec* evt, const double* t, int64_t n, hipStream_t st) {
  hipLaunchKernelGGL(k_sam_fill, dim3(blocks_for(n, 256)), dim3(256), 0, st, d, evt, t, n);
  return hipGetLastError();
}

hipError_t launch_sam_search(const SamDev& d, int end_bin, double* sig, int32_t* n_on, int32_t* n_off,
                             rta_sam_alert* alerts, int max_alerts, int32_t* n_alerts, hipStream_t st) {
  const int64_t G2 = (int64_t)d.grid * d.grid, n = (int64_t)d.n_scales * G2;
  SamJobs jb;
  jb.job0[0] = 0;
  for (int s = 0; s < d.n_scales; ++s) {
    jb.lo[s] = std::max(end_bin - d.scales[s] + 1, 0);
    jb.job0[s + 1] = jb.job0[s] + (end_bin - jb.lo[s] + kSamChunk) / kSamChunk;
  }
  hipLaunchKernelGGL(k_sam_reset, dim3(blocks_for(n, 256)), dim3(256), 0, st, d.win, n, n_alerts);
  hipLaunchKernelGGL(k_sam_window, dim3(blocks_for(jb.job0[d.n_scales] * G2, 256)), dim3(256), 0, st, d, end_bin,
                     jb);
  const int rows = search_rows(d.grid);
  hipLaunchKernelGGL(k_sam_search, dim3((unsigned)((d.grid + rows - 1) / rows), (unsigned)d.n_scales),
                     dim3(kSearchNT), 0, st, d, sig, n_on, n_off, alerts, max_alerts, n_alerts);
  return hipGetLastError();
}

}  // namespace rta
