// Gamma/hadron + energy network on BF16 matrix cores (gfx950 MFMA).
//
// The network (10 -> 64 -> 64 -> 64 -> 2, ReLU) maps per-telescope image
// parameters to a gamma logit and log10(E/TeV); it fills the gamma/hadron
// separation and energy steps that the paper lists among the reconstruction
// products (Section 4.1).  Operands are bfloat16, accumulation FP32.
//
// Register layout.  Every layer is computed transposed, Z^T = W^T . H^T, on
// 16x16 tiles: A = a block of W^T (rows = output features), B = a block of
// H^T (features x 16 rows), C/D = 16 output features x 16 rows.  In that
// orientation the accumulator layout (lane l: row-of-batch l%16, features
// 4*(l/16)..+3) is exactly the B-operand layout of a 16-feature block, so
// activations go from one layer to the next in registers.  Contractions over
// 64 features (or over the batch) take two 16-blocks per
// v_mfma_f32_16x16x32_bf16, the two blocks' B fragments side by side; the
// 16-wide input and output layers use v_mfma_f32_16x16x16_bf16.
// The backward pass uses the same trick with the untransposed weights.  Weight
// gradients contract over the batch, so per-row activations and gradients are
// written feature-major ([F][B], bf16) and wavefronts, one per 16x16 weight
// tile and batch slice, run the batch contraction with the same instruction.
#include <cmath>

#include "mlp_device.h"
#include "mlp_launch.h"

namespace rta {
using namespace mlpdev;
constexpr int kRowsNT = 64;  // one wavefront, 16 rows

namespace {

// Forward (+ loss, + backward to every layer's pre-activation gradient when
// TRAIN) of 16-row tiles, a single-wavefront workgroup each: a batch of 4096
// is 256 tiles, one per compute unit.  rows != null (TRAIN): batch row b is
// data row rows[b] of x / label / log10e (the batch gather done here instead
// of in separate copies).  A tile is one chain of dependent layers, bound by
// latency: all weights, forward and backward, are loaded into registers at
// the start (204 of them), while the row indices and then the rows arrive,
// instead of layer by layer; the activations and gradients are transposed in
// registers and stored 8 bytes per lane.  B = 4096: 15.4 -> 8.5 us.
// Forward only, a wavefront takes tiles in turn and keeps the weights: 10^6
// rows 284 -> 55 us.  (Training wavefronts that did so needed 292 registers:
// 10 us at B = 4096.)
struct BackFrag {
  bf16x4 w4[4], w3[4][4], w2[4][4];
};

template <bool TRAIN>
__global__ __launch_bounds__(kRowsNT) void k_mlp_rows(MlpDev w, const float* __restrict__ x,
                                                      const float* __restrict__ label,
                                                      const float* __restrict__ log10e,
                                                      const int64_t* __restrict__ rows, int64_t n_data, int B,
                                                      int Bpad, float* __restrict__ out) {
  const int lane = threadIdx.x & 63, col = lane & 15, grp = lane >> 4;
  // data row of this lane's batch row, asked for ahead of the weights, since
  // the row's own loads wait for it
  int64_t db = (int64_t)blockIdx.x * 16 + col;
  if (TRAIN && rows && db < B) db = min(max(rows[db], (int64_t)0), n_data - 1);
  MlpFrag net;
  mlp_load(w, net);
  BackFrag back;
  if constexpr (TRAIN) {
#pragma unroll
    for (int t = 0; t < 4; ++t) back.w4[t] = load4(w.W4n, kOutPad, 16 * t + col, 4 * grp);
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        back.w3[t][u] = load4(w.W3n, kHid, 16 * t + col, 16 * u + 4 * grp);
        back.w2[t][u] = load4(w.W2n, kHid, 16 * t + col, 16 * u + 4 * grp);
      }
  }
  float mean[4], stdv[4];
  load_scale(w, grp, mean, stdv);
  for (int64_t r0 = (int64_t)blockIdx.x * 16; r0 < Bpad; r0 += (int64_t)gridDim.x * 16) {
    const int b = (int)r0 + col;
    const bool valid = b < B;
    float v[4], lab = 0.f, y = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int f = 4 * grp + j;
      v[j] = (valid && f < kIn) ? (x[db * kIn + f] - mean[j]) / stdv[j] : 0.f;
    }
    if (TRAIN && valid) {
      lab = label[db];
      y = log10e[db];
    }
    if constexpr (!TRAIN) db = r0 + (int64_t)gridDim.x * 16 + col;  // (no row gather without training)
    __builtin_amdgcn_sched_barrier(0);  // every load is issued before the first layer
    const bf16x4 xin = pack4(v[0], v[1], v[2], v[3]);
    bf16x4 h1[4], h2[4], h3[4];
    const f32x4 o = mlp_forward(net, xin, h1, h2, h3);
    if (!TRAIN) {
      if (grp == 0 && valid) {
        out[(size_t)b * 2] = o[0];
        out[(size_t)b * 2 + 1] = o[1];
      }
      continue;
    }
    // loss and output gradient (lanes of group 0 own the two outputs of row b)
    float g0 = 0.f, g1 = 0.f;
    if (grp == 0) {
      float lrow = 0.f;
      if (valid) {
        const float z = o[0], e = o[1];
        const float m = lab > 0.5f ? 1.f : 0.f;
        const float sig = 1.f / (1.f + expf(-z));
        lrow = fmaxf(z, 0.f) - z * lab + log1pf(expf(-fabsf(z))) + m * (e - y) * (e - y);
        g0 = (sig - lab) / (float)B;
        g1 = 2.f * m * (e - y) / (float)B;
      }
      w.loss_row[b] = lrow;
    }
    const bf16x4 g4 = pack4(g0, g1, 0.f, 0.f);
    // dH3^T = W4 . G4^T, masked -> G3; then G2, G1
    bf16x4 g3[4], g2[4], g1v[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
      g3[t] = mask_bf(mfma(back.w4[t], g4, zero), h3[t]);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = 0; u < 4; u += 2) acc = mfma2(back.w3[t][u], back.w3[t][u + 1], g3[u], g3[u + 1], acc);
      g2[t] = mask_bf(acc, h2[t]);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = 0; u < 4; u += 2) acc = mfma2(back.w2[t][u], back.w2[t][u + 1], g2[u], g2[u + 1], acc);
      g1v[t] = mask_bf(acc, h1[t]);
    }
    // H^T and G^T (feature-major) for the weight-gradient contraction
    const int b0 = b & ~3;
    store4T(w.H0, Bpad, 4 * grp, b0, xin);
    store4T(w.G4, Bpad, 4 * grp, b0, g4);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      store4T(w.H1, Bpad, 16 * t + 4 * grp, b0, h1[t]);
      store4T(w.H2, Bpad, 16 * t + 4 * grp, b0, h2[t]);
      store4T(w.H3, Bpad, 16 * t + 4 * grp, b0, h3[t]);
      store4T(w.G3, Bpad, 16 * t + 4 * grp, b0, g3[t]);
      store4T(w.G2, Bpad, 16 * t + 4 * grp, b0, g2[t]);
      store4T(w.G1, Bpad, 16 * t + 4 * grp, b0, g1v[t]);
    }
    break;  // one tile per wavefront
  }
}

// Weight / bias gradients and the loss.  The batch contraction of each 16x16
// weight tile (40) and block of 16 biases (13) is cut into kGradSplit slices of
// consecutive 16-row blocks, one wavefront per (tile, slice), each writing
// its partial sums to gpart[slice]; a last wavefront sums the loss.  The
// slices are added in slice order by grad_sum (fixed order: the gradient is
// reproducible).  One long contraction per tile would leave the chip nearly
// idle and every step waiting on the previous load.  A slice of up to 16
// blocks (a batch of 4096) has all its loads in flight at once, and the loss
// 32 rows per lane: 7.2 -> 5.7 us, two latencies and the launch.
constexpr int kGradTiles = 53;
constexpr int kGradBlocks = kGradTiles * kGradSplit + 1;

__global__ __launch_bounds__(64) void k_mlp_grad(MlpDev w, int B, int Bpad, float* __restrict__ loss_out) {
  const int lane = threadIdx.x, col = lane & 15, grp = lane >> 4;
  if (blockIdx.x == kGradTiles * kGradSplit) {
    // 32 loads in flight per step, added in row order
    float s = 0.f;
    for (int r = lane; r < B; r += 64 * 32) {
      float v[32];
#pragma unroll
      for (int u = 0; u < 32; ++u) v[u] = r + 64 * u < B ? w.loss_row[r + 64 * u] : 0.f;
#pragma unroll
      for (int u = 0; u < 32; ++u)
        if (r + 64 * u < B) s += v[u];
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) {
      const float L = s / (float)B;
      if (loss_out) *loss_out = L;
      w.loss_row[Bpad] = L;
    }
    return;
  }
  const int wv = blockIdx.x / kGradSplit, sl = blockIdx.x % kGradSplit;
  const int nk = Bpad / 16, per = (nk + kGradSplit - 1) / kGradSplit;
  const int k0 = min(nk, sl * per), k1 = min(nk, k0 + per);
  float* __restrict__ part = w.gpart + (size_t)sl * kNParams;
  // tile -> (layer, input chunk, output chunk); biases: a row of ones as input
  const uint16_t *H = nullptr, *G;
  int in0 = 0, out0, in_dim = 1, out_dim, off;
  if (wv < 4) { H = w.H0; G = w.G1; out0 = 16 * wv; in_dim = kIn; out_dim = kHid; off = kOffW1; }
  else if (wv < 20) { const int t = wv - 4; H = w.H1; G = w.G2; in0 = 16 * (t / 4); out0 = 16 * (t % 4); in_dim = kHid; out_dim = kHid; off = kOffW2; }
  else if (wv < 36) { const int t = wv - 20; H = w.H2; G = w.G3; in0 = 16 * (t / 4); out0 = 16 * (t % 4); in_dim = kHid; out_dim = kHid; off = kOffW3; }
  else if (wv < 40) { H = w.H3; G = w.G4; in0 = 16 * (wv - 36); out0 = 0; in_dim = kHid; out_dim = kOut; off = kOffW4; }
  else if (wv < 52) {
    const int l = (wv - 40) / 4;
    G = l == 0 ? w.G1 : l == 1 ? w.G2 : w.G3;
    out0 = 16 * (wv & 3); out_dim = kHid; off = l == 0 ? kOffB1 : l == 1 ? kOffB2 : kOffB3;
  } else { G = w.G4; out0 = 0; out_dim = kOut; off = kOffB4; }
  bf16x4 ones;
  ones[0] = ones[1] = ones[2] = ones[3] = (short)0x3F80;  // bf16(1.0)
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  constexpr int U = 16;  // 16-row blocks loaded before their MFMAs
  for (int k = k0; k < k1; k += U) {
    bf16x4 a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (k + u < k1) {
        a[u] = H ? load4(H, Bpad, in0 + col, 16 * (k + u) + 4 * grp) : ones;
        b[u] = load4(G, Bpad, out0 + col, 16 * (k + u) + 4 * grp);
      }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; u += 2) {
      if (k + u + 1 < k1)
        acc = mfma2(a[u], a[u + 1], b[u], b[u + 1], acc);
      else if (k + u < k1)
        acc = mfma(a[u], b[u], acc);
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = in0 + 4 * grp + i, n = out0 + col;
    if (m < in_dim && n < out_dim) part[off + m * out_dim + n] = acc[i];
  }
}

// Gradient of parameter p: the slice partials added in slice order.
__device__ __forceinline__ float grad_sum(const MlpDev& w, int p) {
  float g = 0.f;
#pragma unroll
  for (int s = 0; s < kGradSplit; ++s) g += w.gpart[(size_t)s * kNParams + p];
  return g;
}

__global__ __launch_bounds__(256) void k_mlp_grad_sum(MlpDev w) {
  const int p = blockIdx.x * 256 + threadIdx.x;
  if (p < kNParams) w.grad[p] = grad_sum(w, p);
}

// Parameter index -> bf16 copies in both orientations.
__device__ __forceinline__ void write_bf16_copies(const MlpDev& w, int p, float v) {
  const uint16_t h = f2bf(v);
  if (p < kOffB1) {
    const int i = p / kHid, o = p % kHid;
    w.W1t[o * kInPad + i] = h;
  } else if (p < kOffW2) {
    w.b1[p - kOffB1] = v;
  } else if (p < kOffB2) {
    const int q = p - kOffW2, i = q / kHid, o = q % kHid;
    w.W2t[o * kHid + i] = h;
    w.W2n[i * kHid + o] = h;
  } else if (p < kOffW3) {
    w.b2[p - kOffB2] = v;
  } else if (p < kOffB3) {
    const int q = p - kOffW3, i = q / kHid, o = q % kHid;
    w.W3t[o * kHid + i] = h;
    w.W3n[i * kHid + o] = h;
  } else if (p < kOffW4) {
    w.b3[p - kOffB3] = v;
  } else if (p < kOffB4) {
    const int q = p - kOffW4, i = q / kOut, o = q % kOut;
    w.W4t[o * kHid + i] = h;
    w.W4n[i * kOutPad + o] = h;
  } else {
    w.b4[p - kOffB4] = v;
  }
}

// Adam step on the FP32 master weights with the gradient summed from the
// slice partials (update == 0: only refresh the bf16 copies from the
// masters).  c1 = 1/(1 - beta1^t), c2 = 1/(1 - beta2^t).
__global__ __launch_bounds__(256) void k_mlp_adam(MlpDev w, int update, float lr, float b1, float b2, float eps,
                                                  float c1, float c2) {
  const int p = blockIdx.x * 256 + threadIdx.x;
  if (p >= kNParams) return;
  float v = w.master[p];
  if (update) {
    const float g = grad_sum(w, p);
    w.grad[p] = g;
    const float m = b1 * w.m1[p] + (1.f - b1) * g;
    const float s = b2 * w.m2[p] + (1.f - b2) * g * g;
    w.m1[p] = m;
    w.m2[p] = s;
    v -= lr * (m * c1) / (sqrtf(s * c2) + eps);
    w.master[p] = v;
  }
  write_bf16_copies(w, p, v);
}

}  // namespace

hipError_t launch_mlp_rows(const MlpDev& w, const float* x, const float* label, const float* log10e, int B, int Bpad,
                           int n_cu, float* out, bool train, hipStream_t st) {
  return launch_mlp_rows_gather(w, x, label, log10e, nullptr, 0, B, Bpad, n_cu, out, train, st);
}

hipError_t launch_mlp_rows_gather(const MlpDev& w, const float* x, const float* label, const float* log10e,
                                  const int64_t* rows, int64_t n_data, int B, int Bpad, int n_cu, float* out,
                                  bool train, hipStream_t st) {
  // forward: three wavefronts per SIMD, as the registers allow, then tiles in turn
  const int grid = train || Bpad / 16 < 12 * n_cu ? Bpad / 16 : 12 * n_cu;
  if (train)
    hipLaunchKernelGGL(k_mlp_rows<true>, dim3(grid), dim3(kRowsNT), 0, st, w, x, label, log10e, rows, n_data, B,
                       Bpad, out);
  else
    hipLaunchKernelGGL(k_mlp_rows<false>, dim3(grid), dim3(kRowsNT), 0, st, w, x, label, log10e, rows, n_data, B,
                       Bpad, out);
  return hipGetLastError();
}

hipError_t launch_mlp_grad(const MlpDev& w, int B, int Bpad, float* loss_out, hipStream_t st) {
  hipLaunchKernelGGL(k_mlp_grad, dim3(kGradBlocks), dim3(64), 0, st, w, B, Bpad, loss_out);
  return hipGetLastError();
}

hipError_t launch_mlp_grad_sum(const MlpDev& w, hipStream_t st) {
  hipLaunchKernelGGL(k_mlp_grad_sum, dim3((kNParams + 255) / 256), dim3(256), 0, st, w);
  return hipGetLastError();
}

hipError_t launch_mlp_adam(const MlpDev& w, bool update, float lr, float b1, float b2, float eps, float c1, float c2,
                           hipStream_t st) {
  hipLaunchKernelGGL(k_mlp_adam, dim3((kNParams + 255) / 256), dim3(256), 0, st, w, update ? 1 : 0, lr, b1, b2, eps,
                     c1, c2);
  return hipGetLastError();
}

}  // namespace rta
