// Device building blocks of the BF16-MFMA network, shared by the training
// kernels (mlp.hip) and the per-array-event kernel (reco.hip).
#pragma once

#include "rta_internal.h"

namespace rta {
namespace mlpdev {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kIn = 10, kHid = 64, kOut = 2;
constexpr int kInPad = 16, kOutPad = 16;


// float -> bfloat16, round to nearest even (finite inputs).
__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Two values rounded to nearest even by v_cvt_pk_bf16_f32: the bits of f2bf
// for every finite or infinite float (all 2^32 patterns compared); a NaN
// stays a NaN.
__device__ __forceinline__ uint32_t pack2(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ bf16x4 pack4(float a, float b, float c, float d) {
  return __builtin_bit_cast(bf16x4, u32x2{pack2(a, b), pack2(c, d)});
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// One 16x16 tile product over K = 16 (v_mfma_f32_16x16x16_bf16).
__device__ __forceinline__ f32x4 mfma(bf16x4 a, bf16x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// One 16x16 tile product over two K = 16 blocks at once
// (v_mfma_f32_16x16x32_bf16): lane group g supplies eight k slots, the
// four of block 0 then the four of block 1 that the K = 16 layout gives it.
// Both operands use the same slot order, so the contraction is the sum over
// both blocks whatever k each slot stands for.
__device__ __forceinline__ f32x4 mfma2(bf16x4 a0, bf16x4 a1, bf16x4 b0, bf16x4 b1, f32x4 c) {
  const bf16x8 a = __builtin_bit_cast(bf16x8, __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7));
  const bf16x8 b = __builtin_bit_cast(bf16x8, __builtin_shufflevector(b0, b1, 0, 1, 2, 3, 4, 5, 6, 7));
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// A operand: 4 consecutive bf16 of row `row` starting at column `col0`.
__device__ __forceinline__ bf16x4 load4(const uint16_t* M, int ld, int row, int col0) {
  return *reinterpret_cast<const bf16x4*>(M + (size_t)row * ld + col0);
}

__device__ __forceinline__ f32x4 bias4(const float* b, int o) {
  f32x4 v;
  v[0] = b[o]; v[1] = b[o + 1]; v[2] = b[o + 2]; v[3] = b[o + 3];
  return v;
}

// max(a, 0) as the median of a, 0 and infinity: the bits of fmaxf(a, 0) for
// every float (all 2^32 patterns compared) in one instruction, where the
// compiler puts a second one before a maximum of a matrix product to quiet
// signalling NaNs.
__device__ __forceinline__ float relu(float a) { return __builtin_amdgcn_fmed3f(a, 0.f, __builtin_inff()); }

__device__ __forceinline__ bf16x4 relu_bf(f32x4 a) { return pack4(relu(a[0]), relu(a[1]), relu(a[2]), relu(a[3])); }

// g * [h > 0] elementwise, rounded to bf16 (h is a ReLU output, >= 0).
__device__ __forceinline__ bf16x4 mask_bf(f32x4 g, bf16x4 h) {
  return pack4(h[0] ? g[0] : 0.f, h[1] ? g[1] : 0.f, h[2] ? g[2] : 0.f, h[3] ? g[3] : 0.f);
}

// Stores a fragment (lane: row b of the batch, features f0 .. f0 + 3)
// feature-major: the four lanes of a quad exchange halfwords until lane j has
// feature f0 + j of the quad's four rows, one 8-byte store instead of four
// 2-byte ones.  b0: the quad's first row.
__device__ __forceinline__ void store4T(uint16_t* MT, int ldb, int f0, int b0, bf16x4 v) {
  const int j = threadIdx.x & 3;
  const u32x2 d = __builtin_bit_cast(u32x2, v);
  // pairs of rows: even lanes keep features 0 and 2 of two rows, odd 1 and 3
  const uint32_t p0 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)d[0], 0xB1, 0xF, 0xF, false);  // lane ^ 1
  const uint32_t p1 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)d[1], 0xB1, 0xF, 0xF, false);
  const uint32_t sel = (j & 1) ? 0x03020706u : 0x05040100u;  // (partner high, own high) or (own low, partner low)
  const uint32_t a0 = __builtin_amdgcn_perm(p0, d[0], sel), a1 = __builtin_amdgcn_perm(p1, d[1], sel);
  // four rows: lanes 0, 1 keep a0, lanes 2, 3 a1
  const uint32_t r = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(j < 2 ? a1 : a0), 0x4E, 0xF, 0xF, false);
  *reinterpret_cast<u32x2*>(MT + (size_t)(f0 + j) * ldb + b0) = j < 2 ? u32x2{a0, r} : u32x2{r, a1};
}

// A wavefront's share of the network's weights: the A-operand fragments of
// every layer and the biases, 132 registers, which cover the whole network
// over the 64 lanes.  Loaded at once, a forward pass waits for memory once
// instead of once per layer, and a wavefront that takes several tiles reads
// the weights once.
struct MlpFrag {
  bf16x4 w1[4], w2[4][4], w3[4][4], w4[4];
  f32x4 b1[4], b2[4], b3[4], b4;
};

__device__ __forceinline__ void mlp_load(const MlpDev& w, MlpFrag& f) {
  const int lane = threadIdx.x & 63, col = lane & 15, grp = lane >> 4;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    f.w1[t] = load4(w.W1t, kInPad, 16 * t + col, 4 * grp);
    f.b1[t] = bias4(w.b1, 16 * t + 4 * grp);
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
#pragma unroll
    for (int u = 0; u < 4; ++u) f.w2[t][u] = load4(w.W2t, kHid, 16 * t + col, 16 * u + 4 * grp);
    f.b2[t] = bias4(w.b2, 16 * t + 4 * grp);
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
#pragma unroll
    for (int u = 0; u < 4; ++u) f.w3[t][u] = load4(w.W3t, kHid, 16 * t + col, 16 * u + 4 * grp);
    f.b3[t] = bias4(w.b3, 16 * t + 4 * grp);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) f.w4[u] = load4(w.W4t, kHid, col, 16 * u + 4 * grp);
  f.b4 = bias4(w.b4, 4 * grp);
}

// Forward of one 16-row tile by one wavefront.  xin: B-operand tile of the
// standardised inputs (lane: row l%16, features 4*(l/16)..+3).  Returns the
// output accumulator (lanes 0..15: [logit, log10 E, 0, 0] of row l%16) and
// the three hidden activations in B-operand layout.
__device__ __forceinline__ f32x4 mlp_forward(const MlpFrag& f, bf16x4 xin, bf16x4 (&h1)[4], bf16x4 (&h2)[4],
                                             bf16x4 (&h3)[4]) {
#pragma unroll
  for (int t = 0; t < 4; ++t) h1[t] = relu_bf(mfma(f.w1[t], xin, f.b1[t]));
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    f32x4 acc = f.b2[t];
#pragma unroll
    for (int u = 0; u < 4; u += 2) acc = mfma2(f.w2[t][u], f.w2[t][u + 1], h1[u], h1[u + 1], acc);
    h2[t] = relu_bf(acc);
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    f32x4 acc = f.b3[t];
#pragma unroll
    for (int u = 0; u < 4; u += 2) acc = mfma2(f.w3[t][u], f.w3[t][u + 1], h2[u], h2[u + 1], acc);
    h3[t] = relu_bf(acc);
  }
  f32x4 out = f.b4;
#pragma unroll
  for (int u = 0; u < 4; u += 2) out = mfma2(f.w4[u], f.w4[u + 1], h3[u], h3[u + 1], out);
  return out;
}

// The same with each layer's weights loaded when it needs them, for kernels
// whose occupancy the 132 registers would cost.
__device__ __forceinline__ f32x4 mlp_forward_tile(const MlpDev& w, bf16x4 xin, bf16x4 (&h1)[4], bf16x4 (&h2)[4],
                                                  bf16x4 (&h3)[4]) {
  const int lane = threadIdx.x & 63, col = lane & 15, grp = lane >> 4;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    f32x4 acc = bias4(w.b1, 16 * t + 4 * grp);
    acc = mfma(load4(w.W1t, kInPad, 16 * t + col, 4 * grp), xin, acc);
    h1[t] = relu_bf(acc);
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    f32x4 acc = bias4(w.b2, 16 * t + 4 * grp);
#pragma unroll
    for (int u = 0; u < 4; u += 2)
      acc = mfma2(load4(w.W2t, kHid, 16 * t + col, 16 * u + 4 * grp),
                  load4(w.W2t, kHid, 16 * t + col, 16 * (u + 1) + 4 * grp), h1[u], h1[u + 1], acc);
    h2[t] = relu_bf(acc);
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    f32x4 acc = bias4(w.b3, 16 * t + 4 * grp);
#pragma unroll
    for (int u = 0; u < 4; u += 2)
      acc = mfma2(load4(w.W3t, kHid, 16 * t + col, 16 * u + 4 * grp),
                  load4(w.W3t, kHid, 16 * t + col, 16 * (u + 1) + 4 * grp), h2[u], h2[u + 1], acc);
    h3[t] = relu_bf(acc);
  }
  f32x4 out = bias4(w.b4, 4 * grp);
#pragma unroll
  for (int u = 0; u < 4; u += 2)
    out = mfma2(load4(w.W4t, kHid, col, 16 * u + 4 * grp), load4(w.W4t, kHid, col, 16 * (u + 1) + 4 * grp), h3[u],
                h3[u + 1], out);
  return out;
}

// The 10 network inputs of a Hillas record.
__device__ __forceinline__ float record_feature(const rta_hillas_rec& r, int f) {
  switch (f) {
    case 0: return log10f(r.size);
    case 1: return r.length;
    case 2: return r.width;
    case 3: return r.cog_dist;
    case 4: return r.psi;
    case 5: return r.skewness;
    case 6: return r.kurtosis;
    case 7: return r.time_gradient;
    case 8: return r.leakage;
    default: return (float)r.n_islands;
  }
}

// Features 4 grp .. 4 grp + 3 of a record (0 past the tenth) for a lane of
// group grp, by selects: a switch on the lane's feature index makes every
// lane step through the branches of all.
__device__ __forceinline__ void record_features4(const rta_hillas_rec& r, int grp, float (&x)[4]) {
  const float lg = record_feature(r, 0);
  x[0] = grp == 0 ? lg : grp == 1 ? r.psi : grp == 2 ? r.leakage : 0.f;
  x[1] = grp == 0 ? r.length : grp == 1 ? r.skewness : grp == 2 ? (float)r.n_islands : 0.f;
  x[2] = grp == 0 ? r.width : grp == 1 ? r.kurtosis : 0.f;
  x[3] = grp == 0 ? r.cog_dist : grp == 1 ? r.time_gradient : 0.f;
}

// The lane's four standardised inputs of a record; a non-finite one is 0
// (such rows fall back to the box cuts).  mean, stdv: at least 16 entries,
// 0 and 1 past the tenth.
__device__ __forceinline__ bf16x4 record_inputs(const float (&x)[4], const float (&mean)[4], const float (&stdv)[4]) {
  float v[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float z = (x[j] - mean[j]) / stdv[j];
    v[j] = isfinite(z) ? z : 0.f;
  }
  return pack4(v[0], v[1], v[2], v[3]);
}

__device__ __forceinline__ void load_scale(const MlpDev& w, int grp, float (&mean)[4], float (&stdv)[4]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    mean[j] = w.mean[4 * grp + j];
    stdv[j] = w.stdv[4 * grp + j];
  }
}

// Standardised input tile from records rec[r0 .. r0+15] (rows >= n are 0).
__device__ __forceinline__ bf16x4 mlp_record_tile(const MlpDev& w, const rta_hillas_rec* rec, int64_t n, int64_t r0) {
  const int lane = threadIdx.x & 63, col = lane & 15, grp = lane >> 4;
  if (r0 + col >= n) return pack4(0.f, 0.f, 0.f, 0.f);
  float x[4], mean[4], stdv[4];
  load_scale(w, grp, mean, stdv);
  record_features4(rec[r0 + col], grp, x);
  return record_inputs(x, mean, stdv);
}

struct ClassOut {
  float score, log10e;
  int gamma, fallback;
};

// Decision for one record: the network's outputs when in_range, else the box
// cuts.  The bin tables (w_mean, w_std, l_mean, l_std) are given apart, so
// that a kernel can keep them where it likes.
__device__ __forceinline__ ClassOut classify_decide(const rta_hillas_rec& r, const rta_boxcut_desc& bc,
                                                    const float* w_mean, const float* w_std, const float* l_mean,
                                                    const float* l_std, bool in_range, float logit, float mlp_e) {
  ClassOut o;
  const float lgs = log10f(r.size);
  if (in_range) {
    o.score = 1.f / (1.f + expf(-logit));
    o.log10e = mlp_e;
    o.gamma = o.score > bc.mlp_cut;
    o.fallback = 0;
  } else {
    int b = (int)floorf((lgs - bc.lgs_lo) / (bc.lgs_hi - bc.lgs_lo) * (float)bc.n_bins);
    b = b < 0 ? 0 : (b >= bc.n_bins ? bc.n_bins - 1 : b);
    const float sw = (r.width - w_mean[b]) / w_std[b];
    const float sl = (r.length - l_mean[b]) / l_std[b];
    o.gamma = (sw < bc.cut_w) && (sl < bc.cut_l);
    o.score = o.gamma ? 1.f : 0.f;
    o.log10e = bc.e_a + bc.e_b * lgs;
    o.fallback = 1;
  }
  return o;
}

// The same given the network outputs (have_mlp): the network is used when
// every feature is finite and inside the trained range.
__device__ __forceinline__ ClassOut classify_record(const rta_hillas_rec& r, const rta_boxcut_desc& bc, bool have_mlp,
                                                    float logit, float mlp_e) {
  bool in_range = have_mlp;
#pragma unroll
  for (int f = 0; f < kIn; ++f) {
    const float v = record_feature(r, f);
    in_range = in_range && isfinite(v) && v >= bc.feat_lo[f] && v <= bc.feat_hi[f];
  }
  return classify_decide(r, bc, bc.w_mean, bc.w_std, bc.l_mean, bc.l_std, in_range, logit, mlp_e);
}

}  // namespace mlpdev
}  // namespace rta
