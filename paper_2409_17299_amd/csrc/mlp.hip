// mlp.hip -- inference and training kernels of the inverse-CDF surrogate
// (2 -> 64 -> 64 -> 1, SiLU).  One wave evaluates 32 samples at a time: lane l
// and lane l + 32 share sample l % 32 and each holds 32 of the 64 hidden
// features of every layer (the slot mapping of mlp.h).  Layer 2 and the
// back-propagation through it are BF16 MFMA with FP32 accumulation (BF16
// weights; activations as a hi + lo pair of bfloat16 numbers); the weight
// gradients are MFMA products over the sample dimension after an LDS
// transpose.  Reductions over waves are in a fixed order, so a training run is
// deterministic.
#include "mlp.h"
#include "physics.h"

namespace sfqed {

namespace {

__device__ __forceinline__ float sigm(float z) { return __builtin_amdgcn_rcpf(1.f + __expf(-z)); }

__device__ __forceinline__ float silu(float z) { return z * sigm(z); }

__device__ __forceinline__ bf16x8 frag_load(const uint16_t* p) {
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(p));
}

__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ uint16_t bf16_bits(float v) { return __builtin_bit_cast(uint16_t, (__bf16)v); }

// The parameters one lane needs, in registers for the whole kernel.
struct LaneParams {
  bf16x8 w2[2][4];
  float4 p1[32];  // slot s*8+i: W1[phi][0], W1[phi][1], b1[phi], b2[phi]
  float w3[32];
  float b3;
};

__device__ __forceinline__ void load_params(const MlpPacked* W, int lane, LaneParams& P) {
  const int h = lane >> 5;
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int s = 0; s < 4; ++s) P.w2[mt][s] = frag_load(W->w2a[mt][s][lane]);
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int f = mlp_phi(s, h, i);
      P.p1[s * 8 + i] = W->p1[f];
      P.w3[s * 8 + i] = W->w3[f];
    }
  P.b3 = W->b3;
}

// Layer 1 in FP32 and its SiLU.  Each activation leaves as two bfloat16
// numbers, hi = bf16(h) and lo = bf16(h - hi), the B operands of layer 2, so
// that the product sees h to about 16 significant bits (z1 and sigmoid(z1)
// optionally kept for the backward pass).
template <bool kKeep>
__device__ __forceinline__ void layer1(const LaneParams& P, float f1, float f2, bf16x8 hb[4], bf16x8 lb[4],
                                       float* z1, float* s1) {
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float4 q = P.p1[s * 8 + i];
      const float z = fmaf(q.x, f1, fmaf(q.y, f2, q.z));
      const float sg = sigm(z);
      const float h = z * sg;
      const __bf16 hi = (__bf16)h;
      hb[s][i] = hi;
      lb[s][i] = (__bf16)(h - (float)hi);
      if constexpr (kKeep) {
        z1[s * 8 + i] = z;
        s1[s * 8 + i] = sg;
      }
    }
}

// z2 (without bias) = W2 (hi + lo), or W2 b for a single operand.
__device__ __forceinline__ void layer2(const bf16x8 w[2][4], const bf16x8 b[4], const bf16x8* lo, f32x16 acc[2]) {
#pragma unroll
  for (int mt = 0; mt < 2; ++mt) {
    f32x16 c = {};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      c = mfma(w[mt][s], b[s], c);
      if (lo) c = mfma(w[mt][s], lo[s], c);
    }
    acc[mt] = c;
  }
}

// Network output for the lane's sample (both lanes of a sample get it).
__device__ __forceinline__ float forward(const LaneParams& P, float f1, float f2) {
  bf16x8 hb[4], lb[4];
  layer1<false>(P, f1, f2, hb, lb, nullptr, nullptr);
  f32x16 acc[2];
  layer2(P.w2, hb, lb, acc);
  float y = 0.f;
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float z = acc[mt][r] + P.p1[16 * mt + r].w;
      y = fmaf(P.w3[16 * mt + r], z * sigm(z), y);
    }
  y += __shfl_xor(y, 32);
  return y + P.b3;
}

// Inference keeps the weights of layers 1 and 2 and the layer-2 biases in
// registers and reads b1 and w3 (per feature slot) from LDS, where the two
// halves of a wave each read one address: two waves per SIMD.  It is bound by
// issue (128 SiLU a sample; the vector units issue 92% of the time), so what
// counts is instructions: b2 is the C operand of the first product instead of
// an addition, h - bf16(h) is one two-term dot product instead of unpacking and
// subtracting (exact either way), and what comes before and after the network
// is done once per sample (forward_infer).  1e7 samples 444 -> 392 us.
struct InferParams {
  bf16x8 w2[2][4];
  float w1a[32], w1b[32];  // slot s*8+i: feature phi(s, h, i)
  f32x16 b2[2];
  float b3;
};

// For h = 0, 1 and slot = 0..31 (feature f = phi(slot / 8, h, slot % 8)):
// l1[h][slot] = b1[f], l3[h][slot] = w3[f].  The whole block calls this (it
// synchronises).  The weights of layer 1 and the biases go through LDS (p1): read
// by every lane from memory they are 32 loads of 16 bytes a lane, 3 us of a
// wave's start, which calls of 1e5 samples, 32 a wave, do not hide.
__device__ __forceinline__ void load_infer_params(const MlpPacked* W, int lane, InferParams& P, float4* p1,
                                                  float (*l1)[32], float (*l3)[32]) {
  const int h = lane >> 5;
  if (threadIdx.x < 64) {
    const int hh = threadIdx.x >> 5, q = threadIdx.x & 31, f = mlp_phi(q >> 3, hh, q & 7);
    p1[threadIdx.x] = W->p1[threadIdx.x];
    l1[hh][q] = W->p1[f].z;
    l3[hh][q] = W->w3[f];
  }
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int s = 0; s < 4; ++s) P.w2[mt][s] = frag_load(W->w2a[mt][s][lane]);
  P.b3 = W->b3;
  __syncthreads();
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float4 q = p1[mlp_phi(s, h, i)];
      P.w1a[s * 8 + i] = q.x;
      P.w1b[s * 8 + i] = q.y;
      P.b2[s >> 1][(s & 1) * 8 + i] = q.w;
    }
}

// This half-wave's part of the output for the sample of lane l and l + 32
// (features f1, f2).
__device__ __forceinline__ float infer_half(const InferParams& P, const float4* l1h, const float4* l3h, float f1,
                                            float f2) {
  // layer 1 one K-step at a time, each step's activations going straight into
  // its four MFMAs (fewer values live at once); the empty asm keeps the LDS
  // reads here, where kept across samples they would spill
  uint32_t at = 0;
  asm volatile("" : "+v"(at));
  l1h += at;
  l3h += at;
  // (-1, 0) and (0, -1) in bfloat16, from registers: the compiler would write
  // the first as the inline constant -1.0, which the instruction reads as the second
  uint32_t m0 = 0x0000BF80u, m1 = 0xBF800000u;
  asm("" : "+s"(m0), "+s"(m1));
  const bf16x2 minus0 = __builtin_bit_cast(bf16x2, m0), minus1 = __builtin_bit_cast(bf16x2, m1);
  f32x16 acc[2];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    bf16x8 hb, lb;
    const float4 ba = l1h[2 * s], bb = l1h[2 * s + 1];
    const float b1[8] = {ba.x, ba.y, ba.z, ba.w, bb.x, bb.y, bb.z, bb.w};
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
      const int q = s * 8 + i;
      const float h0 = silu(fmaf(P.w1a[q], f1, fmaf(P.w1b[q], f2, b1[i])));
      const float h1 = silu(fmaf(P.w1a[q + 1], f1, fmaf(P.w1b[q + 1], f2, b1[i + 1])));
      const bf16x2 hi = {(__bf16)h0, (__bf16)h1};
      hb[i] = hi[0];
      hb[i + 1] = hi[1];
      lb[i] = (__bf16)__builtin_amdgcn_fdot2_f32_bf16(hi, minus0, h0, false);
      lb[i + 1] = (__bf16)__builtin_amdgcn_fdot2_f32_bf16(hi, minus1, h1, false);
    }
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      acc[mt] = mfma(P.w2[mt][s], hb, s == 0 ? P.b2[mt] : acc[mt]);
      acc[mt] = mfma(P.w2[mt][s], lb, acc[mt]);
    }
  }
  float y = 0.f;
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int r = 0; r < 16; r += 4) {
      const float4 w = l3h[4 * mt + r / 4];
      y = fmaf(w.x, silu(acc[mt][r]), y);
      y = fmaf(w.y, silu(acc[mt][r + 1]), y);
      y = fmaf(w.z, silu(acc[mt][r + 2]), y);
      y = fmaf(w.w, silu(acc[mt][r + 3]), y);
    }
  return y;
}

// x = (x of lanes 0-31, y of lanes 0-31), y = (x of lanes 32-63, y of lanes 32-63)
__device__ __forceinline__ void swap_halves(float& x, float& y) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, y),
                                                  false, false);
  const unsigned lo = r[0], hi = r[1];  // (a bit cast of r[1] itself would read r[0])
  x = __builtin_bit_cast(float, lo);
  y = __builtin_bit_cast(float, hi);
}

// Network output for a sample per lane: the wave evaluates those of lanes 0-31,
// then (two) those of lanes 32-63, so that what comes before and after the
// network (two logarithms, a sigmoid) is computed once per sample.
__device__ __forceinline__ float forward_infer(const InferParams& P, const float4* l1h, const float4* l3h, float f1,
                                               float f2, bool two) {
  float g1 = f1, g2 = f2;
  swap_halves(f1, g1);
  swap_halves(f2, g2);
  float ya = 0.f, yb = 0.f;
#pragma unroll 1
  for (int half = 0; half < (two ? 2 : 1); ++half) {
    yb = infer_half(P, l1h, l3h, half ? g1 : f1, half ? g2 : f2);
    if (half == 0) ya = yb;
  }
  swap_halves(ya, yb);
  return (ya + yb) + P.b3;
}

// A wave takes 64 samples at a time, or 32 where there are too few for every
// wave to have more (there the second half would only add its latency).
__global__ void __launch_bounds__(kMlpThreads, 2) k_mlp_forward(const MlpPacked* W, const float* x, float* y,
                                                                int64_t n) {
  __shared__ __align__(16) float l1[2][32], l3[2][32];
  __shared__ float4 p1[kH];
  const int lane = threadIdx.x & 63;
  InferParams P;
  load_infer_params(W, lane, P, p1, l1, l3);
  const float4* l1h = reinterpret_cast<const float4*>(l1[lane >> 5]);
  const float4* l3h = reinterpret_cast<const float4*>(l3[lane >> 5]);
  const int64_t nw = (int64_t)gridDim.x * (kMlpThreads / 64);
  const bool two = n > 32 * nw;
  const int per = two ? 64 : 32;
  for (int64_t t = (int64_t)blockIdx.x * (kMlpThreads / 64) + (threadIdx.x >> 6); t * per < n; t += nw) {
    const int64_t i = t * per + lane;
    const bool ok = i < n && lane < per;
    const float f1 = ok ? x[2 * i] : 0.f, f2 = ok ? x[2 * i + 1] : 0.f;
    const float v = forward_infer(P, l1h, l3h, f1, f2, two);
    if (ok) y[i] = v;
  }
}

// delta = sigmoid(out_scale y + ln chi) inside the trained chi range, the FP32
// table sampler outside it.
__global__ void __launch_bounds__(kMlpThreads, 2) k_mlp_sample(const MlpPacked* W, MlpGeom g, TableView tab,
                                                              const float* chi, const uint32_t* k, float* delta,
                                                              int64_t n) {
  __shared__ __align__(16) float l1[2][32], l3[2][32];
  __shared__ float4 p1[kH];
  const int lane = threadIdx.x & 63;
  InferParams P;
  load_infer_params(W, lane, P, p1, l1, l3);
  const float4* l1h = reinterpret_cast<const float4*>(l1[lane >> 5]);
  const float4* l3h = reinterpret_cast<const float4*>(l3[lane >> 5]);
  const int64_t nw = (int64_t)gridDim.x * (kMlpThreads / 64);
  const bool two = n > 32 * nw;
  const int per = two ? 64 : 32;
  for (int64_t t = (int64_t)blockIdx.x * (kMlpThreads / 64) + (threadIdx.x >> 6); t * per < n; t += nw) {
    const int64_t i = t * per + lane;
    const bool ok = i < n && lane < per;
    const float c = ok ? chi[i] : 1.f;
    const uint32_t kk = ok ? k[i] : 0x80000000u;
    float lr, lrc;
    log_r32(kk, lr, lrc);
    const float lc = logf(c);
    const float v = forward_infer(P, l1h, l3h, fmaf(lc, g.f1_scale, g.f1_shift), (lr - lrc) * g.f2_scale, two);
    float d = sigm(fmaf(v, g.out_scale, lc));
    if (!(c >= g.chi_lo && c <= g.chi_hi)) {
      float omd;
      sample_rad32(tab.cdf[0].f32, tab.cdf[0], c, kk, d, omd);
    }
    if (ok) delta[i] = d;
  }
}

// ------------------------------------------------------------------ training
constexpr int kGradThreads = 128;  // two waves, one 32-sample tile each
constexpr int kRows = 260;         // LDS rows per wave: dz2, dz1, h2, h1 (64 each), f1, f2, 1, dy
constexpr int kRowDz2 = 0, kRowDz1 = 64, kRowH2 = 128, kRowH1 = 192, kRowX = 256;

__device__ __forceinline__ uint32_t batch_index(int64_t j, int64_t n_data, int64_t base, int seed_mode,
                                                uint64_t seed, uint32_t step) {
  if (seed_mode) {
    const uint4 u = draw(seed, (uint64_t)j, step, 0x4D4C5000u);
    return (uint32_t)(((uint64_t)u.x * (uint64_t)n_data) >> 32);
  }
  int64_t i = base + j;
  if (i >= n_data) i -= n_data;
  return (uint32_t)i;
}

__global__ void __launch_bounds__(kGradThreads) k_mlp_grad(const MlpPacked* W, const float* x, const float* t,
                                                          int64_t n_data, int64_t batch, int64_t base, int seed_mode,
                                                          uint64_t seed, uint32_t step, float* partial) {
  __shared__ __attribute__((aligned(16))) uint16_t lds[kGradThreads / 64][kRows][32];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, h = lane >> 5, col = lane & 31;
  const int64_t tile = (int64_t)blockIdx.x * (kGradThreads / 64) + wv;
  const int64_t j = tile * 32 + col;
  const bool ok = j < batch;
  float f1 = 0.f, f2 = 0.f, tt = 0.f;
  if (ok) {  // ahead of the parameters: the samples lie anywhere in the data and come from HBM
    const uint32_t i = batch_index(j, n_data, base, seed_mode, seed, step);
    f1 = x[2 * (int64_t)i];
    f2 = x[2 * (int64_t)i + 1];
    tt = t[i];
  }
  LaneParams P;
  load_params(W, lane, P);
  bf16x8 w2t[2][4];
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int s = 0; s < 4; ++s) w2t[mt][s] = frag_load(W->w2t[mt][s][lane]);

  // forward, keeping what the backward pass needs
  bf16x8 hb[4], lb[4];
  float z1[32], s1[32];
  layer1<true>(P, f1, f2, hb, lb, z1, s1);
  f32x16 acc[2];
  layer2(P.w2, hb, lb, acc);
  float z2[32], s2[32], y = 0.f;
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int q = 16 * mt + r;
      z2[q] = acc[mt][r] + P.p1[q].w;
      s2[q] = sigm(z2[q]);
      y = fmaf(P.w3[q], z2[q] * s2[q], y);
    }
  y += __shfl_xor(y, 32);
  y += P.b3;
  const float res = ok ? y - tt : 0.f;
  const float dy = res * (2.f / (float)batch);

  // dz2 = dy w3 silu'(z2) -> B operands of dh1 = W2^T dz2
  bf16x8 db[4];
  float dz2[32];
#pragma unroll
  for (int q = 0; q < 32; ++q) {
    dz2[q] = dy * P.w3[q] * s2[q] * fmaf(z2[q], 1.f - s2[q], 1.f);
    db[q >> 3][q & 7] = (__bf16)dz2[q];
  }
  f32x16 dacc[2];
  layer2(w2t, db, nullptr, dacc);

  // transpose through LDS: row = feature (or input), column = sample
  uint16_t(*L)[32] = lds[wv];
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int q = s * 8 + i, f = mlp_phi(s, h, i);
      const float dz1 = dacc[q >> 4][q & 15] * s1[q] * fmaf(z1[q], 1.f - s1[q], 1.f);
      L[kRowDz2 + f][col] = bf16_bits(dz2[q]);
      L[kRowDz1 + f][col] = bf16_bits(dz1);
      L[kRowH2 + f][col] = bf16_bits(z2[q] * s2[q]);
      // the leading bfloat16 part of h1, from the same FP32 value the forward
      // rounded (elements are not read back out of the bf16 vectors)
      L[kRowH1 + f][col] = bf16_bits(z1[q] * s1[q]);
    }
  if (h == 0) {
    L[kRowX + 0][col] = bf16_bits(f1);
    L[kRowX + 1][col] = bf16_bits(f2);
    L[kRowX + 2][col] = bf16_bits(ok ? 1.f : 0.f);
    L[kRowX + 3][col] = bf16_bits(dy);
  }
  __syncthreads();

  // weight gradients: sums over the tile's 32 samples (two K-steps of 16)
  f32x16 gw2[2][2], ge[6];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) gw2[a][b] = f32x16{};
#pragma unroll
  for (int a = 0; a < 6; ++a) ge[a] = f32x16{};
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
    const int c0 = 16 * kk + 8 * h;
    bf16x8 bh[2], bx;
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) bh[nt] = frag_load(&L[kRowH1 + 32 * nt + col][c0]);
    bx = col < 4 ? frag_load(&L[kRowX + col][c0]) : bf16x8{};
#pragma unroll
    for (int a = 0; a < 6; ++a) {
      const bf16x8 af = frag_load(&L[32 * a + col][c0]);
      if (a < 2) {
        gw2[a][0] = mfma(af, bh[0], gw2[a][0]);
        gw2[a][1] = mfma(af, bh[1], gw2[a][1]);
      }
      ge[a] = mfma(bx, af, ge[a]);
    }
  }

  // per-wave partial row
  float* out = partial + tile * kGradRow;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = 8 * (r >> 2) + 4 * h + (r & 3);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) out[kOffW2 + kH * (32 * a + row) + 32 * b + col] = gw2[a][b][r];
  }
  // the products with (f1, f2, 1, dy) have those as rows 0 to 3 (results 0 to 3
  // of the lower half wave) and the features as columns: a store per result,
  // not one masked store per accumulator
  if (h == 0) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      out[kOffB2 + 32 * b + col] = ge[b][2];
      out[kOffW1 + 2 * (32 * b + col)] = ge[2 + b][0];
      out[kOffW1 + 2 * (32 * b + col) + 1] = ge[2 + b][1];
      out[kOffB1 + 32 * b + col] = ge[2 + b][2];
      out[kOffW3 + 32 * b + col] = ge[4 + b][3];
    }
  }
  // b3 and the squared residuals: sums over the 32 samples, fixed order
  float gb = h == 0 ? dy : 0.f, sq = h == 0 ? res * res : 0.f;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    gb += __shfl_xor(gb, o);
    sq += __shfl_xor(sq, o);
  }
  if (lane == 0) {
    out[kOffB3] = gb;
    out[kMlpParams] = sq;
  }
}

// Writes parameter i of the master copy into the packed forms.
__device__ __forceinline__ void pack_one(MlpPacked* P, int i, float v) {
  if (i < kOffB1) {
    float* p = reinterpret_cast<float*>(&P->p1[i >> 1]);
    p[i & 1] = v;
  } else if (i < kOffW2) {
    P->p1[i - kOffB1].z = v;
  } else if (i < kOffB2) {
    const int f = (i - kOffW2) >> 6, k = (i - kOffW2) & 63;
    const uint16_t b = bf16_bits(v);
    // z2 = W2 h1: row f, K index k
    {
      const int s = 2 * (k >> 5) + ((k >> 4) & 1), hh = (k >> 2) & 1, sl = 4 * ((k >> 3) & 1) + (k & 3);
      P->w2a[f >> 5][s][(f & 31) + 32 * hh][sl] = b;
    }
    // dh1 = W2^T dz2: row k, K index f
    {
      const int s = 2 * (f >> 5) + ((f >> 4) & 1), hh = (f >> 2) & 1, sl = 4 * ((f >> 3) & 1) + (f & 3);
      P->w2t[k >> 5][s][(k & 31) + 32 * hh][sl] = b;
    }
  } else if (i < kOffW3) {
    P->p1[i - kOffB2].w = v;
  } else if (i < kOffB3) {
    P->w3[i - kOffW3] = v;
  } else {
    P->b3 = v;
  }
}

__global__ void k_mlp_pack(const float* master, MlpPacked* P) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < kMlpParams) pack_one(P, i, master[i]);
}

// Sum of the partial rows, kReduceCols columns per block.  The pass has few
// columns (4418) and, at the training batch of 16,384, 512 rows of them, so one
// thread per column left 17 blocks walking 512 dependent trips each (129 us);
// here kReduceGroups threads share a column, each adding every
// kReduceGroups-th row (128-byte row segments, 16 loads in flight per thread),
// and the block adds the groups in a fixed order in FP64.
constexpr int kReduceCols = 32, kReduceGroups = 32;
__global__ void __launch_bounds__(kReduceCols* kReduceGroups)
    k_mlp_reduce(const float* partial, int rows, int64_t batch, float* grad_out, float* loss_out, float* master,
                 float* m, float* v, MlpPacked* P, int adam, AdamArgs a) {
  __shared__ double red[kReduceGroups / 2][kReduceCols];
  const int col = threadIdx.x % kReduceCols, grp = threadIdx.x / kReduceCols;
  const int i = blockIdx.x * kReduceCols + col;
  double s = 0.0;
  if (i < kGradRow) {
#pragma unroll 16
    for (int r = grp; r < rows; r += kReduceGroups) s += (double)partial[(int64_t)r * kGradRow + i];
  }
  s += __shfl_xor(s, kReduceCols);  // a wave holds two groups of the same columns
  if ((grp & 1) == 0) red[grp >> 1][col] = s;
  __syncthreads();
  if (threadIdx.x >= kReduceCols || i >= kGradRow) return;
  s = 0.0;
#pragma unroll
  for (int g = 0; g < kReduceGroups / 2; ++g) s += red[g][col];
  if (i == kMlpParams) {
    if (loss_out) *loss_out = (float)(s / (double)batch);
    return;
  }
  const float g = (float)s;
  if (!adam) {
    grad_out[i] = g;
    return;
  }
  const float mi = a.beta1 * m[i] + (1.f - a.beta1) * g;
  const float vi = a.beta2 * v[i] + (1.f - a.beta2) * g * g;
  m[i] = mi;
  v[i] = vi;
  const float p = master[i] - a.lr * (mi / a.bc1) / (sqrtf(vi / a.bc2) + a.eps);
  master[i] = p;
  pack_one(P, i, p);
}

}  // namespace

hipError_t launch_mlp_forward(const MlpPacked* w, const float* x, float* y, int64_t n, int grid, hipStream_t st) {
  hipLaunchKernelGGL(k_mlp_forward, dim3(grid), dim3(kMlpThreads), 0, st, w, x, y, n);
  return hipGetLastError();
}

hipError_t launch_mlp_sample(const MlpPacked* w, MlpGeom g, TableView tab, const float* chi, const uint32_t* k,
                             float* delta, int64_t n, int grid, hipStream_t st) {
  hipLaunchKernelGGL(k_mlp_sample, dim3(grid), dim3(kMlpThreads), 0, st, w, g, tab, chi, k, delta, n);
  return hipGetLastError();
}

hipError_t launch_mlp_grad(const MlpPacked* w, const float* x, const float* t, int64_t n_data, int64_t batch,
                           int64_t base, int seed_mode, uint64_t seed, uint32_t step, float* partial,
                           hipStream_t st) {
  const int64_t blocks = (batch + kGradThreads / 2 - 1) / (kGradThreads / 2);
  hipLaunchKernelGGL(k_mlp_grad, dim3((unsigned)blocks), dim3(kGradThreads), 0, st, w, x, t, n_data, batch, base,
                     seed_mode, seed, step, partial);
  return hipGetLastError();
}

hipError_t launch_mlp_reduce(const float* partial, int rows, int64_t batch, float* grad_out, float* loss_out,
                             float* master, float* m, float* v, MlpPacked* packed, int adam, AdamArgs a,
                             hipStream_t st) {
  hipLaunchKernelGGL(k_mlp_reduce, dim3((kGradRow + kReduceCols - 1) / kReduceCols), dim3(kReduceCols * kReduceGroups),
                     0, st, partial, rows, batch, grad_out, loss_out, master, m, v, packed, adam, a);
  return hipGetLastError();
}

hipError_t launch_mlp_pack(const float* master, MlpPacked* packed, hipStream_t st) {
  hipLaunchKernelGGL(k_mlp_pack, dim3((kMlpParams + 255) / 256), dim3(256), 0, st, master, packed);
  return hipGetLastError();
}

}  // namespace sfqed
