// mhd_mlp.hpp -- the learned interface flux: a 15 -> 64 -> 64 -> 7 GELU
// network that stands in for HLLD at smooth interfaces (HLLD stays in use
// where the pressure or density jump exceeds a threshold), its training
// kernels, and the capture of interface samples.  BF16 operands, FP32
// accumulation on the MFMA units (v_mfma_f32_16x16x16_bf16, and for the
// 64-deep layers inside a step v_mfma_f32_16x16x32_bf16).
//
// Features: the mean of the two face-frame primitive states (rho, vn, vt1,
// vt2, p, Bt1, Bt2), the unit jump and the jump size s, and Bn, all in units
// of rho0 = (rhoL + rhoR)/2, p0 = (pL + pR)/2, v0 = sqrt(p0/rho0),
// B0 = sqrt(p0) (layout at mlp_features); outputs: the dissipative part of
// the flux, F - (F(wl) + F(wr))/2, divided by s (rho0 v0, p0, p0, p0, p0 v0,
// B0 v0, B0 v0); the central part is computed exactly.  Dividing by s keeps
// the BF16 operands of order one.  The normalisation follows the scaling
// symmetry of ideal MHD, under which HLLD is covariant.
//
// Parameters (FP32 master copy, packed): W1[15][64] b1[64] W2[64][64] b2[64]
// W3[64][7] b3[7], [in][out] row-major, 5639 values.
//
// MFMA 16x16x16 operand layout (lane l, 64 lanes): A fragment holds
// A[l % 16][4 (l / 16) + 0..3], B fragment B[4 (l / 16) + 0..3][l % 16],
// accumulator C[4 (l / 16) + 0..3][l % 16].
#pragma once
#include <hip/hip_runtime.h>

#include "mhd_device.hpp"

namespace mhd {

constexpr int kNin = 15, kNh = 64, kNout = 7;
constexpr float kTinyJump = 1e-4f;
constexpr int kParams = 15 * 64 + 64 + 64 * 64 + 64 + 64 * 7 + 7;
constexpr int oW1 = 0, ob1 = 960, oW2 = 1024, ob2 = 5120, oW3 = 5184, ob3 = 5632;

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

// round to the nearest bfloat16, ties to even (gfx950 converts in hardware,
// two values per v_cvt_pk_bf16_f32)
__device__ __forceinline__ unsigned short f2bf(float x) { return __builtin_bit_cast(unsigned short, (__bf16)x); }
__device__ __forceinline__ unsigned f2bf2(float a, float b) {
  return __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a, b}, bf16x2v));
}
// four floats to one MFMA BF16 operand fragment
__device__ __forceinline__ bf16x4 f2bf4(float a, float b, float c, float d) {
  return __builtin_bit_cast(bf16x4, u32x2{f2bf2(a, b), f2bf2(c, d)});
}
__device__ __forceinline__ float bf2f(unsigned short h) { return __uint_as_float((unsigned)h << 16); }

// GELU, tanh form: 0.5 x (1 + tanh u) = x s with s = 1 / (1 + exp(-2u)),
// u = sqrt(2/pi) (x + 0.044715 x^3); exp(-2u) = 2^q with
// q = x (a + b x^2), a = -2 sqrt(2/pi) log2(e), b = 0.044715 a, so one GELU
// is three multiply-adds, v_exp_f32, an add, v_rcp_f32 and a multiply
// (the hardware reciprocal needs no range scaling: a denominator beyond
// 2^126 gives s = 0, the limit).  The derivative is
// s + 2 x s (1 - s) du/dx.
__device__ __forceinline__ float gelu_sig(float x) {
  const float a = -2.302208198144325f, b = -0.1029432395800235f;
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(x * __builtin_fmaf(b, x * x, a)));
}
__device__ __forceinline__ float gelu(float x) { return x * gelu_sig(x); }
__device__ __forceinline__ float gelu_prime(float x) {
  const float sg = gelu_sig(x);
  const float du2 = 1.5957691216057308f * (1.0f + 3.0f * 0.044715f * x * x);   // 2 du/dx
  return sg + x * sg * (1.0f - sg) * du2;
}

__device__ __forceinline__ f32x4 mfma16(bf16x4 a, bf16x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}
// v_mfma_f32_16x16x32_bf16 (gfx950) on two 16-deep fragment pairs: lane l
// supplies k = 8 (l / 16) + 0..7, here the 4 values of the first pair's
// fragment followed by the 4 of the second.  Both operands take their k
// slots in that same order, so the product is the sum of the two 16-deep
// products: half the MFMA issues for the same contraction.
__device__ __forceinline__ f32x4 mfma32(bf16x4 a0, bf16x4 a1, bf16x4 b0, bf16x4 b1, f32x4 c) {
  const bf16x8 a = __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7));
  const bf16x8 b = __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(b0, b1, 0, 1, 2, 3, 4, 5, 6, 7));
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Inference weights as the kernels read them: transposed, BF16, padded.
//   W1t[64][16] (k = 15 zero), W2t[64][64], W3t[16][64] (rows >= 7 zero),
//   biases in FP32: b1[64], b2[64], b3[16].
// Rows lie kP1 and kP2 values apart: sixteen lanes read the same column of
// sixteen rows, which at 16 and 64 values (32 and 128 bytes) share four banks and
// one (each read took sixteen turns); at 40 and 144 bytes they do not.
constexpr int kP1 = 20, kP2 = 72;
struct MlpWeights {
  unsigned short W1t[64 * kP1];
  unsigned short W2t[64 * kP2];
  unsigned short W3t[16 * kP2];
  float b1[64], b2[64], b3[16];
};

// FP32 master parameters -> inference layout
__global__ void __launch_bounds__(256) k_mlp_pack(const float* __restrict__ P, MlpWeights* __restrict__ out) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  if (t < 64 * 16) {
    const int n = t / 16, k = t % 16;
    out->W1t[n * kP1 + k] = f2bf(k < kNin ? P[oW1 + k * kNh + n] : 0.0f);
  }
  if (t < 64 * 64) {
    const int n = t / 64, k = t % 64;
    out->W2t[n * kP2 + k] = f2bf(P[oW2 + k * kNh + n]);
  }
  if (t < 16 * 64) {
    const int n = t / 64, k = t % 64;
    out->W3t[n * kP2 + k] = f2bf(n < kNout ? P[oW3 + k * kNout + n] : 0.0f);
  }
  if (t < 64) {
    out->b1[t] = P[ob1 + t];
    out->b2[t] = P[ob2 + t];
  }
  if (t < 16) out->b3[t] = t < kNout ? P[ob3 + t] : 0.0f;
}

// Per-wave LDS staging of inference: the BF16 features of the wave's 64
// faces (one row per lane) and the 8 padded outputs of each face.
struct MlpStage {
  unsigned short X[64 * 16];
  float Y[64 * 8];
};
// LDS of one 256-thread block: the inference weights and four wave stages.
struct MlpShared {
  MlpWeights w;
  MlpStage st[4];
};

// Block-wide copy of the weights into LDS (a block barrier: every thread of
// the block calls it once, before any inference).
__device__ __forceinline__ void mlp_load_weights(MlpShared& sh, const MlpWeights* __restrict__ g) {
  const uint4* src = reinterpret_cast<const uint4*>(g);
  uint4* dst = reinterpret_cast<uint4*>(&sh.w);
  for (int t = threadIdx.x; t < (int)(sizeof(MlpWeights) / 16); t += blockDim.x) dst[t] = src[t];
  __syncthreads();
}

// ordering of LDS traffic between the lanes of one wave
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Normalised features of one interface (face frame) and the scales the
// network output is multiplied by.  With sc_w = (rho0, v0, v0, v0, p0, B0, B0)
// and d = (wR - wL) / sc_w, s = |d|:
//   x0 mean rho / rho0 (= 1), x1..x3 mean (vn, vt1, vt2) / v0, x4 = s,
//   x5, x6 mean (Bt1, Bt2) / B0, x7..x13 = d / s (0 when s = 0), x14 = Bn / B0;
//   osc = s * (rho0 v0, p0, p0, p0, p0 v0, B0 v0, B0 v0).
__device__ __forceinline__ void mlp_features(const float wl[7], const float wr[7], float bn, float x[16],
                                             float osc[7]) {
  const float rho0 = 0.5f * (wl[0] + wr[0]), p0 = 0.5f * (wl[4] + wr[4]);
  const float v0 = sqrtf(p0 / rho0), b0 = sqrtf(p0);
  const float inv[7] = {1.0f / rho0, 1.0f / v0, 1.0f / v0, 1.0f / v0, 1.0f / p0, 1.0f / b0, 1.0f / b0};
  float d[7], ss = 0.0f;
#pragma unroll
  for (int m = 0; m < 7; ++m) {
    d[m] = (wr[m] - wl[m]) * inv[m];
    ss += d[m] * d[m];
  }
  const float sj = sqrtf(ss);
  const float is = sj > 0.0f ? 1.0f / sj : 0.0f;
  x[0] = 0.5f * (wl[0] + wr[0]) * inv[0];
  x[1] = 0.5f * (wl[1] + wr[1]) * inv[1];
  x[2] = 0.5f * (wl[2] + wr[2]) * inv[2];
  x[3] = 0.5f * (wl[3] + wr[3]) * inv[3];
  x[4] = sj;
  x[5] = 0.5f * (wl[5] + wr[5]) * inv[5];
  x[6] = 0.5f * (wl[6] + wr[6]) * inv[6];
#pragma unroll
  for (int m = 0; m < 7; ++m) x[7 + m] = d[m] * is;
  x[14] = bn * inv[5];
  x[15] = 0.0f;
  osc[0] = sj * rho0 * v0; osc[1] = sj * p0; osc[2] = sj * p0; osc[3] = sj * p0;
  osc[4] = sj * p0 * v0; osc[5] = sj * b0 * v0; osc[6] = sj * b0 * v0;
}

// Network output for the 64 faces of one wave (one face per lane).  All
// lanes of the wave call this together; lanes without a face pass zeros.
// The network runs transposed (H^T = W^T X^T): the weights are the A operand
// (lane (li, lk) reads W^T[16 t + li][16 s + 4 lk + 0..3] from LDS), so the
// accumulator tile of one layer is already the B operand of the next, and
// GELU and the BF16 rounding of each hidden layer act on it in registers.
// Per 16-face tile: 4 MFMA 16x16x16 (layer 1) and 8 + 2 MFMA 16x16x32.
__device__ __forceinline__ void mlp_forward_wave(MlpShared& sh, const float x[16], float y[7]) {
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  MlpStage& S = sh.st[threadIdx.x >> 6];
  const MlpWeights& g = sh.w;
  {
    unsigned pk[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) pk[m] = f2bf2(x[2 * m], x[2 * m + 1]);
    uint4* dst = reinterpret_cast<uint4*>(S.X + lane * 16);
    dst[0] = make_uint4(pk[0], pk[1], pk[2], pk[3]);
    dst[1] = make_uint4(pk[4], pk[5], pk[6], pk[7]);
  }
  wave_sync();
#pragma unroll 1
  for (int ft = 0; ft < 4; ++ft) {
    const bf16x4 xf = *reinterpret_cast<const bf16x4*>(S.X + (16 * ft + li) * 16 + 4 * lk);
    bf16x4 h1[4], h2[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const bf16x4 wa = *reinterpret_cast<const bf16x4*>(g.W1t + (16 * t + li) * kP1 + 4 * lk);
      const f32x4 z = mfma16(wa, xf, f32x4{0.f, 0.f, 0.f, 0.f});
      const float4 bb = *reinterpret_cast<const float4*>(g.b1 + 16 * t + 4 * lk);
      h1[t] = f2bf4(gelu(z[0] + bb.x), gelu(z[1] + bb.y), gelu(z[2] + bb.z), gelu(z[3] + bb.w));
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kc = 0; kc < 2; ++kc) {
        const unsigned short* wr = g.W2t + (16 * t + li) * kP2 + 32 * kc + 4 * lk;
        z = mfma32(*reinterpret_cast<const bf16x4*>(wr), *reinterpret_cast<const bf16x4*>(wr + 16), h1[2 * kc],
                   h1[2 * kc + 1], z);
      }
      const float4 bb = *reinterpret_cast<const float4*>(g.b2 + 16 * t + 4 * lk);
      h2[t] = f2bf4(gelu(z[0] + bb.x), gelu(z[1] + bb.y), gelu(z[2] + bb.z), gelu(z[3] + bb.w));
    }
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kc = 0; kc < 2; ++kc) {
      const unsigned short* wr = g.W3t + li * kP2 + 32 * kc + 4 * lk;
      o = mfma32(*reinterpret_cast<const bf16x4*>(wr), *reinterpret_cast<const bf16x4*>(wr + 16), h2[2 * kc],
                 h2[2 * kc + 1], o);
    }
    // lane (li, lk) holds outputs 4 lk + 0..3 of face 16 ft + li
    if (lk < 2) {
      const float4 b3 = *reinterpret_cast<const float4*>(g.b3 + 4 * lk);
      *reinterpret_cast<float4*>(S.Y + (16 * ft + li) * 8 + 4 * lk) =
          make_float4(o[0] + b3.x, o[1] + b3.y, o[2] + b3.z, o[3] + b3.w);
    }
  }
  wave_sync();
  const float4 y0 = *reinterpret_cast<const float4*>(S.Y + lane * 8);
  const float4 y1 = *reinterpret_cast<const float4*>(S.Y + lane * 8 + 4);
  y[0] = y0.x; y[1] = y0.y; y[2] = y0.z; y[3] = y0.w;
  y[4] = y1.x; y[5] = y1.y; y[6] = y1.z;
  wave_sync();   // the stage is rewritten by the next call
}

// Interface capture: (wl[7], wr[7], bn, flux[7]) of every stride-th face
struct Capture {
  float* buf;                    // [cap][22], nullptr = off
  long long cap;
  unsigned long long* count;     // device counter of attempted writes
  int stride;
};

// the record of a face (its states written), or nullptr when the face is not
// sampled or the buffer is full; capture_flux completes it
__device__ __forceinline__ float* capture_states(const Capture& cp, long long face, const float wl[7],
                                                 const float wr[7], float bn) {
  if (!cp.buf || face % cp.stride) return nullptr;
  const unsigned long long slot = atomicAdd(cp.count, 1ull);
  if ((long long)slot >= cp.cap) return nullptr;
  float* o = cp.buf + slot * 22;
#pragma unroll
  for (int m = 0; m < 7; ++m) {
    o[m] = wl[m];
    o[7 + m] = wr[m];
  }
  o[14] = bn;
  return o;
}
__device__ __forceinline__ void capture_flux(float* o, const float f[7]) {
  if (!o) return;
#pragma unroll
  for (int m = 0; m < 7; ++m) o[15 + m] = f[m];
}
__device__ __forceinline__ void capture_face(const Capture& cp, long long face, const float wl[7], const float wr[7],
                                             float bn, const float f[7]) {
  capture_flux(capture_states(cp, face, wl, wr, bn), f);
}

// Learned flux with HLLD fallback for one face per lane (capture: face id
// `face` recorded with the flux used).  Returns 1 when the face used HLLD (a
// strong jump), 0 when it used the network.  Every lane of the wave calls it
// (lanes without a face pass active = false).  The fallback flux, or the
// exact central part, is computed before the network, so that only the flux
// and the output scales stay live across it.
__device__ __forceinline__ int mlp_or_hlld(MlpShared& sh, bool active, const float wl[7], const float wr[7], float bn,
                                           float gam, float dp, float drho, float f[7], const Capture& cp,
                                           long long face) {
  bool fall = true;
  float x[16], sc[7];
  if (active) {
    const float jp = fabsf(wr[4] - wl[4]) / fminf(wl[4], wr[4]);
    const float jr = fabsf(wr[0] - wl[0]) / fminf(wl[0], wr[0]);
    fall = (jp > dp) || (jr > drho);
  }
  float* rec = nullptr;
  if (active) rec = capture_states(cp, face, wl, wr, bn);
#pragma unroll
  for (int m = 0; m < 7; ++m) f[m] = 0.0f;
  if (active && !fall) {
    mlp_features(wl, wr, bn, x, sc);
    // the network gives the dissipative part; the central part is exact
    const float gm1inv = 1.0f / (gam - 1.0f);
    float ul[7], ur[7], fl[7], fr[7];
    state_and_flux(wl, bn, gm1inv, ul, fl);
    state_and_flux(wr, bn, gm1inv, ur, fr);
#pragma unroll
    for (int m = 0; m < 7; ++m) f[m] = 0.5f * (fl[m] + fr[m]);
  } else {
#pragma unroll
    for (int m = 0; m < 16; ++m) x[m] = 0.0f;
#pragma unroll
    for (int m = 0; m < 7; ++m) sc[m] = 0.0f;
    if (active) riemann_hlld(wl, wr, bn, gam, f);
  }
  float y[7] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  // the network runs when any lane of the wave needs it (wave-uniform test)
  if (__ballot(active && !fall) != 0ull) mlp_forward_wave(sh, x, y);
  if (!active) return 0;
  if (!fall) {
#pragma unroll
    for (int m = 0; m < 7; ++m) f[m] += y[m] * sc[m];
  }
  capture_flux(rec, f);
  return fall ? 1 : 0;
}

// ------------------------------------------------------------ training
// Captured samples -> features X[n][15], targets T[n][7], fallback flags.
__global__ void __launch_bounds__(256) k_mlp_prepare(const float* __restrict__ S, int n, float gam, float dp,
                                                     float drho, float* __restrict__ X, float* __restrict__ T,
                                                     int* __restrict__ flag) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const float* s = S + (long long)i * 22;
  float wl[7], wr[7], x[16], sc[7];
#pragma unroll
  for (int m = 0; m < 7; ++m) {
    wl[m] = s[m];
    wr[m] = s[7 + m];
  }
  mlp_features(wl, wr, s[14], x, sc);
  const float gm1inv = 1.0f / (gam - 1.0f);
  float ul[7], ur[7], fl[7], fr[7];
  state_and_flux(wl, s[14], gm1inv, ul, fl);
  state_and_flux(wr, s[14], gm1inv, ur, fr);
#pragma unroll
  for (int m = 0; m < kNin; ++m) X[(long long)i * kNin + m] = x[m];
#pragma unroll
  for (int m = 0; m < kNout; ++m)
    T[(long long)i * kNout + m] = sc[m] > 0.0f ? (s[15 + m] - 0.5f * (fl[m] + fr[m])) / sc[m] : 0.0f;
  const float jp = fabsf(wr[4] - wl[4]) / fminf(wl[4], wr[4]);
  const float jr = fabsf(wr[0] - wl[0]) / fminf(wl[0], wr[0]);
  // bit 0: strong jump (HLLD at run time); bit 1: jump below kTinyJump, whose
  // target is dominated by the float round-off of the flux difference
  flag[i] = ((jp > dp) || (jr > drho) ? 1 : 0) | (x[4] < kTinyJump ? 2 : 0);
}

// ---- the network on batches of rows
//
// Like the inference above the batch kernels run the network transposed, a wave
// on 16 rows at a time, every layer's accumulator tile being the next layer's B
// operand: activations never leave the registers.  The FP32 master weights are
// rounded to BF16 into LDS by each block.  (One GEMM per layer with FP32
// activations in memory moved 1 KB per row and, at the driver's batch of 4096,
// spent its time on sixteen launches.)
struct BatchWeights {
  unsigned short W1t[64 * kP1], W2t[64 * kP2], W3t[16 * kP2];   // [out][in], as MlpWeights
  float b1[64], b2[64], b3[16];
};

__device__ __forceinline__ void load_batch_weights(BatchWeights& g, const float* __restrict__ P) {
  for (int t = threadIdx.x; t < 64 * 16; t += blockDim.x) {
    const int k = t >> 6, n = t & 63;
    g.W1t[n * kP1 + k] = f2bf(k < kNin ? P[oW1 + k * kNh + n] : 0.0f);
    // W3: k the output (rows past the seventh are zero), n the hidden unit
    g.W3t[k * kP2 + n] = f2bf(k < kNout ? P[oW3 + n * kNout + k] : 0.0f);
  }
  for (int t = threadIdx.x; t < 64 * 64; t += blockDim.x) g.W2t[(t & 63) * kP2 + (t >> 6)] = f2bf(P[oW2 + t]);
  for (int t = threadIdx.x; t < 64; t += blockDim.x) {
    g.b1[t] = P[ob1 + t];
    g.b2[t] = P[ob2 + t];
    if (t < 16) g.b3[t] = t < kNout ? P[ob3 + t] : 0.0f;
  }
}

// two 16-deep products, the first before the second: rounded as a 16-deep loop over
// k, so that no activation falls on the other side of a BF16 rounding point
__device__ __forceinline__ f32x4 mfma16x2(bf16x4 a0, bf16x4 a1, bf16x4 b0, bf16x4 b1, f32x4 c) {
  return mfma16(a1, b1, mfma16(a0, b0, c));
}

__device__ __forceinline__ bf16x4 frag(const unsigned short* p) { return *reinterpret_cast<const bf16x4*>(p); }

// features 4 lk .. 4 lk + 3 of one row of X (zero past the fifteenth and for rows past the batch)
__device__ __forceinline__ bf16x4 row_features(const float* __restrict__ X, long long row, bool on, int lk) {
  float x[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) x[i] = on && 4 * lk + i < kNin ? X[row * kNin + 4 * lk + i] : 0.0f;
  return f2bf4(x[0], x[1], x[2], x[3]);
}

// pre-activations and BF16 activations of both hidden layers and the outputs of 16
// rows: lane (li, lk) holds units 16 t + 4 lk + 0..3 (outputs 4 lk + 0..3) of row li
struct BatchForward {
  f32x4 z1[4], z2[4], o;
  bf16x4 h1[4], h2[4];
};

__device__ __forceinline__ void batch_forward(const BatchWeights& g, bf16x4 xf, int li, int lk, BatchForward& r) {
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const float4 b = *reinterpret_cast<const float4*>(g.b1 + 16 * t + 4 * lk);
    r.z1[t] = mfma16(frag(g.W1t + (16 * t + li) * kP1 + 4 * lk), xf, f32x4{0.f, 0.f, 0.f, 0.f}) +
              f32x4{b.x, b.y, b.z, b.w};
    r.h1[t] = f2bf4(gelu(r.z1[t][0]), gelu(r.z1[t][1]), gelu(r.z1[t][2]), gelu(r.z1[t][3]));
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kc = 0; kc < 2; ++kc) {
      const unsigned short* w = g.W2t + (16 * t + li) * kP2 + 32 * kc + 4 * lk;
      z = mfma16x2(frag(w), frag(w + 16), r.h1[2 * kc], r.h1[2 * kc + 1], z);
    }
    const float4 b = *reinterpret_cast<const float4*>(g.b2 + 16 * t + 4 * lk);
    r.z2[t] = z + f32x4{b.x, b.y, b.z, b.w};
    r.h2[t] = f2bf4(gelu(r.z2[t][0]), gelu(r.z2[t][1]), gelu(r.z2[t][2]), gelu(r.z2[t][3]));
  }
  f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kc = 0; kc < 2; ++kc) {
    const unsigned short* w = g.W3t + li * kP2 + 32 * kc + 4 * lk;
    o = mfma16x2(frag(w), frag(w + 16), r.h2[2 * kc], r.h2[2 * kc + 1], o);
  }
  const float4 b = *reinterpret_cast<const float4*>(g.b3 + 4 * lk);
  r.o = o + f32x4{b.x, b.y, b.z, b.w};
}

// Y = network(X).  250,000 rows: 218 us as three GEMMs, 22 us, of which the GELUs (128
// exponentials and reciprocals a row) take about 12 at the vector units' rate; the rest
// is the start of the launch: each block rounds the weights into its LDS and waits for
// them.  Four blocks per CU at most, so that a block does that once for several tiles.
__global__ void __launch_bounds__(256) k_mlp_forward(const float* __restrict__ P, const float* __restrict__ X, int n,
                                                     float* __restrict__ Y) {
  __shared__ BatchWeights g;
  load_batch_weights(g, P);
  __syncthreads();
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int tiles = (n - 1) / 16 + 1, step = gridDim.x * 4;
  for (int tile = blockIdx.x * 4 + (threadIdx.x >> 6); tile < tiles; tile += step) {
    const long long row = 16LL * tile + li;
    const bool on = row < n;
    BatchForward r;
    batch_forward(g, row_features(X, row, on, lk), li, lk, r);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (on && 4 * lk + i < kNout) Y[row * kNout + 4 * lk + i] = r.o[i];
  }
}

// Gradients of a batch, one partial sum over rows per block.  A block takes 64
// rows at a time: each wave runs 16 of them forward and backward in registers,
// leaves the BF16 operands of the weight gradients transposed in LDS, and the
// block then contracts over its 64 rows, each wave six of the 24 gradient tiles.
// Bias gradients sum the FP32 values.  MSE: dY = 2 (Y - T) / (7 n) and the squared
// error's sum; otherwise T holds dY.  part: kGradPitch floats per block.
// Bound by latency (a block per CU and tile): a training step on 4096 rows takes
// 19.5 us with the reduction (159 us as sixteen launches).
constexpr int kGradPitch = kParams + 1;   // the gradients and the squared error
constexpr int kGradBlocks = 256;          // blocks at most

struct GradShared {
  BatchWeights w;
  unsigned short W2[64 * kP2], W3[64 * kP1];                                  // [in][out]
  unsigned short Xt[16 * kP2], H1t[64 * kP2], H2t[64 * kP2];                  // [unit][row]
  unsigned short D1t[64 * kP2], D2t[64 * kP2], D3t[16 * kP2];
};

template <bool MSE>
__global__ void __launch_bounds__(256) k_mlp_gradients(const float* __restrict__ P, const float* __restrict__ X,
                                                       const float* __restrict__ T, int n, float* __restrict__ part) {
  __shared__ GradShared g;
  load_batch_weights(g.w, P);
  for (int t = threadIdx.x; t < 64 * 64; t += 256) g.W2[(t >> 6) * kP2 + (t & 63)] = f2bf(P[oW2 + t]);
  for (int t = threadIdx.x; t < 64 * 16; t += 256) {
    const int k = t & 15, m = t >> 4;
    g.W3[m * kP1 + k] = f2bf(k < kNout ? P[oW3 + m * kNout + k] : 0.0f);
  }
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4, wv = threadIdx.x >> 6;
  const float total = (float)(7LL * n);
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 gw1 = zero, gw2[4], gw3 = zero, gb1[4], gb2[4], gb3 = zero;
#pragma unroll
  for (int t = 0; t < 4; ++t) gw2[t] = gb1[t] = gb2[t] = zero;
  float err = 0.0f;
  const int tiles = (n - 1) / 64 + 1;
  for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const long long row = 64LL * tile + 16 * wv + li;
    const bool on = row < n;
    __syncthreads();   // weights loaded; the operands of the tile before are read
    const bf16x4 xf = row_features(X, row, on, lk);
    BatchForward r;
    batch_forward(g.w, xf, li, lk, r);
    f32x4 dy = zero;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (!on || 4 * lk + i >= kNout) continue;
      const float t = T[row * kNout + 4 * lk + i];
      if (MSE) {
        const float d = r.o[i] - t;
        dy[i] = 2.0f * d / total;
        err += d * d;
      } else {
        dy[i] = t;
      }
    }
    gb3 += dy;
    const bf16x4 dyf = f2bf4(dy[0], dy[1], dy[2], dy[3]);
    bf16x4 d2[4], d1[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      f32x4 d = mfma16(frag(g.W3 + (16 * t + li) * kP1 + 4 * lk), dyf, zero);
#pragma unroll
      for (int i = 0; i < 4; ++i) d[i] *= gelu_prime(r.z2[t][i]);
      gb2[t] += d;
      d2[t] = f2bf4(d[0], d[1], d[2], d[3]);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      f32x4 d = zero;
#pragma unroll
      for (int kc = 0; kc < 2; ++kc) {
        const unsigned short* w = g.W2 + (16 * t + li) * kP2 + 32 * kc + 4 * lk;
        d = mfma16x2(frag(w), frag(w + 16), d2[2 * kc], d2[2 * kc + 1], d);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) d[i] *= gelu_prime(r.z1[t][i]);
      gb1[t] += d;
      d1[t] = f2bf4(d[0], d[1], d[2], d[3]);
    }
    const int at = 4 * lk * kP2 + 16 * wv + li;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      g.Xt[at + i * kP2] = (unsigned short)xf[i];
      g.D3t[at + i * kP2] = (unsigned short)dyf[i];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int q = at + (16 * t + i) * kP2;
        g.H1t[q] = (unsigned short)r.h1[t][i];
        g.H2t[q] = (unsigned short)r.h2[t][i];
        g.D1t[q] = (unsigned short)d1[t][i];
        g.D2t[q] = (unsigned short)d2[t][i];
      }
    }
    __syncthreads();
    // contractions over the 64 rows: A [unit][row], B [row][unit], both read along
    // the rows
#pragma unroll
    for (int kc = 0; kc < 2; ++kc) {
      const int c = li * kP2 + 32 * kc + 4 * lk, cw = c + 16 * wv * kP2;
      const bf16x4 h0 = frag(g.H1t + cw), h1 = frag(g.H1t + cw + 16);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const unsigned short* d = g.D2t + c + 16 * t * kP2;
        gw2[t] = mfma16x2(h0, h1, frag(d), frag(d + 16), gw2[t]);
      }
      gw1 = mfma16x2(frag(g.Xt + c), frag(g.Xt + c + 16), frag(g.D1t + cw), frag(g.D1t + cw + 16), gw1);
      gw3 = mfma16x2(frag(g.H2t + cw), frag(g.H2t + cw + 16), frag(g.D3t + c), frag(g.D3t + c + 16), gw3);
    }
  }
  float* out = part + (long long)blockIdx.x * kGradPitch;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = 4 * lk + i;
    if (m < kNin) out[oW1 + m * kNh + 16 * wv + li] = gw1[i];
#pragma unroll
    for (int t = 0; t < 4; ++t) out[oW2 + (16 * wv + m) * kNh + 16 * t + li] = gw2[t][i];
    if (li < kNout) out[oW3 + (16 * wv + m) * kNout + li] = gw3[i];
  }
  // bias gradients and the error: over the sixteen rows of a wave, then the waves
  __shared__ float sums[4][64 + 64 + 16 + 4];
  const auto rows = [&](float v) {
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) v += __shfl_xor(v, o, 64);
    return v;
  };
#pragma unroll
  for (int i = 0; i < 4; ++i) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float s1 = rows(gb1[t][i]), s2 = rows(gb2[t][i]);
      if (li == 0) {
        sums[wv][16 * t + 4 * lk + i] = s1;
        sums[wv][64 + 16 * t + 4 * lk + i] = s2;
      }
    }
    const float s3 = rows(gb3[i]);
    if (li == 0) sums[wv][128 + 4 * lk + i] = s3;
  }
  const float se = rows(err);
  if (li == 0) sums[wv][144 + lk] = se;
  __syncthreads();
  const int t = threadIdx.x;
  const auto waves = [&](int q) { return ((sums[0][q] + sums[1][q]) + sums[2][q]) + sums[3][q]; };
  if (t < 64) {
    out[ob1 + t] = waves(t);
    out[ob2 + t] = waves(64 + t);
    if (t < kNout) out[ob3 + t] = waves(128 + t);
    if (t == 0) out[kParams] = ((waves(144) + waves(145)) + waves(146)) + waves(147);
  }
}

// Sum the blocks' partials in a fixed order (32 parameters x 8 segments of the
// blocks per block); ADAM: also the loss and one step of Adam (Kingma & Ba) on the
// FP32 master parameters.
struct AdamArgs {
  float *P, *m, *v, *loss;
  float total, lr, b1, b2, eps, c1, c2;
};

template <bool ADAM>
__global__ void __launch_bounds__(256) k_mlp_reduce(const float* __restrict__ part, int blocks, float* __restrict__ G,
                                                    AdamArgs a) {
  __shared__ float red[8][32];
  const int q = threadIdx.x & 31, seg = threadIdx.x >> 5, i = blockIdx.x * 32 + q;
  const int per = (blocks + 7) / 8, b0 = seg * per, b1 = min(blocks, b0 + per);
  float s = 0.0f;
  if (i < kGradPitch) {
#pragma unroll 8
    for (int b = b0; b < b1; ++b) s += part[(long long)b * kGradPitch + i];
  }
  red[seg][q] = s;
  __syncthreads();
  if (seg || i >= kGradPitch) return;
  float g = red[0][q];
#pragma unroll
  for (int k = 1; k < 8; ++k) g += red[k][q];
  if (i == kParams) {
    if (ADAM && a.loss) *a.loss = g / a.total;
    return;
  }
  G[i] = g;
  if (ADAM) {
    const float mi = a.b1 * a.m[i] + (1.0f - a.b1) * g;
    const float vi = a.b2 * a.v[i] + (1.0f - a.b2) * g * g;
    a.m[i] = mi;
    a.v[i] = vi;
    a.P[i] -= a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
  }
}

}  // namespace mhd
