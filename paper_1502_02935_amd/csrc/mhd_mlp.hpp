// mhd_mlp.hpp -- device side of the learned flux correction: a 32-64-64-8
// MLP with GELU hidden layers, bfloat16 weights and activations, FP32
// accumulation on the matrix cores (v_mfma_f32_16x16x32_bf16 in the step,
// 16x16x16 in the batch kernels), plus the face
// features and the output-to-flux map shared by training and inference.
//
// Parameter vector (FP32 master, 6792 values): W1[64][32], b1[64],
// W2[64][64], b2[64], W3[8][64], b3[8].  Weights are rounded to bfloat16 when
// loaded; biases stay FP32.
//
// MFMA 16x16x16 operand layout (lane l, r = l % 16, q = l / 16):
//   A (16 x 16, M x K): lane holds A[r][4q .. 4q+3]
//   B (16 x 16, K x N): lane holds B[4q .. 4q+3][r]
//   D (16 x 16, M x N): lane holds D[4q .. 4q+3][r]
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mhd {

constexpr int kMlpIn = 32;
constexpr int kMlpHid = 64;
constexpr int kMlpOut = 8;
constexpr int kMlpParams = 6792;
constexpr int kP_W1 = 0;
constexpr int kP_B1 = kP_W1 + 64 * 32;
constexpr int kP_W2 = kP_B1 + 64;
constexpr int kP_B2 = kP_W2 + 64 * 64;
constexpr int kP_W3 = kP_B2 + 64;
constexpr int kP_B3 = kP_W3 + 8 * 64;

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16v2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// float -> bfloat16 bits, round to nearest, ties to even (finite inputs).
__device__ __forceinline__ unsigned short bf16_bits(float x) {
  unsigned u = __float_as_uint(x);
  if ((u & 0x7f800000u) == 0x7f800000u) return (unsigned short)(u >> 16);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf16_float(unsigned short b) {
  return __uint_as_float(((unsigned)b) << 16);
}
__device__ __forceinline__ float bf16_round(float x) { return bf16_float(bf16_bits(x)); }

// Normal CDF Phi(x) = (1 + erf(x / sqrt 2)) / 2 from the Chebyshev-fitted
// erfc of Numerical Recipes (2nd ed., section 6.2; fractional error below
// 1.2e-7 for every argument), taken at |x| so that both tails keep their
// relative accuracy: Phi = 1 - erfc(|x|/sqrt 2)/2 for x >= 0, else
// erfc(|x|/sqrt 2)/2.  About 16 vector instructions against some 50 for the
// library erff; GELU's 128 evaluations per face dominate the MLP's cost.
__device__ __forceinline__ float norm_cdf(float x) {
  const float z = fabsf(x) * 0.70710678118654752f;
  const float t = __builtin_amdgcn_rcpf(1.0f + 0.5f * z);
  float p = 0.17087277f;
  p = fmaf(p, t, -0.82215223f);
  p = fmaf(p, t, 1.48851587f);
  p = fmaf(p, t, -1.13520398f);
  p = fmaf(p, t, 0.27886807f);
  p = fmaf(p, t, -0.18628806f);
  p = fmaf(p, t, 0.09678418f);
  p = fmaf(p, t, 0.37409196f);
  p = fmaf(p, t, 1.00002368f);
  p = fmaf(p, t, -1.26551223f);
  const float e = 0.5f * t * __expf(fmaf(-z, z, p));
  return x >= 0.0f ? 1.0f - e : e;
}

// What the in-step inference reads from LDS: the GELU table (kGeluN pieces, see
// mhd_kernels.hpp), one array per coefficient -- the 64 lanes of a read fetch
// scattered pieces, and one 4-byte word a piece per read spreads them over
// all the banks, where 16-byte pieces fall into eight bank groups and
// conflict four times as often --, and the biases of the three layers.
constexpr int kMlpBiases = 2 * kMlpHid + kMlpOut;
struct alignas(16) MlpLds {
  float c0[kGeluN], c1[kGeluN], c2[kGeluN];
  float b[kMlpBiases];
};
__device__ __forceinline__ void fill_mlp_lds(MlpLds& t, const float4* __restrict__ gelu,
                                             const float* __restrict__ P) {
  for (int e = (int)threadIdx.x; e < kGeluN; e += (int)blockDim.x) {
    const float4 c = gelu[e];
    t.c0[e] = c.x;
    t.c1[e] = c.y;
    t.c2[e] = c.z;
  }
  for (int e = (int)threadIdx.x; e < kMlpBiases; e += (int)blockDim.x)
    t.b[e] = P[e < kMlpHid ? kP_B1 + e
                           : (e < 2 * kMlpHid ? kP_B2 + e - kMlpHid : kP_B3 + e - 2 * kMlpHid)];
}

// GELU(x) = c0 + x (c1 + x c2) of x's piece: adding kGeluMagic rounds x in
// quarters of a piece to an integer in the low mantissa bits, the clamp keeps
// it within the table, and one mask makes it the byte offset of the piece, so
// an evaluation is 5 vector instructions and two LDS reads (8 with a table of
// Phi over the position in the piece; 128 evaluations a face).  Error against
// FP64 over [-8.5, 8.5]: largest 3.4e-7 and rms 5.5e-8, where x Phi(x) had
// 4.9e-7 and 6.4e-8.  A NaN argument reads the lowest piece and stays NaN.
__device__ __forceinline__ float gelu_tab(const MlpLds& t, float x) {
  const float u = __builtin_amdgcn_fmed3f(fmaf(x, 4.0f * kGeluScale, kGeluMagic),
                                          kGeluMagic - 2 * kGeluN, kGeluMagic + 2 * kGeluN - 1);
  const unsigned e = (__float_as_uint(u) & (4u * kGeluN - 4u)) >> 2;
  return fmaf(x, fmaf(x, t.c2[e], t.c1[e]), t.c0[e]);
}

// GELU(x) = x Phi(x) and its derivative Phi(x) + x phi(x).
__device__ __forceinline__ float gelu(float x) { return x * norm_cdf(x); }
__device__ __forceinline__ float gelu_d(float x, float phi) {  // phi: Phi(x)
  return phi + x * __expf(-0.5f * x * x) * 0.39894228040143268f;
}

// Orders a wave's LDS accesses (which the hardware runs in program order):
// what its lanes wrote before is read by its lanes after.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Two values in one hardware conversion (v_cvt_pk_bf16_f32, round to
// nearest even: the same as bf16_bits for finite values), a in the low
// half, b in the high half.
__device__ __forceinline__ unsigned bf16_pair(float a, float b) {
  return __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a, b}, bf16v2));
}

__device__ __forceinline__ bf16x4 pack4(unsigned short a, unsigned short b, unsigned short c,
                                        unsigned short d) {
  bf16x4 v;
  v[0] = (short)a;
  v[1] = (short)b;
  v[2] = (short)c;
  v[3] = (short)d;
  return v;
}

__device__ __forceinline__ f32x4 mfma16(bf16x4 a, bf16x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// B fragment of W^T for a layer y = W x (W row-major [N][K] FP32): column n,
// rows k0 .. k0+3 are W[n][k0 .. k0+3]; rows n >= nvalid are zero.
__device__ __forceinline__ bf16x4 wt_frag(const float* __restrict__ W, int K, int n, int k0,
                                          int nvalid) {
  if (n >= nvalid) return pack4(0, 0, 0, 0);
  const float* w = W + n * K + k0;
  return pack4(bf16_bits(w[0]), bf16_bits(w[1]), bf16_bits(w[2]), bf16_bits(w[3]));
}

// One dense layer for the 64 samples of a wave.  in: LDS bf16 [64][ins]
// (K inputs); W: FP32 [N][K] (first nvalid rows real, the rest zero); out:
// pre-activations + bias for D element (m, n) go to emit(m, n, value).
template <int K, int NB, class Emit>
__device__ __forceinline__ void wave_layer(const unsigned short* in, int ins,
                                           const float* __restrict__ W, const float* __restrict__ b,
                                           int nvalid, Emit emit) {
  const int lane = threadIdx.x & 63;
  const int r = lane & 15, q = lane >> 4;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    bf16x4 bw[K / 16];
#pragma unroll
    for (int kb = 0; kb < K / 16; ++kb) bw[kb] = wt_frag(W, K, nb * 16 + r, kb * 16 + 4 * q, nvalid);
    const int n = nb * 16 + r;
    const float bias = n < nvalid ? b[n] : 0.0f;
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kb = 0; kb < K / 16; ++kb) {
        const bf16x4 a = *(const bf16x4*)(in + (mb * 16 + r) * ins + kb * 16 + 4 * q);
        acc = mfma16(a, bw[kb], acc);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) emit(mb * 16 + 4 * q + i, n, acc[i] + bias);
    }
  }
}

// LDS row strides (bf16 elements), padded to spread banks.
constexpr int kXs = kMlpIn + 4;
constexpr int kHs = kMlpHid + 4;

// Forward pass of a wave's 64 samples.  X: LDS bf16 [64][kXs] (inputs,
// already rounded); H1, H2: LDS bf16 [64][kHs]; Y: LDS float [64][8].
// Every wave of the block must call it (it holds
// block barriers between the layers: lanes read what other lanes wrote).
__device__ __forceinline__ void wave_mlp_forward(const float* __restrict__ P,
                                                 const unsigned short* X, unsigned short* H1,
                                                 unsigned short* H2, float* Y) {
  wave_layer<32, 4>(X, kXs, P + kP_W1, P + kP_B1, 64, [&](int m, int n, float v) {
    H1[m * kHs + n] = bf16_bits(gelu(v));
  });
  __syncthreads();
  wave_layer<64, 4>(H1, kHs, P + kP_W2, P + kP_B2, 64, [&](int m, int n, float v) {
    H2[m * kHs + n] = bf16_bits(gelu(v));
  });
  __syncthreads();
  wave_layer<64, 1>(H2, kHs, P + kP_W3, P + kP_B3, 8, [&](int m, int n, float v) {
    if (n < 8) Y[m * 8 + n] = v;
  });
  __syncthreads();
}

// ---- inference with the activations kept in registers ------------------
// Each layer is computed transposed, H^T = W X^T: the weights are the A
// operand (M = outputs, K = inputs), the samples the B operand (N).  The D
// fragment of output block mb then holds, in lane (r, q), features
// 16 mb + 4q .. 4q+3 of sample r -- exactly the B fragment of the next
// layer's input block kb = mb, so hidden activations never leave the
// registers: bias, GELU and the bf16 rounding happen in place.
//
// Weights are pre-packed (k_mlp_pack, from the FP32 master vector) as bf16
// A fragments of 16 x 32 (v_mfma_f32_16x16x32_bf16, 8 values a lane): the
// contraction's index may run in any order that A and B share, so slot
// (q, j) of block kp stands for feature 32 kp + 4 q + j (j < 4) and 32 kp + 16
// + 4 q + j - 4 (j >= 4) -- a lane's two D fragments of the layer before, side
// by side.  Fragment f holds, in lane l = r + 16 q, those 8 weights of row 16
// mb + r, stored [f][64 lanes][16 bytes] so that one wave fetches a fragment
// with one coalesced 1 KB load.  Rows beyond a layer's outputs (W3 has 8) are
// zero.
constexpr int kFragW1 = 0;            // mb 0..3
constexpr int kFragW2 = kFragW1 + 4;  // mb 0..3 x kp 0..1
constexpr int kFragW3 = kFragW2 + 8;  // kp 0..1
constexpr int kNumFrags = kFragW3 + 2;
constexpr int kFragBytes = kNumFrags * 64 * 16;

typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ bf16x8 frag_of(const u32x4* __restrict__ W, int f, int lane) {
  return __builtin_bit_cast(bf16x8, W[f * 64 + lane]);
}
__device__ __forceinline__ bf16x8 side_by_side(u32x2 a, u32x2 b) {
  return __builtin_bit_cast(bf16x8, u32x4{a[0], a[1], b[0], b[1]});
}
__device__ __forceinline__ f32x4 mfma32(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// The biases of a lane's 4 D values (features 4q .. 4q+3 of the block, in LDS),
// the accumulator's start: the matrix core adds them with the products.
__device__ __forceinline__ f32x4 bias4(const float* b) {
  return *(const f32x4*)b;
}

// GELU (from the LDS table) of the 4 D values of a lane (bias already in),
// rounded to bf16.
__device__ __forceinline__ u32x2 act4(f32x4 d, const MlpLds& t) {
  float g[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) g[i] = gelu_tab(t, d[i]);
  return u32x2{bf16_pair(g[0], g[1]), bf16_pair(g[2], g[3])};
}

// y = MLP(x) for the 64 samples of a wave, 16 at a time.  X: LDS bf16
// [64][kXs], row = sample; the sample's 8 outputs replace the start of its row
// (mlp_out).  Wave-local: the caller orders the writes of X (wave_sync) and of
// t (a barrier) before, and the reads of the outputs (wave_sync) after.
//
// 16x16x32 fragments halve the MFMAs (56 a wave) and the weight loads of
// 16x16x16 ones: k_flux_mlp 199 -> 186 us a launch (128^3, event timing).
// Weights and biases are read again for every 16 samples: held through the loop (the compiler
// hoists them if it may) they take 88 of the registers, and the kernel is bound
// by what its waves overlap of its phases -- the stencil's reads (the address
// unit 69 % busy), the table's LDS reads (77 %, two fifths of it bank
// conflicts), the vector instructions (70 %).  With them reloaded and the
// outputs in place of the inputs 5 waves a SIMD fit where 4 did: 176 -> 162 us a
// launch, both in turn on one card (172 on another; 6 waves, weights from LDS in
// blocks of 512 or 640, two blocks of samples a load: slower than 4 waves).
constexpr int kMlpOutLd = kXs / 2;  // floats from one sample's outputs to the next's
__device__ __forceinline__ const float* mlp_out(const unsigned short* X, int sample) {
  return (const float*)X + sample * kMlpOutLd;
}
__device__ __forceinline__ void wave_mlp_infer(const u32x4* __restrict__ W, unsigned short* X,
                                               const MlpLds& t) {
  const int lane = threadIdx.x & 63;
  const int r = lane & 15, q = lane >> 4;
#pragma unroll 1
  for (int sb = 0; sb < 4; ++sb) {
    const unsigned short* xr = X + (sb * 16 + r) * kXs + 4 * q;
    const bf16x8 x = side_by_side(*(const u32x2*)(xr), *(const u32x2*)(xr + 16));
    u32x2 h1[4], h2[4];
    int f0 = 4 * q;
    asm volatile("" : "+v"(f0));  // keeps the loads of the turn in the turn
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
      h1[mb] = act4(mfma32(frag_of(W, kFragW1 + mb, lane), x, bias4(t.b + 16 * mb + f0)), t);
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
      f32x4 acc = bias4(t.b + kMlpHid + 16 * mb + f0);
#pragma unroll
      for (int kp = 0; kp < 2; ++kp)
        acc = mfma32(frag_of(W, kFragW2 + 2 * mb + kp, lane),
                     side_by_side(h1[2 * kp], h1[2 * kp + 1]), acc);
      h2[mb] = act4(acc, t);
    }
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kp = 0; kp < 2; ++kp)
      acc = mfma32(frag_of(W, kFragW3 + kp, lane), side_by_side(h2[2 * kp], h2[2 * kp + 1]), acc);
    if (q < 2) {
      float* y = (float*)X + (sb * 16 + r) * kMlpOutLd + 4 * q;
#pragma unroll
      for (int i = 0; i < 4; ++i) y[i] = acc[i] + t.b[2 * kMlpHid + f0 + i];
    }
  }
}

// ---- face features and the output <-> flux maps ------------------------
// w8 = rho, vn, vt1, vt2, P, Bn, Bt1, Bt2 of cells i-2 .. i+1 (face i-1/2),
// cell-centred, face-normal frame.  Face means rho_m, v_m, P_m of cells i-1,
// i; c_m = sqrt(gamma P_m / rho_m).

struct FaceScale {
  float rm, cm, sr;  // rho_m, c_m, sqrt(rho_m)
  float vm[3];
};

__device__ __forceinline__ FaceScale face_scale(const float w8[32], float gam) {
  FaceScale s;
  s.rm = 0.5f * (w8[8] + w8[16]);
  for (int d = 0; d < 3; ++d) s.vm[d] = 0.5f * (w8[9 + d] + w8[17 + d]);
  s.cm = __builtin_amdgcn_sqrtf(gam * 0.5f * (w8[12] + w8[20]) / s.rm);
  s.sr = __builtin_amdgcn_sqrtf(s.rm);
  return s;
}

// x = rho/rho_m, (v - v_m)/c_m, P/(rho_m c_m^2), B/(sqrt(rho_m) c_m) per cell.
__device__ __forceinline__ void face_features(const float w8[32], const FaceScale& s,
                                              float x[32]) {
  const float ir = 1.0f / s.rm, ic = 1.0f / s.cm;
  const float ip = ir * ic * ic, ib = ic / s.sr;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const float* w = w8 + 8 * c;
    float* o = x + 8 * c;
    o[0] = w[0] * ir;
    for (int d = 0; d < 3; ++d) o[1 + d] = (w[1 + d] - s.vm[d]) * ic;
    o[4] = w[4] * ip;
    for (int d = 0; d < 3; ++d) o[5 + d] = w[5 + d] * ib;
  }
}

// y (8 outputs) -> flux correction in the face frame (rho, Mn, Mt1, Mt2, E,
// Bt1, Bt2): rho_m c_m, rho_m c_m^2, rho_m c_m^3, sqrt(rho_m) c_m^2 scales and
// the Galilean shift by v_m of the momentum and energy rows; y[5] unused.
__device__ __forceinline__ void out_to_flux(const FaceScale& s, const float y[8], float df[7]) {
  const float fr = s.rm * s.cm * y[0];
  const float k2 = s.rm * s.cm * s.cm;
  const float fm0 = k2 * y[1], fm1 = k2 * y[2], fm2 = k2 * y[3];
  const float fe = k2 * s.cm * y[4];
  const float v2 = s.vm[0] * s.vm[0] + s.vm[1] * s.vm[1] + s.vm[2] * s.vm[2];
  df[0] = fr;
  df[1] = fm0 + s.vm[0] * fr;
  df[2] = fm1 + s.vm[1] * fr;
  df[3] = fm2 + s.vm[2] * fr;
  df[4] = fe + (s.vm[0] * fm0 + s.vm[1] * fm1 + s.vm[2] * fm2) + 0.5f * v2 * fr;
  const float kb = s.sr * s.cm * s.cm;
  df[5] = kb * y[6];
  df[6] = kb * y[7];
}

__device__ __forceinline__ void flux_to_out(const FaceScale& s, const float df[7], float y[8]) {
  const float fr = df[0];
  const float fm0 = df[1] - s.vm[0] * fr, fm1 = df[2] - s.vm[1] * fr, fm2 = df[3] - s.vm[2] * fr;
  const float v2 = s.vm[0] * s.vm[0] + s.vm[1] * s.vm[1] + s.vm[2] * s.vm[2];
  const float fe = df[4] - (s.vm[0] * fm0 + s.vm[1] * fm1 + s.vm[2] * fm2) - 0.5f * v2 * fr;
  const float k2 = s.rm * s.cm * s.cm;
  y[0] = fr / (s.rm * s.cm);
  y[1] = fm0 / k2;
  y[2] = fm1 / k2;
  y[3] = fm2 / k2;
  y[4] = fe / (k2 * s.cm);
  y[5] = 0.0f;
  const float kb = s.sr * s.cm * s.cm;
  y[6] = df[5] / kb;
  y[7] = df[6] / kb;
}

}  // namespace mhd
