// BF16 inference of the learned token offsets on the matrix cores.
//
// For every 9-mer token location t of a letter string (t = 0..n-9) the network
// maps the one-hot of the 8 flanking letters (w[t..t+3], w[t+5..t+8]) to 128
// outputs, o = W2 relu(W1 x + b1) + b2, and keeps the 32 of the middle letter
// w[t+4]: delta[t][k] = o[w[t+4]*32 + k] (0 if the middle letter is not A, C,
// G or T).  Weights and hidden values are rounded to bfloat16 (nearest, ties
// to even); products accumulate in FP32; biases are added in FP32.
//
// Layout on the 32x32x16 bf16 MFMA, one wavefront per tile of 32 tokens, both
// layers transposed so that no data crosses lanes:
//   layer 1: P^T [64 hidden x 32 tokens] = W1 [64 x 32] * X^T [32 x 32]
//            (2 hidden tiles x 2 K steps; X^T is built from the letters in the
//            lane that owns the token column);
//   layer 2: O^T [128 x 32 tokens] = W2 [128 x 64] * H^T [64 x 32]
//            (4 output tiles = the 4 middle letters, 4 K steps).  The B
//            operand of layer 2 is the layer-1 accumulator itself, relu'd and
//            rounded: lane l holds hidden rows 8(v/4) + 4(l/32) + v%4 of its
//            token column, so K step (mt, half) pairs slot j of lane l with
//            hidden 32mt + 16half + 8(j/4) + 4(l/32) + j%4, and W2's fragments
//            are gathered in that order.
// Lane l (column token l%32) then holds 16 of its token's 32 outputs per
// letter tile and keeps the tile of its own middle letter.
#include "rm_internal.h"

namespace rm {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kIn = 32, kHid = 64, kOut = 128;
constexpr int kW1 = 0, kB1 = kHid * kIn, kW2 = kB1 + kHid, kB2 = kW2 + kOut * kHid;
constexpr int kWavesPerBlock = 4;

__device__ __forceinline__ unsigned short bf16_bits(float x) {
  uint32_t u = __float_as_uint(x);
  u += 0x7FFFu + ((u >> 16) & 1u);  // round to nearest, ties to even
  return (unsigned short)(u >> 16);
}

__device__ __forceinline__ bf16x8 as_bf16(u16x8 v) { return __builtin_bit_cast(bf16x8, v); }

// The letters t..t+8 of a lane's token.
struct Letters {
  uint32_t first, last;  // w[t..t+3], w[t+5..t+8], one byte each
  int mid;
};

__device__ __forceinline__ Letters load_letters(const uint8_t* __restrict__ seq, int64_t t,
                                                int64_t n_tok) {
  Letters l{0x04040404u, 0x04040404u, 4};
  if (t < n_tok) {
    __builtin_memcpy(&l.first, seq + t, 4);
    __builtin_memcpy(&l.last, seq + t + 5, 4);
    l.mid = seq[t + 4];
  }
  return l;
}

// One letter's four inputs, 1.0 at the letter's and none beyond the fourth.
__device__ __forceinline__ uint2 onehot(uint32_t letter) {
  const uint64_t v = letter < 4 ? (uint64_t)0x3F80 << (16 * letter) : 0;
  return make_uint2((uint32_t)v, (uint32_t)(v >> 32));
}

// Bound by its stores (128 bytes a token) and VALU issue.  Lane l holds 16-byte
// pieces of a token's row; they go through LDS, so that a store instruction
// writes 1 KB in a row and not halves of 32 lines, and the next tile's letters
// are loaded (three loads) before this tile's products.  10^7 letters: 400 us,
// 3.2 TB/s; 700 us with 16-byte stores 32
// bytes apart, nine byte loads in the chain, and the rounding done in integers.
__global__ __launch_bounds__(64 * kWavesPerBlock, 2) void mlp_infer_kernel(
    const float* __restrict__ params, const uint8_t* __restrict__ seq, int64_t n_tok,
    float* __restrict__ delta) {
  __shared__ float sb2[kOut + 32];  // the last row, of other letters, is 0
  __shared__ float rows[kWavesPerBlock][32][36];  // 36: 16 lanes' 16 bytes on 64 banks
  for (int i = threadIdx.x; i < kOut + 32; i += blockDim.x) sb2[i] = i < kOut ? params[kB2 + i] : 0.f;
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 5, col = lane & 31;

  // the biases of the lane's hidden rows, the first products' addend
  floatx16 b1[2];
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int v = 0; v < 16; ++v)
      b1[mt][v] = params[kB1 + 32 * mt + 8 * (v >> 2) + 4 * g + (v & 3)];
  // weight fragments (A operands), rounded once per wavefront
  bf16x8 w1f[2][2];
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      u16x8 v;
      const float* src = params + kW1 + (32 * mt + col) * kIn + 16 * ks + 8 * g;
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = bf16_bits(src[j]);
      w1f[mt][ks] = as_bf16(v);
    }
  bf16x8 w2f[4][4];
#pragma unroll
  for (int mo = 0; mo < 4; ++mo)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int mt = ks >> 1, half = ks & 1;
      u16x8 v;
      const float* src = params + kW2 + (32 * mo + col) * kHid + 32 * mt + 16 * half + 4 * g;
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = bf16_bits(src[8 * (j >> 2) + (j & 3)]);
      w2f[mo][ks] = as_bf16(v);
    }

  const int64_t n_tiles = (n_tok + 31) / 32;
  const int64_t step = (int64_t)gridDim.x * kWavesPerBlock;
  int64_t tile = (int64_t)blockIdx.x * kWavesPerBlock + wave;
  Letters next = load_letters(seq, tile * 32 + col, n_tok);
  for (; tile < n_tiles; tile += step) {
    const Letters let = next;  // of token 32 tile + col
    next = load_letters(seq, (tile + step) * 32 + col, n_tok);

    // layer 1.  Inputs 16ks + 8g + j: flank 4ks + 2g + j/4, letter j%4
    floatx16 acc1[2] = {b1[0], b1[1]};
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const uint32_t w = (ks ? let.last : let.first) >> (16 * g);
      const uint2 lo = onehot(w & 255), hi = onehot(w >> 8 & 255);
      const bf16x8 xb = __builtin_bit_cast(bf16x8, make_uint4(lo.x, lo.y, hi.x, hi.y));
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
        acc1[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1f[mt][ks], xb, acc1[mt], 0, 0, 0);
    }
    // hidden values, relu'd and rounded: the B operands of layer 2
    bf16x8 hf[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int mt = ks >> 1, half = ks & 1;
#pragma unroll
      for (int j = 0; j < 8; ++j) hf[ks][j] = (__bf16)__builtin_amdgcn_fmed3f(acc1[mt][8 * half + j], 0.f, INFINITY);
    }
    // layer 2, one letter tile at a time; keep the middle letter's
    const int mid = let.mid;
    floatx16 res;
#pragma unroll
    for (int v = 0; v < 16; ++v) res[v] = 0.f;
#pragma unroll
    for (int mo = 0; mo < 4; ++mo) {
      floatx16 acc2;
#pragma unroll
      for (int v = 0; v < 16; ++v) acc2[v] = 0.f;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        acc2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w2f[mo][ks], hf[ks], acc2, 0, 0, 0);
#pragma unroll
      for (int v = 0; v < 16; ++v) res[v] = mid == mo ? acc2[v] : res[v];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 b = *reinterpret_cast<const float4*>(&sb2[32 * min(mid, 4) + 8 * q + 4 * g]);
      *reinterpret_cast<float4*>(&rows[wave][col][8 * q + 4 * g]) = make_float4(
          res[4 * q] + b.x, res[4 * q + 1] + b.y, res[4 * q + 2] + b.z, res[4 * q + 3] + b.w);
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = 8 * q + (lane >> 3);
      const int64_t t = tile * 32 + r;
      if (t < n_tok)
        *reinterpret_cast<float4*>(delta + t * 32 + 4 * (lane & 7)) =
            *reinterpret_cast<const float4*>(&rows[wave][r][4 * (lane & 7)]);
    }
    __builtin_amdgcn_wave_barrier();  // the rows are rewritten by the next tile
  }
}

}  // namespace

hipError_t launch_mlp_infer(const float* params, const uint8_t* seq, int64_t n_letters,
                            float* delta, hipStream_t s) {
  const int64_t n_tok = n_letters - 8;
  const int64_t tiles = (n_tok + 31) / 32;
  int64_t blocks = (tiles + kWavesPerBlock - 1) / kWavesPerBlock;
  if (blocks > 512) blocks = 512;  // all resident: a wavefront loads the weights once
  hipLaunchKernelGGL(mlp_infer_kernel, dim3((unsigned)blocks), dim3(64 * kWavesPerBlock), 0, s,
                     params, seq, n_tok, delta);
  return hipGetLastError();
}

}  // namespace rm
