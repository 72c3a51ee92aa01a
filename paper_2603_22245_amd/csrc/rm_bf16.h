// Products of one-hot (string, letter) rows with the FP32 phase table on
// 32x32x16 bfloat16 MFMAs, shared by the rescore and threshold kernels.
//
// Component (k, L) of a string's RoPE vector sums the table entries
// omega^(f_k p) over the positions p holding letter L (§2.1-§2.2), so the
// vectors of a set of strings are the product of their one-hot rows with the
// table [p][factor].  The table splits exactly into three bfloat16 parts and
// the indicators are exact in bfloat16, so three bf16 MFMAs with FP32
// accumulation give the FP32 direct sums up to the order of the additions.
#pragma once

#include "rm_internal.h"

namespace rm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Exact split of an FP32 value into three bfloat16 bit patterns, x = hi + mid +
// lo: hi keeps the sign, exponent and top 7 stored mantissa bits of x
// (truncated), so x - hi is exact and has at most 16 significant bits; mid
// keeps the top 8 of those, and the exact remainder has at most 8 (bfloat16
// has the exponent range of FP32, so no part underflows).
__device__ __forceinline__ void split_bf16x3(float x, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
  const uint32_t h = __float_as_uint(x) & 0xffff0000u;
  const float r1 = x - __uint_as_float(h);
  const uint32_t m = __float_as_uint(r1) & 0xffff0000u;
  const float r2 = r1 - __uint_as_float(m);
  hi = h >> 16;
  mid = m >> 16;
  lo = __float_as_uint(r2) >> 16;
}

// One 64-position chunk (positions pb .. pb+63, zero past N) of the table
// [N][64 reals] as its three parts in LDS: tparts[part][column block][8
// positions][column] holds the 8 bf16 of positions 8 pg .. 8 pg + 7 (the B
// fragment layout of the 32x32x16 bf16 MFMA).  Block-cooperative: 512
// fragments over `nthreads` threads.
__device__ __forceinline__ void stage_table_parts(const float* __restrict__ tab, int pb, int N,
                                                  u32x4 (*tparts)[2][8][32], int tid,
                                                  int nthreads) {
#pragma unroll 2
  for (int f = tid; f < 512; f += nthreads) {
    const int c = f & 31, pg = (f >> 5) & 7, cb = f >> 8;
    float x[8];  // loads without a branch, so that all are in flight together
#pragma unroll
    for (int jj = 0; jj < 8; ++jj)
      x[jj] = tab[(int64_t)min(pb + 8 * pg + jj, N - 1) * 64 + cb * 32 + c];
    uint32_t hi[8], mid[8], lo[8];
#pragma unroll
    for (int jj = 0; jj < 8; ++jj)
      split_bf16x3(pb + 8 * pg + jj < N ? x[jj] : 0.f, hi[jj], mid[jj], lo[jj]);
    tparts[0][cb][pg][c] = u32x4{hi[0] | hi[1] << 16, hi[2] | hi[3] << 16, hi[4] | hi[5] << 16,
                                 hi[6] | hi[7] << 16};
    tparts[1][cb][pg][c] = u32x4{mid[0] | mid[1] << 16, mid[2] | mid[3] << 16,
                                 mid[4] | mid[5] << 16, mid[6] | mid[7] << 16};
    tparts[2][cb][pg][c] = u32x4{lo[0] | lo[1] << 16, lo[2] | lo[3] << 16, lo[4] | lo[5] << 16,
                                 lo[6] | lo[7] << 16};
  }
}

// A fragment of eight positions of one (string, letter) row: `w` holds the
// string's letters there (bytes 0..3, 4 for none), `onehot_tab` has byte L =
// 0x40 for the row's letter L and 0 elsewhere; the result is bf16 2.0 where the
// letter matches, else 0 (2 keeps one byte of the pattern: sums come out
// doubled, which halving undoes exactly).
__device__ __forceinline__ bf16x8 onehot_fragment(uint2 w, uint32_t onehot_tab) {
  const uint32_t h0 = __builtin_amdgcn_perm(0u, onehot_tab, w.x);  // bytes 0x40 / 0
  const uint32_t h1 = __builtin_amdgcn_perm(0u, onehot_tab, w.y);
  const u32x4 av{__builtin_amdgcn_perm(0u, h0, 0x010c000cu), __builtin_amdgcn_perm(0u, h0, 0x030c020cu),
                 __builtin_amdgcn_perm(0u, h1, 0x010c000cu), __builtin_amdgcn_perm(0u, h1, 0x030c020cu)};
  return __builtin_bit_cast(bf16x8, av);
}

// ---- fidelities of eight strings from a row block of the product
// Row 4 s + L of a block holds string s's sums for letter L, 64 reals (re, im per
// factor); rows of kMatRow floats keep 16-byte reads aligned and the lanes'
// rows in different banks.
constexpr int kMatRow = 68;

// F = |<x|c>|^2 / (X C) of the block's strings with the head x (rows `head`,
// squared norm X; zero where X or C is below `lowest`), string s in lanes 8 s
// .. 8 s + 7.  A lane takes four factors of its string: three sums of 32 reals in
// registers, then three exchanges.  The additions are those of wave_sum over
// lanes that hold a factor's two letter pairs each (pairs, then neighbours at
// distance 2, 4, 8, 16 and 32), in its order, and every term is formed as it
// was there, so F keeps its bits; a wavefront sum per string and per
// term took 97 instructions a string, this takes about 19.
__device__ __forceinline__ float strings_fidelity(const float (*mat)[kMatRow],
                                                  const float (*head)[kMatRow], float X,
                                                  float lowest, int lane) {
  const int s = lane >> 3, c0 = 8 * (lane & 7);
  float m[4][8], x[4][8];
#pragma unroll
  for (int L = 0; L < 4; ++L)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      *reinterpret_cast<float4*>(&m[L][4 * i]) =
          *reinterpret_cast<const float4*>(&mat[4 * s + L][c0 + 4 * i]);
      *reinterpret_cast<float4*>(&x[L][4 * i]) = *reinterpret_cast<const float4*>(&head[L][c0 + 4 * i]);
    }
  float C[4], R[4], I[4];
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    float c[2], r[2], q[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float ax = m[2 * h][2 * f], ay = m[2 * h][2 * f + 1];
      const float bx = m[2 * h + 1][2 * f], by = m[2 * h + 1][2 * f + 1];
      const float px = x[2 * h][2 * f], py = x[2 * h][2 * f + 1];
      const float qx = x[2 * h + 1][2 * f], qy = x[2 * h + 1][2 * f + 1];
      c[h] = __builtin_fmaf(by, by, __builtin_fmaf(bx, bx, __builtin_fmaf(ax, ax, ay * ay)));
      r[h] = __builtin_fmaf(qy, by, __builtin_fmaf(qx, bx, __builtin_fmaf(px, ax, py * ay)));
      q[h] = __builtin_fmaf(-qy, bx, __builtin_fmaf(qx, by, __builtin_fmaf(px, ay, -(py * ax))));
    }
    C[f] = c[0] + c[1];
    R[f] = r[0] + r[1];
    I[f] = q[0] + q[1];
  }
  auto total = [&](const float (&v)[4]) {
    float t = (v[0] + v[1]) + (v[2] + v[3]);
    t += dpp<0xB1>(t);   // quad_perm [1,0,3,2]
    t += dpp<0x4E>(t);   // quad_perm [2,3,0,1]
    t += dpp<0x141>(t);  // row_half_mirror
    return t;
  };
  const float c = total(C), re = total(R), im = total(I);
  return X < lowest || c < lowest ? 0.f : __builtin_fmaf(re, re, im * im) / (X * c);
}

// Squared norm of the head in rows `head`, summed like the strings' above, in
// every lane.
__device__ __forceinline__ float head_norm2(const float (*head)[kMatRow], int lane) {
  const int k = lane >> 1, h = lane & 1;
  const float2 a = *reinterpret_cast<const float2*>(&head[2 * h][2 * k]);
  const float2 b = *reinterpret_cast<const float2*>(&head[2 * h + 1][2 * k]);
  return wave_sum(__builtin_fmaf(
      b.y, b.y, __builtin_fmaf(b.x, b.x, __builtin_fmaf(a.x, a.x, a.y * a.y))));
}

}  // namespace rm
