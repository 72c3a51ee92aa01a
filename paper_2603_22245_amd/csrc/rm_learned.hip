// Learned angle offsets: forward encoding, pair fidelity, ranking loss,
// backward pass and Adam update, all FP32.
//
// The learned encoding (the paper has none; it notes that token definitions,
// initial encodings or rotations could be altered, §2.10): 9-mer tokens at
// locations p = 0..n-9 (s-mer locations, §2.1); the middle letter L picks the
// component; the 8 flanking letters, one-hot (32 inputs), go through
// o = W2 relu(W1 x + b1) + b2 (128 outputs = 4 letters x 32 factors); the
// token adds exp(i (theta_k p + o[L*32+k])) to component (k, L), theta_k =
// 2 pi (k+1) / N (§2.2) with N the nominal length.  Fidelity (§2.4) of pairs,
// and a pairwise logistic ranking loss on Levenshtein labels.
//
// Parameters: W1 [64][32], b1 [64], W2 [128][64], b2 [128], row-major, FP32.
//
// A block of eight wavefronts takes up to eight strings.  Their tokens are
// sorted by middle letter, two wavefronts per letter, so that the second layer
// of a wavefront's tokens is one product with the letter's 32 rows of W2, and
// go through the matrix cores 16 at a time:
//   layer 1: P^T [64 x 16 tokens] = W1 [64 x 32] X^T [32 x 16].  X is one-hot,
//     exact in bfloat16, and W1 is the exact sum of three bfloat16 parts, so
//     three bf16 MFMAs per product are FP32 sums up to the order of additions;
//   layer 2: O^T [32 x 16] = W2_L [32 x 64] H^T [64 x 16], both split: of the
//     nine products of parts all but low x low (2^-32 of the product) are
//     added.  Lane l of an accumulator holds rows 16 rb + 4 (l / 16) + v of
//     column l % 16; eight such rows of a lane are the K entries of the next
//     product's B operand (its A operand lists them in the same order), so no
//     data moves;
//   a lane then owns 8 factors of its token: phase, sine and cosine.
// FP32 MFMAs would need no splits, but run at a sixteenth of the bf16 rate:
// for layer 2 they cost 6 % of a step more at the same error (0.97e-7 against
// 0.96e-7 of the gradient's 2-norm, 1.1e-7 with VALU sums).  In the backward
// products the split doubled the error (2e-7) and is not used.
// A step of 1,024 pairs of 150 letters takes 113 us (encoder 32, ranking 6,
// backward 70, reduction and Adam 5); 706 us with one token at a time on the
// VALU (189, 84, 416, 13).
#include <algorithm>

#include "rm_bf16.h"
#include "rm_internal.h"

namespace rm {

namespace {

constexpr int kIn = 32, kHid = 64, kOut = 128;
constexpr int kW1 = 0, kB1 = kHid * kIn, kW2 = kB1 + kHid, kB2 = kW2 + kOut * kHid;
constexpr int kParams = kB2 + kOut;  // 10,432
constexpr int kMaxLen = 256;         // letters of a string kept in LDS
constexpr int kMaxTok = kMaxLen - 8;
constexpr int kStrings = 8;          // strings of a block, at most
constexpr int kWaves = 8;
constexpr float kInvTau = 20.f;  // of the ranking loss, 1 / 0.05

static_assert(kParams == RM_LEARNED_PARAMS, "parameter count");

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

// What every wavefront of a block reads of the network: W1's three bfloat16
// parts as A fragments (rows 16 rb + lane % 16, inputs 8 (lane / 16) + 0..7),
// and the biases.
struct Net {
  u32x4 w1[3][4][64];
  float b1[kHid];
  float b2[kOut];
  uint32_t odd[5];  // 1 where the wavefront's part of W1, or b1, holds an infinity or no number
};

__device__ __forceinline__ void load_net(Net& net, const float* __restrict__ p) {
  const int t = threadIdx.x;
  if (t < 256) {
    const int rb = t >> 6, lane = t & 63;
    const float* src = p + kW1 + (16 * rb + (lane & 15)) * kIn + 8 * (lane >> 4);
    uint32_t part[3][8];
#pragma unroll
    for (int j = 0; j < 8; ++j) split_bf16x3(src[j], part[0][j], part[1][j], part[2][j]);
    bool finite = true;
#pragma unroll
    for (int j = 0; j < 8; ++j) finite &= fabsf(src[j]) < INFINITY;
    const uint32_t odd = __ballot(!finite) != 0;
    if (lane == 0) net.odd[rb] = odd;
#pragma unroll
    for (int q = 0; q < 3; ++q)
      net.w1[q][rb][lane] =
          u32x4{part[q][0] | part[q][1] << 16, part[q][2] | part[q][3] << 16,
                part[q][4] | part[q][5] << 16, part[q][6] | part[q][7] << 16};
  } else if (t < 256 + kHid) {  // the fifth wavefront
    const float b = p[kB1 + t - 256];
    net.b1[t - 256] = b;
    const uint32_t odd = __ballot(!(fabsf(b) < INFINITY)) != 0;
    if (t == 256) net.odd[4] = odd;
  } else if (t < 256 + kHid + kOut) {
    net.b2[t - 256 - kHid] = p[kB2 + t - 256 - kHid];
  }
}

// Whether W1 or b1 holds an infinity or no number; uniform, after the barrier.
__device__ __forceinline__ bool odd_net(const Net& net) {
  return __builtin_amdgcn_readfirstlane(net.odd[0] | net.odd[1] | net.odd[2] | net.odd[3] |
                                        net.odd[4]) != 0;
}

// max(x, 0) as one integer maximum (a positive NaN would stay, but settle leaves
// none; fmaxf would take two instructions to quiet it).
__device__ __forceinline__ float relu(float x) {
  return __uint_as_float((uint32_t)max(__float_as_int(x), 0));
}

// Sine and cosine of z quarter turns: z = q + f with q the nearest integer (f
// is exact), then the Taylor series in f on |f| <= 1/2, whose first left-out
// terms are below 2e-9 (sine) and 2e-10 (cosine).
__device__ __forceinline__ void sine_cosine(float z, float* sn, float* cs) {
  const float q = rintf(z), f = z - q;
  const float f2 = f * f;
  float s = __builtin_fmaf(f2, 1.6044118e-4f, -4.6817541e-3f);
  s = __builtin_fmaf(f2, s, 7.9692626e-2f);
  s = __builtin_fmaf(f2, s, -6.4596410e-1f);
  s = __builtin_fmaf(f2, s, 1.5707964f);
  s *= f;
  float c = __builtin_fmaf(f2, -2.5202042e-5f, 9.1926027e-4f);
  c = __builtin_fmaf(f2, c, -2.0863481e-2f);
  c = __builtin_fmaf(f2, c, 2.5366951e-1f);
  c = __builtin_fmaf(f2, c, -1.2337006f);
  c = __builtin_fmaf(f2, c, 1.f);
  const int n = (int)q;
  const float a = (n & 1) ? c : s, b = (n & 1) ? s : c;
  *sn = __uint_as_float(__float_as_uint(a) ^ ((uint32_t)(n & 2) << 30));
  *cs = __uint_as_float(__float_as_uint(b) ^ ((uint32_t)((n + 1) & 2) << 30));
}

// The three bfloat16 parts of eight values, packed in order.
__device__ __forceinline__ void split8(const float (&x)[8], u32x4 (&part)[3]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint32_t lo[3], hi[3];
    split_bf16x3(x[2 * i], lo[0], lo[1], lo[2]);
    split_bf16x3(x[2 * i + 1], hi[0], hi[1], hi[2]);
#pragma unroll
    for (int q = 0; q < 3; ++q) part[q][i] = lo[q] | hi[q] << 16;
  }
}
__device__ __forceinline__ void split4(const f32x4& x, s16x4 (&part)[3]) {
  uint32_t p[3][4];
#pragma unroll
  for (int i = 0; i < 4; ++i) split_bf16x3(x[i], p[0][i], p[1][i], p[2][i]);
#pragma unroll
  for (int q = 0; q < 3; ++q)
    part[q] = __builtin_bit_cast(s16x4, make_uint2(p[q][0] | p[q][1] << 16, p[q][2] | p[q][3] << 16));
}

__device__ __forceinline__ f32x4 mfma32(const u32x4& a, const u32x4& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Parts (a, b) of the eight products of two split operands, smallest first.
constexpr int kTerms = 8;
constexpr int kTermA[kTerms] = {1, 2, 0, 2, 1, 0, 1, 0};
constexpr int kTermB[kTerms] = {2, 1, 2, 0, 1, 1, 0, 0};

// Flanks 2g and 2g + 1 of the 9-mer at `let` as a one-hot B fragment of layer 1
// (inputs 4 i + letter of flank i; a code above 3 selects none).
__device__ __forceinline__ u32x4 flank_fragment(const uint8_t* let, int g) {
  const int i = 2 * g + (g > 1);  // letter 4 is the middle one
  const uint32_t f0 = let[i], f1 = let[i + 1];
  const uint64_t h0 = f0 < 4 ? 0x3F80ull << (16 * f0) : 0ull;
  const uint64_t h1 = f1 < 4 ? 0x3F80ull << (16 * f1) : 0ull;
  return u32x4{(uint32_t)h0, (uint32_t)(h0 >> 32), (uint32_t)h1, (uint32_t)(h1 >> 32)};
}

// A pre-activation this close to zero (a few dozen ulps of the summands) is
// summed again in FP32 in the order of the flanks, so that its sign -- whether
// the unit is on and passes gradients -- does not depend on how the matrix
// cores add.  About one tile in 400 has one.  With a weight that is infinite or no
// number all are: a product with a one-hot zero would spread it over every token,
// and a sum of the chosen weights leaves it to those that choose it, where a unit
// that is no number is off.
constexpr float kNearZero = 1.0f / 1048576.0f;

// Settles a lane's 16 pre-activations h[i / 4][i % 4]: unit(i) is the hidden unit
// and letters(i) the 9-mer of entry i.  One at a time, so that the rare path
// needs few registers.
template <typename Unit, typename Letters>
__device__ __forceinline__ void settle(const float* __restrict__ p, bool every, f32x4 (&h)[4],
                                       Unit unit, Letters letters) {
  float least = every ? 0.f : 1.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) least = fminf(least, fabsf(h[i >> 2][i & 3]));
  if (!__ballot(least < kNearZero)) return;
  uint32_t todo = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) todo |= (uint32_t)(every || fabsf(h[i >> 2][i & 3]) < kNearZero) << i;
#pragma unroll 1
  while (todo) {
    const int at = __builtin_ctz(todo);
    todo &= todo - 1;
    const int u = unit(at);
    const uint8_t* let = letters(at);
    float pre = p[kB1 + u];
#pragma unroll 1
    for (int i = 0; i < 8; ++i) {
      const int f = let[i + (i > 3)];
      if (f < 4) pre += p[kW1 + u * kIn + 4 * i + f];
    }
    pre = isnan(pre) ? 0.f : pre;
#pragma unroll
    for (int i = 0; i < 16; ++i) h[i >> 2][i & 3] = at == i ? pre : h[i >> 2][i & 3];
  }
}

// The letter's rows of W2 as A fragments of layer 2: rows 16 ob + lane % 16,
// K entry j of step st = hidden unit 16 (2 st + j / 4) + 4 (lane / 16) + j % 4.
__device__ __forceinline__ void load_w2(const float* __restrict__ p, int L, int lane,
                                        u32x4 (&w2)[2][2][3]) {
#pragma unroll
  for (int ob = 0; ob < 2; ++ob)
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      const float* src = p + kW2 + (L * 32 + 16 * ob + (lane & 15)) * kHid + 32 * st + 4 * (lane >> 4);
      float x[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = src[16 * (j >> 2) + (j & 3)];
      split8(x, w2[ob][st]);
    }
}

// Phases of the lane's token (9-mer at `let`, its one-hot flanks x, location p): sine and cosine of
// theta_k p + delta_k for its factors k - 1 = 16 ob + 4 g + v, index 4 ob + v.
// k p is reduced mod N exactly: k p - q N is exact in FP32 (k p < 2^13; for an
// N that FP32 does not hold, q = 0).  The offset's whole turns are taken off
// before it is rounded as quarter turns, whose constant is the sum of two FP32
// values: the phase is off by at most 5e-7 (1e-7 root mean square) for offsets
// up to 10^5 rad.  Scaled at once the offset alone would cost 4.4e-7 at 8 rad
// and 1.0e-6 at 20, and the FP32 sum of both angles 2.8e-7 and 5.4e-7.
__device__ __forceinline__ void token_phases(const float* __restrict__ params, const Net& net, bool every,
                                             const u32x4 (&w2)[2][2][3], int L, const uint8_t* let,
                                             const u32x4& x, int p, float Nf, float inv_n,
                                             float turn, int lane, float (&sn)[8], float (&cs)[8]) {
  const int g = lane >> 4;
  f32x4 h[4];
#pragma unroll
  for (int rb = 0; rb < 4; ++rb) {
    h[rb] = *reinterpret_cast<const f32x4*>(&net.b1[16 * rb + 4 * g]);
#pragma unroll
    for (int q = 2; q >= 0; --q) h[rb] = mfma32(net.w1[q][rb][lane], x, h[rb]);  // small parts first
  }
  settle(params, every, h, [&](int i) { return 16 * (i >> 2) + 4 * g + (i & 3); },
         [&](int) { return let; });
  u32x4 hp[2][3];
#pragma unroll
  for (int st = 0; st < 2; ++st) {
    float hv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) hv[j] = relu(h[2 * st + (j >> 2)][j & 3]);
    split8(hv, hp[st]);
  }
  // smallest terms first over both K steps, the bias last: an accumulator
  // that is already large loses more in each further addition
  f32x4 o[2] = {f32x4{}, f32x4{}};
#pragma unroll
  for (int q = 0; q < kTerms; ++q)
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int ob = 0; ob < 2; ++ob)
        o[ob] = mfma32(w2[ob][st][kTermA[q]], hp[st][kTermB[q]], o[ob]);
#pragma unroll
  for (int ob = 0; ob < 2; ++ob)
    o[ob] += *reinterpret_cast<const f32x4*>(&net.b2[L * 32 + 16 * ob + 4 * g]);
  const float pf = (float)p;
#pragma unroll
  for (int ob = 0; ob < 2; ++ob)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float kp = (float)(16 * ob + 4 * g + v + 1) * pf;
      const float r = __builtin_fmaf(-rintf(kp * inv_n), Nf, kp);
      const float whole = 4.f * rintf(o[ob][v] * 0.15915494f);
      const float part = __builtin_fmaf(o[ob][v], 2.5682553e-8f,
                                        __builtin_fmaf(o[ob][v], 0.63661977f, -whole));
      sine_cosine(__builtin_fmaf(r, turn, part), &sn[4 * ob + v], &cs[4 * ob + v]);
    }
}

// Strings come from one set (string s = seq[off[s] .. off[s+1])) or, for
// pairs, from two: string s is string s/2 of set a (s even) or of set b (s odd).
struct Strings {
  const uint8_t* a;
  const int64_t* aoff;
  const uint8_t* b;  // null: one set
  const int64_t* boff;
};

// Letters of string sidx (at most kMaxLen) into LDS; returns its tokens.
__device__ __forceinline__ int load_string(uint8_t* let, const Strings& st, int64_t sidx,
                                           int lane) {
  const uint8_t* seq = st.a;
  const int64_t* off = st.aoff;
  if (st.b != nullptr) {
    if (sidx & 1) {
      seq = st.b;
      off = st.boff;
    }
    sidx >>= 1;
  }
  const int64_t a = off[sidx];
  const int n = (int)min<int64_t>(off[sidx + 1] - a, kMaxLen);
  for (int i = lane; i < n; i += 64) let[i] = seq[a + i];
  __builtin_amdgcn_wave_barrier();
  return max(n - 8, 0);
}

// Sum over the 16 lanes of a lane group (a DPP row), in every lane of it.
__device__ __forceinline__ float row_sum(float v) {
  v += dpp<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp<0x141>(v);  // row_half_mirror
  v += dpp<0x140>(v);  // row_mirror
  return v;
}

// F of a pair of encodings, a lane's four reals of each.
__device__ __forceinline__ float fidelity(float4 a, float4 b) {
  // z = sum conj(a) b
  const float zr = wave_sum(a.x * b.x + a.y * b.y + a.z * b.z + a.w * b.w);
  const float zi = wave_sum(a.x * b.y - a.y * b.x + a.z * b.w - a.w * b.z);
  const float A = wave_sum(a.x * a.x + a.y * a.y + a.z * a.z + a.w * a.w);
  const float B = wave_sum(b.x * b.x + b.y * b.y + b.z * b.z + b.w * b.w);
  return (A > 0.f && B > 0.f) ? (zr * zr + zi * zi) / (A * B) : 0.f;
}

// Learned encodings c of n_strings strings: out[s][256] (k*4+letter, re/im);
// for pairs (F not null) also F of strings 2i and 2i + 1.  A block takes `per`
// strings at a time.  A string's tokens of one letter fill their own 16-token
// tiles, so a lane sums its factors over the tiles in registers and the 16 lanes
// are added once per string and letter.  Where all the strings' tokens of the
// letter fit one tile they share it, and each string adds the lanes of its own.
//
// Bound by VALU issue (the phases and the splits).  100,000 strings of 150
// letters 1.24 ms (6.9 with a token at a time); of 12 letters, four tokens, 267
// us (364 with a token at a time, 573 with a tile for each string and letter).
__global__ __launch_bounds__(64 * kWaves, 2) void learned_encode_kernel(
    const float* __restrict__ params, Strings st, int32_t n_strings, int per, float Nf,
    float inv_n, float turn, float* __restrict__ out, float* __restrict__ F) {
  __shared__ Net net;
  __shared__ uint8_t letters[kStrings][kMaxLen + 8];
  __shared__ uint8_t place[4][kStrings][kMaxLen];  // locations of a letter's tokens
  __shared__ int tokens[4][kStrings];
  __shared__ __align__(16) float c[kStrings][256];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int L = wave >> 1, g = lane >> 4;
  load_net(net, params);
  u32x4 w2[2][2][3];
  load_w2(params, L, lane, w2);
  for (int64_t first = (int64_t)blockIdx.x * per; first < n_strings;
       first += (int64_t)gridDim.x * per) {
    const int n_own = (int)min<int64_t>(per, n_strings - first);
    if (wave < n_own) {
      const int n = load_string(letters[wave], st, first + wave, lane);
      int have[4] = {0, 0, 0, 0};
      for (int p0 = 0; p0 < n; p0 += 64) {
        const int mid = p0 + lane < n ? (int)letters[wave][p0 + lane + 4] : 4;
#pragma unroll
        for (int L = 0; L < 4; ++L) {
          const uint64_t m = __ballot(mid == L);
          if (mid == L)
            place[L][wave][have[L] + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                         __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0))] =
                (uint8_t)(p0 + lane);
          have[L] += __builtin_popcountll(m);
        }
      }
      if (lane < 4) tokens[lane][wave] = lane == 0 ? have[0] : lane == 1 ? have[1] : lane == 2 ? have[2] : have[3];
    }
    __syncthreads();

    const bool every = odd_net(net);
    int total = 0;
    for (int s = 0; s < n_own; ++s) total += tokens[L][s];
    const bool pooled = total <= 16;
    for (int s = wave & 1; s < n_own; s += 2) {
      const int n = pooled ? total : tokens[L][s];
      int from = pooled ? -1 : s;  // the string of the lane's token
      float re[8], im[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) re[i] = im[i] = 0.f;
      for (int t = 0; t < n; t += 16) {
        const int i = t + (lane & 15);
        const bool valid = i < n;
        int at = valid ? i : 0;
        if (pooled) {
          from = 0;
          while (at >= tokens[L][from]) at -= tokens[L][from++];
        }
        const int p = place[L][from][at];
        float sn[8], cs[8];
        const uint8_t* let = &letters[from][p];
        token_phases(params, net, every, w2, L, let, flank_fragment(let, g), p, Nf, inv_n, turn, lane, sn, cs);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          re[q] += valid ? cs[q] : 0.f;
          im[q] += valid ? sn[q] : 0.f;
        }
      }
#pragma unroll 1
      do {  // the string's sums, or those of all this wavefront's strings
        float sr[8], si[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) sr[q] = si[q] = 0.f;
        if (tokens[L][s] != 0) {  // uniform
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            sr[q] = row_sum(from == s ? re[q] : 0.f);
            si[q] = row_sum(from == s ? im[q] : 0.f);
          }
        }
        if ((lane & 15) == 0) {
#pragma unroll
          for (int q = 0; q < 8; ++q)
            *reinterpret_cast<float2*>(&c[s][((16 * (q >> 2) + 4 * g + (q & 3)) * 4 + L) * 2]) =
                make_float2(sr[q], si[q]);
        }
      } while (pooled && (s += 2) < n_own);
    }
    __syncthreads();
    if (wave < n_own)
      reinterpret_cast<float4*>(out + (first + wave) * 256)[lane] =
          *reinterpret_cast<const float4*>(&c[wave][4 * lane]);
    if (F != nullptr && 2 * wave + 1 < n_own) {
      const float f = fidelity(*reinterpret_cast<const float4*>(&c[2 * wave][4 * lane]),
                               *reinterpret_cast<const float4*>(&c[2 * wave + 1][4 * lane]));
      if (lane == 0) F[(first >> 1) + wave] = f;
    }
    // (The next strings' letters and lists were last read before the barrier above,
    // and their sums are written after the next one.)
  }
}

// The plain encoding (§2.2, s = 1) of whole strings in FP32, for comparison:
// letter p adds exp(i theta_k p) to component (k, letter), p = 0..n-1.
__global__ __launch_bounds__(256) void plain_encode_kernel(const uint8_t* __restrict__ seq,
                                                           const int64_t* __restrict__ off,
                                                           int32_t n_strings, int N,
                                                           float* __restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int64_t s = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (s >= n_strings) return;
  const int64_t a = off[s], n = off[s + 1] - a;
  const int k = lane >> 1, hh = lane & 1;
  const int64_t fk = k + 1;
  float2 c0 = make_float2(0.f, 0.f), c1 = make_float2(0.f, 0.f);
  for (int64_t p = 0; p < n; ++p) {
    const int L = seq[a + p];
    if ((L >> 1) != hh) continue;
    float sn, cs;
    sincospif(2.f * (float)((fk * p) % N) / (float)N, &sn, &cs);
    if (L & 1) { c1.x += cs; c1.y += sn; } else { c0.x += cs; c0.y += sn; }
  }
  reinterpret_cast<float4*>(out + s * 256)[lane] = make_float4(c0.x, c0.y, c1.x, c1.y);
}

// F of pairs of encodings ca[i * stride], cb[i * stride]; one wavefront per pair.
__global__ __launch_bounds__(256) void pair_fidelity_kernel(const float* __restrict__ ca,
                                                            const float* __restrict__ cb,
                                                            int64_t stride, int32_t n_pairs,
                                                            float* __restrict__ F) {
  const int lane = threadIdx.x & 63;
  const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= n_pairs) return;
  const float f = fidelity(reinterpret_cast<const float4*>(ca + i * stride)[lane],
                           reinterpret_cast<const float4*>(cb + i * stride)[lane]);
  if (lane == 0) F[i] = f;
}

// Ranking loss: per pair i, over all j, the loss terms softplus(z) and count
// for d_i < d_j (z = -(F_i - F_j) / tau), and the unscaled dLoss/dF_i
// contributions -sigma(z_ij) (d_i < d_j) and +sigma(z_ji) (d_j < d_i), with
// e = exp(-|z|): softplus = max(z, 0) + log1p(e), sigma = 1 / (1 + e) or
// e / (1 + e).  A block of four wavefronts per i (79 us for 1,024 pairs with a
// lane per i and an eighth of the j's, 14 us with a wavefront per i): a lane
// adds its j's in order, the lanes in wave_sum's fixed order, the wavefronts in
// theirs.  A training step's count (step, if not null) advances here, before
// the kernel that uses it.
constexpr int kRankWaves = 4;

__global__ __launch_bounds__(64 * kRankWaves) void ranking_kernel(
    const float* __restrict__ F, const int32_t* __restrict__ ld, int32_t n,
    float* __restrict__ g_out, float* __restrict__ loss_out, int32_t* __restrict__ cnt_out,
    float* __restrict__ step) {
  __shared__ float part[3][kRankWaves];
  const int i = blockIdx.x;
  if (step != nullptr && i == 0 && threadIdx.x == 0) *step += 1.f;
  const float Fi = F[i];
  const int Li = ld[i];
  float g = 0.f, l = 0.f, cnt = 0.f;
  for (int j = threadIdx.x; j < n; j += 64 * kRankWaves) {
    const int Lj = ld[j];
    if (Li == Lj) continue;
    const bool lower = Li < Lj;  // want F_i > F_j
    const float z = (lower ? F[j] - Fi : Fi - F[j]) * kInvTau;
    const float e = expf(-fabsf(z));
    const float sigma = (z > 0.f ? 1.f : e) / (1.f + e);
    if (lower) {
      l += fmaxf(z, 0.f) + log1pf(e);
      cnt += 1.f;
      g -= sigma;
    } else {
      g += sigma;
    }
  }
  g = wave_sum(g);
  l = wave_sum(l);
  cnt = wave_sum(cnt);  // at most 1,024: exact
  if ((threadIdx.x & 63) == 0) {
    part[0][threadIdx.x >> 6] = g;
    part[1][threadIdx.x >> 6] = l;
    part[2][threadIdx.x >> 6] = cnt;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    g_out[i] = (part[0][0] + part[0][1]) + (part[0][2] + part[0][3]);
    loss_out[i] = (part[1][0] + part[1][1]) + (part[1][2] + part[1][3]);
    cnt_out[i] = (int)(part[2][0] + part[2][1] + part[2][2] + part[2][3]);
  }
}

// Backward: per string, dLoss/dc = dLoss/dF * dF/dc (dLoss/dF_i = g_i over tau
// and the count of ordered pairs), then through the tokens and the network.
// The block's tokens are sorted by middle letter over all its strings (little
// of a 16-token tile is padding), two wavefronts per letter taking every other
// tile:
//   the forward up to the phases, tokens as columns;
//   d delta_k = -G_r sin + G_i cos, in the layer-2 accumulator layout;
//   dH [16 x 64] = dD [16 x 32] W2_L [32 x 64] in FP32 MFMAs, whose A operand
//     is d delta as it lies, masked by H [16 x 64] = relu(X W1^T): layer 1 once
//     more with its operands swapped.  Both leave four tokens of one hidden
//     unit in a lane, so they are B operands of the sums over tokens:
//   dW2_L [32 x 64] += dD^T H in FP32 MFMAs (d delta goes through LDS once to
//     become the A operand) and dW1^T [32 x 64] += X^T dP as three bf16 MFMAs
//     (one-hot X, dP split exactly).
// A wavefront keeps its letter's dW2 block, a dW1 and the bias sums in
// registers over all its tiles.  The wavefronts are added in a fixed order
// through LDS, and the per-block partials in block order by the reduction
// kernel: deterministic.  Bound by issue: the FP32 MFMAs (2,048 cycles a tile)
// and the VALU work of phases and splits (about 2,400) hardly overlap.
constexpr int kRowD = 48;  // floats of a token's d delta in LDS (conflict-free columns)
struct Sums {
  float w1[kWaves][kIn * kHid];  // dW1^T of every wavefront
  float w2[4][32 * kHid];        // dW2 of a letter's second wavefront
  float b1[kWaves][kHid];
  float b2[kWaves][32];
};

__global__ __launch_bounds__(64 * kWaves, 2) void learned_backward_kernel(
    const float* __restrict__ params, Strings st, int32_t n_pairs, int per, float Nf, float inv_n,
    float turn, const float* __restrict__ c, const float* __restrict__ rank_g,
    const int32_t* __restrict__ cnt, float* __restrict__ partial) {
  __shared__ Net net;
  __shared__ uint8_t letters[kStrings][kMaxLen + 8];
  __shared__ uint16_t list[4][kStrings * kMaxTok];  // string << 8 | location
  __shared__ int tokens[4][kStrings];
  __shared__ __align__(16) float2 G[kStrings][4][32];
  __shared__ union {
    struct {
      f32x4 w2t[4][2][4][64];  // W2_L's rows as B fragments of dH
      float d[kWaves][16 * kRowD];
    } run;
    Sums sum;
  } u;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t first = (int64_t)blockIdx.x * per;
  const int n_own = (int)min<int64_t>(per, 2 * (int64_t)n_pairs - first);
  load_net(net, params);
  // hidden units 16 cb + lane % 16, K entry j = factor 16 (j / 4) + 4 (lane / 16) + j % 4
  for (int i = wave; i < 16; i += kWaves) {
    const int L = i >> 2, cb = i & 3;
    const float* src = params + kW2 + (L * 32 + 4 * (lane >> 4)) * kHid + 16 * cb + (lane & 15);
    float x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = src[(16 * (j >> 2) + (j & 3)) * kHid];
    u.run.w2t[L][0][cb][lane] = f32x4{x[0], x[1], x[2], x[3]};
    u.run.w2t[L][1][cb][lane] = f32x4{x[4], x[5], x[6], x[7]};
  }
  int n = 0;
  if (wave < n_own) {
    const int64_t pr = (first + wave) >> 1;
    const bool is_b = wave & 1;  // `per` is even
    // dF/dc for this side: F = |z|^2/(AB), z = <a|b>
    const float4 a = reinterpret_cast<const float4*>(c + (2 * pr) * 256)[lane];
    const float4 b = reinterpret_cast<const float4*>(c + (2 * pr + 1) * 256)[lane];
    const float zr = wave_sum(a.x * b.x + a.y * b.y + a.z * b.z + a.w * b.w);
    const float zi = wave_sum(a.x * b.y - a.y * b.x + a.z * b.w - a.w * b.z);
    const float A = wave_sum(a.x * a.x + a.y * a.y + a.z * a.z + a.w * a.w);
    const float B = wave_sum(b.x * b.x + b.y * b.y + b.z * b.z + b.w * b.w);
    float g0r = 0.f, g0i = 0.f, g1r = 0.f, g1i = 0.f;
    int pairs = 0;  // ordered pairs of the batch: every wavefront adds them up
    for (int i = lane; i < n_pairs; i += 64) pairs += cnt[i];
    pairs = (int)wave_sum((float)pairs);  // at most 2^19: exact
    if (A > 0.f && B > 0.f && pairs > 0) {
      const float d = rank_g[pr] * (kInvTau / (float)pairs);
      const float F = (zr * zr + zi * zi) / (A * B), AB = A * B;
      if (!is_b) {  // G_a = 2 conj(z) b / (AB) - 2 F a / A
        g0r = d * (2.f * (zr * b.x + zi * b.y) / AB - 2.f * F * a.x / A);
        g0i = d * (2.f * (zr * b.y - zi * b.x) / AB - 2.f * F * a.y / A);
        g1r = d * (2.f * (zr * b.z + zi * b.w) / AB - 2.f * F * a.z / A);
        g1i = d * (2.f * (zr * b.w - zi * b.z) / AB - 2.f * F * a.w / A);
      } else {      // G_b = 2 z a / (AB) - 2 F b / B
        g0r = d * (2.f * (zr * a.x - zi * a.y) / AB - 2.f * F * b.x / B);
        g0i = d * (2.f * (zr * a.y + zi * a.x) / AB - 2.f * F * b.y / B);
        g1r = d * (2.f * (zr * a.z - zi * a.w) / AB - 2.f * F * b.z / B);
        g1i = d * (2.f * (zr * a.w + zi * a.z) / AB - 2.f * F * b.w / B);
      }
    }
    // lane (k, hh) holds G of components (k, 2hh) and (k, 2hh+1)
    G[wave][2 * (lane & 1)][lane >> 1] = make_float2(g0r, g0i);
    G[wave][2 * (lane & 1) + 1][lane >> 1] = make_float2(g1r, g1i);
    n = load_string(letters[wave], st, first + wave, lane);
    int have[4] = {0, 0, 0, 0};
    for (int p0 = 0; p0 < n; p0 += 64) {
      const int mid = p0 + lane < n ? (int)letters[wave][p0 + lane + 4] : 4;
#pragma unroll
      for (int L = 0; L < 4; ++L) have[L] += __builtin_popcountll(__ballot(mid == L));
    }
    if (lane < 4) tokens[lane][wave] = lane == 0 ? have[0] : lane == 1 ? have[1] : lane == 2 ? have[2] : have[3];
  }
  __syncthreads();
  if (wave < n_own) {
    int at[4] = {0, 0, 0, 0};
    for (int s = 0; s < wave; ++s)
#pragma unroll
      for (int L = 0; L < 4; ++L) at[L] += tokens[L][s];
    for (int p0 = 0; p0 < n; p0 += 64) {
      const int mid = p0 + lane < n ? (int)letters[wave][p0 + lane + 4] : 4;
#pragma unroll
      for (int L = 0; L < 4; ++L) {
        const uint64_t m = __ballot(mid == L);
        if (mid == L)
          list[L][at[L] + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                              __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0))] =
              (uint16_t)(wave << 8 | (p0 + lane));
        at[L] += __builtin_popcountll(m);
      }
    }
  }
  __syncthreads();

  const int L = wave >> 1, g = lane >> 4, col = lane & 15;
  const bool every = odd_net(net);
  int n_tok = 0;
  for (int s = 0; s < n_own; ++s) n_tok += tokens[L][s];
  u32x4 w2[2][2][3];
  load_w2(params, L, lane, w2);
  f32x4 gw2[2][4], gw1[2][4], gb2[2];
  float gb1[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    gb2[i] = f32x4{};
#pragma unroll
    for (int j = 0; j < 4; ++j) gw2[i][j] = gw1[i][j] = f32x4{};
  }
  float* dbuf = u.run.d[wave];

  for (int t = 16 * (wave & 1); t < n_tok; t += 32) {
    const bool valid = t + col < n_tok;
    const float live = valid ? 1.f : 0.f;  // a padding column repeats a token, with no weight
    const int e = list[L][valid ? t + col : t];
    const int s = e >> 8, p = e & 255;
    const u32x4 x = flank_fragment(&letters[s][p], g);
    float dd[8];
    {
      float sn[8], cs[8];
      token_phases(params, net, every, w2, L, &letters[s][p], x, p, Nf, inv_n, turn, lane, sn, cs);
#pragma unroll
      for (int ob = 0; ob < 2; ++ob)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float2 Gk = G[s][L][16 * ob + 4 * g + v];
          const float d = live * (Gk.y * cs[4 * ob + v] - Gk.x * sn[4 * ob + v]);
          dd[4 * ob + v] = d;
          gb2[ob][v] += d;
        }
    }
#pragma unroll
    for (int ob = 0; ob < 2; ++ob)
      *reinterpret_cast<f32x4*>(&dbuf[col * kRowD + 16 * ob + 4 * g]) =
          f32x4{dd[4 * ob], dd[4 * ob + 1], dd[4 * ob + 2], dd[4 * ob + 3]};
    __builtin_amdgcn_wave_barrier();
    // d delta of tokens 4 g + j, factor 16 ob + col
    f32x4 df[2];
#pragma unroll
    for (int ob = 0; ob < 2; ++ob) {
      f32x4 d;
#pragma unroll
      for (int j = 0; j < 4; ++j) d[j] = dbuf[(4 * g + j) * kRowD + 16 * ob + col];
      df[ob] = d;
    }
    // one-hot of tokens 4 g + j, input 16 rb + col = 4 i + letter of flank i
    s16x4 hot[2];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int ej = list[L][min(t + 4 * g + j, n_tok - 1)];  // past the end: dP is zero
      const uint8_t* let = &letters[ej >> 8][ej & 255];
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) {
        const int i = 4 * rb + (col >> 2);
        hot[rb][j] = let[i + (i > 3)] == (col & 3) ? (short)0x3F80 : (short)0;
      }
    }
    f32x4 hid[4];  // tokens 4 g + v, hidden units 16 cb + col
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
      const float b1 = net.b1[16 * cb + col];
      hid[cb] = f32x4{b1, b1, b1, b1};
#pragma unroll
      for (int q = 2; q >= 0; --q) hid[cb] = mfma32(x, net.w1[q][cb][lane], hid[cb]);
    }
    settle(params, every, hid, [&](int i) { return 16 * (i >> 2) + col; },
           [&](int i) {
             const int ei = list[L][min(t + 4 * g + (i & 3), n_tok - 1)];
             return &letters[ei >> 8][ei & 255];
           });
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
      f32x4 h = hid[cb];
      f32x4 dh{};
      const f32x4 wa = u.run.w2t[L][0][cb][lane], wb = u.run.w2t[L][1][cb][lane];
#pragma unroll
      for (int j = 0; j < 8; ++j)
        dh = __builtin_amdgcn_mfma_f32_16x16x4f32(dd[j], j < 4 ? wa[j] : wb[j - 4], dh, 0, 0, 0);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        dh[v] = h[v] > 0.f ? dh[v] : 0.f;
        gb1[cb] += dh[v];
        h[v] = relu(h[v]);
      }
      s16x4 pp[3];
      split4(dh, pp);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int ob = 0; ob < 2; ++ob)
          gw2[ob][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(df[ob][j], h[j], gw2[ob][cb], 0, 0, 0);
#pragma unroll
      for (int q = 2; q >= 0; --q)
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
          gw1[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(hot[rb], pp[q], gw1[rb][cb], 0, 0, 0);
    }
    __builtin_amdgcn_wave_barrier();  // dbuf is rewritten by the next tile
  }

  __syncthreads();  // every wavefront is done with the run's LDS
  Sums& sum = u.sum;
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        sum.w1[wave][(16 * rb + 4 * g + v) * kHid + 16 * cb + col] = gw1[rb][cb][v];
        if (wave & 1) sum.w2[L][(16 * rb + 4 * g + v) * kHid + 16 * cb + col] = gw2[rb][cb][v];
      }
#pragma unroll
  for (int cb = 0; cb < 4; ++cb) {  // the four lane groups hold four tokens each
    float b = gb1[cb];
    b += __shfl_xor(b, 16, 64);
    b += __shfl_xor(b, 32, 64);
    if (g == 0) sum.b1[wave][16 * cb + col] = b;
  }
#pragma unroll
  for (int ob = 0; ob < 2; ++ob)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float b = row_sum(gb2[ob][v]);
      if (col == 0) sum.b2[wave][16 * ob + 4 * g + v] = b;
    }
  __syncthreads();
  // partial gradient of this block, parameter order
  float* out = partial + (int64_t)blockIdx.x * kParams;
  if (!(wave & 1)) {
#pragma unroll
    for (int ob = 0; ob < 2; ++ob)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = 16 * ob + 4 * g + v, j = 16 * cb + col;
          out[kW2 + (L * 32 + r) * kHid + j] = gw2[ob][cb][v] + sum.w2[L][r * kHid + j];
        }
  }
  for (int i = threadIdx.x; i < kIn * kHid; i += blockDim.x) {
    float w = sum.w1[0][i];
#pragma unroll
    for (int q = 1; q < kWaves; ++q) w += sum.w1[q][i];
    out[kW1 + (i % kHid) * kIn + i / kHid] = w;
  }
  if (threadIdx.x < kHid) {
    float b = sum.b1[0][threadIdx.x];
#pragma unroll
    for (int q = 1; q < kWaves; ++q) b += sum.b1[q][threadIdx.x];
    out[kB1 + threadIdx.x] = b;
  } else if (threadIdx.x < kHid + kOut) {
    const int i = threadIdx.x - kHid;
    out[kB2 + i] = sum.b2[i / 32 * 2][i % 32] + sum.b2[i / 32 * 2 + 1][i % 32];
  }
}

// Sum of the per-block partial gradients (block: 64 parameters x 16 subsets
// of the partials, summed in a fixed order); then either the gradient is
// written (grad != nullptr) or an Adam step is applied to state = [params | m
// | v | t].  One more block sums the loss terms, over the number of ordered
// pairs.  The step count t is advanced by the ranking of the same step.
constexpr int kRedParams = 64, kRedParts = 16;
constexpr int kRedBlocks = (kParams + kRedParams - 1) / kRedParams;

__global__ __launch_bounds__(kRedParams * kRedParts) void reduce_adam_kernel(
    const float* __restrict__ partial, int n_blocks, const float* __restrict__ lossv,
    const int32_t* __restrict__ cnt, int32_t n, float* __restrict__ loss,
    float* __restrict__ grad, float* __restrict__ state, float lr) {
  __shared__ float red[kRedParts][kRedParams];
  const int tp = threadIdx.x % kRedParams, q = threadIdx.x / kRedParams;
  if (blockIdx.x == kRedBlocks) {
    const bool has = (int)threadIdx.x < n;
    const float l = wave_sum(has ? lossv[threadIdx.x] : 0.f);
    const float c = wave_sum(has ? (float)cnt[threadIdx.x] : 0.f);
    if (tp == 0) {
      red[0][q] = l;
      red[1][q] = c;
    }
    __syncthreads();
    if (q == 0) {  // the sixteen parts as a tree: a running sum rounds its largest values most often
      const float sum = wave_sum(tp < kRedParts ? red[0][tp] : 0.f);
      const float pairs = wave_sum(tp < kRedParts ? red[1][tp] : 0.f);
      if (tp == 0) *loss = pairs > 0.f ? sum / pairs : 0.f;
    }
    return;
  }
  const int i = blockIdx.x * kRedParams + tp;
  float g = 0.f;
  if (i < kParams) {
    int b = q;
    for (; b + 3 * kRedParts < n_blocks; b += 4 * kRedParts) {  // 4 loads in flight
      const float v0 = partial[(int64_t)b * kParams + i];
      const float v1 = partial[(int64_t)(b + kRedParts) * kParams + i];
      const float v2 = partial[(int64_t)(b + 2 * kRedParts) * kParams + i];
      const float v3 = partial[(int64_t)(b + 3 * kRedParts) * kParams + i];
      g += v0;
      g += v1;
      g += v2;
      g += v3;
    }
    for (; b < n_blocks; b += kRedParts) g += partial[(int64_t)b * kParams + i];
  }
  red[q][tp] = g;
  __syncthreads();
  if (q != 0 || i >= kParams) return;
  for (int r = 1; r < kRedParts; ++r) g += red[r][tp];
  if (grad != nullptr) {
    grad[i] = g;
    return;
  }
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  const float t = state[3 * kParams];
  float m = b1 * state[kParams + i] + (1.f - b1) * g;
  float v = b2 * state[2 * kParams + i] + (1.f - b2) * g * g;
  state[kParams + i] = m;
  state[2 * kParams + i] = v;
  float mh = m / (1.f - powf(b1, t));
  float vh = v / (1.f - powf(b2, t));
  state[i] -= lr * mh / (sqrtf(vh) + eps);
}

static_assert(kRedParams == 64 && RM_LEARNED_MAX_PAIRS <= kRedParams * kRedParts,
              "the loss block's layout");

// Blocks of an encoding, at most: one per CU, which is what their registers allow
// at a time, so that each splits the weights once (100,000 strings of 12 letters
// in tiles of their own 482 us, with 4,096 blocks 522).
constexpr int64_t kEncodeBlocks = 256;

// Strings per block: a block per CU from 1,024 pairs on, two pairs at least.
int strings_per_block(int64_t n_strings) { return n_strings > 1024 ? kStrings : kStrings / 2; }

// The nominal length as the phases use it: a position's part of a turn in
// quarter turns.
struct Nominal {
  float n, inv, turn;
  explicit Nominal(int N)
      : n((float)N), inv((float)(1.0 / N)), turn((float)(4.0 / N)) {}
};

}  // namespace

size_t learned_workspace_bytes(int32_t n_pairs) {
  int64_t strings = 2 * (int64_t)n_pairs;
  int64_t blocks = (strings + 3) / 4;              // at least the blocks of a step
  size_t bytes = 0;
  bytes += (size_t)strings * 256 * sizeof(float);  // encodings
  bytes += (size_t)n_pairs * sizeof(float) * 4;    // F, dF, per-i loss, per-i count
  bytes += 256;                                    // loss
  bytes += (size_t)blocks * kParams * sizeof(float);
  return (bytes + 255) / 256 * 256 + 1024;
}

hipError_t launch_learned_encode(const float* params, const uint8_t* seq, const int64_t* off,
                                 int32_t n_strings, int N, float* out, hipStream_t s) {
  if (params == nullptr) {
    hipLaunchKernelGGL(plain_encode_kernel, dim3((unsigned)(((int64_t)n_strings + 3) / 4)),
                       dim3(256), 0, s, seq, off, n_strings, N, out);
    return hipGetLastError();
  }
  const int per = strings_per_block(n_strings);
  const Nominal nom(N);
  const int64_t groups = ((int64_t)n_strings + per - 1) / per;
  const unsigned blocks = (unsigned)std::min<int64_t>(groups, kEncodeBlocks);
  hipLaunchKernelGGL(learned_encode_kernel, dim3(blocks), dim3(64 * kWaves), 0, s, params,
                     Strings{seq, off, nullptr, nullptr}, n_strings, per, nom.n, nom.inv, nom.turn,
                     out, (float*)nullptr);
  return hipGetLastError();
}

hipError_t launch_pair_fidelity(const float* ca, const float* cb, int32_t n_pairs, float* F,
                                hipStream_t s) {
  unsigned blocks = (unsigned)(((int64_t)n_pairs + 3) / 4);
  hipLaunchKernelGGL(pair_fidelity_kernel, dim3(blocks), dim3(256), 0, s, ca, cb, (int64_t)256,
                     n_pairs, F);
  return hipGetLastError();
}

// One training (or gradient-only) step over n_pairs pairs (a_i, b_i); the
// workspace holds the encodings of a_i and b_i as rows 2i and 2i+1.
hipError_t launch_learned_step(float* state, float lr, const uint8_t* a, const int64_t* aoff,
                               const uint8_t* b, const int64_t* boff, const int32_t* ld,
                               int32_t n_pairs, int N, void* ws, float* grad_out,
                               float* loss_out, hipStream_t s) {
  const int64_t strings = 2 * (int64_t)n_pairs;
  const int per = strings_per_block(strings);
  const unsigned blocks = (unsigned)((strings + per - 1) / per);
  const Strings st{a, aoff, b, boff};
  const Nominal nom(N);
  uint8_t* base = static_cast<uint8_t*>(ws);
  float* c = reinterpret_cast<float*>(base);
  float* F = c + strings * 256;
  float* dF = F + n_pairs;
  float* lossv = dF + n_pairs;
  int32_t* cntv = reinterpret_cast<int32_t*>(lossv + n_pairs);
  float* loss_ws = reinterpret_cast<float*>(cntv + n_pairs);
  float* partial = reinterpret_cast<float*>(
      (reinterpret_cast<uintptr_t>(loss_ws + 64) + 255) / 256 * 256);
  hipLaunchKernelGGL(learned_encode_kernel, dim3(blocks), dim3(64 * kWaves), 0, s, state, st,
                     (int32_t)strings, per, nom.n, nom.inv, nom.turn, c, F);
  hipLaunchKernelGGL(ranking_kernel, dim3((unsigned)n_pairs), dim3(64 * kRankWaves), 0, s, F, ld,
                     n_pairs, dF, lossv, cntv, grad_out ? nullptr : state + 3 * kParams);
  hipLaunchKernelGGL(learned_backward_kernel, dim3(blocks), dim3(64 * kWaves), 0, s, state, st,
                     n_pairs, per, nom.n, nom.inv, nom.turn, c, dF, cntv, partial);
  hipLaunchKernelGGL(reduce_adam_kernel, dim3(kRedBlocks + 1), dim3(kRedParams * kRedParts), 0, s,
                     partial, (int)blocks, lossv, cntv, n_pairs, loss_out ? loss_out : loss_ws,
                     grad_out, grad_out ? nullptr : state, lr);
  return hipGetLastError();
}

}  // namespace rm
