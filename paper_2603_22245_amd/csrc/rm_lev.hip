// Exact Levenshtein distance of string pairs (the labels of the learned
// ranking loss, and the reference the Spearman correlation is taken against).
//
// Bit-parallel dynamic programme over the columns of the text: Myers (J. ACM
// 46(3), 1999) with the block decomposition of the same paper, in its
// global-distance form (the horizontal delta entering row 0 is +1 at every
// column, the vertical deltas of column 0 are all +1).  The shorter string is
// the pattern, at most 256 letters = 4 words of 64 bits; the score at the last
// pattern row starts at m and follows the horizontal delta leaving the last
// block.
//
// A lane per word: lane w of a pair works on column t - w in step t, so the
// delta that word w - 1 left in step t - 1 is the one entering this column, and
// a step costs one word instead of up to four in a chain.  A block takes 64
// pairs with one, two or four lanes a pair, as the longest of their patterns
// needs (its other wavefronts end at once).  A pair's first lane loads its text
// eight letters at a time, eight columns ahead, and hands each letter down with
// the deltas.  Bound by the serial chain of the columns, and by VALU issue from
// about 10^5 pairs on.  Pairs of 150 letters: 8,192 in 30 us, 10^6 in 0.94 ms
// (126 us and 4.5 ms with a lane per pair); of 16 letters: 10^6 in 39 us (44 us
// with a lane per pair, 187 us with four lanes for patterns of one word).
#include <algorithm>

#include "rm_internal.h"

namespace rm {

namespace {

constexpr int kWords = 4;   // of a pattern, and wavefronts of a block
constexpr int kPairs = 64;  // pairs of a block
constexpr int kOther = 4;   // a letter that matches nothing

// Letters at .. at + 7 of a string of n, one per byte from the low end; kOther past its end.
__device__ __forceinline__ uint64_t eight_letters(const uint8_t* s, int64_t at, int64_t n) {
  uint64_t v = 0x0101010101010101ull * kOther;
  if (at + 8 <= n) {
    __builtin_memcpy(&v, s + at, 8);
  } else {
    for (int i = 0; at + i < n; ++i)
      v ^= (uint64_t)(s[at + i] ^ kOther) << (8 * i);
  }
  return v;
}

// Bit 0 of every byte, as eight bits.
__device__ __forceinline__ uint64_t low_bits(uint64_t bytes) {
  return ((bytes & 0x0101010101010101ull) * 0x0102040810204080ull) >> 56;
}

// A pattern word: bits 0 and 1 of its letters, and which of them are one of the four.
struct Word {
  uint64_t b0, b1, letter;
};

__device__ __forceinline__ Word load_word(const uint8_t* P, int64_t m, int64_t first) {
  Word p{0, 0, 0};
  for (int q = 0; q < 64 && first + q < m; q += 8) {
    const uint64_t v = eight_letters(P, first + q, m);
    const uint64_t high = v & 0xfcfcfcfcfcfcfcfcull;  // no carry leaves a byte below
    const uint64_t other = (((high >> 2) + 0x3f3f3f3f3f3f3f3full) >> 6);
    p.b0 |= low_bits(v) << q;
    p.b1 |= low_bits(v >> 1) << q;
    p.letter |= low_bits(~other) << q;
  }
  return p;
}

// Distance of the lane's pair, whose KW lanes are aligned; every lane of the
// wavefront takes part, and all lanes of a pair return its result.  live: the
// pair exists.
template <int KW>
__device__ __forceinline__ int32_t distance(const uint8_t* A, int64_t la, const uint8_t* B,
                                            int64_t lb, bool live, int w) {
  const bool swap = la > lb;
  const uint8_t* P = swap ? B : A;
  const uint8_t* T = swap ? A : B;
  const int64_t m = swap ? lb : la;
  const int64_t tn = live && m > 0 && m <= 64 * kWords ? (swap ? la : lb) : 0;
  const Word word = load_word(P, tn > 0 ? m : 0, 64 * w);
  const bool last = 64 * w < m && 64 * (w + 1) >= m;  // the word holds the last pattern row
  const uint64_t high = 1ull << (last ? (int)((m - 1) & 63) : 63);
  const int64_t steps = (int64_t)wave_max_u64((uint64_t)(tn > 0 ? tn + KW - 1 : 0));
  uint64_t pv = ~0ull, mv = 0;
  int score = (int)m, hout = 0, c = kOther;
  uint64_t next = w == 0 && tn > 0 ? eight_letters(T, 0, tn) : 0x0101010101010101ull * kOther;
  for (int64_t t0 = 0; t0 < steps; t0 += 8) {
    uint64_t text = next;
    if (w == 0 && t0 + 8 < tn) next = eight_letters(T, t0 + 8, tn);
    const int left = (int)min<int64_t>(tn + w - t0, 8);  // steps of this lane's columns
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      // What the word above left in the last step.  Before its first column a
      // word sees no letter and no delta, which leave its state as it is.
      const int letter = (int)(text >> (8 * i)) & 255;
      int hin = 1;  // row 0: D[0][j] = j
      if constexpr (KW > 1) {
        constexpr int kAbove = KW == 4 ? 0x90 : 0xA0;  // quad_perm [0,0,1,2] or [0,0,2,2]
        const int above_c = __builtin_amdgcn_update_dpp(0, c, kAbove, 0xf, 0xf, false);
        const int above_h = __builtin_amdgcn_update_dpp(0, hout, kAbove, 0xf, 0xf, false);
        c = w == 0 ? letter : above_c;
        hin = w == 0 ? 1 : above_h;
      } else {
        c = letter;
      }
      const uint64_t s0 = (uint64_t)(int64_t)-(c & 1), s1 = (uint64_t)(int64_t)-(c >> 1 & 1);
      uint64_t eq = c < 4 ? ~(word.b0 ^ s0) & ~(word.b1 ^ s1) & word.letter : 0;
      const uint64_t xv = eq | mv;
      if (hin < 0) eq |= 1;
      const uint64_t xh = (((eq & pv) + pv) ^ pv) | eq;
      uint64_t ph = mv | ~(xh | pv);
      uint64_t mh = pv & xh;
      hout = (ph & high) ? 1 : (mh & high) ? -1 : 0;
      ph = (ph << 1) | (hin > 0 ? 1 : 0);
      mh = (mh << 1) | (hin < 0 ? 1 : 0);
      pv = mh | ~(xv | ph);
      mv = ph & xv;
      score += i < left ? hout : 0;
    }
  }
  // the last word's score, in every lane of the pair
  int res = last ? score : 0;
  if constexpr (KW > 1) res += __builtin_amdgcn_update_dpp(0, res, 0xB1, 0xf, 0xf, false);  // [1,0,3,2]
  if constexpr (KW > 2) res += __builtin_amdgcn_update_dpp(0, res, 0x4E, 0xf, 0xf, false);  // [2,3,0,1]
  if (m <= 0) return (int32_t)max<int64_t>(swap ? la : lb, 0);
  return m > 64 * kWords ? -1 : res;
}

__global__ __launch_bounds__(64 * kWords) void levenshtein_kernel(
    const uint8_t* __restrict__ a, const int64_t* __restrict__ aoff,
    const uint8_t* __restrict__ b, const int64_t* __restrict__ boff, int64_t n,
    int32_t* __restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t i0 = (int64_t)blockIdx.x * kPairs;
  // lanes per pair: the words of the block's longest pattern
  const int64_t own = min(i0 + lane, n - 1);
  const int64_t m = min(aoff[own + 1] - aoff[own], boff[own + 1] - boff[own]);
  const bool two = m > 64 && m <= 64 * kWords, four = m > 128 && m <= 64 * kWords;
  const int kw = __ballot(four) != 0 ? 4 : __ballot(two) != 0 ? 2 : 1;  // uniform
  if (wave >= kw) return;
  const int64_t pair = i0 + (wave * 64 + lane) / kw;
  const bool live = pair < n;
  const int64_t i = live ? pair : n - 1;
  const int w = lane & (kw - 1);
  const int64_t a0 = aoff[i], la = aoff[i + 1] - a0;
  const int64_t b0 = boff[i], lb = boff[i + 1] - b0;
  int32_t d;
  if (kw == 1) d = distance<1>(a + a0, la, b + b0, lb, live, w);
  else if (kw == 2) d = distance<2>(a + a0, la, b + b0, lb, live, w);
  else d = distance<4>(a + a0, la, b + b0, lb, live, w);
  if (live && w == 0) out[i] = d;
}

}  // namespace

hipError_t launch_levenshtein(const uint8_t* a, const int64_t* aoff, const uint8_t* b,
                              const int64_t* boff, int64_t n, int32_t* out, hipStream_t s) {
  // a launch has fewer than 2^32 threads, four per pair
  constexpr int64_t kMost = (int64_t)1 << 29;
  for (int64_t i = 0; i < n; i += kMost) {
    const int64_t some = std::min(n - i, kMost);
    hipLaunchKernelGGL(levenshtein_kernel, dim3((unsigned)((some + kPairs - 1) / kPairs)),
                       dim3(64 * kWords), 0, s, a, aoff + i, b, boff + i, some, out + i);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace rm
