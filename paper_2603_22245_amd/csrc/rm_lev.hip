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
// Four lanes per pair, one word each: lane w works on column t - w in step t,
// so the delta that word w - 1 left in step t - 1 is the one entering this
// column, and a step costs one word instead of up to four in a chain.  A
// wavefront's 16 pairs are contiguous in memory and are copied to LDS first
// (coalesced; a column's letter is then one LDS read, issued a step ahead).
// Bound by the serial chain of the columns: 8,192 pairs of 150 letters in 55
// us, 10^6 in 1.42 ms (139 us and 4.4 ms with a lane per pair and letters read
// from global memory).
#include "rm_internal.h"

namespace rm {

namespace {

constexpr int kWords = 4;
constexpr int kPairs = 64 / kWords;  // pairs of a wavefront
constexpr int kStage = 6144;         // LDS bytes for their letters, per side

// Distance of the lane's pair; every lane of the wavefront takes part, and
// lane 0 of a pair's four returns its result.  live: the pair exists.
__device__ __forceinline__ int32_t distance(const uint8_t* A, int64_t la, const uint8_t* B,
                                            int64_t lb, bool live, int w) {
  const bool swap = la > lb;
  const uint8_t* P = swap ? B : A;
  const uint8_t* T = swap ? A : B;
  const int64_t m = swap ? lb : la, tn = swap ? la : lb;
  const bool run = live && m > 0 && m <= 64 * kWords;
  // match masks of this lane's word
  uint64_t eqA = 0, eqC = 0, eqG = 0, eqT = 0;
  const int q1 = run ? (int)min<int64_t>(m - 64 * w, 64) : 0;
  for (int q = 0; q < q1; ++q) {
    const uint8_t c = P[64 * w + q];
    const uint64_t bit = 1ull << q;
    eqA |= c == 0 ? bit : 0;
    eqC |= c == 1 ? bit : 0;
    eqG |= c == 2 ? bit : 0;
    eqT |= c == 3 ? bit : 0;
  }
  const bool mine = q1 > 0;                        // this word holds pattern rows
  const bool last = mine && 64 * (w + 1) >= m;     // ... the last of them
  const uint64_t high = 1ull << (last ? (int)((m - 1) & 63) : 63);
  uint64_t pv = ~0ull, mv = 0;
  int64_t score = m;
  int hout = 0;
  int64_t j = -(int64_t)w;  // this lane's column
  int c = mine && w == 0 && tn > 0 ? T[0] : 4;
  while (__ballot(mine && j < tn)) {
    // letter of the lane's next column
    const int next = mine && j + 1 >= 0 && j + 1 < tn ? T[j + 1] : 4;
    // the delta leaving the word above in the last step (quad_perm [0,0,1,2])
    const int above = __builtin_amdgcn_update_dpp(0, hout, 0x90, 0xf, 0xf, false);
    const int hin = w == 0 ? 1 : above;  // row 0: D[0][j] = j
    if (mine && j >= 0 && j < tn) {
      uint64_t eq = c == 0 ? eqA : c == 1 ? eqC : c == 2 ? eqG : c == 3 ? eqT : 0;
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
      score += hout;
    }
    c = next;
    ++j;
  }
  // the last word's score, in every lane of the four
  int res = last ? (int)score : 0;
  res += __builtin_amdgcn_update_dpp(0, res, 0xB1, 0xf, 0xf, false);  // quad_perm [1,0,3,2]
  res += __builtin_amdgcn_update_dpp(0, res, 0x4E, 0xf, 0xf, false);  // quad_perm [2,3,0,1]
  if (m <= 0) return (int32_t)max<int64_t>(tn, 0);
  return m > 64 * kWords ? -1 : res;
}

__global__ __launch_bounds__(64) void levenshtein_kernel(
    const uint8_t* __restrict__ a, const int64_t* __restrict__ aoff,
    const uint8_t* __restrict__ b, const int64_t* __restrict__ boff, int64_t n,
    int32_t* __restrict__ out) {
  __shared__ uint8_t sa[kStage], sb[kStage];
  const int lane = threadIdx.x, w = lane % kWords;
  const int64_t i0 = (int64_t)blockIdx.x * kPairs;
  const int64_t i1 = min(n, i0 + kPairs);
  const bool live = i0 + lane / kWords < i1;
  const int64_t i = live ? i0 + lane / kWords : i0;
  const int64_t a0 = aoff[i], la = aoff[i + 1] - a0;
  const int64_t b0 = boff[i], lb = boff[i + 1] - b0;
  const int64_t abase = aoff[i0], na = aoff[i1] - abase;
  const int64_t bbase = boff[i0], nb = boff[i1] - bbase;
  int32_t d;
  if (na <= kStage && nb <= kStage) {  // uniform
    for (int q = lane; q < (int)na; q += 64) sa[q] = a[abase + q];
    for (int q = lane; q < (int)nb; q += 64) sb[q] = b[bbase + q];
    __syncthreads();
    d = distance(sa + (a0 - abase), la, sb + (b0 - bbase), lb, live, w);
  } else {  // long strings: letters straight from global memory
    d = distance(a + a0, la, b + b0, lb, live, w);
  }
  if (live && w == 0) out[i] = d;
}

}  // namespace

hipError_t launch_levenshtein(const uint8_t* a, const int64_t* aoff, const uint8_t* b,
                              const int64_t* boff, int64_t n, int32_t* out, hipStream_t s) {
  const unsigned blocks = (unsigned)((n + kPairs - 1) / kPairs);
  hipLaunchKernelGGL(levenshtein_kernel, dim3(blocks), dim3(64), 0, s, a, aoff, b, boff, n, out);
  return hipGetLastError();
}

}  // namespace rm
