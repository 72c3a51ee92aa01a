// Scoring GEMM with fused per-read top-k (§3.1): FP32 and FP8 instantiations,
// the work plan, the launch sequence and the merge of per-chunk lists.  The
// kernel itself is in rm_score_kernel.h; FP16 is instantiated in
// rm_score_f16.hip.
#include "rm_score_kernel.h"

#include <algorithm>
#include <cmath>

namespace rm {

namespace {

// Clears the work counter and every group's shared per-read thresholds and
// slots ("no information" = 0).
__global__ void clear_state(ScoreLaunch L) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) *L.counter = 0;
  for (int gi = 0; gi < L.n_groups; ++gi)
    if (i < L.g[gi].R) {
      L.g[gi].gthr[i] = 0u;
      uint4* slot = reinterpret_cast<uint4*>(L.g[gi].gslot + i * kScoreSlots);
#pragma unroll
      for (int u = 0; u < kScoreSlots / 2; ++u) slot[u] = make_uint4(0, 0, 0, 0);
    }
}

// Keys per read that merge_kernel takes, and that merge_block_kernel takes.
constexpr int kMergeKeys = 1024, kMergeKeysWide = 16384;
// One block per CU of the chip; the reads of a single group up to which read
// tiles hold 128.
constexpr int64_t kChipBlocks = 256;
constexpr int32_t kFewReads = 1024;
// Reads up to which a launch only streams the index; those up to which (a group),
// or twice which, lists that are not seeded cost little.
constexpr int32_t kStreamReads = 32, kColdReads = 8;

// Merge the P per-chunk lists of each read into its k_fetch best (keys are
// unique per read).  One wavefront per read (all its lanes active): each lane
// sorts the EMAX keys it holds (descending), then every round takes the
// wavefront maximum of the lanes' heads and the lane that held it drops its
// head.  Lane `out` keeps the
// round-`out` winner, so the k_fetch results are written with one coalesced
// store each.  wave_best: that reduction of n keys.
template <int EMAX>
__device__ __forceinline__ uint64_t wave_best(const uint64_t* __restrict__ src, int n, int k,
                                              int lane) {
  uint64_t mine[EMAX];
#pragma unroll
  for (int e = 0; e < EMAX; ++e) {
    int i = e * 64 + lane;
    mine[e] = i < n ? src[i] : 0;
  }
  // odd-even transposition sort, descending (EMAX rounds make it complete)
#pragma unroll
  for (int p = 0; p < EMAX; ++p)
#pragma unroll
    for (int e = p & 1; e + 1 < EMAX; e += 2) {
      uint64_t x = mine[e], y = mine[e + 1];
      mine[e] = x > y ? x : y;
      mine[e + 1] = x > y ? y : x;
    }
  uint64_t res = 0;
  for (int out = 0; out < k; ++out) {
    const uint64_t gbest = wave_max_u64(mine[0]);
    if (gbest != 0 && mine[0] == gbest) {
#pragma unroll
      for (int e = 0; e + 1 < EMAX; ++e) mine[e] = mine[e + 1];
      mine[EMAX - 1] = 0;
    }
    if (lane == out) res = gbest;
  }
  return res;
}

template <int EMAX>
__global__ __launch_bounds__(256) void merge_kernel(const uint64_t* __restrict__ ws, int n_per_read,
                                                    int32_t R, int k_fetch,
                                                    int32_t* __restrict__ cand_idx,
                                                    float* __restrict__ cand_score) {
  const int lane = threadIdx.x & 63;
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= R) return;
  const uint64_t res = wave_best<EMAX>(ws + r * n_per_read, n_per_read, k_fetch, lane);
  if (lane < k_fetch) {
    write_list_entry(res, &cand_idx[r * k_fetch + lane], &cand_score[r * k_fetch + lane]);
  }
}

// The same merge for few reads with many chunks (n_per_read up to
// kMergeKeysWide, 16 keys per lane of the block): 16 wavefronts per read, each
// reducing a sixteenth of the keys to its k_fetch best, then the first
// wavefront those.  Latency bound; one wavefront per read would hold 256 keys
// per lane.
constexpr int kMergeWaves = 16;
template <int EMAX>
__global__ __launch_bounds__(64 * kMergeWaves) void merge_block_kernel(
    const uint64_t* __restrict__ ws, int n_per_read, int k_fetch, int32_t* __restrict__ cand_idx,
    float* __restrict__ cand_score) {
  __shared__ uint64_t best[kMergeWaves * RM_MAX_KFETCH];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t r = blockIdx.x;
  const int per = (n_per_read + kMergeWaves - 1) / kMergeWaves, from = wave * per;
  const uint64_t key = wave_best<EMAX>(ws + r * n_per_read + from, min(per, n_per_read - from),
                                       k_fetch, lane);
  if (lane < k_fetch) best[wave * k_fetch + lane] = key;
  __syncthreads();
  if (wave != 0) return;
  const uint64_t res = wave_best<16>(best, kMergeWaves * k_fetch, k_fetch, lane);
  if (lane < k_fetch) {
    write_list_entry(res, &cand_idx[r * k_fetch + lane], &cand_score[r * k_fetch + lane]);
  }
}

// Seeds the reads' slots before the scoring launch, so that no chunk starts
// without a threshold.  A block of eight wavefronts scores 128 reads against
// seed_tiles of the 32-window tiles sampled evenly over the index; a lane
// keeps, per read, the largest F of its column over these tiles, with no
// lists and no test.  Windows of different columns are different windows
// (slot = id mod 32 = column), so the columns' maxima are exactly what the
// slots hold, and the KP-th largest of them bounds the read's KP-th best
// from below (slot_bounds, at the start of every scoring item).  A key's low
// word names a window, but the bound only uses its F.
// Without it every chunk of a small launch fills its own lists from nothing
// (16 to 60 appends and 2 to 4 merges per read and chunk), which took most of
// the time: 200 reads against 20,000 FP16 windows 318 -> 71 us, 1,000 reads
// against 100,000 339 -> 218 us, 100 reads against 10^7 2.4 -> 1.1 ms.  Both
// operands come straight from global memory (the block's wavefronts read the
// same window rows): latency and L1 bound, about a third of the scoring
// kernel's rate per score; seed_windows weighs that.
template <int PREC, int KR>
__global__ __launch_bounds__(512) void seed_kernel(ScoreLaunch L) {
  using RF = RowFmt<PREC, KR>;
  constexpr bool kFp8 = PREC == RM_FP8_E4M3;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 5, col = lane & 31;
  int gi = 0;
  while (gi + 1 < L.n_groups && (int)blockIdx.x >= L.g[gi + 1].seed_begin) ++gi;
  const ScoreGroup& G = L.g[gi];
  const int local = blockIdx.x - G.seed_begin;
  const int seg = local % G.seed_segs;
  const int64_t R = G.R, W = G.W;
  const int64_t read0 = ((int64_t)(local / G.seed_segs) * 8 + wave) * 16;
  if (read0 >= R) return;
  uint4 a[1][RF::AU4];
  const int64_t arow = 2 * read0 + col;
#pragma unroll
  for (int u = 0; u < RF::AU4; ++u)
    a[0][u] = arow < 2 * R ? reinterpret_cast<const uint4*>(G.reads + arow * RF::RB)[RF::lane_chunk(g, u)]
                           : make_uint4(0, 0, 0, 0);
  float m[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) m[q] = -1.f;
  const int64_t all = (W + kBlkW - 1) / kBlkW, n = (int64_t)G.seed_segs * G.seed_tiles;
  for (int t = 0; t < G.seed_tiles; ++t) {
    const int64_t j = ((int64_t)seg * G.seed_tiles + t) * all / n * kBlkW + col;
    const int64_t row = min(j, W - 1);
    const uint4* src = reinterpret_cast<const uint4*>(G.index + row * RF::RB);
    uint4 b[RF::AU4];
#pragma unroll
    for (int u = 0; u < RF::AU4; ++u) b[u] = src[RF::lane_chunk(g, u)];
    f32x16 acc{};
    mfma_regs<PREC, KR>(a[0], b, acc);
    float sj2 = 1.f;
    if constexpr (kFp8) {
      const float sc = G.win_scale[row];
      sj2 = sc * sc;
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const float re = acc[2 * q], im = acc[2 * q + 1];
      const float F = (re * re + im * im) * sj2;
      m[q] = j < W ? fmaxf(m[q], F) : m[q];
    }
  }
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int64_t r = read0 + 4 * (q >> 1) + 2 * g + (q & 1);
    if (r >= R || m[q] < 0.f) continue;
    float F = m[q];
    if constexpr (kFp8) F *= G.read_scale[r] * G.read_scale[r];
    const uint64_t key = make_key(F, -1);
    unsigned long long* slot =
        reinterpret_cast<unsigned long long*>(&G.gslot[r * kScoreSlots + col]);
    if (key > __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMax(slot, (unsigned long long)key);
  }
}

template <int PREC>
hipError_t launch_seed(bool reduced, int blocks, const ScoreLaunch& L, hipStream_t s) {
  hipLaunchKernelGGL((reduced ? seed_kernel<PREC, kRealReduced> : seed_kernel<PREC, kReal>),
                     dim3((unsigned)blocks), dim3(512), 0, s, L);
  return hipGetLastError();
}

// Instantiations: (precision, reads per block, list length, row format) ->
// (fragments per wavefront, list+buffer entries, ring stages, column blocks);
// LDS stays within 160 KB.
template <int KR>
hipError_t dispatch_f8(int read_tile, int kp, const ScoreLaunch& L, hipStream_t s) {
  if (read_tile == 256) {
    switch (kp) {
      case 8: return launch_persistent<RM_FP8_E4M3, 2, 8, 32, 4, 2, KR>(L, s);
      case 16: return launch_persistent<RM_FP8_E4M3, 2, 16, 32, 4, 2, KR>(L, s);
      default: return launch_persistent<RM_FP8_E4M3, 2, 32, 48, 3, 2, KR>(L, s);
    }
  }
  switch (kp) {
    case 8: return launch_persistent<RM_FP8_E4M3, 1, 8, 32, 4, 1, KR>(L, s);
    case 16: return launch_persistent<RM_FP8_E4M3, 1, 16, 32, 4, 1, KR>(L, s);
    case 32: return launch_persistent<RM_FP8_E4M3, 1, 32, 64, 4, 1, KR>(L, s);
    // 64-key lists with a 32-slot buffer: 96 KB of lists
    default: return launch_persistent<RM_FP8_E4M3, 1, 64, 96, 4, 1, KR>(L, s);
  }
}

template <int KR>
hipError_t dispatch_f32(int kp, const ScoreLaunch& L, hipStream_t s) {
  switch (kp) {
    case 8: return launch_persistent<RM_FP32, 1, 8, 32, 3, 1, KR>(L, s);
    case 16: return launch_persistent<RM_FP32, 1, 16, 32, 3, 1, KR>(L, s);
    case 32: return launch_persistent<RM_FP32, 1, 32, 64, 2, 1, KR>(L, s);
    // 64-key lists with a 16-slot buffer (80 KB) and two stages of at most 32 KB
    default: return launch_persistent<RM_FP32, 1, 64, 80, 2, 1, KR>(L, s);
  }
}

hipError_t dispatch(int precision, bool reduced, int read_tile, int kp, const ScoreLaunch& L,
                    hipStream_t s) {
  if (precision == RM_FP32)
    return reduced ? dispatch_f32<kRealReduced>(kp, L, s) : dispatch_f32<kReal>(kp, L, s);
  if (precision == RM_FP16) return dispatch_score_f16(read_tile, kp, reduced, L, s);
  return reduced ? dispatch_f8<kRealReduced>(read_tile, kp, L, s)
                 : dispatch_f8<kReal>(read_tile, kp, L, s);
}

}  // namespace

bool read_tile_ok(int precision, int kp, int read_tile) {
  if (read_tile == 128) return true;
  if (read_tile == 256) return precision != RM_FP32 && kp <= 32;  // 64-key lists: 128 reads
  return false;
}

static size_t align256(size_t v) { return (v + 255) / 256 * 256; }

// Reads of a block tile where the caller names none.  128-read tiles leave room
// for two blocks per CU and lose less to a part-filled tile: up to 1,024 reads
// they are the faster ones (FP16, 200 reads x 20,000 windows 101 -> 86 us, 1,000
// x 100,000 238 -> 225 us, 100 x 10^7 1.18 -> 1.11 ms), beyond that the wider
// tile's reuse of each window is (2,000 x 10^6: 1.79 against 1.84 ms).
static int default_read_tile(int precision, int kp, int n_groups, int64_t R0) {
  const bool few = n_groups == 1 && R0 <= kFewReads;
  return !few && read_tile_ok(precision, kp, 256) ? 256 : 128;
}

// A group's read tiles.  256-read tiles run two fragments per wavefront; a group
// that would leave a quarter or more of its padded reads empty takes 128-read
// tiles (one fragment per wavefront, half the work per tile) in the same launch.
static void tile_reads(int64_t R, int rt, GroupPlan& gp) {
  gp.read_tiles = (int)((R + rt - 1) / rt);
  gp.thin = 0;
  if (rt == 256) {
    const int64_t t128 = (R + 127) / 128;
    if (4 * 128 * t128 <= 3 * 256 * (int64_t)gp.read_tiles) {
      gp.thin = 1;
      gp.read_tiles = (int)t128;
    }
  }
}

// Chunks for about 30 items per CU of a 256-CU chip (a short last round), at least
// 64 tile units each, at most 1024 keys per read for the merge; fewer, longer items
// leave an uneven last round, more items repeat each read's top-k warm-up in more
// chunks.
static int64_t long_chunks(int64_t tiles, int read_tiles, int kp) {
  const int64_t P = (kChipBlocks * 30 + read_tiles - 1) / read_tiles;
  return std::max<int64_t>(std::min<int64_t>({P, (tiles + 63) / 64, kMergeKeys / kp}), 1);
}

// Whether long chunks, `items` of them in a launch and the longest of `longest` tile
// units, leave CUs idle for more than it costs to fill the lists of shorter ones.
static bool chip_idle(int precision, int64_t items, int64_t longest, bool only) {
  if (precision == RM_FP32) return items < 2 * kChipBlocks;
  return items < kChipBlocks / 2 || (items < kChipBlocks && (only || longest > 256));
}

// A group's chunks, with chunk_tiles 64-window units per chunk or the default
// rule (<= 0).  share: the group's part of kChipBlocks by its work; idle: of the
// launch (chip_idle).
static void cut_windows(int64_t R, int64_t tiles, int64_t chunk_tiles, int64_t share, bool only,
                        bool idle, int precision, int kp, GroupPlan& gp) {
  int64_t ct = chunk_tiles, most = kMergeKeys / kp;
  if (ct <= 0) {
    int64_t P = long_chunks(tiles, gp.read_tiles, kp), Q = 0;
    most = std::max<int64_t>(most, kMergeKeysWide / kp);
    // Few read tiles: that rule gives 64 chunks of 16-key lists at most,
    // and one per 4,096 windows (10 items for 200 FP32 reads against
    // 20,000 windows).  Here a group gets its share of eight items per CU
    // with chunks of 2,048 windows or more, but at least its share of one
    // per CU, and a single group fills whole rounds of the chip.  Measured
    // (chunks before -> now): FP32 200 x 20,000 1,330 -> 165 us (5 -> 104),
    // FP16 8 x 10^7 2,310 -> 725 us (64 -> 512), 300 x 10^6 970 -> 440 us.
    // Up to 32 reads the launch only streams the index, and shorter
    // chunks cost more than they balance (8 x 10^7: 512 chunks 724 us,
    // 1,024 775 us).
    // No seed starts lists of 64 keys (seed_windows): every chunk fills its own
    // from nothing, so they are only shorter where CUs would be idle, and two
    // items per CU (FP16 and FP8 groups: one).  FP32 scores cost more against the same
    // lists; elsewhere few reads of a group take 1,024 windows at least, and
    // in FP16 a read tile of 17 reads or more 128 chunks at most, unless 256 are one
    // tile unit each.  With long chunks / eight items per CU / as here: FP16
    // 3,000 reads x 200,000 windows 2.56 / 3.30 / 2.57 ms, 8,000 x 42,000 1.85 / 2.85 / 1.91,
    // 60 x 200,000 1.40 / 1.78 / 1.03, 1 x 10^6 1.07 / 0.23 / 0.22; seven groups of 2,950
    // reads in all, a reference of 226,000 letters, 1.93 / 2.77 / 1.95 (FP32 6.10 /
    // 5.72 / 4.61), of 300 reads and 400,000 letters 1.36 / 1.35 / 1.16.
    const bool cold = kp > kScoreSlots, f32 = precision == RM_FP32;
    if (!cold || idle) {
      const int64_t own = (share + gp.read_tiles - 1) / gp.read_tiles;
      Q = std::min((!cold ? 8 : only || f32 ? 2 : 1) * share / gp.read_tiles, (tiles + 31) / 32);
      Q = std::max(Q, cold && !only && !f32 && R <= kColdReads ? std::min(own, (tiles + 15) / 16) : own);
      if (R <= kStreamReads) Q = std::min<int64_t>(Q, 2 * kChipBlocks);
      if (only) {
        const int64_t rounds = (Q * gp.read_tiles + kChipBlocks - 1) / kChipBlocks;
        Q = std::max(Q, rounds * kChipBlocks / gp.read_tiles);
      }
      if (cold && precision == RM_FP16 && R > 2 * kColdReads && gp.read_tiles == 1 && tiles > most)
        Q = std::min<int64_t>(Q, kChipBlocks / 2);
    }
    P = std::max(P, std::min({Q, most, tiles}));
    ct = (tiles + P - 1) / P;
  }
  if (ct < 1) ct = 1;
  int64_t P = (tiles + ct - 1) / ct;
  if (P > most) {  // keep the merge within its keys per read
    P = most;
    ct = (tiles + P - 1) / P;
    P = (tiles + ct - 1) / ct;
  }
  gp.chunk_windows = ct * kPlanW;
  gp.chunks = (int)P;
}

static int list_keys(int k_fetch) {
  return k_fetch <= 8 ? 8 : k_fetch <= 16 ? 16 : k_fetch <= 32 ? 32 : 64;
}

static size_t list_bytes(int64_t lists, int kp) {
  return align256((size_t)lists * (size_t)kp * sizeof(uint64_t));
}

ScorePlan plan_score(int precision, int n_groups, const int64_t* W, const int32_t* R, int k_fetch,
                     Tuning t) {
  ScorePlan p{};
  p.kp = list_keys(k_fetch);
  const int rt = t.read_tile ? t.read_tile : default_read_tile(precision, p.kp, n_groups, R[0]);
  if (!read_tile_ok(precision, p.kp, rt) || n_groups < 1 || n_groups > kMaxGroups) return p;
  p.read_tile = rt;
  p.n_groups = n_groups;
  // work of a group: 64-window units x 128-read halves of its read tiles
  int64_t work[kMaxGroups], total_work = 0, items1 = 0, longest = 0;
  for (int i = 0; i < n_groups; ++i) {
    GroupPlan& gp = p.g[i];
    tile_reads(R[i], rt, gp);
    const int64_t tiles = (W[i] + kPlanW - 1) / kPlanW;
    const int64_t P = long_chunks(tiles, gp.read_tiles, p.kp);
    items1 += gp.read_tiles * P;
    longest = std::max(longest, (tiles + P - 1) / P);
    work[i] = (W[i] + kPlanW - 1) / kPlanW * gp.read_tiles * (rt == 256 && !gp.thin ? 2 : 1);
    total_work += work[i];
  }
  size_t off = 0;
  int64_t items = 0;
  for (int i = 0; i < n_groups; ++i) {
    GroupPlan& gp = p.g[i];
    cut_windows(R[i], (W[i] + kPlanW - 1) / kPlanW, t.chunk_tiles,
                (work[i] * kChipBlocks + total_work - 1) / total_work, n_groups == 1,
                chip_idle(precision, items1, longest, n_groups == 1), precision, p.kp, gp);
    gp.lists_offset = off;
    off += list_bytes((int64_t)R[i] * gp.chunks, p.kp);
    gp.thr_offset = off;
    off = align256(off + (size_t)R[i] * sizeof(uint32_t));
    gp.slot_offset = off;
    off = align256(off + (size_t)R[i] * kScoreSlots * sizeof(uint64_t));
    items += (int64_t)gp.read_tiles * gp.chunks;
  }
  p.counter_offset = off;
  p.ws_bytes = off + 256;
  p.total_items = items;
  p.ok = items > 0 && items < INT32_MAX;
  return p;
}

// What every launch of at most these reads needs.  The default rule gives fewer
// reads more chunks, so a plan of its own reads alone would be too small for some
// smaller batches (FP16, 20,000 windows, 16 candidates: 14,114 reads 18.1 MB,
// 13,372 reads 18.8 MB).
size_t score_workspace_bytes(int precision, int n_groups, const int64_t* W, const int32_t* R,
                             int k_fetch, Tuning t) {
  const ScorePlan p = plan_score(precision, n_groups, W, R, k_fetch, t);
  if (!p.ok) return 0;
  if (t.chunk_tiles > 0) return p.ws_bytes;  // chunks of a given length: as many for any reads
  // The most lists of a group over its smaller read counts.  Chunks change with
  // the read tiles only, so the counts that matter are the last of each.  From
  // kChipBlocks * 30 tiles on there is one chunk.
  int64_t sum = 0;
  size_t rest = 256, lists = 0;
  for (int i = 0; i < n_groups; ++i) {
    const int64_t tiles = (W[i] + kPlanW - 1) / kPlanW;
    int64_t most = 0;
    const auto at = [&](int64_t r) {
      GroupPlan g{};
      tile_reads(r, t.read_tile ? t.read_tile : default_read_tile(precision, p.kp, n_groups, r), g);
      const int64_t P = long_chunks(tiles, g.read_tiles, p.kp);
      const bool idle = n_groups > 1 || chip_idle(precision, g.read_tiles * P, (tiles + P - 1) / P, true);
      cut_windows(r, tiles, 0, kChipBlocks, n_groups == 1, idle, precision, p.kp, g);
      most = std::max(most, r * g.chunks);
    };
    at(std::min<int64_t>(R[i], kColdReads));
    at(std::min<int64_t>(R[i], 2 * kColdReads));
    at(std::min<int64_t>(R[i], kStreamReads));
    for (int64_t r = 128; r < std::min<int64_t>(R[i], kChipBlocks * 30 * 256 + 1); r += 128) at(r);
    at(R[i]);
    sum += most;
    lists += list_bytes(most, p.kp);
    rest += align256((size_t)R[i] * sizeof(uint32_t)) +
            align256((size_t)R[i] * kScoreSlots * sizeof(uint64_t));
  }
  if (n_groups > 1) {
    // The groups share the chip: a group with share s has at most 8 s tiles' worth
    // of lists (or a list a read), and the shares add up to kChipBlocks and one
    // for each group; besides these at most those of the 30 items per CU.
    int64_t shared = 8 * (kChipBlocks + n_groups) * p.read_tile;
    for (int i = 0; i < n_groups; ++i) {
      const int64_t chunks = std::min<int64_t>((W[i] + 64 * kPlanW - 1) / (64 * kPlanW),
                                               kMergeKeys / p.kp);
      shared += R[i] + std::min<int64_t>(R[i] * std::max<int64_t>(chunks, 1),
                                         kChipBlocks * 30 * p.read_tile + R[i]);
    }
    if (shared < sum) lists = list_bytes(shared, p.kp) + 256 * (size_t)n_groups;
  }
  return lists + rest;
}

// Windows that the seed pass samples for a group of `items` work items (0: none).
//
// A sample of S windows costs S scores a read, and leaves the lists that start from
// it about kp W / S keys to take in: the best S grows with the root of W and, since
// longer lists are also dearer to fill, FP16 and FP8 with kp^(3/4), FP32 with its
// root.  It is bounded by what many reads pay for it (from 10,000 reads on the best S falls
// with their number; a 300th of the windows costs 1 % at any), is a power of two
// (whole rounds of the chip for the pass), and a launch of more than 12 rounds
// takes none: later rounds start from the earlier ones' slots and the first round's
// lists cost no more than the sample.  Nor do few windows: with fewer than a list
// holds a sample bounds nothing (FP16, one window, 200 reads, 16 keys: 41 us without,
// 50 with it; 100 windows 90 and 60).  The factors are those of the least time over
// eight samples of 512 to 65,536 windows and none, 5 to 10 window counts of 1,000
// to 10^7 by 10 to 14 read counts of 1 to 100,000, in the three precisions and with
// 8, 16 and 32 keys: over 957 of these shapes 1.4 % above the best in the mean, 18 %
// at most in FP16, 30 in FP8 (1,000 reads x 42,000 windows, 32 keys), 28 in FP32 (one
// read, below 80 us), and at most 12 % above the larger sample below, which is 2.1
// times the best elsewhere.  FP16, 16 keys: without a sample / with
// this one / with at least 8,192 windows and a 64th of them:
//   200 reads x 20,000 windows     318     71     84 us
//   1,000 x 300,000                571    432    431 us
//   20,000 x 20,000                958    878  1,165 us
//   100,000 x 5,000              1,726  1,625  2,680 us
// FP32 scores cost eight times as much against the same lists: 200 x 20,000 288,
// 149 and 159 us; 20,000 x 5,000 1,238 us without, as here, and 2,311 with 8,192.
//
// Groups share the chip's rounds, which leaves more of their lists cold: a 16th of
// the windows and 8,192 at least (seven groups of 5,000 reads in all, FP8, a
// reference of 10^7 letters: 11.7 ms without, 7.0 with a single launch's sample,
// 5.5 with twice that and with the 16th; of 10^6 letters 3.96, 1.33, 1.29 and 1.22).
static int64_t seed_windows(int precision, int kp, int64_t W, int64_t R, bool grouped,
                            int64_t items) {
  if (kp > kScoreSlots || items > 12 * kChipBlocks || W <= 2 * kp) return 0;
  const bool f32 = precision == RM_FP32;
  const double w = (double)W, r = (double)R;
  if (grouped && !f32)
    return (int64_t)std::max(std::min({std::max(w / 16.0, 8192.0), 1e8 / r, 65536.0}), 512.0);
  const double factor = f32 ? (grouped ? 32.0 : 16.0) : precision == RM_FP16 ? 28.0 : 40.0;
  const double lists = kp / 16.0;
  double S = std::max(factor * std::sqrt(w) * std::pow(lists, f32 ? 0.5 : 0.75), f32 ? 0.0 : 1024.0);
  S = std::min({S, std::max((f32 ? 2.5e6 : 5e7 * lists) / r, w / 300.0), 65536.0});
  if (S < 512.0) return f32 ? 0 : 512;
  return (int64_t)1 << (int)std::log2(S);
}

hipError_t launch_score_topk(const rm_index* idx, const ScorePlan& plan,
                             const void* const* read_emb, const float* const* read_scale,
                             const int32_t* R, int k_fetch, int32_t* const* cand_idx,
                             float* const* cand_score, void* ws, hipStream_t s) {
  uint8_t* base = static_cast<uint8_t*>(ws);
  ScoreLaunch L{};
  L.n_groups = plan.n_groups;
  L.total_items = (int32_t)plan.total_items;
  L.counter = reinterpret_cast<int*>(base + plan.counter_offset);
  int32_t item = 0;
  int32_t maxR = 0;
  int32_t seed_blocks = 0;
  for (int i = 0; i < plan.n_groups; ++i) {
    const GroupPlan& gp = plan.g[i];
    ScoreGroup& G = L.g[i];
    G.index = static_cast<const uint8_t*>(idx[i].d_emb);
    G.win_scale = idx[i].d_scale;
    G.W = idx[i].n_windows;
    G.reads = static_cast<const uint8_t*>(read_emb[i]);
    G.read_scale = read_scale ? read_scale[i] : nullptr;
    G.R = R[i];
    G.read_tiles = gp.read_tiles;
    G.chunk_windows = gp.chunk_windows;
    G.P = gp.chunks;
    G.item_begin = item;
    G.thin = gp.thin;
    G.seed_begin = seed_blocks;
    const int64_t sample = seed_windows(idx[0].p.precision, plan.kp, G.W, R[i], plan.n_groups > 1,
                                        (int64_t)gp.read_tiles * gp.chunks);
    if (sample > 0) {
      const int64_t n = (std::min(G.W, sample) + kBlkW - 1) / kBlkW, tiles = ((int64_t)R[i] + 127) / 128;
      // 2 to 8 tiles per block, fewer where that fills the chip twice
      G.seed_tiles = (int)std::min<int64_t>(std::max<int64_t>(n * tiles / (2 * kChipBlocks), 2), 8);
      G.seed_segs = (int)((n + G.seed_tiles - 1) / G.seed_tiles);
      seed_blocks += G.seed_segs * (int)tiles;
    }
    G.lists = reinterpret_cast<uint64_t*>(base + gp.lists_offset);
    G.gthr = reinterpret_cast<uint32_t*>(base + gp.thr_offset);
    G.gslot = reinterpret_cast<uint64_t*>(base + gp.slot_offset);
    item += gp.read_tiles * gp.chunks;
    if (R[i] > maxR) maxR = R[i];
  }
  hipLaunchKernelGGL(clear_state, dim3((unsigned)(((int64_t)maxR + 255) / 256)), dim3(256), 0, s, L);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (seed_blocks > 0) {
    const bool red = reduced_rows(idx[0].p);
    e = idx[0].p.precision == RM_FP32   ? launch_seed<RM_FP32>(red, seed_blocks, L, s)
        : idx[0].p.precision == RM_FP16 ? launch_seed<RM_FP16>(red, seed_blocks, L, s)
                                        : launch_seed<RM_FP8_E4M3>(red, seed_blocks, L, s);
    if (e != hipSuccess) return e;
  }
  e = dispatch(idx[0].p.precision, reduced_rows(idx[0].p), plan.read_tile, plan.kp, L, s);
  if (e != hipSuccess) return e;
  for (int i = 0; i < plan.n_groups; ++i) {
    int n_per_read = plan.g[i].chunks * plan.kp;
    const uint64_t* lists = reinterpret_cast<const uint64_t*>(base + plan.g[i].lists_offset);
    if (n_per_read > kMergeKeys) {  // at most kMergeKeysWide (plan_score)
      auto wide = n_per_read <= kMergeKeysWide / 4 ? merge_block_kernel<4> : merge_block_kernel<16>;
      hipLaunchKernelGGL(wide, dim3((unsigned)R[i]), dim3(64 * kMergeWaves), 0, s, lists, n_per_read,
                         k_fetch, cand_idx[i], cand_score[i]);
      e = hipGetLastError();
      if (e != hipSuccess) return e;
      continue;
    }
    unsigned blocks = (unsigned)(((int64_t)R[i] + 3) / 4);
    auto kern = n_per_read <= 256 ? merge_kernel<4> : n_per_read <= 512 ? merge_kernel<8>
                                                                        : merge_kernel<16>;
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(256), 0, s, lists, n_per_read, R[i], k_fetch,
                       cand_idx[i], cand_score[i]);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace rm
