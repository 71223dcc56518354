// Shared pieces of the two attention-decode kernels (MSD over the INT8 cache, attn.hip; the
// dequantise-then-BF16 comparison kernel, attn_dequant.hip): launch parameters, the flash-decode
// split plan, the 16-lane row reductions and the partial-result merge.
#pragma once
#include "kernels.hpp"

namespace msd {

struct AttnParams {
  const uint16_t* q;
  const int8_t* K;
  const int8_t* V;
  const float* k_scale;
  const float* v_scale;
  const int32_t* kv_len;
  int B, Hq, Hkv, G;
  int64_t L;
  int nsplit;
  int64_t tokens_per_split;
  int balanced;   // the splits follow the lengths (balanced_splits) instead of L / nsplit
  float* part_o;  // [B*Hkv][nsplit][G][128]
  float* part_m;  // [B*Hkv][nsplit][G]
  float* part_l;
  int32_t* part_of;  // balanced splits: first slot and slot count of every entry, [B][2]
  void* out;
  int out_bf16;
  int8_t* tap_q1;
  int8_t* tap_q2;
  float* tap_alpha;
  int32_t* tap_s1;
  int32_t* tap_s2;
  int8_t* tap_p1;  // codes of the decomposed softmax numerator [B][Hq][L] (nullable pair)
  int8_t* tap_p2;
};

constexpr int kD = 128;
constexpr int kTile = 64;
constexpr int kAttnWaves = 4;
constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ v4i mfma_s8(v4i a, v4i b, v4i c) {
  return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
}

// All-reduce over the 16 lanes sharing lane/16 (one DPP row): four rotate-and-combine steps.
__device__ __forceinline__ float row16_max(float v) {
  v = fmaxf(v, row16_ror<8>(v));
  v = fmaxf(v, row16_ror<4>(v));
  v = fmaxf(v, row16_ror<2>(v));
  return fmaxf(v, row16_ror<1>(v));
}
__device__ __forceinline__ float row16_sum(float v) {
  v += row16_ror<8>(v);
  v += row16_ror<4>(v);
  v += row16_ror<2>(v);
  return v + row16_ror<1>(v);
}

// 4x4 byte transpose: in[t] = 4 channel bytes of token t; out[c] = 4 token bytes of channel c
__device__ __forceinline__ void transpose4x4(uint32_t a, uint32_t b, uint32_t c, uint32_t d,
                                             uint32_t (&o)[4]) {
  const uint32_t ab_lo = __builtin_amdgcn_perm(b, a, 0x05010400u);
  const uint32_t ab_hi = __builtin_amdgcn_perm(b, a, 0x07030602u);
  const uint32_t cd_lo = __builtin_amdgcn_perm(d, c, 0x05010400u);
  const uint32_t cd_hi = __builtin_amdgcn_perm(d, c, 0x07030602u);
  o[0] = __builtin_amdgcn_perm(cd_lo, ab_lo, 0x05040100u);
  o[1] = __builtin_amdgcn_perm(cd_lo, ab_lo, 0x07060302u);
  o[2] = __builtin_amdgcn_perm(cd_hi, ab_hi, 0x05040100u);
  o[3] = __builtin_amdgcn_perm(cd_hi, ab_hi, 0x07060302u);
}

// KV splits per (batch, KV head) of the comparison kernel: about two workgroups per CU, at least two rounds of the
// four waves per split
inline int attn_dequant_plan_nsplit(int B, int Hkv, int64_t L) {
  const int64_t pairs = (int64_t)B * Hkv;
  int64_t ns = cdiv(512, pairs);
  int64_t max_by_len = L / (kAttnWaves * kTile * 2);
  if (max_by_len < 1) max_by_len = 1;
  if (ns > max_by_len) ns = max_by_len;
  if (ns > 64) ns = 64;
  if (ns < 1) ns = 1;
  return (int)ns;
}

// KV splits of a call, by what a split costs.  `pairs` workgroups per split run on 256 CUs; a CU takes
// ceil(workgroups / 256) of them one after the other or, up to `resident`, side by side, which takes as long (either
// way it streams their tokens at its rate); each takes a prologue and an epilogue, shared while they are resident
// together; and more than one split means a merge launch.  So the number of workgroups should be a little below a
// multiple of 256, and a split is worth its merge only from a few hundred tokens on.  `round` tokens (one tile of
// every wave or token stream) take round_ns.
constexpr int kCus = 256;
constexpr int kMaxParts = 64;
struct SplitCost {
  int round;           // tokens per round
  int64_t round_ns;    // one round
  int resident;        // workgroups per CU
  int64_t wg_ns;       // prologue and epilogue of the workgroups resident together ...
  int64_t overlap_ns;  // ... less what two of them hide of each other's
  int64_t merge_ns;    // the merge launch ...
  int64_t part_ns;     // ... and what one more partial result per row adds
};
inline int plan_nsplit(int64_t pairs, int64_t L, const SplitCost& c) {
  int best = 1;
  int64_t best_ns = INT64_MAX;
  for (int ns = 1; ns <= kMaxParts && (ns == 1 || (int64_t)(ns - 1) * c.round < L); ++ns) {
    const int64_t gens = cdiv(pairs * ns, kCus), rounds = cdiv(cdiv(L > 0 ? L : 1, ns), c.round);
    const int64_t t = gens * rounds * c.round_ns + cdiv(gens, c.resident) * (c.wg_ns - (gens > 1 ? c.overlap_ns : 0)) +
                      (ns > 1 ? c.merge_ns + ns * c.part_ns : 0);
    if (t < best_ns) best_ns = t, best = ns;
  }
  return best;
}
// The grouped-query kernel.  Up to 8 heads per KV head: two workgroups per CU and 2.5 us per round of 256 tokens
// (10 ns per token: the stream); beyond, one workgroup per CU and 5 us per fragment of 8 heads (the vector ALU).
// The merge launch is 4 to 5 us.  Measured against about 512 workgroups and at least
// 512 tokens per split whatever the batch (us): 5 x 8 KV heads x 1079 tokens 13.9 -> 9.8, 1 x 8 x 32768 38.6 -> 20.6,
// 32 x 8 x 3000 with 12 heads each 62.8 -> 51.9, 13 x 1 x 17679 with 12 heads 52.1 -> 24.3; 16 x 8 x 4096 unchanged (28.5).
inline int attn_plan_nsplit(int B, int Hkv, int G, int64_t L) {
  const int frags = G <= 8 ? 1 : (G + 7) / 8;
  const SplitCost c = {kAttnWaves * kTile, frags == 1 ? 2500 : 2500 * frags, frags == 1 ? 2 : 1, frags == 1 ? 4000 : 8000, frags == 1 ? 2000 : 0, 5000, 20};
  return plan_nsplit((int64_t)B * Hkv, L, c);
}

// ---- splits that follow the lengths of a ragged batch.  Splits sized by the capacity L leave the workgroups of
// short contexts idle while those of the longest ones set the time of the call; here the same number of
// workgroups shares the tiles that exist: entry b gets n_b = clamp(ceil(tiles_b / u), 1, kMaxParts) consecutive
// slots, u being the smallest split size (in tiles) with sum n_b <= slots.  Every wave of every workgroup finds u by
// itself from the lengths (one lane per entry, a binary search of a few steps: about a microsecond) and the first
// split of an entry leaves its slots in the workspace for the merge kernel.  Measured (us, splits of L -> balanced): 16
// entries of 2048..4096 tokens, 8 KV heads 27.5 -> 25.9.
constexpr int kBalancedMaxB = 64;  // one lane per entry; larger batches average out over their entries

__device__ __forceinline__ int wave_sum_int(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x128, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x124, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x122, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x121, 0xF, 0xF, false);
  return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) + __builtin_amdgcn_readlane(v, 32) +
         __builtin_amdgcn_readlane(v, 48);
}

struct BalancedSplits {  // lane b: entry b (nothing beyond B)
  int len, tiles, n, start;
};
// slots > B; unit = tokens per tile.  All 64 lanes take part.
__device__ __forceinline__ BalancedSplits balanced_splits(const int32_t* kv_len, int64_t L, int B, int slots, int unit,
                                                          int lane) {
  BalancedSplits r;
  const bool have = lane < B;
  r.len = have ? (int)max((int64_t)0, min((int64_t)kv_len[min(lane, B - 1)], L)) : 0;
  r.tiles = (int)(((uint32_t)r.len + unit - 1) / (uint32_t)unit);
  const uint32_t total = (uint32_t)wave_sum_int(r.tiles);
  auto parts = [&](uint32_t u) { return have ? (int)min(max(((uint32_t)r.tiles + u - 1) / u, 1u), (uint32_t)kMaxParts) : 0; };
  uint32_t lo = max(1u, (total + slots - 1) / (uint32_t)slots);
  uint32_t hi = max(lo, (total + (slots - B) - 1) / (uint32_t)(slots - B));  // n_b <= tiles_b / u + 1: always enough
  while (lo < hi) {
    const uint32_t mid = (lo + hi) / 2;
    if (wave_sum_int(parts(mid)) <= slots) hi = mid;
    else lo = mid + 1;
  }
  r.n = parts(lo);
  int x = r.n;  // inclusive prefix sum over the lanes
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);
  const int r0 = __builtin_amdgcn_readlane(x, 15), r1 = __builtin_amdgcn_readlane(x, 31), r2 = __builtin_amdgcn_readlane(x, 47);
  x += (lane >= 16 ? r0 : 0) + (lane >= 32 ? r1 : 0) + (lane >= 48 ? r2 : 0);
  r.start = x - r.n;
  return r;
}
// The entry whose slots hold `slot`, its split number and its token range [t_begin, t_end); false: an unused slot.
__device__ __forceinline__ bool balanced_slot(const BalancedSplits& s, int B, int slot, int unit, int lane, int& b,
                                              int& split, int64_t& t_begin, int64_t& t_end) {
  const unsigned long long at = __ballot(lane < B && s.start <= slot);
  b = 63 - __builtin_clzll(at);
  split = slot - __builtin_amdgcn_readlane(s.start, b);
  const int n = __builtin_amdgcn_readlane(s.n, b);
  if (split >= n) return false;
  const uint32_t tiles = (uint32_t)__builtin_amdgcn_readlane(s.tiles, b);
  t_begin = (int64_t)(uint32_t)(tiles * (uint32_t)split / (uint32_t)n) * unit;
  t_end = min((int64_t)__builtin_amdgcn_readlane(s.len, b),
              (int64_t)(uint32_t)(tiles * (uint32_t)(split + 1) / (uint32_t)n) * unit);
  return true;
}

// fills the split plan, the partial-result pointers inside the workspace and the output fields of p
void attn_fill_params(const AttnArgs& a, int nsplit, AttnParams& p);
// launches the kernel instances for more than 8 query heads per KV head (attn_wide.hip)
int launch_attn_wide(const AttnParams& p, dim3 grid, bool per_token, bool lowprec, hipStream_t stream);
// merges the split partials into p.out (attn.hip); call only when p.nsplit > 1
int launch_attn_combine(const AttnParams& p, int per_channel, hipStream_t stream);

}  // namespace msd
