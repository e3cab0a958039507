// Selection of experts from logits that arrive in hand-over slots, and the reports of a routing launch, as device functions:
// for the launches that route a layer (fused_kernels.hip) and for the estimator's (estimator_kernels.hip).
#pragma once
#include <cstddef>

#include "device_utils.h"
#include "kernels.h"
#include "launch_rules.h"

namespace moe_spec {
namespace {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / kWave;
static_assert(kWaves == kRouteWaves, "the launch rules count wavefronts");
// Development aid, compiled in with -DMOE_SPEC_STAGE_CLOCK only: workgroup 0 of token 0 notes the
// constant-rate clock (100 MHz) at the stages of the routing kernel.
#ifdef MOE_SPEC_STAGE_CLOCK
#define STAGE(i) do { if (a.stage_clock && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) a.stage_clock[i] = wall_clock64(); } while (0)
#else
#define STAGE(i) do { } while (0)
#endif

// ---------------------------------------------------------------------------------------------
// Routing

struct SelectShared {
  unsigned long long keys[kMaxExperts];   // the token's logits as order-preserving integers
  alignas(16) uint32_t high[kMaxExperts + 64];   // their high words, in parts (select_ids)
  int cnt[kWaves][kMaxExperts];           // partial rank counts of the four wavefronts, where high words are not enough
  unsigned int filled[kMaxTopK];          // candidates that count as this rank by their high words
  double top_z[kMaxTopK];
  double top_e[kWaves][kMaxTopK];         // exp(z_j - z_0), 0 beyond k; every wavefront has its own
  int top_i[kMaxTopK];
  int hits;
};
static_assert(alignof(SelectShared) % 16 == 0 && offsetof(SelectShared, high) % 16 == 0, "high is read 16 bytes at a time");

struct RouteShared {
  double red[2][kWaves];                  // one per norm
  double part[kWaves];
  SelectShared sel;
};

// Sum over the workgroup, the same value in every thread.  red[] is written before the barrier and read behind it: a
// second sum takes another array.
__device__ __forceinline__ double block_sum(double v, double *red, int lane, int wave) {
  v = wave_sum(v);
  if (lane == 0) red[wave] = v;
  __syncthreads();
  double tot = 0.0;
#pragma unroll
  for (int x = 0; x < kWaves; ++x) tot += red[x];
  return tot;
}

// Ranks by whole logits: larger logit first, equal logits by lower index.  Every wavefront holds all candidates in
// registers (element i = r*64 + lane, R per lane) and counts, for each of its candidates, how many candidates broadcast
// from source lanes [16 wave, 16 wave + 16) rank before it; the four partial counts of a candidate add up to its position.
template <int R>
__device__ void rank_whole(int E, int k, SelectShared &sel, int lane, int wave) {
  constexpr int kSrcPerWave = kWave / kWaves;
  unsigned long long key[R];
  int cnt[R];
#pragma unroll
  for (int r = 0; r < R; ++r) { key[r] = sel.keys[r * kWave + lane]; cnt[r] = 0; }
  for (int j = wave * kSrcPerWave; j < (wave + 1) * kSrcPerWave; ++j) {
    const bool after = lane > j;                 // same register: the source has the lower index
#pragma unroll
    for (int r2 = 0; r2 < R; ++r2) {
      const unsigned long long sj = readlane(key[r2], j);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        bool before;                             // does (r2, j) rank before (r, lane)?
        if (r2 < r) before = sj >= key[r];
        else if (r2 > r) before = sj > key[r];
        else before = sj > key[r] || (after && sj == key[r]);
        cnt[r] += before ? 1 : 0;
      }
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) sel.cnt[wave][r * kWave + lane] = cnt[r];
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int i = r * kWave + lane;
      const int rk = (sel.cnt[0][i] + sel.cnt[1][i]) + (sel.cnt[2][i] + sel.cnt[3][i]);
      if (i < E && rk < k) { sel.top_z[rk] = unsortable(key[r]); sel.top_i[rk] = i; }
    }
  }
  __syncthreads();
}

// Top-k of one token's E logits, read from their slots as they arrive: larger logit first, equal logits by lower index.
// Fills sel.top_i / sel.top_z (by descending logit) and sel.top_e, the same in every workgroup that calls it.
// A chain of dependent steps of one wavefront per SIMD, so instructions count: candidates are ranked by the high words of
// their keys (sign, exponent, 20 bits), one compare instead of a 64-bit one with its ties, read from LDS as broadcasts of
// four, and the lanes that share a candidate sit in one wavefront, which needs no barrier to add them up.  If two of the
// first k have the same high word, some rank is taken twice and another not at all (or one too many is below k): then all
// wavefronts see that and rank whole keys.  64 / 128 / 256 experts: 645 / 1370 / 3015 -> 360 / 595 / 1615 ns a selection.
template <int R>
__device__ void select_ids(const RoutePairArgs &a, int stage, const unsigned long long *slots, int E, int k,
                           SelectShared &sel, int tid, int32_t *post) {
  const int lane = tid & (kWave - 1), wave = tid / kWave;
  constexpr int kParts = kWaves / R;             // lanes that share a candidate
  constexpr int kCands = kWave / kParts;         // candidates of a wavefront
  constexpr int kSrc = R * kWave / kParts;       // sources of a lane
  // thread i waits for logit i (one look at every slot per workgroup, not one per wavefront) and shares it
  // through LDS
  static_assert(kMaxExperts == kBlock, "one thread per candidate");
  unsigned long long mine = 0ull;                // padding ranks below every logit, minus infinity included
  // A logit needs more than a microsecond to get from its producer to here, so the first look comes 0.4 us after
  // this workgroup's own logits went out.  Fewer polls in flight across the device let the stores themselves get
  // through sooner: both routings 12.9 -> 11.7 us on 128 experts (8 to 25 units of 64 cycles measure alike,
  // 45 units 12.7 us).
  __builtin_amdgcn_s_sleep(16);
  if (tid < E) {
    const double zi = __longlong_as_double(static_cast<long long>(await64(slots + tid, a.spin_limit, a.status)));
    // a logit that is not a number (an empty slot after a wait that ran out) sorts as minus infinity: the
    // order stays total whatever the input, so the k ids are distinct and inside [0, E)
    mine = sortable(zi == zi ? zi : -INFINITY);
  }
  sel.keys[tid] = mine;
  if (tid < R * kWave) sel.high[tid + tid / kSrc * 4] = uint32_t(mine >> 32);    // parts 16 bytes apart: on other banks
  if (tid < kMaxTopK) sel.filled[tid] = 0u;
  if (tid == 0) sel.hits = 0;
  __syncthreads();
  STAGE(stage);
  {
    const int c = wave * kCands + lane % kCands, part = lane / kCands;
    const unsigned long long key = sel.keys[c];
    const uint32_t high = uint32_t(key >> 32);
    const uint4 *src = reinterpret_cast<const uint4 *>(sel.high + part * (kSrc + 4));
    int n[4] = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < kSrc / 4; ++j) {
      const uint4 s = src[j];
      n[0] += s.x > high ? 1 : 0;
      n[1] += s.y > high ? 1 : 0;
      n[2] += s.z > high ? 1 : 0;
      n[3] += s.w > high ? 1 : 0;
    }
    int rk = (n[0] + n[1]) + (n[2] + n[3]);
    if (kParts >= 4) rk = add_lanes_16_apart(rk);
    if (kParts >= 2) rk = add_lanes_32_apart(rk);
    if (part == 0 && rk < k) {
      sel.top_z[rk] = unsortable(key);
      sel.top_i[rk] = c;
      atomicAdd(&sel.filled[rk], 1u);
    }
  }
  __syncthreads();
  if (__ballot(lane < k && sel.filled[lane < k ? lane : 0] != 1u)) rank_whole<R>(E, k, sel, lane, wave);
  if (wave == 0 && lane < k && post) post[lane] = sel.top_i[lane];   // the host, if it waits for the ids, goes first
  if (lane < kMaxTopK) sel.top_e[wave][lane] = lane < k ? exp(sel.top_z[lane] - sel.top_z[0]) : 0.0;
}

__device__ __forceinline__ void select_ids_any(const RoutePairArgs &a, int stage, const unsigned long long *slots,
                                               int E, int k, SelectShared &sel, int tid, int32_t *post = nullptr) {
  if (E <= kWave) select_ids<1>(a, stage, slots, E, k, sel, tid, post);
  else if (E <= 2 * kWave) select_ids<2>(a, stage, slots, E, k, sel, tid, post);
  else select_ids<4>(a, stage, slots, E, k, sel, tid, post);
}

// Softmax over the k selected logits: top_e[wave] holds the numerators; returns their sum (the same in every thread).
__device__ __forceinline__ double select_gates(int k, const SelectShared &sel, int tid) {
  const double *e = sel.top_e[tid / kWave];
  double denom = 0.0;
  for (int q = 0; q < k; q += 4) denom = (((denom + e[q]) + e[q + 1]) + e[q + 2]) + e[q + 3];
  return denom;
}

// The true routing of token b, written out by the workgroup that reports it.
__device__ __forceinline__ void report_true(const RoutePairArgs &a, int b, SelectShared &sel, double denom, int tid,
                                            const SlotTable *resident) {
  const int k = a.k;
  if (tid < k) {
    const int id = sel.top_i[tid];
    const double g64 = sel.top_e[0][tid] / denom;
    const float g = static_cast<float>(g64);
    const size_t o = size_t(b) * k + tid;
    if (a.mb_true) a.mb_true->ids[o] = id;     // the host waits for every word it armed
    a.true_ids[o] = id;
    if (resident && a.slots_out) a.slots_out[o] = resident->slot[id];
    a.true_gates[o] = g;
    if (a.true_gates64) a.true_gates64[o] = g64;
    if (a.user_true_ids) a.user_true_ids[o] = id;
    if (a.user_true_gates) a.user_true_gates[o] = g;
    if (a.cmp_ids) {                           // recall@k of the prediction made one layer earlier (Sec. 3.3)
      int hit = 0;
      for (int j = 0; j < k; ++j) hit |= (a.cmp_ids[size_t(b) * k + j] == id);
      if (hit) atomicAdd(&sel.hits, 1);
    }
  }
  if (a.cmp_ids) {
    __syncthreads();
    if (tid == 0) {
      atomicAdd(&a.diag->hits, static_cast<unsigned long long>(sel.hits));
      atomicAdd(&a.diag->preds, static_cast<unsigned long long>(k));
    }
  }
}

// The prediction of token b, written out (its ids went to the host when they were selected).
__device__ __forceinline__ void report_next(const RoutePairArgs &a, int b, SelectShared &sel, double denom, int tid) {
  if (tid < a.k) {
    const int id = sel.top_i[tid];
    const float g = static_cast<float>(sel.top_e[0][tid] / denom);
    const size_t o = size_t(b) * a.k + tid;
    a.next_ids[o] = id;
    a.next_gates[o] = g;
    if (a.user_next_ids) a.user_next_ids[o] = id;
    if (a.user_next_gates) a.user_next_gates[o] = g;
  }
}

}  // namespace
}  // namespace moe_spec
