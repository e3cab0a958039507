// The expert FFN of a batch on the matrix cores, as a device function: expert_kernels.hip launches it by itself,
// fused_kernels.hip beside the routing of the same layer.
#pragma once
#include <type_traits>

#include "device_utils.h"
#include "kernels.h"
#include "launch_rules.h"

namespace moe_spec {

constexpr int kMfmaBlock = 256;
constexpr int kMfmaWaves = kMfmaBlock / kWave;

// Positions f = b*k + j of the id table that name expert e, in ascending order, by wavefront 0.
// All of the table's words a lane looks at are requested before the first is examined, so the
// scan costs one memory latency whatever the size of the table (at most 64 x 16 ids).
__device__ __forceinline__ void gather_tokens(const int32_t *ids, int n_ids, int e, int *list,
                                              int *n_list, int tid) {
  constexpr int kPerLane = kMaxBatch * kMaxTopK / kWave;
  if (tid < kWave) {
    int v[kPerLane];
#pragma unroll
    for (int i = 0; i < kPerLane; ++i) {
      const int f = i * kWave + tid;
      v[i] = f < n_ids ? ids[f] : -1;
    }
    int count = 0;
#pragma unroll
    for (int i = 0; i < kPerLane; ++i) {
      if (i * kWave < n_ids) {                 // uniform over the wavefront
        const bool match = v[i] == e;
        const unsigned long long mask = __ballot(match);
        if (match) list[count + __popcll(mask & ((1ull << tid) - 1ull))] = i * kWave + tid;
        count += __popcll(mask);
      }
    }
    if (tid == 0) *n_list = count;
  }
  __syncthreads();
}

// Matrix-core kernels for decode batches of two and more (bf16 weights) and for prefill: the
// expert FFN as 16x16x32 bf16 MFMA tiles.  The launches stay HBM-bound, but one weight fragment
// meets up to 16 tokens per instruction, where the general kernels above fetch every token's
// activations from LDS for every weight chunk and are LDS-bound from a few tokens on.
// A operand = 16 weight rows, B operand = up to 16 tokens routed to the expert; K walks the reduction 128 columns per
// step.  HBM decides how the weights are read: a load that takes 64 bytes of each of 16 rows, as the operand wants them,
// streams at 5.5 to 5.8 TB/s however it is split (read-only kernel, 700 and 300 MB), one that takes 256 bytes of each of
// four rows at 6.6 to 6.8, past the caches.  So lane (r, p) = (lane % 4, lane / 4) loads one chunk of 16 bytes of rows
// r, 4 + r, 8 + r and 12 + r, and the four registers are turned in place (rows_to_lanes) until lane (m, g) =
// (lane % 16, lane / 16) holds what lanes p = 4 g .. 4 g + 3 loaded of row m: 48 moves for 4 KB, a seventh of the time
// these take to arrive.  Place p takes the chunk at column chunk_column(p), so that a row's sum adds 64 columns after 64
// columns, the even chunks of each 64 and then the odd ones, however wide a step is.  The B operand is read with the same
// column assignment.
// Gate/up and down of 21 experts of 2880 x 2880, 12 positions of each most: 117.5 -> 101.5 us (6.9 TB/s) and
// 64.4 -> 54.0; 48 experts of 768 x 2048, 32 tokens: 56.0 -> 47.7 and 31.1 -> 28.2; 8 of 14336 x 4096, 64 tokens: 349 ->
// 352 and 232 -> 201.
// Accumulator layout: lane holds token column lane % 16, rows 4 (lane / 16) .. +3.

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

__device__ __forceinline__ bf16x8_t load_bf16x8(const uint16_t *p, bool valid) {
  uint4 v = make_uint4(0u, 0u, 0u, 0u);
  if (valid) v = *reinterpret_cast<const uint4 *>(p);
  return __builtin_bit_cast(bf16x8_t, v);
}

// One step of the reduction for one wavefront, 128 columns: 16 weight rows in four loads, tokens of up to NT tiles.
template <bool GATEUP, int NT>
struct MfmaStep {
  uint4 w0[4], w1[4];          // rows of W_gate (or W_down), rows of W_up
  bf16x8_t x[NT][4];
};

// Lane bit (SHIFT / 4's bit 2 or 3) against the choice between two registers: afterwards a holds what both registers
// had in the lanes with the bit clear, b what they had in the others.
template <int SHIFT, int HIGH, int LOW>
__device__ __forceinline__ void swap_lanes(uint32_t &a, uint32_t &b) {
  const uint32_t from_a = a;
  a = __builtin_amdgcn_update_dpp(a, b, 0x110 + SHIFT, 0xf, HIGH, false);          // row_shr
  b = __builtin_amdgcn_update_dpp(b, from_a, 0x100 + SHIFT, 0xf, LOW, false);      // row_shl
}

// w[i], lane (r, p) = (lane % 4, lane / 4): chunk p of row 4 i + r  ->  w[s], lane (m, g): chunk 4 g + s of row m.
__device__ __forceinline__ void rows_to_lanes(uint4 (&w)[4]) {
#define MOE_SWAP(f)                                                              \
  swap_lanes<4, 0xa, 0x5>(w[0].f, w[1].f); swap_lanes<4, 0xa, 0x5>(w[2].f, w[3].f); \
  swap_lanes<8, 0xc, 0x3>(w[0].f, w[2].f); swap_lanes<8, 0xc, 0x3>(w[1].f, w[3].f);
  MOE_SWAP(x) MOE_SWAP(y) MOE_SWAP(z) MOE_SWAP(w)
#undef MOE_SWAP
}

// Column, within a step of 128, of the chunk of 8 at place p = 0 .. 15: lane group g gets chunks 2 g and 2 g + 1 of the
// first 64 columns, then of the second.
__device__ __forceinline__ int chunk_column(int p) { return 16 * (p >> 2) + 64 * ((p >> 1) & 1) + 8 * (p & 1); }

template <bool STREAM>
__device__ __forceinline__ uint4 load_weights(const char *p) {
  return STREAM ? load_stream<uint4>(p) : *reinterpret_cast<const uint4 *>(p);
}

// GATEUP: hq[f, row] = bf16(silu(W_gate[row,:] . s_b) * (W_up[row,:] . s_b)),  act_q = s_l as bf16 [tokens, K]
// else  : y[f, row]  = W_down[row,:] . hq[f,:],                                  act_q = hq [tokens*k, K]
template <bool GATEUP, int NT, int KSPLIT>
struct ExpertMfmaShared {
  int list[kMaxBatch];         // prefill
  // partial accumulators of the wavefronts that share a tile: [wave][token tile][gate | up][register][lane]
  float partial[KSPLIT > 1 ? kMfmaWaves : 1][NT][GATEUP ? 2 : 1][4][kWave];
};

// The positions f = b*k + j routed to an expert: in a decode batch from the host's lists (no search, so the first
// weights are on their way at once), in prefill from
// per-expert lists on the device over any number of tokens, 64 positions per grid plane.
// STREAM: weights, read once, bypass the caches (nontemporal).  Not where two steps share a line of a row, and not in
// prefill, where the planes of an expert share its weights through the caches.
template <bool STREAM>
struct DecodeTokens {
  const TokenLists &lists;
  int by;
  static constexpr bool kStream = STREAM, kEarly = true;
  __device__ __forceinline__ int slot() const { return int(lists.expert[by] >> 16); }
  __device__ __forceinline__ int count(const ExpertArgs &, int *, int) const {
    return int(lists.expert[by + 1] & 0xffff) - int(lists.expert[by] & 0xffff);
  }
  __device__ __forceinline__ int position(const int *, int i) const { return lists.pos[(lists.expert[by] & 0xffff) + i]; }
  __device__ __forceinline__ static int f_of(int p) { return p & 1023; }
  __device__ __forceinline__ static int token_of(int p, int) { return p >> 10; }
};
struct PrefillTokens {
  const ActiveList &act;
  int by, bz;
  static constexpr bool kStream = false, kEarly = false;
  __device__ __forceinline__ int slot() const { return act.slot[by]; }
  __device__ __forceinline__ int count(const ExpertArgs &a, int *list, int tid) const {
    const int e = act.expert[by], first = bz * kMaxBatch;
    const int n = min(kMaxBatch, a.pos_count[e] - first);
    if (n > 0) {                               // the same for the whole workgroup
      if (tid < n) list[tid] = a.pos_list[size_t(e) * a.list_stride + first + tid];
      __syncthreads();
    }
    return n;
  }
  __device__ __forceinline__ int position(const int *list, int i) const { return list[i]; }
  __device__ __forceinline__ static int f_of(int p) { return p; }
  __device__ __forceinline__ static int token_of(int p, int k) { return p / k; }
};

// How a wavefront sums its part of a row: in one chain, in two (of every 64 columns alternately), or, where it has the whole
// row, in a chain for each of four equal parts: the sum that four wavefronts come to.
constexpr int kOneChain = 1, kTwoChains = 2, kFourParts = 4;

// One workgroup: row block bx of the expert that tok names.
template <bool GATEUP, int NT, int KSPLIT, int CHAINS, typename Tokens>
__device__ __forceinline__ void expert_mfma_body(const ExpertArgs &a, const Tokens &tok, const uint16_t *act_q,
                                                 uint16_t *hq_out, const int bx,
                                                 ExpertMfmaShared<GATEUP, NT, KSPLIT> &sh) {
  auto &partial = sh.partial;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int m = lane & 15, g = lane >> 4;
  const int K = GATEUP ? a.H : a.I;            // reduction length
  const int R = GATEUP ? a.I : a.H;            // output rows

  const uint16_t *wbase = reinterpret_cast<const uint16_t *>(a.pool + size_t(tok.slot()) * a.slot_bytes);
  static_assert(CHAINS == kOneChain || !GATEUP, "the second accumulator is W_up's");
  static_assert(CHAINS != kFourParts || KSPLIT == 1, "four parts of the whole row");
  // KSPLIT wavefronts share 16 output rows: they split the reduction dimension into equal parts
  // (of whole 64 columns) and add their partial tiles in LDS: many short chains of dependent loads
  // keep HBM busier than few long ones.  Short reductions are not split: the launcher picks KSPLIT.
  const int row_base = (bx * (kMfmaWaves / KSPLIT) + wave / KSPLIT) * 16;
  const int part = wave % KSPLIT;
  const bool rows_inside = row_base < R;       // a workgroup's last tiles may lie past the matrix
  constexpr int kParts = CHAINS == kFourParts ? 4 : KSPLIT;
  const int k_part = (K + kParts * 64 - 1) / (kParts * 64) * 64;
  const int k_begin = part * k_part, k_end = rows_inside ? min(K, k_begin + kParts / KSPLIT * k_part) : k_begin;
  // base and column in scalar registers, a lane's rows as byte offsets (an expert block is smaller than 4 GB)
  const char *p0 = reinterpret_cast<const char *>(wbase + (GATEUP ? size_t(0) : size_t(2) * a.I * a.H));
  const char *p1 = p0 + size_t(2) * a.I * a.H;             // W_up (GATEUP only)
  const int w_col = chunk_column(lane >> 2), x_col = chunk_column(4 * g);
  uint32_t woff[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) woff[i] = (uint32_t(min(row_base + 4 * i + (lane & 3), R - 1)) * uint32_t(K) + w_col) * 2;

  // columns past the wavefront's part load nothing and contribute zeros, so the staged loop
  // below may run one step beyond the end
  auto fetch_w = [&](int k0, MfmaStep<GATEUP, NT> &st) {
#pragma unroll
    for (int i = 0; i < 4; ++i) { st.w0[i] = make_uint4(0u, 0u, 0u, 0u); if (GATEUP) st.w1[i] = make_uint4(0u, 0u, 0u, 0u); }
    if (k0 + w_col < k_end) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        st.w0[i] = load_weights<Tokens::kStream>(p0 + size_t(k0) * 2 + woff[i]);
        if (GATEUP) st.w1[i] = load_weights<Tokens::kStream>(p1 + size_t(k0) * 2 + woff[i]);
      }
    }
  };
  MfmaStep<GATEUP, NT> even, odd;              // the loads of one step are in flight during the other's MFMAs
  constexpr bool kEarlyWeights = Tokens::kEarly || (!GATEUP && NT <= 2);
  if (kEarlyWeights) fetch_w(k_begin, even);

  const int n = tok.count(a, sh.list, tid);
  if (n <= 0) return;                          // the same for the whole workgroup
  if (KSPLIT == 1 && !rows_inside) return;     // nothing to share, nobody waits for this wavefront
  const int ntiles = (n + 15) / 16;

  const uint16_t *bp[NT];
  bool bvalid[NT];
  int fpos[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int idx = t * 16 + m;
    bvalid[t] = idx < n;
    const int p = bvalid[t] ? tok.position(sh.list, idx) : 0;
    fpos[t] = Tokens::f_of(p);
    bp[t] = act_q + size_t(GATEUP ? Tokens::token_of(p, a.k) : fpos[t]) * K;
  }
  f32x4_t acc0[NT], acc1[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc0[t] = acc1[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  int chain_end = k_part;                      // kFourParts: acc1 is the sum of the chains that have ended

  auto fetch_x = [&](int k0, MfmaStep<GATEUP, NT> &st) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (t < ntiles) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int col = k0 + x_col + chunk_column(c);
          st.x[t][c] = load_bf16x8(bp[t] + col, col < k_end && bvalid[t]);
        }
      }
    }
  };
  auto multiply = [&](int k0, MfmaStep<GATEUP, NT> &st) {
    rows_to_lanes(st.w0);
    if (GATEUP) rows_to_lanes(st.w1);
#pragma unroll
    for (int half = 0; half < 2; ++half) {                 // 64 columns each
      if (CHAINS == kFourParts && k0 + 64 * half == chain_end) {
        chain_end += k_part;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          acc1[t] += acc0[t];
          acc0[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (t < ntiles) {
#pragma unroll
          for (int c = 2 * half; c < 2 * half + 2; ++c) {
            f32x4_t &acc = CHAINS == kTwoChains && half == 1 ? acc1[t] : acc0[t];
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, st.w0[c]), st.x[t][c], acc, 0, 0, 0);
            if (GATEUP)
              acc1[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, st.w1[c]), st.x[t][c], acc1[t], 0, 0, 0);
          }
        }
      }
    }
  };
  if (!kEarlyWeights) fetch_w(k_begin, even);
  for (int k0 = k_begin; k0 < k_end; k0 += 256) {
    fetch_x(k0, even);
    fetch_w(k0 + 128, odd);
    multiply(k0, even);
    fetch_x(k0 + 128, odd);
    fetch_w(k0 + 256, even);
    multiply(k0 + 128, odd);
  }

  if (CHAINS != kOneChain) {
#pragma unroll
    for (int t = 0; t < NT; ++t) acc0[t] = acc1[t] + acc0[t];
  }
  if (KSPLIT > 1) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (t < ntiles) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          partial[wave][t][0][i][lane] = acc0[t][i];
          if (GATEUP) partial[wave][t][GATEUP ? 1 : 0][i][lane] = acc1[t][i];
        }
      }
    }
    __syncthreads();
  }

  // Of the wavefronts that share a tile, number p finishes token tiles p, p + KSPLIT, ...  The
  // accumulator layout is as the MFMA left it: lane = token column lane % 16, rows 4 (lane / 16) .. + 3.
  const int r0 = row_base + 4 * g;             // this lane's four output rows, all inside or all outside
  if (r0 >= R) return;
  const int w0 = wave - part;                  // first of the wavefronts that share this tile
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    if (t % KSPLIT == part && t < ntiles && bvalid[t]) {
      float s0[4], s1[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (KSPLIT == 1) {
          s0[i] = acc0[t][i];
          s1[i] = acc1[t][i];
        } else {
          s0[i] = 0.f;
          s1[i] = 0.f;
#pragma unroll
          for (int p = 0; p < KSPLIT; ++p) {
            s0[i] += partial[w0 + p][t][0][i][lane];
            if (GATEUP) s1[i] += partial[w0 + p][t][GATEUP ? 1 : 0][i][lane];
          }
        }
      }
      const int f = fpos[t];
      if (GATEUP) {
        uint16_t q[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float hv = round_to_bf16(s0[i] / (1.f + expf(-s0[i])) * s1[i]);
          q[i] = uint16_t(__float_as_uint(hv) >> 16);
        }
        uint2 packed;
        packed.x = uint32_t(q[0]) | (uint32_t(q[1]) << 16);
        packed.y = uint32_t(q[2]) | (uint32_t(q[3]) << 16);
        *reinterpret_cast<uint2 *>(hq_out + size_t(f) * R + r0) = packed;
      } else {
        *reinterpret_cast<float4 *>(a.y + size_t(f) * R + r0) = make_float4(s0[0], s0[1], s0[2], s0[3]);
      }
    }
  }
}

template <int V> using int_c = std::integral_constant<int, V>;

// Calls f with the wavefronts per 16-row tile as a constant.
template <typename F>
hipError_t with_ksplit(int ksplit, F f) {
  if (ksplit == 4) return f(int_c<4>());
  if (ksplit == 2) return f(int_c<2>());
  return f(int_c<1>());
}

// Decode batches: tiles of 16 positions of the expert that has most (1, 2 or 4), and whether two steps of a row never
// share a line, so that the weights may bypass the caches.
inline int decode_tiles(int most) { return most <= 16 ? 1 : most <= 32 ? 2 : 4; }
inline bool whole_lines(int K) { return K % 64 == 0; }

// Calls f with the tiles, wavefronts per tile and chains of the down projection of a decode batch, as constants.
template <typename F>
hipError_t with_down_form(const ExpertArgs &a, const TokenLists &lists, int cus, F f) {
  const int tiles = (a.B + 15) / 16, positions = int(lists.expert[lists.n] & 0xffff);
  auto of_tiles = [&](auto nt) {
    return with_ksplit(down_ksplit(a.I, tiles, a.H, lists.n, positions, cus), [&](auto ksplit) {
      if constexpr (ksplit() == 1)
        if (a.I >= 1024) return f(nt, ksplit, int_c<kFourParts>());
      if constexpr (ksplit() == 2 && nt() == 1)
        if (tiles == 1) return f(nt, ksplit, int_c<kTwoChains>());
      return f(nt, ksplit, int_c<kOneChain>());
    });
  };
  switch (decode_tiles(lists.most)) {
    case 1: return of_tiles(int_c<1>());
    case 2: return of_tiles(int_c<2>());
    default: return of_tiles(int_c<4>());
  }
}

}  // namespace moe_spec
