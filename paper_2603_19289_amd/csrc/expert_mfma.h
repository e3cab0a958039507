// The expert FFN of a batch on the matrix cores, as a device function: expert_kernels.hip launches it by itself,
// fused_kernels.hip beside the routing of the same layer.
#pragma once
#include "device_utils.h"
#include "kernels.h"

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
// activations from LDS for every weight chunk and are LDS-bound from a few tokens on.  A operand = 16 weight rows, B operand = up to 16 tokens routed to the expert, K walks
// the reduction dimension 64 columns per step: lane (m, g) = (lane % 16, lane / 16) loads the 32
// contiguous bytes at column k0 + 16 g of row m (so four lanes cover one 128-byte line) and
// feeds the first 8 columns to one MFMA and the next 8 to a second one; the B operand is read
// with the same column assignment, which is all that the contraction needs.
// Accumulator layout: lane holds token column lane % 16, rows 4 (lane / 16) .. +3.

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

__device__ __forceinline__ bf16x8_t load_bf16x8(const uint16_t *p, bool valid) {
  uint4 v = make_uint4(0u, 0u, 0u, 0u);
  if (valid) v = *reinterpret_cast<const uint4 *>(p);
  return __builtin_bit_cast(bf16x8_t, v);
}

// One step of the reduction for one wavefront: the weight fragments of its 16 rows and the token
// fragments of up to NT tiles, each the 2 x 16 bytes a lane feeds to two MFMAs.
template <bool GATEUP, int NT>
struct MfmaStep {
  bf16x8_t w0[2], w1[2];       // rows of W_gate (or W_down), rows of W_up
  bf16x8_t x[NT][2];
};

// GATEUP: hq[f, row] = bf16(silu(W_gate[row,:] . s_b) * (W_up[row,:] . s_b)),  act_q = s_l as bf16 [tokens, K]
// else  : y[f, row]  = W_down[row,:] . hq[f,:],                                  act_q = hq [tokens*k, K]
// The positions f = b*k + j routed to the expert come either from the [B,k] id table of a decode
// batch (B <= 64, one grid plane) or, with a.pos_list, from per-expert lists over any number of
// tokens, 64 positions per plane.  Weights are read with ordinary loads: a lane's
// two 16-byte loads of a step take alternate quarters of the same 128-byte lines, and the planes
// of an expert share its weights through the caches; streaming loads measured 8-10 % slower here.
template <bool GATEUP, int NT, int KSPLIT>
struct ExpertMfmaShared {
  int list[kMaxBatch];
  int n_list;
  // partial accumulators of the wavefronts that share a tile: [wave][token tile][gate | up][register][lane]
  float partial[KSPLIT > 1 ? kMfmaWaves : 1][NT][GATEUP ? 2 : 1][4][kWave];
};

// One workgroup: row block bx, expert by of the active list, plane bz of 64 positions.
template <bool GATEUP, int NT, int KSPLIT>
__device__ __forceinline__ void expert_mfma_body(const ExpertArgs &a, const ActiveList &act, const uint16_t *act_q,
                                                 uint16_t *hq_out, const int bx, const int by, const int bz,
                                                 ExpertMfmaShared<GATEUP, NT, KSPLIT> &sh) {
  int (&list)[kMaxBatch] = sh.list;
  auto &partial = sh.partial;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int m = lane & 15, g = lane >> 4;
  const int K = GATEUP ? a.H : a.I;            // reduction length
  const int R = GATEUP ? a.I : a.H;            // output rows

  const int e = act.expert[by];
  const uint16_t *wbase = reinterpret_cast<const uint16_t *>(a.pool + size_t(act.slot[by]) * a.slot_bytes);
  // KSPLIT wavefronts share 16 output rows: they split the reduction dimension into equal parts
  // (whole 64-column steps) and add their partial tiles in LDS.  Many short chains of dependent
  // loads that start at different columns keep HBM busier than few long ones that walk their rows
  // in step: a read-only probe of this access pattern reaches 6.2 TB/s with four wavefronts per 16
  // rows against 4.6 TB/s with one.  Short reductions are not split: the launcher picks KSPLIT.
  const int row_base = (bx * (kMfmaWaves / KSPLIT) + wave / KSPLIT) * 16;
  const int part = wave % KSPLIT;
  const bool rows_inside = row_base < R;       // a workgroup's last tiles may lie past the matrix
  const int k_part = (K + KSPLIT * 64 - 1) / (KSPLIT * 64) * 64;
  const int k_begin = part * k_part, k_end = rows_inside ? min(K, k_begin + k_part) : k_begin;
  const int my_row = min(row_base + m, R - 1);
  const uint16_t *p0 = wbase + (GATEUP ? size_t(0) : size_t(2) * a.I * a.H) + size_t(my_row) * K;
  const uint16_t *p1 = p0 + size_t(a.I) * a.H;             // W_up row (GATEUP only)

  // columns past the wavefront's part load nothing and contribute zeros, so the staged loop
  // below may run one step beyond the end
  auto fetch_w = [&](int k0, MfmaStep<GATEUP, NT> &st) {
    const int kk = k0 + 16 * g;
    const bool v0 = kk < k_end, v1 = kk + 8 < k_end;
    st.w0[0] = load_bf16x8(p0 + kk, v0);
    st.w0[1] = load_bf16x8(p0 + kk + 8, v1);
    if (GATEUP) { st.w1[0] = load_bf16x8(p1 + kk, v0); st.w1[1] = load_bf16x8(p1 + kk + 8, v1); }
  };
  MfmaStep<GATEUP, NT> even, odd;              // the loads of one step are in flight during the other's MFMAs
  // down projection with up to two token tiles: the first weights are on their way while the token list is
  // built (measured: 6 % faster there; 7 % slower in the gate/up kernel, which has twice the weight registers
  // per step, and 20 % slower with four token tiles, as in prefill)
  constexpr bool kEarlyWeights = !GATEUP && NT <= 2;
  if (kEarlyWeights) fetch_w(k_begin, even);

  int n;
  if (a.pos_list) {
    const int first = bz * kMaxBatch;
    n = min(kMaxBatch, a.pos_count[e] - first);
    if (n <= 0) return;                        // the same for the whole workgroup
    if (tid < n) list[tid] = a.pos_list[size_t(e) * a.list_stride + first + tid];
    __syncthreads();
  } else {
    gather_tokens(a.exec_ids, a.B * a.k, e, list, &sh.n_list, tid);
    n = sh.n_list;
  }
  if (n == 0) return;                          // the same for the whole workgroup
  if (KSPLIT == 1 && !rows_inside) return;     // nothing to share, nobody waits for this wavefront
  const int ntiles = (n + 15) / 16;

  const uint16_t *bp[NT];
  bool bvalid[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int idx = t * 16 + m;
    bvalid[t] = idx < n;
    const int f = bvalid[t] ? list[idx] : 0;
    bp[t] = act_q + size_t(GATEUP ? f / a.k : f) * K;
  }
  f32x4_t acc0[NT], acc1[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) { acc0[t] = f32x4_t{0.f, 0.f, 0.f, 0.f}; acc1[t] = f32x4_t{0.f, 0.f, 0.f, 0.f}; }

  auto fetch_x = [&](int k0, MfmaStep<GATEUP, NT> &st) {
    const int kk = k0 + 16 * g;
    const bool v0 = kk < k_end, v1 = kk + 8 < k_end;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (t < ntiles) {
        st.x[t][0] = load_bf16x8(bp[t] + kk, v0 && bvalid[t]);
        st.x[t][1] = load_bf16x8(bp[t] + kk + 8, v1 && bvalid[t]);
      }
    }
  };
  auto fetch = [&](int k0, MfmaStep<GATEUP, NT> &st) { fetch_w(k0, st); fetch_x(k0, st); };
  auto multiply = [&](const MfmaStep<GATEUP, NT> &st) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (t < ntiles) {
        acc0[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(st.w0[0], st.x[t][0], acc0[t], 0, 0, 0);
        acc0[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(st.w0[1], st.x[t][1], acc0[t], 0, 0, 0);
        if (GATEUP) {
          acc1[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(st.w1[0], st.x[t][0], acc1[t], 0, 0, 0);
          acc1[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(st.w1[1], st.x[t][1], acc1[t], 0, 0, 0);
        }
      }
    }
  };
  if (kEarlyWeights) fetch_x(k_begin, even);
  else fetch(k_begin, even);
  for (int k0 = k_begin; k0 < k_end; k0 += 128) {
    fetch(k0 + 64, odd);
    multiply(even);
    fetch(k0 + 128, even);
    multiply(odd);
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
      const int f = list[t * 16 + m];
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

// Wavefronts per 16-row tile by the length of the reduction: each should still walk at least eight
// 64-column steps, below that the shared start-up (token lists, partial sums) outweighs what the extra
// parallelism wins.  With a single tile of tokens there is less to start up and two steps are enough: down
// projection of about 30 experts of 2048 x 768, 4 tokens, 21.2 / 18.9 / 18.1 us with 1 / 2 / 4 wavefronts (with
// 32 tokens, two tiles, 27.5 / 28.6 / 31.7 us).
inline int mfma_ksplit(int K, int token_tiles) {
  const int steps = (K + 63) / 64;
  if (steps >= 32 || (token_tiles == 1 && steps >= 8)) return 4;
  return steps >= 16 ? 2 : 1;
}

}  // namespace moe_spec
