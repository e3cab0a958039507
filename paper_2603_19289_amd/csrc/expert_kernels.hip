// Expert kernels: SwiGLU expert GEMVs gathered over the device cache slots of one layer, and
// the gate-weighted combine (paper: Algorithm 1, O <- MoE_l(X, ids, g, C_l); Sec. 4 for which ids
// and gates are executed).
//
// A launch covers the experts of one cache wave.  blockIdx.y picks the expert, blockIdx.x a
// block of output rows.  Each workgroup finds the tokens routed to its expert by scanning the
// [B,k] id table, stages their activation vectors in LDS, and each wavefront streams whole
// weight rows with 16-byte loads per lane, reducing across the 64 lanes with shuffles.
// Weights are read once per token tile; at batch 1 that is exactly once.
#include "device_utils.h"
#include "expert_mfma.h"
#include "gateup_b1.h"
#include "kernels.h"
#include "launch_rules.h"

namespace moe_spec {
namespace {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / kWave;

// h[f, row] = silu(W_gate[row,:] . s_b) * (W_up[row,:] . s_b) for every position f routed to the expert.
template <typename WT, int TT>
__global__ __launch_bounds__(kBlock) void gateup_kernel(const ExpertArgs a, const ActiveList act,
                                                        const int rpw) {
  extern __shared__ float act_rows[];          // [TT][H]
  __shared__ int list[kMaxBatch];
  __shared__ int n_list;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int H = a.H, I = a.I;
  constexpr int VN = Packed<WT>::N;

  const int e = act.expert[blockIdx.y];
  const WT *wg = reinterpret_cast<const WT *>(a.pool + size_t(act.slot[blockIdx.y]) * a.slot_bytes);
  const WT *wu = wg + size_t(I) * H;
  gather_tokens(a.exec_ids, a.B * a.k, e, list, &n_list, tid);
  const int n = n_list;
  const int row0 = (blockIdx.x * kWaves + wave) * rpw;

  for (int t0 = 0; t0 < n; t0 += TT) {
    const int nt = min(TT, n - t0);
    for (int t = 0; t < nt; ++t) {
      const float *src = a.s + size_t(list[t0 + t] / a.k) * H;
      for (int i = tid * 4; i < H; i += kBlock * 4)
        *reinterpret_cast<float4 *>(act_rows + size_t(t) * H + i) = *reinterpret_cast<const float4 *>(src + i);
    }
    __syncthreads();
    for (int rr = 0; rr < rpw; ++rr) {
      const int row = row0 + rr;
      if (row >= I) break;
      float ag[TT], au[TT];
#pragma unroll
      for (int t = 0; t < TT; ++t) { ag[t] = 0.f; au[t] = 0.f; }
      const WT *pg = wg + size_t(row) * H;
      const WT *pu = wu + size_t(row) * H;
#pragma unroll 4
      for (int c = lane * VN; c < H; c += kWave * VN) {
        float fg[VN], fu[VN];
        Packed<WT>::unpack(load_stream<typename Packed<WT>::Raw>(pg + c), fg);
        Packed<WT>::unpack(load_stream<typename Packed<WT>::Raw>(pu + c), fu);
#pragma unroll
        for (int t = 0; t < TT; ++t) {
          if (t < nt) {
            const float *sv = act_rows + size_t(t) * H + c;
#pragma unroll
            for (int x = 0; x < VN; ++x) { ag[t] += fg[x] * sv[x]; au[t] += fu[x] * sv[x]; }
          }
        }
      }
#pragma unroll
      for (int t = 0; t < TT; ++t) {
        if (t < nt) {
          const float g = wave_sum(ag[t]);
          const float u = wave_sum(au[t]);
          if (lane == 0) {
            float hv = g / (1.f + expf(-g)) * u;
            if (a.bf16) hv = round_to_bf16(hv);
            a.h[size_t(list[t0 + t]) * I + row] = hv;
          }
        }
      }
    }
    __syncthreads();
  }
}

// y[f, row] = W_down[row,:] . h[f,:] for every position f routed to the expert.
template <typename WT, int TT>
__global__ __launch_bounds__(kBlock) void down_kernel(const ExpertArgs a, const ActiveList act,
                                                      const int rpw) {
  extern __shared__ float act_rows[];          // [TT][I]
  __shared__ int list[kMaxBatch];
  __shared__ int n_list;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int H = a.H, I = a.I;
  constexpr int VN = Packed<WT>::N;

  const int e = act.expert[blockIdx.y];
  const WT *wd = reinterpret_cast<const WT *>(a.pool + size_t(act.slot[blockIdx.y]) * a.slot_bytes) +
                 size_t(2) * I * H;
  gather_tokens(a.exec_ids, a.B * a.k, e, list, &n_list, tid);
  const int n = n_list;
  const int row0 = (blockIdx.x * kWaves + wave) * rpw;

  for (int t0 = 0; t0 < n; t0 += TT) {
    const int nt = min(TT, n - t0);
    for (int t = 0; t < nt; ++t) {
      const float *src = a.h + size_t(list[t0 + t]) * I;
      for (int i = tid * 4; i < I; i += kBlock * 4)
        *reinterpret_cast<float4 *>(act_rows + size_t(t) * I + i) = *reinterpret_cast<const float4 *>(src + i);
    }
    __syncthreads();
    for (int rr = 0; rr < rpw; ++rr) {
      const int row = row0 + rr;
      if (row >= H) break;
      float acc[TT];
#pragma unroll
      for (int t = 0; t < TT; ++t) acc[t] = 0.f;
      const WT *pw = wd + size_t(row) * I;
#pragma unroll 4
      for (int c = lane * VN; c < I; c += kWave * VN) {
        float fw[VN];
        Packed<WT>::unpack(load_stream<typename Packed<WT>::Raw>(pw + c), fw);
#pragma unroll
        for (int t = 0; t < TT; ++t) {
          if (t < nt) {
            const float *hv = act_rows + size_t(t) * I + c;
#pragma unroll
            for (int x = 0; x < VN; ++x) acc[t] += fw[x] * hv[x];
          }
        }
      }
#pragma unroll
      for (int t = 0; t < TT; ++t) {
        if (t < nt) {
          const float v = wave_sum(acc[t]);
          if (lane == 0) a.y[size_t(list[t0 + t]) * H + row] = v;
        }
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------------------------
// Batch-1 kernels: no token lists, no staging barrier in the gate/up kernel, combine fused into
// the down kernel.  These are the kernels of the headline workload.

// The slots of a launch that was queued behind the routing without waiting for its ids (BY_ROUTING): a lane for each of the k
// positions, or "absent" if an expert is in none; the host, which learns the same ids meanwhile, copies it and launches again.
__device__ __forceinline__ bool routed_slots(const ExpertArgs &a, int lane, int *slot) {
  *slot = a.slots[lane < a.k ? lane : 0];
  return __ballot(*slot < 0) == 0;
}

template <typename WT, int NCH, bool BY_ROUTING>
__global__ __launch_bounds__(kBlock) void gateup_b1_kernel(const ExpertArgs a, const ActiveList act,
                                                           const int rpw) {
  int slot = 0;
  if (BY_ROUTING) {
    if (!routed_slots(a, threadIdx.x & (kWave - 1), &slot)) return;
    slot = __builtin_amdgcn_readlane(slot, blockIdx.y);
  } else {
    slot = act.slot[blockIdx.y];
  }
  gateup_b1_body<WT, NCH, false>(a, slot, blockIdx.y, blockIdx.x, rpw, 0, a.I, nullptr, nullptr);
}

template <typename WT, int NCH, bool BY_ROUTING>
__global__ __launch_bounds__(kBlock) void gateup_b1_pair_kernel(const ExpertArgs a, const ActiveList act) {
  int slot = 0;
  if (BY_ROUTING) {
    if (!routed_slots(a, threadIdx.x & (kWave - 1), &slot)) return;
    slot = __builtin_amdgcn_readlane(slot, blockIdx.y);
  } else {
    slot = act.slot[blockIdx.y];
  }
  gateup_b1_pair_body<WT, NCH>(a, slot, blockIdx.y, blockIdx.x);
}

// O[row] = sum_j gate_j * (W_down_{e_j}[row,:] . hq[j,:]) for the one token of the batch: the down
// projection of all k executed experts and the gate-weighted combine in one pass.  SPLIT
// wavefronts share one output row.  The k rows it needs (one per expert, I values each) are
// walked as one flat list of 16-byte chunks so that all 64 lanes load on every iteration
// whatever I is; each lane folds the gate of its chunk's expert into its partial sum, one
// reduction per wavefront remains, and the SPLIT partial sums meet in LDS.  `act` is in
// execution-position order.
template <typename WT, int SPLIT, int UNROLL, bool BY_ROUTING>
__global__ __launch_bounds__(kBlock) void down_combine_b1_kernel(const ExpertArgs a, const ActiveList act,
                                                                 const float inv_chunks) {
  using R = Packed<WT>;
  constexpr int VN = R::N;
  __shared__ float part_sum[kWaves];
  __shared__ int slots[BY_ROUTING ? kWaves : 1][kWave];      // every wavefront has its own
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  if (BY_ROUTING) {
    int slot;
    if (!routed_slots(a, lane, &slot)) return;
    slots[wave][lane] = slot;
  }
  const int H = a.H, I = a.I, k = a.k;
  const int row = blockIdx.x * (kWaves / SPLIT) + wave / SPLIT;
  const int part = wave % SPLIT;
  const bool valid = row < H;
  const int chunks = I / VN;                   // per expert row
  const int total = chunks * k;
  const WT *hq = reinterpret_cast<const WT *>(a.h);
  const size_t down_off = (size_t(2) * I * H + size_t(valid ? row : 0) * I) * sizeof(WT);
  float acc = 0.f;
  if (valid) {
#pragma unroll UNROLL
    for (int t = part * kWave + lane; t < total; t += kWave * SPLIT) {
      int j = int(float(t) * inv_chunks);      // t / chunks, fixed up below (t < 2^24 is exact in float)
      j -= (j * chunks > t);
      j += ((j + 1) * chunks <= t);
      const int c = (t - j * chunks) * VN;
      const int slot = BY_ROUTING ? slots[BY_ROUTING ? wave : 0][j] : act.slot[j];
      const char *base = a.pool + size_t(slot) * a.slot_bytes + down_off;
      const typename R::Raw w = load_stream<typename R::Raw>(base + size_t(c) * sizeof(WT));
      const typename R::Raw hh = *reinterpret_cast<const typename R::Raw *>(hq + size_t(j) * I + c);
      acc += a.exec_gates[j] * dot_chunk(w, hh, 0.f);
    }
  }
  const float v = wave_sum(acc);
  if (SPLIT == 1) {
    if (lane == 0 && valid) a.out[row] = v;
  } else {
    if (lane == 0) part_sum[wave] = v;
    __syncthreads();
    if (lane == 0 && part == 0 && valid) {
      float tot = 0.f;
#pragma unroll
      for (int p = 0; p < SPLIT; ++p) tot += part_sum[wave + p];
      a.out[row] = tot;
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Matrix-core kernels for decode batches of two and more (bf16 weights) and for prefill
template <bool GATEUP, int NT, int KSPLIT, int CHAINS, bool STREAM>
__global__ __launch_bounds__(kBlock) void expert_mfma_kernel(const ExpertArgs a, const TokenLists lists,
                                                             const uint16_t *act_q, uint16_t *hq_out) {
  __shared__ ExpertMfmaShared<GATEUP, NT, KSPLIT> sh;
  expert_mfma_body<GATEUP, NT, KSPLIT, CHAINS>(a, DecodeTokens<STREAM>{lists, int(blockIdx.y)}, act_q, hq_out, blockIdx.x, sh);
}

template <bool GATEUP, int NT, int KSPLIT>
__global__ __launch_bounds__(kBlock) void expert_mfma_lists_kernel(const ExpertArgs a, const ActiveList act,
                                                                   const uint16_t *act_q, uint16_t *hq_out) {
  __shared__ ExpertMfmaShared<GATEUP, NT, KSPLIT> sh;
  expert_mfma_body<GATEUP, NT, KSPLIT, kOneChain>(a, PrefillTokens{act, int(blockIdx.y), int(blockIdx.z)}, act_q, hq_out,
                                                  blockIdx.x, sh);
}

// ---------------------------------------------------------------------------------------------
// Prefill with many positions per expert: the expert FFN as a tiled matrix product.  A workgroup
// owns 128 positions of one expert and 256 weight rows (gate/up: 128 rows of W_gate and the same 128
// of W_up, so that both factors of the SwiGLU product meet in one lane; down: 256 rows of W_down), and
// walks the reduction 64 columns at a time through two LDS buffers: the next 64 columns travel to
// registers while the current ones are multiplied.  A wavefront multiplies 64 positions with 64 weight
// rows.  expert_mfma_lists_kernel, which feeds every MFMA from global memory, re-reads each weight row once
// per 64 positions and stops where the caches do.
// Sums: every 512 columns the accumulators are added to a second set and start again from zero, so that
// no float32 chain is longer than those of the other kernels from 2048 columns on (one chain of 4096 columns moved half as
// many SwiGLU values more to the neighbouring bf16 value).
// The tiles of all experts of the launch form one list that one workgroup per compute unit walks:
// positions per expert are known on the device only.
constexpr int kTileBlock = 512;
constexpr int kTilePos = 128, kTileRows = 256, kTileK = 64;
constexpr int kTileSteps = 8;                  // steps of 64 columns per chain of sums
constexpr int kTileGroup = 8;                  // row tiles that share a group of position tiles in an L2

template <bool GATEUP>
__global__ __launch_bounds__(kTileBlock, 2) void expert_tile_kernel(const ExpertArgs a, const ActiveList act,
                                                                    const uint16_t *act_q, uint16_t *hq_out) {
  // rows of 64 columns: positions first, then weight rows.  The 16-byte chunk c of row r lies at chunk
  // c ^ (r % 8): eight lanes that read the same chunk of eight rows touch all banks once.
  constexpr int kBuf = (kTilePos + kTileRows) * (kTileK / 8);
  __shared__ uint4 tile[2 * kBuf];
  __shared__ int list[kTilePos];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int m = lane & 15, g = lane >> 4;
  const int K = GATEUP ? a.H : a.I;
  const int R = GATEUP ? a.I : a.H;
  constexpr int kRowsOut = GATEUP ? kTileRows / 2 : kTileRows;         // output rows per tile
  const int r_first = a.row_first, r_end = a.row_end ? a.row_end : R;
  const int row_tiles = (r_end - r_first + kRowsOut - 1) / kRowsOut;
  const int chunk = tid & 7, ld_row = tid >> 3;                        // this thread's chunk and first row when loading
  const int ld_at = ld_row * 8 + (chunk ^ (ld_row & 7));
  const int wave_pos = (wave & 1) * 64;
  const int wave_row = (wave >> 1) * (GATEUP ? 32 : 64);
  // workgroups go round the eight XCDs: the ones of an XCD take neighbouring tiles, which share rows and positions
  const int per_xcd = gridDim.x / 8;
  const int slot = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;

  for (long t = slot;; t += gridDim.x) {
    // ---- which expert, positions and rows
    long left = t;
    int e = -1, n_all = 0, n_pt = 0, which = 0;
    for (int i = 0; i < act.n; ++i) {
      const int cnt = a.pos_count[act.expert[i]];
      const int pt = (cnt + kTilePos - 1) / kTilePos;
      const long tiles = long(pt) * row_tiles;
      if (left < tiles) { e = act.expert[i]; n_all = cnt; n_pt = pt; which = i; break; }
      left -= tiles;
    }
    if (e < 0) return;                         // past the last tile: the same for the whole workgroup
    const int group = int(left / (long(kTileGroup) * n_pt));
    const int in_group = int(left - long(group) * kTileGroup * n_pt);
    const int group_rows = min(kTileGroup, row_tiles - group * kTileGroup);
    const int pos0 = in_group / group_rows * kTilePos;
    const int row0 = r_first + (group * kTileGroup + in_group % group_rows) * kRowsOut;
    const int n = min(kTilePos, n_all - pos0);
    __syncthreads();                           // the previous tile's readers of list and tile are done
    if (tid < n) list[tid] = a.pos_list[size_t(e) * a.list_stride + pos0 + tid];
    __syncthreads();

    const uint16_t *wbase = reinterpret_cast<const uint16_t *>(a.pool + size_t(act.slot[which]) * a.slot_bytes) +
                            (GATEUP ? size_t(0) : size_t(2) * a.I * a.H);
    const uint16_t *xp[2];
    uint32_t woff[4];                          // an expert block holds fewer than 2^30 weights
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int p = ld_row + 64 * i;
      const int f = list[p < n ? p : 0];       // rows past the end repeat one and are not stored
      xp[i] = act_q + size_t(GATEUP ? f / a.k : f) * K + chunk * 8;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = ld_row + 64 * i;
      const int in = r & (kRowsOut - 1);
      woff[i] = uint32_t(min(row0 + in, r_end - 1)) * uint32_t(K) + (GATEUP && r >= kRowsOut ? uint32_t(a.I) * uint32_t(a.H) : 0u) + chunk * 8;
    }
    f32x4_t total[4][4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int p = 0; p < 4; ++p) total[j][p] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    uint4 held[6];
    auto fetch = [&](int k0) {                 // columns past the end are zeros on both sides
      const bool inside = k0 + chunk * 8 < K;
#pragma unroll
      for (int i = 0; i < 6; ++i) held[i] = make_uint4(0u, 0u, 0u, 0u);
      if (inside) {
#pragma unroll
        for (int i = 0; i < 2; ++i) held[i] = *reinterpret_cast<const uint4 *>(xp[i] + k0);
#pragma unroll
        for (int i = 0; i < 4; ++i) held[2 + i] = *reinterpret_cast<const uint4 *>(wbase + woff[i] + k0);
      }
    };
    auto keep = [&](int buf) {
#pragma unroll
      for (int i = 0; i < 6; ++i) tile[buf * kBuf + ld_at + i * 64 * 8] = held[i];
    };
    fetch(0);
    keep(0);
    __syncthreads();
    int buf = 0;
    for (int k_first = 0; k_first < K; k_first += kTileSteps * kTileK) {
      f32x4_t acc[4][4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int p = 0; p < 4; ++p) acc[j][p] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      const int k_end = min(K, k_first + kTileSteps * kTileK);
      for (int k0 = k_first; k0 < k_end; k0 += kTileK) {
        const bool more = k0 + kTileK < K;
        if (more) fetch(k0 + kTileK);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          const uint4 *at = tile + buf * kBuf + m * 8 + ((kk * 4 + g) ^ (m & 7));
          bf16x8_t x[4], w[4];
#pragma unroll
          for (int p = 0; p < 4; ++p) x[p] = __builtin_bit_cast(bf16x8_t, at[(wave_pos + p * 16) * 8]);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int r = GATEUP ? wave_row + (j & 1) * 16 + (j >> 1) * kRowsOut : wave_row + j * 16;
            w[j] = __builtin_bit_cast(bf16x8_t, at[(kTilePos + r) * 8]);
          }
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int p = 0; p < 4; ++p) acc[j][p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[j], x[p], acc[j][p], 0, 0, 0);
        }
        buf ^= 1;
        if (more) keep(buf);                   // its last readers passed the barrier of the step before
        __syncthreads();
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int p = 0; p < 4; ++p) total[j][p] += acc[j][p];
    }

    // ---- accumulator layout: lane = position lane % 16, rows 4 (lane / 16) .. + 3
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const int idx = wave_pos + p * 16 + m;
      if (idx < n) {
        const int f = list[idx];
#pragma unroll
        for (int j = 0; j < (GATEUP ? 2 : 4); ++j) {
          const int r = row0 + wave_row + j * 16 + 4 * g;             // four rows, all inside or all outside
          if (r < r_end) {
            if (GATEUP) {
              uint16_t q[4];
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                const float s0 = total[j][p][i], s1 = total[GATEUP ? j + 2 : j][p][i];
                q[i] = uint16_t(__float_as_uint(round_to_bf16(s0 / (1.f + expf(-s0)) * s1)) >> 16);
              }
              uint2 packed;
              packed.x = uint32_t(q[0]) | (uint32_t(q[1]) << 16);
              packed.y = uint32_t(q[2]) | (uint32_t(q[3]) << 16);
              *reinterpret_cast<uint2 *>(hq_out + size_t(f) * R + r) = packed;
            } else {
              *reinterpret_cast<float4 *>(a.y + size_t(f) * R + r) =
                  make_float4(total[j][p][0], total[j][p][1], total[j][p][2], total[j][p][3]);
            }
          }
        }
      }
    }
  }
}

// Positions f = b*k + j of an id table [tokens, k], grouped by expert, ascending inside a group:
// pos[e*stride + i] for i < count[e].  One workgroup per expert; each wavefront counts and then
// writes its own contiguous quarter of the table.
__global__ __launch_bounds__(kBlock) void expert_lists_kernel(const int32_t *ids, int n_ids, int stride,
                                                              int32_t *pos, int32_t *count) {
  __shared__ int wave_count[kWaves];
  const int e = blockIdx.x, tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int per_wave = (n_ids + kBlock - 1) / kBlock * kWave;
  const int lo = wave * per_wave, hi = min(n_ids, lo + per_wave);
  int c = 0;
  for (int base = lo; base < hi; base += kWave) {
    const int f = base + lane;
    c += __popcll(__ballot(f < hi && ids[f] == e));
  }
  if (lane == 0) wave_count[wave] = c;
  __syncthreads();
  int off = 0, total = 0;
  for (int w = 0; w < kWaves; ++w) { if (w < wave) off += wave_count[w]; total += wave_count[w]; }
  for (int base = lo; base < hi; base += kWave) {
    const int f = base + lane;
    const bool match = f < hi && ids[f] == e;
    const unsigned long long mask = __ballot(match);
    if (match) pos[size_t(e) * stride + off + __popcll(mask & ((1ull << lane) - 1ull))] = f;
    off += __popcll(mask);
  }
  if (tid == 0) count[e] = total;
}

// Default-vector statistics (paper: Sec. 3.1, the offline aggregation behind d_{l,e}): for every
// position f routed to an expert of this launch, sum[e,:] += y[f,:] and cnt[e] += 1.
__global__ __launch_bounds__(kBlock) void accumulate_defaults_kernel(const ExpertArgs a, const ActiveList act,
                                                                     double *sum, unsigned long long *cnt) {
  const int f = blockIdx.y;
  const int e = a.exec_ids[f];
  bool mine = false;
  for (int i = 0; i < act.n; ++i) mine |= act.expert[i] == e;
  if (!mine) return;
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i < a.H) atomicAdd(sum + size_t(e) * a.H + i, double(a.y[size_t(f) * a.H + i]));
  if (i == 0) atomicAdd(cnt + e, 1ull);
}

__global__ __launch_bounds__(kBlock) void default_means_kernel(const double *sum, const unsigned long long *cnt,
                                                               float *mean, int H) {
  const int e = blockIdx.y, i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= H) return;
  const unsigned long long n = cnt[e];
  mean[size_t(e) * H + i] = n ? float(sum[size_t(e) * H + i] / double(n)) : 0.f;
}

// Measurement aid: reads a range of 16-byte units of the launch's slots and does nothing else (the
// sum is never stored unless it hits an impossible value).  What a kernel can reach on these bytes.
__global__ __launch_bounds__(kBlock) void stream_read_kernel(const ExpertArgs a, const ActiveList act, size_t first16,
                                                             size_t n16, float *sink) {
  const uint4 *p = reinterpret_cast<const uint4 *>(a.pool + size_t(act.slot[blockIdx.y]) * a.slot_bytes) + first16;
  const size_t stride = size_t(gridDim.x) * kBlock;
  float acc = 0.f;
  for (size_t i = size_t(blockIdx.x) * kBlock + threadIdx.x; i < n16; i += stride) {
    const uint4 v = load_stream<uint4>(p + i);
    acc += __uint_as_float(v.x ^ v.y ^ v.z ^ v.w);
  }
  if (acc == 1.2345e-30f) *sink = acc;
}

// O[b, i] = sum_j gates[b, j] * y[b, j, i], V columns per thread: one in decode batches (four gain nothing there, the
// launch is as short as a launch of dependent loads gets), four in prefill, where it is a stream (32768 tokens, 2 experts,
// 4096 columns 450 -> 232 us, 6.9 TB/s).
template <int V>
__global__ __launch_bounds__(kBlock) void combine_kernel(const ExpertArgs a) {
  const int i = (blockIdx.x * kBlock + threadIdx.x) * V;
  const int b = blockIdx.y;
  if (i >= a.H) return;
  float acc[V] = {};
  for (int j = 0; j < a.k; ++j) {
    const float gate = a.exec_gates[b * a.k + j];
    const float *y = a.y + (size_t(b) * a.k + j) * a.H + i;
    float v[V];
    if (V == 4) {
      const float4 f = __builtin_bit_cast(float4, load_stream<uint4>(y));
      v[0] = f.x; v[V > 1 ? 1 : 0] = f.y; v[V > 2 ? 2 : 0] = f.z; v[V > 3 ? 3 : 0] = f.w;
    } else {
      v[0] = *y;
    }
#pragma unroll
    for (int x = 0; x < V; ++x) acc[x] += gate * v[x];
  }
  float *o = a.out + size_t(b) * a.H + i;
  if (V == 4) *reinterpret_cast<float4 *>(o) = make_float4(acc[0], acc[V > 1 ? 1 : 0], acc[V > 2 ? 2 : 0], acc[V > 3 ? 3 : 0]);
  else *o = acc[0];
}

// Host-to-device copy of whole expert blocks by a few workgroups that read the pinned pool
// directly.  blockIdx.y picks the block, the workgroups of a row share it in 16-byte units.
// kCopyUnroll loads are in flight per lane; the launch keeps the bytes in flight near the link's
// bandwidth-delay product, because host reads that queue up in the memory system delay the
// HBM requests of kernels running beside the copy.
constexpr int kCopyWorkgroups = 16, kCopyUnroll = 2;      // 16 x 256 lanes x 2 x 16 B = 128 KB in flight
__global__ __launch_bounds__(kBlock) void gather_copy_kernel(const CopyList cl) {
  const uint4 *src = static_cast<const uint4 *>(cl.src[blockIdx.y]);
  uint4 *dst = static_cast<uint4 *>(cl.dst[blockIdx.y]);
  const uint32_t n = cl.n16;
  const uint32_t stride = gridDim.x * kBlock;
  uint32_t i = blockIdx.x * kBlock + threadIdx.x;
  for (; i + (kCopyUnroll - 1) * stride < n; i += kCopyUnroll * stride) {
    uint4 v[kCopyUnroll];
#pragma unroll
    for (int u = 0; u < kCopyUnroll; ++u) v[u] = src[i + u * stride];
#pragma unroll
    for (int u = 0; u < kCopyUnroll; ++u) dst[i + u * stride] = v[u];
  }
  for (; i < n; i += stride) dst[i] = src[i];
}

int pick_tok_tile(int B, int row_len) {
  int tt = 1;
  while (tt < B && tt < 8) tt <<= 1;
  while (tt > 1 && size_t(tt) * row_len * sizeof(float) > (size_t(60) << 10)) tt >>= 1;
  return tt;
}

int pick_rows_per_wave(int rows, int n_active) {
  // aim for about 2048 workgroups so that all 256 compute units hold several
  const long total = long(rows) * n_active;
  long rpw = total / (long(kWaves) * 2048);
  if (rpw < 1) rpw = 1;
  if (rpw > 8) rpw = 8;
  return int(rpw);
}

template <typename WT>
hipError_t launch_gateup_t(const ExpertArgs &a, const ActiveList &act, hipStream_t st) {
  const int tt = pick_tok_tile(a.B, a.H);
  const int rpw = pick_rows_per_wave(a.I, act.n);
  const size_t lds = size_t(tt) * a.H * sizeof(float);
  const dim3 grid((a.I + kWaves * rpw - 1) / (kWaves * rpw), act.n), block(kBlock);
  switch (tt) {
    case 1: hipLaunchKernelGGL((gateup_kernel<WT, 1>), grid, block, lds, st, a, act, rpw); break;
    case 2: hipLaunchKernelGGL((gateup_kernel<WT, 2>), grid, block, lds, st, a, act, rpw); break;
    case 4: hipLaunchKernelGGL((gateup_kernel<WT, 4>), grid, block, lds, st, a, act, rpw); break;
    default: hipLaunchKernelGGL((gateup_kernel<WT, 8>), grid, block, lds, st, a, act, rpw); break;
  }
  return hipGetLastError();
}

template <typename WT>
hipError_t launch_down_t(const ExpertArgs &a, const ActiveList &act, hipStream_t st) {
  const int tt = pick_tok_tile(a.B, a.I);
  const int rpw = pick_rows_per_wave(a.H, act.n);
  const size_t lds = size_t(tt) * a.I * sizeof(float);
  const dim3 grid((a.H + kWaves * rpw - 1) / (kWaves * rpw), act.n), block(kBlock);
  switch (tt) {
    case 1: hipLaunchKernelGGL((down_kernel<WT, 1>), grid, block, lds, st, a, act, rpw); break;
    case 2: hipLaunchKernelGGL((down_kernel<WT, 2>), grid, block, lds, st, a, act, rpw); break;
    case 4: hipLaunchKernelGGL((down_kernel<WT, 4>), grid, block, lds, st, a, act, rpw); break;
    default: hipLaunchKernelGGL((down_kernel<WT, 8>), grid, block, lds, st, a, act, rpw); break;
  }
  return hipGetLastError();
}

template <typename WT, int NCH>
void launch_gateup_b1_n(const ExpertArgs &a, const ActiveList &act, hipStream_t st) {
  const GateupSplit split = gateup_b1_split(NCH, a.I, act.n);
  const dim3 grid(split.blocks, act.n), block(kBlock);
  if (split.rpw == 0 && a.slots) hipLaunchKernelGGL((gateup_b1_pair_kernel<WT, NCH, true>), grid, block, 0, st, a, act);
  else if (split.rpw == 0) hipLaunchKernelGGL((gateup_b1_pair_kernel<WT, NCH, false>), grid, block, 0, st, a, act);
  else if (a.slots) hipLaunchKernelGGL((gateup_b1_kernel<WT, NCH, true>), grid, block, 0, st, a, act, split.rpw);
  else hipLaunchKernelGGL((gateup_b1_kernel<WT, NCH, false>), grid, block, 0, st, a, act, split.rpw);
}

// Returns false when H needs more register chunks than the batch-1 kernel is built for.
template <typename WT>
bool launch_gateup_b1(const ExpertArgs &a, const ActiveList &act, hipStream_t st) {
  constexpr int VN = Packed<WT>::N;
  const int need = (a.H + kWave * VN - 1) / (kWave * VN);
  if (need <= 1) launch_gateup_b1_n<WT, 1>(a, act, st);
  else if (need <= 2) launch_gateup_b1_n<WT, 2>(a, act, st);
  else if (need <= 4) launch_gateup_b1_n<WT, 4>(a, act, st);
  else if (need <= 6) launch_gateup_b1_n<WT, 6>(a, act, st);
  else if (need <= 8) launch_gateup_b1_n<WT, 8>(a, act, st);
  else if (need <= 16) launch_gateup_b1_n<WT, 16>(a, act, st);
  else return false;
  return true;
}

template <typename WT, int SPLIT, int UNROLL>
void launch_down_combine_b1_n(const ExpertArgs &a, const ActiveList &act, hipStream_t st) {
  const dim3 grid((a.H + kWaves / SPLIT - 1) / (kWaves / SPLIT)), block(kBlock);
  const float inv_chunks = 1.0f / float(a.I / Packed<WT>::N);
  if (a.slots) hipLaunchKernelGGL((down_combine_b1_kernel<WT, SPLIT, UNROLL, true>), grid, block, 0, st, a, act, inv_chunks);
  else hipLaunchKernelGGL((down_combine_b1_kernel<WT, SPLIT, UNROLL, false>), grid, block, 0, st, a, act, inv_chunks);
}

// The loop of a wavefront is unrolled UNROLL times, so that many loads per lane are in flight
// together; where a row's chunk list is short enough, SPLIT is chosen so that each wavefront's
// share is exactly one such batch (iterations beyond a multiple of UNROLL run one by one).
// Otherwise four wavefronts per row and batches of four, the best measured on the 1440- and
// 3584-chunk rows of the larger workloads.
template <typename WT>
void launch_down_combine_b1(const ExpertArgs &a, const ActiveList &act, hipStream_t st) {
  const long chunks = long(a.I / Packed<WT>::N) * a.k;
  const long iters = chunks % kWave == 0 ? chunks / kWave : 0;      // per row, for one wavefront
  if (iters == 4) launch_down_combine_b1_n<WT, 1, 4>(a, act, st);
  else if (iters == 6) launch_down_combine_b1_n<WT, 1, 6>(a, act, st);
  else if (iters == 8) launch_down_combine_b1_n<WT, 2, 4>(a, act, st);
  else if (iters == 12) launch_down_combine_b1_n<WT, 2, 6>(a, act, st);
  else launch_down_combine_b1_n<WT, 4, 4>(a, act, st);
}

// Compute units of the current device.
hipError_t compute_units(int *n) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  return e != hipSuccess ? e : hipDeviceGetAttribute(n, hipDeviceAttributeMultiprocessorCount, dev);
}

template <bool GATEUP, int NT, int KSPLIT, int CHAINS>
hipError_t launch_expert_mfma(const ExpertArgs &a, const TokenLists &lists, const uint16_t *act_q, uint16_t *hq, hipStream_t st) {
  constexpr int rows_per_wg = 16 * kWaves / KSPLIT;
  const dim3 grid(((GATEUP ? a.I : a.H) + rows_per_wg - 1) / rows_per_wg, lists.n), block(kBlock);
  if (whole_lines(GATEUP ? a.H : a.I))
    hipLaunchKernelGGL((expert_mfma_kernel<GATEUP, NT, KSPLIT, CHAINS, true>), grid, block, 0, st, a, lists, act_q, hq);
  else
    hipLaunchKernelGGL((expert_mfma_kernel<GATEUP, NT, KSPLIT, CHAINS, false>), grid, block, 0, st, a, lists, act_q, hq);
  return hipGetLastError();
}

template <int NT>
hipError_t launch_gateup_mfma_t(const ExpertArgs &a, const TokenLists &lists, const uint16_t *s_q, uint16_t *hq, hipStream_t st) {
  return with_ksplit(gateup_ksplit(a.H, (a.B + 15) / 16),
                     [&](auto ksplit) { return launch_expert_mfma<true, NT, ksplit(), kOneChain>(a, lists, s_q, hq, st); });
}

// The same over position lists on the device (prefill), 64 positions per grid plane.
template <bool GATEUP, int KSPLIT>
hipError_t launch_expert_mfma_lists_k(const ExpertArgs &a, const ActiveList &act, const uint16_t *act_q, uint16_t *hq,
                                      hipStream_t st) {
  const int rows = GATEUP ? a.I : a.H;
  const int rows_per_wg = 16 * kWaves / KSPLIT;
  const int planes = (a.list_tokens + kMaxBatch - 1) / kMaxBatch;
  const dim3 grid((rows + rows_per_wg - 1) / rows_per_wg, act.n, planes), block(kBlock);
  switch ((std::min(a.list_tokens, kMaxBatch) + 15) / 16) {
    case 1: hipLaunchKernelGGL((expert_mfma_lists_kernel<GATEUP, 1, KSPLIT>), grid, block, 0, st, a, act, act_q, hq); break;
    case 2: hipLaunchKernelGGL((expert_mfma_lists_kernel<GATEUP, 2, KSPLIT>), grid, block, 0, st, a, act, act_q, hq); break;
    case 3: hipLaunchKernelGGL((expert_mfma_lists_kernel<GATEUP, 3, KSPLIT>), grid, block, 0, st, a, act, act_q, hq); break;
    default: hipLaunchKernelGGL((expert_mfma_lists_kernel<GATEUP, 4, KSPLIT>), grid, block, 0, st, a, act, act_q, hq); break;
  }
  return hipGetLastError();
}

// Prefill: the tiled kernel, or position lists through expert_mfma_lists_kernel?  A tile takes about 1.5 us per 64
// columns however many of its positions are real (one workgroup per compute unit, the loads of one step in
// flight), the other kernel's time goes with the positions (about 170 TFLOP/s once its weights are read): tiles
// pay once a round of them holds about a quarter of the device's worth of real positions, taking the experts as
// equally loaded.  Measured, expert_mfma_lists_kernel against tiles: gate/up of 8 experts 768 x 2048 with 128
// positions each 50 / 58 us, with 256 87 / 58 us; down (2048 x 768) with 64 24 / 28, with 128 38 / 30; one expert
// 14336 x 4096 with 64 positions 120 / 101, with 128 201 / 101, its down with 256 259 / 341, with 8192 7784 / 1428
// (gate/up 9492 / 2618 us, 735 TFLOP/s).
bool tiles_pay(const ExpertArgs &a, int n_experts, bool gateup, int cus) {
  const long rows = gateup ? a.I : a.H, rows_out = gateup ? kTileRows / 2 : kTileRows;
  const long row_tiles = (rows + rows_out - 1) / rows_out;
  const long pos = long(a.list_tokens) * a.k / a.E;      // per expert
  const long tiles = n_experts * ((pos + kTilePos - 1) / kTilePos) * row_tiles;
  const long rounds = (tiles + cus - 1) / cus;
  return pos > 0 && n_experts * pos * row_tiles * 4 >= rounds * cus * kTilePos;
}

template <bool GATEUP>
hipError_t launch_expert_mfma_lists(const ExpertArgs &a, const ActiveList &act, const uint16_t *act_q, uint16_t *hq,
                                    hipStream_t st) {
  int cus = 0;
  if (hipError_t e = compute_units(&cus); e != hipSuccess) return e;
  if (a.row_end > 0 || tiles_pay(a, act.n, GATEUP, cus)) {
    const int wgs = (cus + 7) / 8 * 8;                   // one per compute unit: 97 KB of LDS
    hipLaunchKernelGGL((expert_tile_kernel<GATEUP>), dim3(wgs), dim3(kTileBlock), 0, st, a, act, act_q, hq);
    return hipGetLastError();
  }
  const int ksplit = gateup_ksplit(GATEUP ? a.H : a.I, (std::min(a.list_tokens, kMaxBatch) + 15) / 16);
  if (ksplit == 4) return launch_expert_mfma_lists_k<GATEUP, 4>(a, act, act_q, hq, st);
  if (ksplit == 2) return launch_expert_mfma_lists_k<GATEUP, 2>(a, act, act_q, hq, st);
  return launch_expert_mfma_lists_k<GATEUP, 1>(a, act, act_q, hq, st);
}

template <typename K>
hipError_t allow_big_lds(K kernel) {
  return hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                             hipFuncAttributeMaxDynamicSharedMemorySize, 128 << 10);
}

}  // namespace

hipError_t launch_gateup(const ExpertArgs &a, const ActiveList &act, int dtype, hipStream_t st) {
  if (act.n <= 0) return hipSuccess;
  return dtype == 1 ? launch_gateup_t<uint16_t>(a, act, st) : launch_gateup_t<float>(a, act, st);
}

// Batch 1, `act` in execution-position order.  H up to 64*16 chunks (8192 bf16 / 4096 float32 columns).
bool b1_supported(int H, int dtype) { return H <= kWave * 16 * (dtype == 1 ? 8 : 4); }

hipError_t launch_gateup_b1(const ExpertArgs &a, const ActiveList &act, int dtype, hipStream_t st) {
  const bool ok = dtype == 1 ? launch_gateup_b1<uint16_t>(a, act, st) : launch_gateup_b1<float>(a, act, st);
  return ok ? hipGetLastError() : hipErrorInvalidValue;
}

// Batch 1: down projection and combine in one kernel (the k executed experts are always one cache
// wave); reads the hq written by launch_gateup_b1.
hipError_t launch_down_combine_b1(const ExpertArgs &a, const ActiveList &act, int dtype, hipStream_t st) {
  if (dtype == 1) launch_down_combine_b1<uint16_t>(a, act, st);
  else launch_down_combine_b1<float>(a, act, st);
  return hipGetLastError();
}

hipError_t launch_down(const ExpertArgs &a, const ActiveList &act, int dtype, hipStream_t st) {
  if (act.n <= 0) return hipSuccess;
  return dtype == 1 ? launch_down_t<uint16_t>(a, act, st) : launch_down_t<float>(a, act, st);
}

// bf16 weights, batch >= kMfmaMinBatch: s_q is s_l as bf16 [B,H]; hq (bf16 [B,k,I]) is written by the gate/up
// launch and read by the down launch.
hipError_t launch_gateup_mfma(const ExpertArgs &a, const TokenLists &lists, const uint16_t *s_q, uint16_t *hq,
                              hipStream_t st) {
  if (lists.n <= 0) return hipSuccess;
  switch (decode_tiles(lists.most)) {
    case 1: return launch_gateup_mfma_t<1>(a, lists, s_q, hq, st);
    case 2: return launch_gateup_mfma_t<2>(a, lists, s_q, hq, st);
    default: return launch_gateup_mfma_t<4>(a, lists, s_q, hq, st);
  }
}

hipError_t launch_down_mfma(const ExpertArgs &a, const TokenLists &lists, const uint16_t *hq, hipStream_t st) {
  if (lists.n <= 0) return hipSuccess;
  int cus = 0;
  if (hipError_t e = compute_units(&cus); e != hipSuccess) return e;
  return with_down_form(a, lists, cus, [&](auto nt, auto ksplit, auto chains) {
    return launch_expert_mfma<false, nt(), ksplit(), chains()>(a, lists, hq, nullptr, st);
  });
}

hipError_t launch_gateup_prefill(const ExpertArgs &a, const ActiveList &act, const uint16_t *s_q, uint16_t *hq,
                                 hipStream_t st) {
  return act.n <= 0 ? hipSuccess : launch_expert_mfma_lists<true>(a, act, s_q, hq, st);
}

hipError_t launch_down_prefill(const ExpertArgs &a, const ActiveList &act, const uint16_t *hq, hipStream_t st) {
  return act.n <= 0 ? hipSuccess : launch_expert_mfma_lists<false>(a, act, hq, nullptr, st);
}

hipError_t launch_expert_lists(const int32_t *ids, int tokens, int k, int E, int32_t *pos, int32_t *count,
                               hipStream_t st) {
  hipLaunchKernelGGL(expert_lists_kernel, dim3(E), dim3(kBlock), 0, st, ids, tokens * k, tokens, pos, count);
  return hipGetLastError();
}

hipError_t launch_gather_copy(const CopyList &cl, hipStream_t st) {
  if (cl.n <= 0) return hipSuccess;
  const int wg_per_block = (kCopyWorkgroups + cl.n - 1) / cl.n;
  hipLaunchKernelGGL(gather_copy_kernel, dim3(wg_per_block, cl.n), dim3(kBlock), 0, st, cl);
  return hipGetLastError();
}

hipError_t launch_accumulate_defaults(const ExpertArgs &a, const ActiveList &act, double *sum,
                                      unsigned long long *cnt, hipStream_t st) {
  const dim3 grid((a.H + kBlock - 1) / kBlock, a.B * a.k), block(kBlock);
  hipLaunchKernelGGL(accumulate_defaults_kernel, grid, block, 0, st, a, act, sum, cnt);
  return hipGetLastError();
}

hipError_t launch_default_means(const double *sum, const unsigned long long *cnt, float *mean, int E, int H,
                                hipStream_t st) {
  const dim3 grid((H + kBlock - 1) / kBlock, E), block(kBlock);
  hipLaunchKernelGGL(default_means_kernel, grid, block, 0, st, sum, cnt, mean, H);
  return hipGetLastError();
}

hipError_t launch_stream_read(const ExpertArgs &a, const ActiveList &act, size_t first16, size_t n16, hipStream_t st) {
  hipLaunchKernelGGL(stream_read_kernel, dim3(768, act.n), dim3(kBlock), 0, st, a, act, first16, n16, a.out);
  return hipGetLastError();
}

hipError_t launch_combine(const ExpertArgs &a, hipStream_t st) {
  const int v = a.B > kMaxBatch && reinterpret_cast<uintptr_t>(a.out) % 16 == 0 ? 4 : 1;   // the caller's rows
  const dim3 grid((a.H + kBlock * v - 1) / (kBlock * v), a.B), block(kBlock);
  if (v == 4) hipLaunchKernelGGL(combine_kernel<4>, grid, block, 0, st, a);
  else hipLaunchKernelGGL(combine_kernel<1>, grid, block, 0, st, a);
  return hipGetLastError();
}

hipError_t init_route_kernels();

hipError_t init_kernels() {
  hipError_t e = init_route_kernels();
#define MOE_SPEC_ALLOW(k) if (e == hipSuccess) e = allow_big_lds(k)
  MOE_SPEC_ALLOW((gateup_kernel<uint16_t, 1>)); MOE_SPEC_ALLOW((gateup_kernel<uint16_t, 2>));
  MOE_SPEC_ALLOW((gateup_kernel<uint16_t, 4>)); MOE_SPEC_ALLOW((gateup_kernel<uint16_t, 8>));
  MOE_SPEC_ALLOW((gateup_kernel<float, 1>)); MOE_SPEC_ALLOW((gateup_kernel<float, 2>));
  MOE_SPEC_ALLOW((gateup_kernel<float, 4>)); MOE_SPEC_ALLOW((gateup_kernel<float, 8>));
  MOE_SPEC_ALLOW((down_kernel<uint16_t, 1>)); MOE_SPEC_ALLOW((down_kernel<uint16_t, 2>));
  MOE_SPEC_ALLOW((down_kernel<uint16_t, 4>)); MOE_SPEC_ALLOW((down_kernel<uint16_t, 8>));
  MOE_SPEC_ALLOW((down_kernel<float, 1>)); MOE_SPEC_ALLOW((down_kernel<float, 2>));
  MOE_SPEC_ALLOW((down_kernel<float, 4>)); MOE_SPEC_ALLOW((down_kernel<float, 8>));
#undef MOE_SPEC_ALLOW
  return e;
}

}  // namespace moe_spec
