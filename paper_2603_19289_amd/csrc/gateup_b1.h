// Gate/up projection and SwiGLU of a batch of one, as device functions: expert_kernels.hip launches them by
// themselves, fused_kernels.hip beside the routing of the same layer.
#pragma once
#include "device_utils.h"
#include "kernels.h"
#include "launch_rules.h"

namespace moe_spec {

constexpr int kB1Block = 256;
static_assert(kB1Waves == kB1Block / kWave, "the launch rules count wavefronts");

// s_l = LN_l(r_l), rounded as the router input is, into LDS [H] by the whole workgroup: the routing of the layer
// runs beside this workgroup and cannot hand its own copy over in time.  Both sum the squares in double precision, from
// a thread's second group of columns on in another order.  NG = groups of 256 chunks per row.  Split in two so that the
// weight loads can be issued between the loads of r_l and the waits of the reduction.
template <typename WT, int NG>
struct InputNorm {
  static constexpr int VN = Packed<WT>::N;
  float r[NG][VN], gain[NG][VN];

  __device__ __forceinline__ void load(const ExpertArgs &a, int tid) {
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      const int c = (q * kB1Block + tid) * VN;
      const int at = c < a.H ? c : 0;
#pragma unroll
      for (int x = 0; x < VN; x += 4) {
        const float4 f = *reinterpret_cast<const float4 *>(a.r + at + x);
        const float4 g = *reinterpret_cast<const float4 *>(a.gain + at + x);
        r[q][x] = f.x; r[q][x + 1] = f.y; r[q][x + 2] = f.z; r[q][x + 3] = f.w;
        gain[q][x] = g.x; gain[q][x + 1] = g.y; gain[q][x + 2] = g.z; gain[q][x + 3] = g.w;
      }
    }
  }
  __device__ __forceinline__ void finish(const ExpertArgs &a, float *s_lds, double *red, int tid) {
    double ss = 0.0;
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      if ((q * kB1Block + tid) * VN < a.H) {
#pragma unroll
        for (int x = 0; x < VN; ++x) ss += double(r[q][x]) * double(r[q][x]);
      }
    }
    ss = wave_sum(ss);
    if ((tid & (kWave - 1)) == 0) red[tid / kWave] = ss;
    __syncthreads();
    double tot = 0.0;
#pragma unroll
    for (int w = 0; w < kB1Waves; ++w) tot += red[w];
    const double inv = 1.0 / sqrt(tot / double(a.H) + double(a.eps));
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      const int c = (q * kB1Block + tid) * VN;
      if (c < a.H) {
        float n[VN];
#pragma unroll
        for (int x = 0; x < VN; ++x) {
          double v = double(r[q][x]) * double(gain[q][x]) * inv;
          if (a.bf16) v = round_to_bf16_fast(v);
          n[x] = float(v);
        }
#pragma unroll
        for (int x = 0; x < VN; x += 4)
          *reinterpret_cast<float4 *>(s_lds + c + x) = make_float4(n[x], n[x + 1], n[x + 2], n[x + 3]);
      }
    }
    __syncthreads();
  }
};

// One row of each matrix times the vector, a lane's part.  bf16: two-element dot instructions on packed values, half the
// instructions of unpacking to float (one wavefront per SIMD issues an instruction per 8 clocks, so beside the routing they
// set the pace: 8 of 128 experts of 768 x 2048, a layer step, 22.3 -> 21.2 us; the launch by itself takes as long as
// before).  Two sums by turns, shorter chains: rms error against 64 bits at 512 / 1024 / 2048 / 4096 columns 6.3 / 6.6 / 7.5 /
// 8.3 -> 6.3 / 6.6 / 7.2 / 7.8 e-8 of the sum.
template <typename WT, int NCH>
__device__ __forceinline__ void row_sums(const typename Packed<WT>::Raw (&g)[NCH], const typename Packed<WT>::Raw (&u)[NCH],
                                         const typename Packed<WT>::Raw (&s)[NCH], float &gate, float &up) {
  float sum_g[2] = {0.f, 0.f}, sum_u[2] = {0.f, 0.f};
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
    sum_g[ch & 1] = dot_chunk(g[ch], s[ch], sum_g[ch & 1]);
    sum_u[ch & 1] = dot_chunk(u[ch], s[ch], sum_u[ch & 1]);
  }
  gate = wave_sum(sum_g[0] + sum_g[1]);
  up = wave_sum(sum_u[0] + sum_u[1]);
}

// A lane's columns of the vector s (float, rounded to the weight dtype) in the weight dtype; zeros where it has none.
template <typename WT, int NCH>
__device__ __forceinline__ void load_vector(const float *s, const int (&col)[NCH], const bool (&live)[NCH],
                                            typename Packed<WT>::Raw (&out)[NCH]) {
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
    const float4 lo = *reinterpret_cast<const float4 *>(s + col[ch]);
    if constexpr (sizeof(WT) == 2) {
      const float4 hi = *reinterpret_cast<const float4 *>(s + col[ch] + 4);
      auto pack = [&](float a, float b) { return live[ch] ? (__float_as_uint(a) >> 16) | (__float_as_uint(b) & 0xffff0000u) : 0u; };
      out[ch] = make_uint4(pack(lo.x, lo.y), pack(lo.z, lo.w), pack(hi.x, hi.y), pack(hi.z, hi.w));
    } else {
      out[ch] = live[ch] ? lo : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
}

template <typename WT>
__device__ __forceinline__ void store_product(const ExpertArgs &a, WT *at, float g, float u) {
  float hv = g / (1.f + expf(-g)) * u;
  if (a.bf16) hv = round_to_bf16(hv);
  *at = Packed<WT>::pack_one(hv);
}

// hq[pos, row] for the one token of the batch, stored in the weight dtype for the down kernel.
// slot is that of the expert at execution position pos; rows [first, last) of the expert.  Each lane keeps its NCH chunks of s_l in registers; a wavefront owns
// `rpw` consecutive rows and keeps the 2*NCH 16-byte loads of the next row in flight while it reduces the
// current one (two rows: no faster, a compute unit has as many requests on their way as it can).  NORM: s_l is formed here from
// a.r (LDS s_lds, red), else read from a.s.
template <typename WT, int NCH, bool NORM>
__device__ __forceinline__ void gateup_b1_body(const ExpertArgs &a, int slot, int pos, int block, int rpw,
                                               int first, int last, float *s_lds, double *red) {
  using R = Packed<WT>;
  constexpr int VN = R::N;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int H = a.H, I = a.I;
  const int row0 = first + (block * kB1Waves + wave) * rpw;
  if (!NORM && row0 >= last) return;
  const int row_end = min(row0 + rpw, last);
  const WT *wg = reinterpret_cast<const WT *>(a.pool + size_t(slot) * a.slot_bytes);
  const WT *wu = wg + size_t(I) * H;
  WT *hq = reinterpret_cast<WT *>(a.h) + size_t(pos) * I;
  InputNorm<WT, (NCH + 3) / 4> norm;
  if (NORM) norm.load(a, tid);

  int col[NCH];
  bool live[NCH];
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
    col[ch] = (ch * kWave + lane) * VN;
    live[ch] = col[ch] < H;
    if (!live[ch]) col[ch] = 0;                // dead lanes re-read column 0 and multiply by zero
  }
  typename R::Raw rg[NCH], ru[NCH];
  const size_t at0 = size_t(NORM ? min(row0, I - 1) : row0) * H;
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
    rg[ch] = load_stream<typename R::Raw>(wg + at0 + col[ch]);
    ru[ch] = load_stream<typename R::Raw>(wu + at0 + col[ch]);
  }
  if (NORM) norm.finish(a, s_lds, red, tid);
  typename R::Raw sv[NCH];
  load_vector<WT, NCH>(NORM ? s_lds : a.s, col, live, sv);
  for (int row = row0; row < row_end; ++row) {
    typename R::Raw fg[NCH], fu[NCH];
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) { fg[ch] = rg[ch]; fu[ch] = ru[ch]; }
    if (row + 1 < row_end) {
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        rg[ch] = load_stream<typename R::Raw>(wg + size_t(row + 1) * H + col[ch]);
        ru[ch] = load_stream<typename R::Raw>(wu + size_t(row + 1) * H + col[ch]);
      }
    }
    float g, u;
    row_sums<WT, NCH>(fg, fu, sv, g, u);
    if (lane == 0) store_product<WT>(a, hq + row, g, u);
  }
}

// Small launches (all wavefronts resident at once): a wavefront owns two consecutive rows and
// issues the 4*NCH 16-byte loads of both before it reduces anything.
template <typename WT, int NCH>
__device__ __forceinline__ void gateup_b1_pair_body(const ExpertArgs &a, int slot, int pos, int block) {
  using R = Packed<WT>;
  constexpr int VN = R::N;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int H = a.H, I = a.I;
  const int row0 = (block * kB1Waves + wave) * 2;
  if (row0 >= I) return;
  const WT *wg = reinterpret_cast<const WT *>(a.pool + size_t(slot) * a.slot_bytes);
  const WT *wu = wg + size_t(I) * H;
  WT *hq = reinterpret_cast<WT *>(a.h) + size_t(pos) * I;

  int col[NCH];
  bool live[NCH];
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
    col[ch] = (ch * kWave + lane) * VN;
    live[ch] = col[ch] < H;
    if (!live[ch]) col[ch] = 0;                // dead lanes re-read column 0 and multiply by zero
  }
  typename R::Raw rg[2][NCH], ru[2][NCH];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int row = min(row0 + r, I - 1);      // an odd last row is loaded twice and stored once
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      rg[r][ch] = load_stream<typename R::Raw>(wg + size_t(row) * H + col[ch]);
      ru[r][ch] = load_stream<typename R::Raw>(wu + size_t(row) * H + col[ch]);
    }
  }
  typename R::Raw sv[NCH];
  load_vector<WT, NCH>(a.s, col, live, sv);
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    if (row0 + r >= I) break;
    float g, u;
    row_sums<WT, NCH>(rg[r], ru[r], sv, g, u);
    if (lane == 0) store_product<WT>(a, hq + row0 + r, g, u);
  }
}

}  // namespace moe_spec
