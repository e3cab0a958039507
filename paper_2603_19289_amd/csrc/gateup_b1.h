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

// hq[pos, row] for the one token of the batch, stored in the weight dtype for the down kernel.
// `act` is in execution-position order; rows [first, last) of the expert.  Each lane keeps its NCH chunks of s_l in registers; a wavefront owns
// `rpw` consecutive rows and keeps the 2*NCH 16-byte loads of the next row in flight while it reduces the
// current one.  NORM: s_l is formed here from a.r (LDS s_lds, red), else read from a.s.
template <typename WT, int NCH, bool NORM>
__device__ __forceinline__ void gateup_b1_body(const ExpertArgs &a, const ActiveList &act, int pos, int block, int rpw,
                                               int first, int last, float *s_lds, double *red) {
  using R = Packed<WT>;
  constexpr int VN = R::N;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int H = a.H, I = a.I;
  const int row0 = first + (block * kB1Waves + wave) * rpw;
  if (!NORM && row0 >= last) return;
  const int row_end = min(row0 + rpw, last);
  const WT *wg = reinterpret_cast<const WT *>(a.pool + size_t(act.slot[pos]) * a.slot_bytes);
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
  const float *s = NORM ? s_lds : a.s;
  float sv[NCH][VN];
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
#pragma unroll
    for (int x = 0; x < VN; x += 4) {
      const float4 f = *reinterpret_cast<const float4 *>(s + col[ch] + x);
      const float m = live[ch] ? 1.f : 0.f;
      sv[ch][x] = f.x * m; sv[ch][x + 1] = f.y * m; sv[ch][x + 2] = f.z * m; sv[ch][x + 3] = f.w * m;
    }
  }
  for (int row = row0; row < row_end; ++row) {
    float ag = 0.f, au = 0.f;
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      float fg[VN], fu[VN];
      R::unpack(rg[ch], fg);
      R::unpack(ru[ch], fu);
#pragma unroll
      for (int x = 0; x < VN; ++x) { ag += fg[x] * sv[ch][x]; au += fu[x] * sv[ch][x]; }
    }
    if (row + 1 < row_end) {
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch) {
        rg[ch] = load_stream<typename R::Raw>(wg + size_t(row + 1) * H + col[ch]);
        ru[ch] = load_stream<typename R::Raw>(wu + size_t(row + 1) * H + col[ch]);
      }
    }
    const float g = wave_sum(ag);
    const float u = wave_sum(au);
    if (lane == 0) {
      float hv = g / (1.f + expf(-g)) * u;
      if (a.bf16) hv = round_to_bf16(hv);
      hq[row] = R::pack_one(hv);
    }
  }
}

// Small launches (all wavefronts resident at once): a wavefront owns two consecutive rows and
// issues the 4*NCH 16-byte loads of both before it reduces anything.
template <typename WT, int NCH>
__device__ __forceinline__ void gateup_b1_pair_body(const ExpertArgs &a, const ActiveList &act, int pos, int block) {
  using R = Packed<WT>;
  constexpr int VN = R::N;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int H = a.H, I = a.I;
  const int row0 = (block * kB1Waves + wave) * 2;
  if (row0 >= I) return;
  const WT *wg = reinterpret_cast<const WT *>(a.pool + size_t(act.slot[pos]) * a.slot_bytes);
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
  float sv[NCH][VN];
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
#pragma unroll
    for (int x = 0; x < VN; x += 4) {
      const float4 f = *reinterpret_cast<const float4 *>(a.s + col[ch] + x);
      const float m = live[ch] ? 1.f : 0.f;
      sv[ch][x] = f.x * m; sv[ch][x + 1] = f.y * m; sv[ch][x + 2] = f.z * m; sv[ch][x + 3] = f.w * m;
    }
  }
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    if (row0 + r >= I) break;
    float ag = 0.f, au = 0.f;
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      float fg[VN], fu[VN];
      R::unpack(rg[r][ch], fg);
      R::unpack(ru[r][ch], fu);
#pragma unroll
      for (int x = 0; x < VN; ++x) { ag += fg[x] * sv[ch][x]; au += fu[x] * sv[ch][x]; }
    }
    const float g = wave_sum(ag);
    const float u = wave_sum(au);
    if (lane == 0) {
      float hv = g / (1.f + expf(-g)) * u;
      if (a.bf16) hv = round_to_bf16(hv);
      hq[row0 + r] = R::pack_one(hv);
    }
  }
}

}  // namespace moe_spec
