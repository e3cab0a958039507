// route_pair_kernel: the true routing of layer l AND the prediction for layer l+1 in one launch
// (paper: Sec. 3.1-3.3; Algorithm 1, TopK(Gate_l(X)) and GetNextExperts): RMSNorm, router l, top-k, gates,
// d_l, q_l, router l+1, top-k, gates.
//
// Logits are handed from the workgroups that compute them to the workgroups that need them inside
// the launch.  The hand-over is "the data is the flag": a slot of global memory holds a bit pattern that
// no result can have (all ones: a NaN) until its producer overwrites it with one relaxed device-scope
// atomic store; consumers read the slot with relaxed device-scope atomic loads until it no longer holds
// that pattern.  Each slot is a single atomic object, so nothing has to be ordered against anything
// else: no fence, no counter, no wait for a store's acknowledgement.  Slots come in two sets used by
// alternate launches; a launch re-arms the set the next launch will use (the previous launch, which
// read that set, has ended).  Every wait is bounded: after `spin_limit` polls a waiter gives up, raises
// the status word and finishes with whatever it has, so every wavefront reaches its end.
// Who may wait for whom: a workgroup only waits for the other workgroups of its own token, which the
// launcher checks to fit on the device together (groups are dispatched in order, so the earliest
// unfinished group always gets the next free compute units).
#include <type_traits>

#include "device_utils.h"
#include "expert_mfma.h"
#include "gateup_b1.h"
#include "kernels.h"
#include "launch_rules.h"
#include "route_select.h"

namespace moe_spec {
namespace {

// Products of rows first, first + stride, ... of mat [n_rows,H] with the vector in LDS (laid out as in route_pair_body)
// by one wavefront: sink(row, sum) in every lane.  Four chunks of two rows per step, the next step's on their way
// meanwhile.  AS_FLOAT: the products take the vector's values as float, as it is handed on wherever it is stored.
template <typename WT, bool AS_FLOAT, typename Sink>
__device__ __forceinline__ void rows_dot(const WT *mat, int n_rows, int H, int first, int stride, const double *vec_lds,
                                         Sink sink) {
  using P = Packed<WT>;
  using Raw = typename P::Raw;
  constexpr int VN = P::N;
  const int lane = threadIdx.x & (kWave - 1), G = H / VN;
  const int steps = (H + 4 * kWave * VN - 1) / (4 * kWave * VN);
  const int mine = first < n_rows ? (n_rows - 1 - first) / stride + 1 : 0;
  const int total = (mine + 1) / 2 * steps;
  auto fetch = [&](int i, Raw (&dst)[2][4]) {  // step i of this wavefront's list of row pairs x steps
#pragma unroll
    for (int p = 0; p < 2; ++p) {              // an odd last row is read twice
      const WT *src = mat + size_t(first + min(i / steps * 2 + p, mine - 1) * stride) * H;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int c = ((i % steps * 4 + u) * kWave + lane) * VN;
        dst[p][u] = *reinterpret_cast<const Raw *>(src + (c < H ? c : 0));
      }
    }
  };
  Raw cur[2][4], next[2][4];
  if (mine > 0) fetch(0, cur);
  double acc[2] = {0.0, 0.0};
  for (int i = 0; i < total; ++i) {
    if (i + 1 < total) fetch(i + 1, next);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = ((i % steps * 4 + u) * kWave + lane) * VN;
      if (c < H) {
        float w0[VN], w1[VN];
        P::unpack(cur[0][u], w0);
        P::unpack(cur[1][u], w1);
#pragma unroll
        for (int x = 0; x < VN; ++x) {
          double v = vec_lds[x * G + c / VN];
          if (AS_FLOAT) v = double(float(v));
          acc[0] += double(w0[x]) * v;
          acc[1] += double(w1[x]) * v;
        }
      }
    }
    if (i % steps == steps - 1) {
      const int j = i / steps * 2;
      sink(first + j * stride, wave_sum(acc[0]));
      const double second = wave_sum(acc[1]);
      if (j + 1 < mine) sink(first + (j + 1) * stride, second);
      acc[0] = acc[1] = 0.0;
    }
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int u = 0; u < 4; ++u) cur[p][u] = next[p][u];
  }
}

// The hand-over slots of the launch that takes proj_out further.
__device__ __forceinline__ void arm_estimator(const RoutePairArgs &a, int first, int stride) {
  for (int i = first; i < a.est_t_count; i += stride) arm64(a.est_t + i);
  for (int i = first; i < a.est_v_count; i += stride) arm64(a.est_v + i);
}

// proj_out = proj q_l + proj_add, the rows of one wavefront.
template <typename WT>
__device__ __forceinline__ void project_rows(const RoutePairArgs &a, int b, int first, int stride, const double *vec_lds) {
  constexpr int VN = Packed<WT>::N;
  const int lane = threadIdx.x & (kWave - 1);
  rows_dot<WT, true>(static_cast<const WT *>(a.proj), a.proj_rows, a.H, first, stride, vec_lds, [&](int r, double sum) {
    if (lane == 0) {
      float add[VN];
      load_chunk<WT>(static_cast<const WT *>(a.proj_add) + r / VN * VN, add);
      a.proj_out[size_t(b) * a.proj_rows + r] = sum + double(add[r % VN]);
    }
  });
}

// SPLIT wavefronts share one router row (4 / SPLIT rows per workgroup); NCH 16-byte chunks of the row
// per lane, loaded into registers for both routers at the top of the kernel so that their latency
// overlaps the normalisation.  b is the token; the workgroups of a token form a group that
// exchanges logits through the token's slots and computes everything else redundantly (the norm, the
// top-k, the default-vector sum), so that nothing but the 8-byte logits crosses between workgroups.
// Workgroup 0 of a token finishes the prediction; the last one reports the true routing, off the path
// that the prediction waits on.
// PROJ: the estimator's projection takes the place of the prediction (a kernel of its own: the other path measured 3 %
// slower with the branch in it).
template <typename WT, int SPLIT, int NCH, int ROWS, bool PROJ>
__device__ __forceinline__ void route_pair_body(const RoutePairArgs &a, const int wg, const int n_wg, const int b,
                                                const int n_tokens, double *vec_lds, RouteShared &sh,
                                                const SlotTable *resident = nullptr) {
  static_assert(ROWS == 1 || SPLIT == 1, "several rows per wavefront only with one wavefront per row");
  // The router input being built, double precision, H values.  Threads own groups of VN consecutive columns (in
  // the norms: group tid, tid + 256, ...; in the products: the groups of the wavefront's chunks); column x of
  // group o lives at word x * G + o, so that the lanes of a wavefront, which hold consecutive groups, touch
  // consecutive words whatever x is (with the columns in their natural order every access of a wavefront fell
  // on a few banks)
  using P = Packed<WT>;
  using Raw = typename P::Raw;
  constexpr int VN = P::N;
  constexpr int RPW = kWaves / SPLIT * ROWS;   // rows per workgroup

  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int H = a.H, E = a.E, k = a.k;
  const int G = H / VN;                        // column groups (H is a multiple of 8)
  const double inv_h = 1.0 / double(H);
#define V(c, x) vec_lds[(x) * G + (c) / VN]
  const int row = wg * RPW + wave / SPLIT * ROWS, part = wave % SPLIT;   // this wavefront's (first) row
  const bool pred = PROJ || a.w_next != nullptr;
  const WT *wt = static_cast<const WT *>(a.w_true);
  const WT *wn = static_cast<const WT *>(a.w_next);
  const float *rrow = a.r + size_t(b) * H;
  const int c0 = tid * VN;                     // this thread's columns of the first pass over the row
  STAGE(0);

  // ---- loads that depend on nothing, in the order they are needed: r_l and the gain first, then this
  // wavefront's part of its router rows (waited for at the products only)
  float r0[VN], g0[VN];
  if (c0 < H) {
#pragma unroll
    for (int x = 0; x < VN; x += 4) {
      const float4 f = *reinterpret_cast<const float4 *>(rrow + c0 + x);
      const float4 g = *reinterpret_cast<const float4 *>(a.gain_true + c0 + x);
      r0[x] = f.x; r0[x + 1] = f.y; r0[x + 2] = f.z; r0[x + 3] = f.w;
      g0[x] = g.x; g0[x + 1] = g.y; g0[x + 2] = g.z; g0[x + 3] = g.w;
    }
  }
  Raw rt[NCH], rn[NCH];                        // one row per wavefront: both routers' rows travel in registers
  if (ROWS == 1 && row < E) {
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      const int c = ((ch * SPLIT + part) * kWave + lane) * VN;
      rt[ch] = *reinterpret_cast<const Raw *>(wt + size_t(row) * H + (c < H ? c : 0));
      if (!PROJ && pred) rn[ch] = *reinterpret_cast<const Raw *>(wn + size_t(row) * H + (c < H ? c : 0));
    }
  }
  // re-arm the whole set of slots the next launch will use (last read by the previous launch, which has
  // ended), for every token the context allows: the next launch may carry a larger batch than this one
  for (int i = (b * n_wg + wg) * kBlock + tid; i < a.arm_count; i += n_wg * n_tokens * kBlock) {
    arm64(a.z_true_next + i);
    arm64(a.z_pred_next + i);
  }
  if constexpr (PROJ) arm_estimator(a, (b * n_wg + wg) * kBlock + tid, n_wg * n_tokens * kBlock);

  // ---- s_l = LN_l(r_l)
  {
    double ss = 0.0;
    double v0[VN];                               // this thread's first columns stay in registers until they are final
    if (c0 < H) {
#pragma unroll
      for (int x = 0; x < VN; ++x) { v0[x] = double(r0[x]) * double(g0[x]); ss += double(r0[x]) * double(r0[x]); }
    }
    for (int c = c0 + kBlock * VN; c < H; c += kBlock * VN) {
#pragma unroll
      for (int x = 0; x < VN; x += 4) {
        const float4 f = *reinterpret_cast<const float4 *>(rrow + c + x);
        const float4 g = *reinterpret_cast<const float4 *>(a.gain_true + c + x);
        V(c, x) = double(f.x) * double(g.x); V(c, x + 1) = double(f.y) * double(g.y);
        V(c, x + 2) = double(f.z) * double(g.z); V(c, x + 3) = double(f.w) * double(g.w);
        ss += double(f.x) * double(f.x) + double(f.y) * double(f.y) + double(f.z) * double(f.z) + double(f.w) * double(f.w);
      }
    }
    const double inv = rsqrt(block_sum(ss, sh.red[0], lane, wave) * inv_h + double(a.eps));
    for (int c = c0; c < H; c += kBlock * VN) {
#pragma unroll
      for (int x = 0; x < VN; ++x) {
        double n = (c == c0 ? v0[x] : V(c, x)) * inv;
        if (a.bf16) n = round_to_bf16_fast(n);
        V(c, x) = n;
      }
      if (wg == 0) {                             // s_l for the expert kernels, 16 bytes per store
#pragma unroll
        for (int x = 0; x < VN; x += 4)
          *reinterpret_cast<float4 *>(a.s_out + size_t(b) * H + c + x) =
              make_float4(float(V(c, x)), float(V(c, x + 1)), float(V(c, x + 2)), float(V(c, x + 3)));
        if (a.s_out_q) {
#pragma unroll
          for (int x = 0; x < VN; x += 2)
            *reinterpret_cast<uint32_t *>(a.s_out_q + size_t(b) * H + c + x) =
                (__float_as_uint(float(V(c, x))) >> 16) | (__float_as_uint(float(V(c, x + 1))) & 0xffff0000u);
        }
      }
    }
    __syncthreads();
  }
  STAGE(1);
  // ---- logits of a router: one row per SPLIT wavefronts from the registers loaded above, or (batches) ROWS
  //      rows per wavefront read where they are used, the router being in L2 after the first tokens
  auto dot_row = [&](const Raw (&w)[NCH]) {
    double acc = 0.0;
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      const int c = ((ch * SPLIT + part) * kWave + lane) * VN;
      if (c < H) {
        float wf[VN];
        P::unpack(w[ch], wf);
#pragma unroll
        for (int x = 0; x < VN; ++x) acc += double(wf[x]) * V(c, x);
      }
    }
    return wave_sum(acc);
  };
  auto publish_rows = [&](const Raw (&held)[NCH], const WT *wmat, unsigned long long *slots) {
    if (ROWS > 1) {
      Raw w[2][NCH];
      auto fetch = [&](int rr, Raw (&dst)[NCH]) {
        const int rclamped = min(row + rr, E - 1);
#pragma unroll
        for (int ch = 0; ch < NCH; ++ch) {
          const int c = (ch * kWave + lane) * VN;
          dst[ch] = *reinterpret_cast<const Raw *>(wmat + size_t(rclamped) * H + (c < H ? c : 0));
        }
      };
      fetch(0, w[0]);
#pragma unroll
      for (int rr = 0; rr < ROWS; ++rr) {
        if (rr + 1 < ROWS) fetch(rr + 1, w[(rr + 1) & 1]);
        const double acc = dot_row(w[rr & 1]);
        if (lane == 0 && row + rr < E) publish64(slots + size_t(b) * E + row + rr, acc);
      }
    } else if (SPLIT == 1) {
      const double acc = row < E ? dot_row(held) : 0.0;
      if (lane == 0 && row < E) publish64(slots + size_t(b) * E + row, acc);
    } else {
      const double acc = row < E ? dot_row(held) : 0.0;
      if (lane == 0) sh.part[wave] = acc;
      __syncthreads();
      if (tid < RPW && wg * RPW + tid < E) {
        double s = 0.0;
#pragma unroll
        for (int p = 0; p < SPLIT; ++p) s += sh.part[tid * SPLIT + p];
        publish64(slots + size_t(b) * E + wg * RPW + tid, s);
      }
    }
  };
  publish_rows(rt, wt, a.z_true);
  STAGE(2);
  const int reporter = n_wg - 1;
  if (!pred && wg != reporter) return;

  // ---- (E_l, G_l): every workgroup of the token selects for itself
  select_ids_any(a, 3, a.z_true + size_t(b) * E, E, k, sh.sel, tid);
  STAGE(4);
  // the first eight default-vector rows, asked for as soon as the ids are known; the gates follow meanwhile
  const WT *dv = static_cast<const WT *>(a.dvec);
  Raw dr0[8];
  if (pred && c0 < H) {
#pragma unroll
    for (int q = 0; q < 8; ++q) dr0[q] = *reinterpret_cast<const Raw *>(dv + size_t(sh.sel.top_i[min(q, k - 1)]) * H + c0);
  }
  float gn0[VN];
  if (pred && c0 < H) {
#pragma unroll
    for (int x = 0; x < VN; x += 4) {
      const float4 g = *reinterpret_cast<const float4 *>(a.gain_next + c0 + x);
      gn0[x] = g.x; gn0[x + 1] = g.y; gn0[x + 2] = g.z; gn0[x + 3] = g.w;
    }
  }
  const double denom = select_gates(k, sh.sel, tid);
  if (wg == reporter) report_true(a, b, sh.sel, denom, tid, resident);
  STAGE(5);
  if (!pred) return;

  // ---- d_l = sum_j g_j d_{l,e_j};  q_l = LN_{l+1}(r_l + d_l)   (or s_l + d_l, the caption's reading)
  {
    const double inv_denom = 1.0 / denom;
    double ss = 0.0;
    double q0[VN];                               // as in the first norm: the first columns stay in registers
    for (int c = c0; c < H; c += kBlock * VN) {
      const bool first = c == c0;
      double u[VN];
      if (a.from_normalized) {
#pragma unroll
        for (int x = 0; x < VN; ++x) u[x] = V(c, x);
      } else if (first) {
#pragma unroll
        for (int x = 0; x < VN; ++x) u[x] = r0[x];
      } else {
#pragma unroll
        for (int x = 0; x < VN; x += 4) {
          const float4 f = *reinterpret_cast<const float4 *>(rrow + c + x);
          u[x] = f.x; u[x + 1] = f.y; u[x + 2] = f.z; u[x + 3] = f.w;
        }
      }
      double d[VN];
#pragma unroll
      for (int x = 0; x < VN; ++x) d[x] = 0.0;
      for (int j0 = 0; j0 < k; j0 += 8) {              // eight default-vector rows in flight
        Raw dr[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          if (first && j0 == 0) dr[q] = dr0[q];
          else dr[q] = *reinterpret_cast<const Raw *>(dv + size_t(sh.sel.top_i[min(j0 + q, k - 1)]) * H + c);
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          if (j0 + q < k) {
            const double g = sh.sel.top_e[wave][j0 + q] * inv_denom;
            float dvf[VN];
            P::unpack(dr[q], dvf);
#pragma unroll
            for (int x = 0; x < VN; ++x) d[x] += g * double(dvf[x]);
          }
        }
      }
      float gf[VN];
      if (first) {
#pragma unroll
        for (int x = 0; x < VN; ++x) gf[x] = gn0[x];
      } else {
#pragma unroll
        for (int x = 0; x < VN; x += 4) {
          const float4 g = *reinterpret_cast<const float4 *>(a.gain_next + c + x);
          gf[x] = g.x; gf[x + 1] = g.y; gf[x + 2] = g.z; gf[x + 3] = g.w;
        }
      }
#pragma unroll
      for (int x = 0; x < VN; ++x) {
        const double ux = u[x] + d[x];
        if (first) q0[x] = ux * double(gf[x]);
        else V(c, x) = ux * double(gf[x]);
        ss += ux * ux;
      }
    }
    STAGE(6);
    const double inv = rsqrt(block_sum(ss, sh.red[1], lane, wave) * inv_h + double(a.eps));
    for (int c = c0; c < H; c += kBlock * VN) {
#pragma unroll
      for (int x = 0; x < VN; ++x) {
        double n = (c == c0 ? q0[x] : V(c, x)) * inv;
        if (a.bf16) n = round_to_bf16_fast(n);
        V(c, x) = n;
      }
    }
    __syncthreads();
  }
  STAGE(7);
  if constexpr (PROJ) {
    // The wavefronts of the token's workgroups take the projection's rows in pairs, in turn; the launcher sizes their
    // number for that.  q_l is here anyway: 4 tokens of 128 experts of 2048 columns, latent size 512, 15.0 us in this
    // launch, against 9.1 us for the true routing alone, 14.7 us for a second routing that only yields q_l and 7.4 us
    // for the product by itself.
    project_rows<WT>(a, b, wg * kWaves + wave, n_wg * kWaves, vec_lds);
    return;
  }
  publish_rows(rn, wn, a.z_pred);
  STAGE(8);
  if (wg != 0) return;

  // ---- (E^_{l+1}, G^_{l+1})
  select_ids_any(a, 9, a.z_pred + size_t(b) * E, E, k, sh.sel, tid,
                 a.mb_next ? a.mb_next->ids + size_t(b) * k : nullptr);                  // the host starts the prefetch on these
  const double denom_next = select_gates(k, sh.sel, tid);
  STAGE(10);
  report_next(a, b, sh.sel, denom_next, tid);
  STAGE(11);
#undef V
}

template <typename WT, int SPLIT, int NCH, int ROWS, bool PROJ>
__global__ __launch_bounds__(kBlock) void route_pair_kernel(const RoutePairArgs a, const SlotTable resident) {
  extern __shared__ double vec_lds[];
  __shared__ RouteShared sh;
  route_pair_body<WT, SPLIT, NCH, ROWS, PROJ>(a, blockIdx.x, gridDim.x, blockIdx.y, gridDim.y, vec_lds, sh, &resident);
}

// The same routing for a launch in which expert workgroups hide its latency: nothing is kept in registers or asked for
// early, so that it does not take registers away from them (about 200 in route_pair_body).  The double-precision sums are
// those of route_pair_body in its order, but for the squares of a norm, which it adds in fours from a thread's second
// group of columns on.  Router rows are dealt over the wavefronts of the token's n_wg workgroups, any number of them.
template <typename WT, bool PROJ>
__device__ __forceinline__ void route_lean_body(const RoutePairArgs &a, const int wg, const int n_wg, const int b,
                                                const int n_tokens, double *vec_lds, RouteShared &sh) {
  using P = Packed<WT>;
  using Raw = typename P::Raw;
  constexpr int VN = P::N;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int H = a.H, E = a.E, k = a.k, G = H / VN;
  const double inv_h = 1.0 / double(H);
#define V(c, x) vec_lds[(x) * G + (c) / VN]
  const bool pred = PROJ || a.w_next != nullptr;
  const float *rrow = a.r + size_t(b) * H;
  const int c0 = tid * VN, first = wg * kWaves + wave, stride = n_wg * kWaves;
  for (int i = (b * n_wg + wg) * kBlock + tid; i < a.arm_count; i += n_wg * n_tokens * kBlock) {
    arm64(a.z_true_next + i);
    arm64(a.z_pred_next + i);
  }
  if constexpr (PROJ) arm_estimator(a, (b * n_wg + wg) * kBlock + tid, n_wg * n_tokens * kBlock);
  auto finish_norm = [&](double ss, double *red, bool write) {      // V holds x * gain
    const double inv = rsqrt(block_sum(ss, red, lane, wave) * inv_h + double(a.eps));
    for (int c = c0; c < H; c += kBlock * VN) {
#pragma unroll
      for (int x = 0; x < VN; ++x) {
        double n = V(c, x) * inv;
        if (a.bf16) n = round_to_bf16_fast(n);
        V(c, x) = n;
      }
      if (write) {
#pragma unroll
        for (int x = 0; x < VN; x += 4)
          *reinterpret_cast<float4 *>(a.s_out + size_t(b) * H + c + x) =
              make_float4(float(V(c, x)), float(V(c, x + 1)), float(V(c, x + 2)), float(V(c, x + 3)));
      }
    }
    __syncthreads();
  };
  double ss = 0.0;
  for (int c = c0; c < H; c += kBlock * VN) {
#pragma unroll
    for (int x = 0; x < VN; ++x) {
      const double r = double(rrow[c + x]);
      V(c, x) = r * double(a.gain_true[c + x]);
      ss += r * r;
    }
  }
  finish_norm(ss, sh.red[0], wg == 0);
  auto publish_rows = [&](const void *router, unsigned long long *slots) {
    rows_dot<WT, false>(static_cast<const WT *>(router), E, H, first, stride, vec_lds, [&](int r, double sum) {
      if (lane == 0) publish64(slots + size_t(b) * E + r, sum);
    });
  };
  publish_rows(a.w_true, a.z_true);
  const int reporter = n_wg - 1;
  if (!pred && wg != reporter) return;

  select_ids_any(a, 3, a.z_true + size_t(b) * E, E, k, sh.sel, tid);
  const double denom = select_gates(k, sh.sel, tid);
  if (wg == reporter) report_true(a, b, sh.sel, denom, tid, nullptr);
  if (!pred) return;

  const WT *dv = static_cast<const WT *>(a.dvec);
  const double inv_denom = 1.0 / denom;
  ss = 0.0;
  for (int c = c0; c < H; c += kBlock * VN) {
    double d[VN];
#pragma unroll
    for (int x = 0; x < VN; ++x) d[x] = 0.0;
    for (int j0 = 0; j0 < k; j0 += 4) {                // four default-vector rows in flight
      Raw dr[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) dr[q] = *reinterpret_cast<const Raw *>(dv + size_t(sh.sel.top_i[min(j0 + q, k - 1)]) * H + c);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (j0 + q < k) {
          const double g = sh.sel.top_e[wave][j0 + q] * inv_denom;
          float dvf[VN];
          P::unpack(dr[q], dvf);
#pragma unroll
          for (int x = 0; x < VN; ++x) d[x] += g * double(dvf[x]);
        }
      }
    }
#pragma unroll
    for (int x = 0; x < VN; ++x) {
      const double ux = (a.from_normalized ? V(c, x) : double(rrow[c + x])) + d[x];
      V(c, x) = ux * double(a.gain_next[c + x]);
      ss += ux * ux;
    }
  }
  finish_norm(ss, sh.red[1], false);
  if constexpr (PROJ) {
    project_rows<WT>(a, b, first, stride, vec_lds);
    return;
  }
  publish_rows(a.w_next, a.z_pred);
  if (wg != 0) return;

  select_ids_any(a, 9, a.z_pred + size_t(b) * E, E, k, sh.sel, tid, a.mb_next ? a.mb_next->ids + size_t(b) * k : nullptr);
  const double denom_next = select_gates(k, sh.sel, tid);
  report_next(a, b, sh.sel, denom_next, tid);
#undef V
}

// The routing of a layer and the gate/up projection of its experts, which were predicted one layer earlier, in one
// launch for a batch of one.  The first n_route workgroups route (they are dispatched first, so they are resident
// together), the others stream expert rows; these form s_l themselves.  NCH: chunks of a weight row per lane.
// A compute unit streams up to 28 GB/s from memory however many loads it has in flight, so each one that routes instead is
// missed: two router rows per workgroup.  8 of 128 experts of 768 x 2048, a layer step, 1 / 2 / 4 rows per workgroup:
// 23.9 / 22.3 / 22.4 us, with the dot instructions of row_sums 24.5 / 21.2 / 21.6 (128 / 64 / 32 workgroups; 4 of 32
// of 2880 x 2880 and 2 of 8 of 14336 x 4096 within 1 % of one another).
template <typename WT, int NCH>
__global__ __launch_bounds__(kBlock, 2)
void route_gateup_b1_kernel(const RoutePairArgs ra, const ExpertArgs a, const ActiveList act, const int n_route,
                            const SharedSplit split) {
  extern __shared__ double vec_lds[];
  __shared__ RouteShared sh;
  int i = int(blockIdx.x) - n_route, blocks = split.stream.blocks, rpw = split.stream.rpw, first = 0, last = split.first_tail;
  if (i < 0) {
    route_pair_body<WT, kJointSplit, (NCH + kJointSplit - 1) / kJointSplit, 1, false>(ra, blockIdx.x, n_route, 0, 1, vec_lds, sh);
    i = int(blockIdx.x) - 1;
    blocks = split.tail_blocks;
    if (i < 0 || i >= blocks * act.n) return;
    rpw = split.tail_rpw;
    first = last;
    last = a.I;
    __syncthreads();                           // the routing's last readers of the shared memory are done
  }
  float *s_lds = reinterpret_cast<float *>(vec_lds);
  gateup_b1_body<WT, NCH, true>(a, act.slot[i / blocks], i / blocks, i % blocks, rpw, first, last, s_lds, sh.red[0]);
}

// s_l = LN_l(r_l) as bf16, one workgroup per token: what the expert workgroups of the launch below read.
template <int NG>
__global__ __launch_bounds__(kBlock) void norm_rows_kernel(const ExpertArgs a, uint16_t *s_q) {
  extern __shared__ float s_lds[];
  __shared__ double red[kWaves];
  const int tid = threadIdx.x, b = blockIdx.x;
  ExpertArgs row = a;
  row.r = a.r + size_t(b) * a.H;
  InputNorm<uint16_t, NG> norm;
  norm.load(row, tid);
  norm.finish(row, s_lds, red, tid);
  for (int c = tid * 8; c < a.H; c += kBlock * 8) {
    uint32_t w[4];
#pragma unroll
    for (int x = 0; x < 4; ++x)
      w[x] = (__float_as_uint(s_lds[c + 2 * x]) >> 16) | (__float_as_uint(s_lds[c + 2 * x + 1]) & 0xffff0000u);
    *reinterpret_cast<uint4 *>(s_q + size_t(b) * a.H + c) = make_uint4(w[0], w[1], w[2], w[3]);
  }
}

// The routing of a layer and the matrix-core gate/up projection of its experts, predicted one layer earlier, in one
// launch.  The first n_route workgroups route, n_wg per token (dispatched first: a token's are resident together).
// Measured, routing + gate/up as two launches against this one and the norm before it: 8 tokens of 32 experts of
// 2880 x 2880 15.5 + 114 / 4.7 + 106 us, 32 tokens of 128 experts of 768 x 2048 20 + 42 / 4.2 + 47 to 51 us, 4 tokens of
// those with the estimator's projection 13 + 32 / 4 + 32 us.  One router row and two default-vector rows in flight
// per wavefront instead of two and four: 4 % slower for the second.  Three wavefronts per SIMD with one token tile: the
// gate/up body holds 151 registers.
template <int NT, int KSPLIT, bool PROJ>
__global__ __launch_bounds__(kBlock, NT <= 1 ? 3 : NT == 4 && KSPLIT == 1 ? 1 : 2)
void route_gateup_mfma_kernel(const RoutePairArgs ra, const ExpertArgs a, const TokenLists lists, const uint16_t *s_q,
                              uint16_t *hq, const int n_wg, const int n_route, const int row_blocks, const int stream) {
  extern __shared__ __align__(16) unsigned char beside_lds[];
  if (int(blockIdx.x) < n_route) {
    RouteShared &sh = *reinterpret_cast<RouteShared *>(beside_lds);
    double *vec_lds = reinterpret_cast<double *>(beside_lds + (sizeof(RouteShared) + 15) / 16 * 16);
    route_lean_body<uint16_t, PROJ>(ra, blockIdx.x % n_wg, n_wg, blockIdx.x / n_wg, n_route / n_wg, vec_lds, sh);
    return;
  }
  const int i = blockIdx.x - n_route;
  ExpertMfmaShared<true, NT, KSPLIT> &sh = *reinterpret_cast<ExpertMfmaShared<true, NT, KSPLIT> *>(beside_lds);
  if (stream) expert_mfma_body<true, NT, KSPLIT, kOneChain>(a, DecodeTokens<true>{lists, i / row_blocks}, s_q, hq, i % row_blocks, sh);
  else expert_mfma_body<true, NT, KSPLIT, kOneChain>(a, DecodeTokens<false>{lists, i / row_blocks}, s_q, hq, i % row_blocks, sh);
}

// ---------------------------------------------------------------------------------------------
// Launchers

int g_compute_units = 0;

template <typename K>
hipError_t prepare_kernel(K kernel, size_t lds, int *blocks_per_cu) {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, 96 << 10);
  if (e != hipSuccess) return e;
  if (g_compute_units == 0) {
    int dev = 0;
    if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
    if ((e = hipDeviceGetAttribute(&g_compute_units, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
  }
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, kernel, kBlock, lds);
}

template <typename WT, int SPLIT, int NCH, int ROWS, bool PROJ>
hipError_t launch_route_pair_p(const RoutePairArgs &a, hipStream_t st) {
  constexpr int RPW = kWaves / SPLIT * ROWS;
  const size_t lds = size_t(a.H) * sizeof(double);
  static int blocks_per_cu = -1;               // per instantiation
  static size_t checked_lds = 0;
  if (blocks_per_cu < 0 || lds > checked_lds) {
    int n = 0;
    hipError_t e = prepare_kernel(route_pair_kernel<WT, SPLIT, NCH, ROWS, PROJ>, lds, &n);
    if (e != hipSuccess) return e;
    blocks_per_cu = n;
    checked_lds = lds;
  }
  const int n_wg = routing_workgroups(a.E, RPW, PROJ ? a.proj_rows : 0, a.B, g_compute_units);
  // the workgroups of a token wait for one another: they must fit on the device together
  if (long(n_wg) > long(blocks_per_cu) * g_compute_units) return hipErrorLaunchOutOfResources;
  hipLaunchKernelGGL((route_pair_kernel<WT, SPLIT, NCH, ROWS, PROJ>), dim3(n_wg, a.B), dim3(kBlock), lds, st, a,
                     a.slots_out ? *a.resident : SlotTable());
  return hipGetLastError();
}

template <typename WT, int SPLIT, int NCH, int ROWS>
hipError_t launch_route_pair_n(const RoutePairArgs &a, hipStream_t st) {
  return a.proj ? launch_route_pair_p<WT, SPLIT, NCH, ROWS, true>(a, st)
                : launch_route_pair_p<WT, SPLIT, NCH, ROWS, false>(a, st);
}

template <typename WT, int SPLIT, int ROWS>
hipError_t launch_route_pair_s(const RoutePairArgs &a, int need, hipStream_t st) {
  if (need <= 1) return launch_route_pair_n<WT, SPLIT, 1, ROWS>(a, st);
  if (need <= 2) return launch_route_pair_n<WT, SPLIT, 2, ROWS>(a, st);
  if (need <= 4) return launch_route_pair_n<WT, SPLIT, 4, ROWS>(a, st);
  if (need <= 8) return launch_route_pair_n<WT, SPLIT, 8, ROWS>(a, st);
  return hipErrorInvalidValue;
}

template <typename WT>
hipError_t launch_route_pair_t(const RoutePairArgs &a, hipStream_t st) {
  const int chunks = (a.H + Packed<WT>::N - 1) / Packed<WT>::N;
  const int need1 = (chunks + kWave - 1) / kWave;              // per lane, one wavefront per row
  const int need4 = (chunks + 4 * kWave - 1) / (4 * kWave);    // four wavefronts per row
  // One token: a workgroup per router row, E workgroups (measured on 128 experts of 2048 columns: 11.4 us per
  // launch).  A batch: its tokens already fill the device, and every workgroup repeats its token's norm, top-k
  // and default-vector sum, so the more tokens, the more rows per workgroup: 4 up to about 512 workgroups per
  // launch, 16 beyond (measured before the polls were thinned out, which took about another
  // 0.5 us off each: 8 tokens x 128 experts: 13.5 us with 4 rows per workgroup, 14.4 with 8, 16.7 with 16;
  // 32 tokens: 28.6, 17.3, 17.3 us; 64 tokens: 53.8, 31.7, 21.2 us; 32 rows per workgroup: 21 to 22 us at all three).
  if (a.B > 1 && need1 <= 8) {
    const long wgs4 = long(a.B) * ((a.E + 3) / 4);
    if (wgs4 <= 512) return launch_route_pair_s<WT, 1, 1>(a, need1, st);
    return launch_route_pair_s<WT, 1, 4>(a, need1, st);
  }
  return launch_route_pair_s<WT, 4, 1>(a, need4, st);
}

// Workgroups of the joint batch-one launch that a compute unit holds.
template <typename WT, int NCH>
hipError_t route_gateup_b1_per_cu(int H, int *n) {
  const size_t lds = size_t(H) * sizeof(double);
  static int blocks_per_cu = -1;               // per instantiation
  static size_t checked_lds = 0;
  if (blocks_per_cu < 0 || lds > checked_lds) {
    int now = 0;
    hipError_t e = prepare_kernel(route_gateup_b1_kernel<WT, NCH>, lds, &now);
    if (e != hipSuccess) return e;
    blocks_per_cu = now;
    checked_lds = lds;
  }
  *n = blocks_per_cu;
  return hipSuccess;
}

template <typename WT, int NCH>
hipError_t launch_route_gateup_b1_n(const RoutePairArgs &ra, const ExpertArgs &a, const ActiveList &act, hipStream_t st) {
  const size_t lds = size_t(ra.H) * sizeof(double);
  const int n_route = joint_routing_workgroups(ra.E);
  int blocks_per_cu = 0;
  if (hipError_t e = route_gateup_b1_per_cu<WT, NCH>(ra.H, &blocks_per_cu); e != hipSuccess) return e;
  // the routing workgroups wait for one another: they must fit on the device together
  if (long(n_route) > long(blocks_per_cu) * g_compute_units) return hipErrorLaunchOutOfResources;
  const GateupSplit split = beside_routing_split(NCH, a.I, a.H, act.n, sizeof(WT), n_route, blocks_per_cu, g_compute_units);
  const SharedSplit shared = share_with_routing(split, a.I, a.H, act.n, sizeof(WT), n_route, g_compute_units);
  hipLaunchKernelGGL((route_gateup_b1_kernel<WT, NCH>), dim3(n_route + shared.stream.blocks * act.n), dim3(kBlock), lds, st,
                     ra, a, act, n_route, shared);
  return hipGetLastError();
}

// Calls f with the chunks of a weight row per lane (a constant, rounded up to what the kernel is built for).
template <typename WT, typename F>
hipError_t with_row_chunks(int H, F f) {
  const int need = (H + kWave * Packed<WT>::N - 1) / (kWave * Packed<WT>::N);
  if (need <= 1) return f(std::integral_constant<int, 1>());
  if (need <= 2) return f(std::integral_constant<int, 2>());
  if (need <= 4) return f(std::integral_constant<int, 4>());
  if (need <= 6) return f(std::integral_constant<int, 6>());
  if (need <= 8) return f(std::integral_constant<int, 8>());
  return hipErrorInvalidValue;
}

template <typename WT>
hipError_t launch_route_gateup_b1_t(const RoutePairArgs &ra, const ExpertArgs &a, const ActiveList &act, hipStream_t st) {
  return with_row_chunks<WT>(a.H, [&](auto nch) { return launch_route_gateup_b1_n<WT, nch()>(ra, a, act, st); });
}

template <typename WT>
hipError_t route_gateup_b1_per_cu_t(int H, int *n) {
  return with_row_chunks<WT>(H, [&](auto nch) { return route_gateup_b1_per_cu<WT, nch()>(H, n); });
}

template <int NT, int KSPLIT, bool PROJ>
hipError_t launch_route_gateup_mfma_n(const RoutePairArgs &ra, const ExpertArgs &a, const TokenLists &lists,
                                      const uint16_t *s_q, uint16_t *hq, hipStream_t st) {
  const size_t route_lds = (sizeof(RouteShared) + 15) / 16 * 16 + size_t(ra.H) * sizeof(double);
  const size_t lds = std::max(route_lds, sizeof(ExpertMfmaShared<true, NT, KSPLIT>));
  static int blocks_per_cu = -1;               // per instantiation
  static size_t checked_lds = 0;
  if (blocks_per_cu < 0 || lds > checked_lds) {
    int n = 0;
    hipError_t e = prepare_kernel(route_gateup_mfma_kernel<NT, KSPLIT, PROJ>, lds, &n);
    if (e != hipSuccess) return e;
    blocks_per_cu = n;
    checked_lds = lds;
  }
  const int n_wg = beside_experts_workgroups(ra.E, PROJ ? ra.proj_rows : 0, ra.B, g_compute_units);
  if (long(n_wg) > long(blocks_per_cu) * g_compute_units) return hipErrorLaunchOutOfResources;
  constexpr int rows_per_wg = 16 * kMfmaWaves / KSPLIT;
  const int row_blocks = (a.I + rows_per_wg - 1) / rows_per_wg, n_route = n_wg * ra.B;
  hipLaunchKernelGGL((route_gateup_mfma_kernel<NT, KSPLIT, PROJ>), dim3(n_route + row_blocks * lists.n), dim3(kBlock), lds,
                     st, ra, a, lists, s_q, hq, n_wg, n_route, row_blocks, int(whole_lines(a.H)));
  return hipGetLastError();
}

template <int NT, bool PROJ>
hipError_t launch_route_gateup_mfma_t(const RoutePairArgs &ra, const ExpertArgs &a, const TokenLists &lists,
                                      const uint16_t *s_q, uint16_t *hq, hipStream_t st) {
  return with_ksplit(gateup_ksplit(a.H, (a.B + 15) / 16), [&](auto ksplit) {
    return launch_route_gateup_mfma_n<NT, ksplit(), PROJ>(ra, a, lists, s_q, hq, st);
  });
}

}  // namespace

// Rows of up to 8 chunks per lane: beyond, the LDS that the routing needs would leave the gate/up workgroups too few
// places.  The routing workgroups have to fit on the device together, which a small partition of it may not have room for.
bool route_gateup_b1_supported(int H, int E, int dtype) {
  int per_cu = 0;
  if (H > kWave * 8 * (dtype == 1 ? 8 : 4)) return false;
  const hipError_t e = dtype == 1 ? route_gateup_b1_per_cu_t<uint16_t>(H, &per_cu) : route_gateup_b1_per_cu_t<float>(H, &per_cu);
  return e == hipSuccess && long(joint_routing_workgroups(E)) <= long(per_cu) * g_compute_units;
}

hipError_t launch_route_gateup_b1(const RoutePairArgs &ra, const ExpertArgs &a, const ActiveList &act, int dtype,
                                  hipStream_t st) {
  return dtype == 1 ? launch_route_gateup_b1_t<uint16_t>(ra, a, act, st) : launch_route_gateup_b1_t<float>(ra, a, act, st);
}

bool route_gateup_mfma_supported(int H) { return H <= 4096; }   // beyond, LDS for two workgroups per compute unit only

hipError_t launch_route_gateup_mfma(const RoutePairArgs &ra, const ExpertArgs &a, const TokenLists &lists, uint16_t *s_q,
                                    uint16_t *hq, hipStream_t st) {
  const size_t lds = size_t(a.H) * sizeof(float);
  if (a.H <= 2048) hipLaunchKernelGGL(norm_rows_kernel<1>, dim3(a.B), dim3(kBlock), lds, st, a, s_q);
  else hipLaunchKernelGGL(norm_rows_kernel<2>, dim3(a.B), dim3(kBlock), lds, st, a, s_q);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  if (ra.proj) {
    // The estimator's launch is built for the tiles of the batch, not for those of the fullest expert: with 17 tokens and
    // more it may hold more registers than its experts need.  Tiles by the expert were not measured here.
    switch ((a.B + 15) / 16) {
      case 1: return launch_route_gateup_mfma_t<1, true>(ra, a, lists, s_q, hq, st);
      case 2: return launch_route_gateup_mfma_t<2, true>(ra, a, lists, s_q, hq, st);
      case 3: return launch_route_gateup_mfma_t<3, true>(ra, a, lists, s_q, hq, st);
      default: return launch_route_gateup_mfma_t<4, true>(ra, a, lists, s_q, hq, st);
    }
  }
  switch (decode_tiles(lists.most)) {
    case 1: return launch_route_gateup_mfma_t<1, false>(ra, a, lists, s_q, hq, st);
    case 2: return launch_route_gateup_mfma_t<2, false>(ra, a, lists, s_q, hq, st);
    default: return launch_route_gateup_mfma_t<4, false>(ra, a, lists, s_q, hq, st);
  }
}

// H up to 64 * 4 * 8 chunks of 16 bytes per row (8192 columns of either dtype).
bool route_pair_supported(int H, int dtype) {
  const int vn = dtype == 1 ? 8 : 4;
  return (H + vn - 1) / vn <= 4 * kWave * 8;
}

hipError_t launch_route_pair(const RoutePairArgs &a, int dtype, hipStream_t st) {
  return dtype == 1 ? launch_route_pair_t<uint16_t>(a, st) : launch_route_pair_t<float>(a, st);
}

}  // namespace moe_spec
