// Forward pass of the neural expert estimator (paper: Sec. 6 and Appendix A): project the
// predicting signal to a latent size, add the layer's embedding, feed forward with SiLU and a
// residual connection, LayerNorm, linear head to E logits.  The projection rides in the launch that routes the layer; the
// rest is one launch (estimator_body), by itself or beside the down projection of the layer's experts.  Where that launch
// does not reach (per-layer diagnostics, the baseline signal as input, vectors beyond 4096 values): the double-precision
// GEMV below for each product; LayerNorm, head, top-k and gates then run in the routing kernel (its input mode 3).
// Everything is double precision: these logits decide expert indices.
#include "device_utils.h"
#include "expert_mfma.h"
#include "kernels.h"
#include "launch_rules.h"
#include "route_select.h"

namespace moe_spec {
namespace {

constexpr int kTokTile = 4;

// y[b, row] = act( W[row,:] . x[b,:] + add_w[row] ) + add_f64[b, row]; one wavefront per row.
template <typename WT>
__global__ __launch_bounds__(kBlock) void gemv64_kernel(const GemvArgs a) {
  using P = Packed<WT>;
  constexpr int VN = P::N;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int row = blockIdx.x * kWaves + wave;
  if (row >= a.rows) return;
  const WT *w = static_cast<const WT *>(a.w) + size_t(row) * a.cols;
  double bias = 0.0;
  if (a.add_w) {
    float one[VN];
    const WT *src = static_cast<const WT *>(a.add_w) + (row / VN) * VN;
    load_chunk<WT>(src, one);
    bias = double(one[row % VN]);
  }
  for (int b0 = 0; b0 < a.B; b0 += kTokTile) {
    const int nb = min(kTokTile, a.B - b0);
    double acc[kTokTile];
#pragma unroll
    for (int t = 0; t < kTokTile; ++t) acc[t] = 0.0;
#pragma unroll 2
    for (int c = lane * VN; c < a.cols; c += kWave * VN) {
      float wf[VN];
      load_chunk<WT>(w + c, wf);
#pragma unroll
      for (int t = 0; t < kTokTile; ++t) {
        if (t < nb) {
          const size_t at = size_t(b0 + t) * a.cols + c;
#pragma unroll
          for (int x = 0; x < VN; ++x)
            acc[t] += double(wf[x]) * (a.x_f64 ? a.x_f64[at + x] : double(a.x_f32[at + x]));
        }
      }
    }
#pragma unroll
    for (int t = 0; t < kTokTile; ++t) {
      if (t < nb) {
        double v = wave_sum(acc[t]) + bias;
        if (a.silu) v = v / (1.0 + exp(-v));
        if (lane == 0) {
          const size_t o = size_t(b0 + t) * a.rows + row;
          if (a.add_f64) v += a.add_f64[o];
          a.y[o] = v;
        }
      }
    }
  }
}

constexpr int kEstTokens = 2, kEstRows = 4;    // tokens of a group, rows of a wavefront at a time

// Eight sums over the wavefront at once: the first three steps halve the number of values a lane holds instead of adding up
// each of them over all lanes (13 exchanges and additions instead of 48).  Lane l ends with the sum of a[l / 8].
__device__ __forceinline__ double wave_sums8(double (&a)[8]) {
  const int lane = threadIdx.x & (kWave - 1);
  auto exchange = [](double x, double y, auto swap) {       // half of the lanes get x's sum, the other half y's
    const auto lo = swap(__double2loint(x), __double2loint(y));
    const auto hi = swap(__double2hiint(x), __double2hiint(y));
    return __hiloint2double(int(hi[0]), int(lo[0])) + __hiloint2double(int(hi[1]), int(lo[1]));
  };
#pragma unroll
  for (int i = 0; i < 4; ++i)
    a[i] = exchange(a[i], a[i + 4], [](int x, int y) { return __builtin_amdgcn_permlane32_swap(x, y, false, false); });
#pragma unroll
  for (int i = 0; i < 2; ++i)
    a[i] = exchange(a[i], a[i + 2], [](int x, int y) { return __builtin_amdgcn_permlane16_swap(x, y, false, false); });
  const bool upper = lane & 8;
  double s = (upper ? a[1] : a[0]) + dpp_move<0x128>(upper ? a[0] : a[1]);       // row_ror 8
  s += dpp_move<0x141>(s);
  s += dpp_move<0xB1>(s);
  return s + dpp_move<0x4E>(s);
}

// Rows of w [rows, cols] times the vectors of up to two tokens in LDS, by one wavefront: four rows at a time (group first,
// first + stride, ...), so that what is read from LDS meets four rows, one chunk per lane and row a step and the next step's
// on their way meanwhile.  The first step is asked for where this is made, before the vectors are there.  vec: token after
// token, column x of column group o at x * cols / VN + o (lanes that read the same x of consecutive groups touch
// consecutive words).
template <typename WT>
struct RowProducts {
  using P = Packed<WT>;
  using Raw = typename P::Raw;
  static constexpr int VN = P::N, kRows = kEstRows;
  static_assert(kEstRows * kEstTokens == 8, "wave_sums8");
  const WT *w;
  int rows, cols, first, stride, groups, lane;
  Raw cur[kRows];

  __device__ __forceinline__ void fetch(int group, int c, Raw (&dst)[kRows]) const {
#pragma unroll
    for (int q = 0; q < kRows; ++q)
      dst[q] = *reinterpret_cast<const Raw *>(w + size_t(min(group * kRows + q, rows - 1)) * cols + (c < cols ? c : 0));
  }
  __device__ __forceinline__ RowProducts(const void *w_, int rows_, int cols_, int first_, int stride_)
      : w(static_cast<const WT *>(w_)), rows(rows_), cols(cols_), first(first_), stride(stride_), groups((rows_ + kRows - 1) / kRows),
        lane(threadIdx.x & (kWave - 1)) {
    if (first < groups) fetch(first, lane * VN, cur);
  }
  // Which row of a group and which token a lane ends with; every eighth lane hands it on.
  __device__ __forceinline__ int my_row() const { return (lane >> 3) / kEstTokens; }
  __device__ __forceinline__ int my_token() const { return (lane >> 3) % kEstTokens; }
  // sink(row, token, sum), a lane for each
  template <typename Sink>
  __device__ __forceinline__ void run(const double *vec, int nb, Sink sink) {
    const int G = cols / VN;
    const double *of[kEstTokens];                  // tokens past nb repeat the last: no condition on what is read
#pragma unroll
    for (int t = 0; t < kEstTokens; ++t) of[t] = vec + min(t, nb - 1) * cols;
    for (int group = first; group < groups; group += stride) {
      double acc[kRows * kEstTokens] = {};
      for (int o = lane; o - lane < G; o += kWave) {
        Raw next[kRows];
        const bool more = o - lane + kWave < G;          // the same in every lane
        if (more || group + stride < groups) fetch(more ? group : group + stride, (more ? o + kWave : lane) * VN, next);
        if (o < G) {
          float wf[kRows][VN];
#pragma unroll
          for (int q = 0; q < kRows; ++q) P::unpack(cur[q], wf[q]);
#pragma unroll
          for (int x = 0; x < VN; ++x) {
            double v[kEstTokens];
#pragma unroll
            for (int t = 0; t < kEstTokens; ++t) v[t] = of[t][x * G + o];
#pragma unroll
            for (int q = 0; q < kRows; ++q) {
              const double wd = double(wf[q][x]);
#pragma unroll
              for (int t = 0; t < kEstTokens; ++t) acc[q * kEstTokens + t] += wd * v[t];
            }
          }
        }
#pragma unroll
        for (int q = 0; q < kRows; ++q) cur[q] = next[q];
      }
      const double s = wave_sums8(acc);
      const int row = group * kRows + my_row();
      if ((lane & 7) == 0 && my_token() < nb && row < rows) sink(row, my_token(), s);
    }
  }
};

// The estimator from its feed-forward on for nb tokens from b0 on, by n_wg workgroups that hand t, v and the logits to one
// another through slots that are their own flags; each asks for its next weights before it waits.  A chain of latencies: 4
// tokens of 128 experts of 2048 columns 13.5 us (load 1.3, a product with its hand-over 2.5 to 3.3 each, LayerNorm 1.4,
// selection 1.2), as three launches 6.9 + 6.9 + 8.6, and beside the down projection (16.6 by itself) 20.  Microseconds per
// layer step, separate launches / one: 1 token 39.9 / 35.9, 2 57.7 / 49.5, 4 74.0 / 61.7, 16 150 / 120, 64 348 / 241; 8
// experts of 4096 columns, 1 token 49.6 / 47.1, 8 122 / 91, 64 430 / 217.
template <typename WT>
__device__ __forceinline__ void estimator_body(const EstimatorArgs &e, const RoutePairArgs &ra, const int wg, const int n_wg,
                                               const int group, const int groups, const int b0, const int nb, double *vec,
                                               RouteShared &sh) {
  constexpr int VN = Packed<WT>::N;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int first = wg * kWaves + wave, stride = n_wg * kWaves;
  const int dm = e.dm, F = e.F, E = ra.E;
  for (int i = (group * n_wg + wg) * kBlock + tid; i < ra.arm_count; i += groups * n_wg * kBlock) {
    arm64(ra.z_true_next + i);
    arm64(ra.z_pred_next + i);
  }
  // value c of token t of [nb, cols] goes where RowProducts reads it
  auto place = [](int t, int c, int cols) { return t * cols + c % VN * (cols / VN) + c / VN; };
  // vectors [nb, cols] of the group's tokens to LDS: get fills a thread's values, at(i) being where the i-th is
  auto fill_vectors = [&](int cols, auto get) {
    auto with = [&](auto tokens, auto per_thread) {      // of each token, both at least what there are
      constexpr int N = tokens() * per_thread();
      double got[N];
      get(got, [&](int i) {
        return size_t(b0 + min(i / per_thread(), nb - 1)) * cols + min(i % per_thread() * kBlock + tid, cols - 1);
      });
      __syncthreads();                           // the readers of the vectors before are done
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int t = i / per_thread(), c = i % per_thread() * kBlock + tid;
        if (t < nb && c < cols) vec[place(t, c, cols)] = got[i];
      }
    };
    if (cols <= kBlock) with(int_c<2>(), int_c<1>());
    else if (cols <= 2 * kBlock) with(int_c<2>(), int_c<2>());
    else if (cols <= 4 * kBlock) with(int_c<2>(), int_c<4>());
    else if (cols <= 8 * kBlock) with(int_c<2>(), int_c<8>());
    else with(int_c<1>(), int_c<16>());          // nb * cols <= 4096
    __syncthreads();
  };
  auto await_vectors = [&](const unsigned long long *slots, int cols) {
    fill_vectors(cols, [&](auto &got, auto at) { await_all64(slots, at, ra.spin_limit, ra.status, got); });
  };

  // ---- t = silu(ffn_in u)
  {
    RowProducts<WT> rows(e.ffn_in, F, dm, first, stride);
    fill_vectors(dm, [&](auto &got, auto at) {
#pragma unroll
      for (int i = 0; i < int(sizeof(got) / sizeof(double)); ++i) got[i] = e.u[at(i)];
    });
    rows.run(vec, nb, [&](int r, int t, double s) { publish_value64(e.t + size_t(b0 + t) * F + r, s / (1.0 + exp(-s))); });
  }
  // ---- v = u + ffn_out t
  {
    RowProducts<WT> rows(e.ffn_out, dm, F, first, stride);
    const int row0 = first * RowProducts<WT>::kRows + rows.my_row();
    const double u0 = e.u[size_t(b0 + min(rows.my_token(), nb - 1)) * dm + min(row0, dm - 1)];
    await_vectors(e.t, F);
    rows.run(vec, nb, [&](int r, int t, double s) {
      publish_value64(e.v + size_t(b0 + t) * dm + r, s + (r == row0 ? u0 : e.u[size_t(b0 + t) * dm + r]));
    });
  }
  // ---- LayerNorm, a token per wavefront, and the head
  {
    RowProducts<WT> rows(e.head, E, dm, first, stride);
    await_vectors(e.v, dm);
    if (wave < nb) {
      double *x = vec + size_t(wave) * dm, sum = 0.0, sq = 0.0;
      for (int i = lane; i < dm; i += kWave) sum += x[i];
      const double mean = wave_sum(sum) / double(dm);
      for (int i = lane; i < dm; i += kWave) { const double d = x[i] - mean; sq += d * d; }
      const double inv = rsqrt(wave_sum(sq) / double(dm) + double(e.ln_eps));
      const int G = dm / VN;
      for (int o = lane; o < G; o += kWave) {
#pragma unroll
        for (int q = 0; q < VN; ++q)
          x[q * G + o] = (x[q * G + o] - mean) * inv * double(e.ln_gain[o * VN + q]) + double(e.ln_bias[o * VN + q]);
      }
    }
    __syncthreads();
    rows.run(vec, nb, [&](int r, int t, double s) { publish64(ra.z_pred + size_t(b0 + t) * E + r, s); });
  }
  // ---- a workgroup per token selects and reports
  if (wg >= nb) return;
  __syncthreads();                               // the selection's shared memory is that of the vectors
  const int b = b0 + wg;
  select_ids_any(ra, 9, ra.z_pred + size_t(b) * E, E, ra.k, sh.sel, tid, ra.mb_next ? ra.mb_next->ids + size_t(b) * ra.k : nullptr);
  report_next(ra, b, sh.sel, select_gates(ra.k, sh.sel, tid), tid);
}

template <typename WT>
__device__ __forceinline__ void estimator_workgroup(const EstimatorArgs &e, const RoutePairArgs &ra, const EstimatorSplit &split,
                                                    unsigned char *lds) {
  const int group = blockIdx.x / split.wgs, b0 = group * split.tokens;
  estimator_body<WT>(e, ra, blockIdx.x % split.wgs, split.wgs, group, split.groups, b0, min(split.tokens, ra.B - b0),
                     reinterpret_cast<double *>(lds), *reinterpret_cast<RouteShared *>(lds));
}

template <typename WT>
__global__ __launch_bounds__(kBlock) void estimator_kernel(const EstimatorArgs e, const RoutePairArgs ra, const EstimatorSplit split) {
  extern __shared__ __align__(16) unsigned char lds[];
  estimator_workgroup<WT>(e, ra, split, lds);
}

// The first workgroups carry the estimator on (dispatched first: they are on the device together), the others are those of
// expert_mfma_kernel<GATEUP, ...>, which is built for the down projection.
template <bool GATEUP, int NT, int KSPLIT, int CHAINS>
__global__ __launch_bounds__(kBlock, NT == 1 ? 4 : 2) void down_estimator_kernel(const EstimatorArgs e, const RoutePairArgs ra, const EstimatorSplit split,
                                                                const ExpertArgs a, const TokenLists lists, const uint16_t *act_q,
                                                                const int row_blocks, const int stream) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int n_est = split.wgs * split.groups;
  if (int(blockIdx.x) < n_est) {
    estimator_workgroup<uint16_t>(e, ra, split, lds);
    return;
  }
  const int i = blockIdx.x - n_est;
  ExpertMfmaShared<GATEUP, NT, KSPLIT> &sh = *reinterpret_cast<ExpertMfmaShared<GATEUP, NT, KSPLIT> *>(lds);
  if (stream) expert_mfma_body<GATEUP, NT, KSPLIT, CHAINS>(a, DecodeTokens<true>{lists, i / row_blocks}, act_q, nullptr, i % row_blocks, sh);
  else expert_mfma_body<GATEUP, NT, KSPLIT, CHAINS>(a, DecodeTokens<false>{lists, i / row_blocks}, act_q, nullptr, i % row_blocks, sh);
}

hipError_t compute_units(int *n) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  return e != hipSuccess ? e : hipDeviceGetAttribute(n, hipDeviceAttributeMultiprocessorCount, dev);
}

// The split and the shared memory of an estimator workgroup; refused where the kernel's estimator workgroups do not fit on the
// device together.  known: what the runtime said for this kernel.
struct Fit {
  int per_cu = -1;
  size_t lds = 0;
};
template <typename K>
hipError_t prepare_estimator(K kernel, Fit &known, const EstimatorArgs &e, int B, size_t others_lds, EstimatorSplit *split, size_t *lds) {
  int cus = 0;
  if (hipError_t r = compute_units(&cus); r != hipSuccess) return r;
  *split = estimator_split(e.dm, e.F, B, cus);
  if (split->wgs < 1) return hipErrorInvalidValue;
  *lds = std::max(std::max(sizeof(RouteShared), others_lds), size_t(split->tokens) * std::max(e.dm, e.F) * sizeof(double));
  if (known.per_cu < 0 || *lds > known.lds) {
    int n = 0;
    if (hipError_t r = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, kBlock, *lds); r != hipSuccess) return r;
    known = {n, *lds};
  }
  return long(split->wgs) * split->groups > long(known.per_cu) * cus ? hipErrorLaunchOutOfResources : hipSuccess;
}

template <typename WT>
hipError_t prepare_alone(const EstimatorArgs &e, int B, EstimatorSplit *split, size_t *lds) {
  static Fit known;
  return prepare_estimator(estimator_kernel<WT>, known, e, B, 0, split, lds);
}

template <typename WT>
hipError_t launch_estimator_t(const EstimatorArgs &e, const RoutePairArgs &ra, hipStream_t st) {
  EstimatorSplit split;
  size_t lds = 0;
  if (hipError_t r = prepare_alone<WT>(e, ra.B, &split, &lds); r != hipSuccess) return r;
  hipLaunchKernelGGL(estimator_kernel<WT>, dim3(split.wgs * split.groups), dim3(kBlock), lds, st, e, ra, split);
  return hipGetLastError();
}

}  // namespace

bool estimator_supported(int dm, int F, int B, int dtype) {
  EstimatorArgs e{};
  e.dm = dm;
  e.F = F;
  EstimatorSplit split;
  size_t lds = 0;
  return (dtype == 1 ? prepare_alone<uint16_t>(e, B, &split, &lds) : prepare_alone<float>(e, B, &split, &lds)) == hipSuccess;
}

hipError_t launch_estimator(const EstimatorArgs &e, const RoutePairArgs &ra, int dtype, hipStream_t st) {
  return dtype == 1 ? launch_estimator_t<uint16_t>(e, ra, st) : launch_estimator_t<float>(e, ra, st);
}

hipError_t launch_down_estimator(const EstimatorArgs &e, const RoutePairArgs &ra, const ExpertArgs &a, const TokenLists &lists,
                                 const uint16_t *hq, hipStream_t st) {
  int cus = 0;
  if (hipError_t r = compute_units(&cus); r != hipSuccess) return r;
  return with_down_form(a, lists, cus, [&](auto nt, auto ksplit, auto chains) {
    static Fit known;                            // per instantiation
    auto kernel = down_estimator_kernel<false, nt(), ksplit(), chains()>;
    EstimatorSplit split;
    size_t lds = 0;
    if (hipError_t r = prepare_estimator(kernel, known, e, ra.B, sizeof(ExpertMfmaShared<false, nt(), ksplit()>), &split, &lds);
        r != hipSuccess)
      return r;
    constexpr int rows_per_wg = 16 * kMfmaWaves / ksplit();
    const int row_blocks = (a.H + rows_per_wg - 1) / rows_per_wg;
    hipLaunchKernelGGL(kernel, dim3(split.wgs * split.groups + row_blocks * lists.n), dim3(kBlock), lds, st, e, ra, split, a, lists,
                       hq, row_blocks, int(whole_lines(a.I)));
    return hipGetLastError();
  });
}

hipError_t launch_gemv64(const GemvArgs &a, int dtype, hipStream_t st) {
  const dim3 grid((a.rows + kWaves - 1) / kWaves), block(kBlock);
  if (dtype == 1) hipLaunchKernelGGL(gemv64_kernel<uint16_t>, grid, block, 0, st, a);
  else hipLaunchKernelGGL(gemv64_kernel<float>, grid, block, 0, st, a);
  return hipGetLastError();
}

}  // namespace moe_spec
