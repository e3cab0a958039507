// How much work a launch gives each workgroup: arithmetic on sizes alone, host code without a GPU call in it.
#pragma once
#include <algorithm>
#include <cstddef>

namespace moe_spec {

constexpr int kB1Waves = 4;                    // wavefronts per workgroup of the batch-one gate/up projection
constexpr int kRouteWaves = 4;                 // and of the routing launches

// How a gate/up launch of its own deals the I rows of each of n experts to wavefronts.  Up to 4096 wavefronts of two
// rows each are all resident at once (137 registers at NCH = 4): pairs.  Beyond, one row per wavefront until that would
// exceed about 6144 wavefronts (24 per compute unit), then more rows each.
struct GateupSplit {
  int rpw;                                     // 0: pairs
  int blocks;                                  // workgroups per expert
};
inline GateupSplit gateup_b1_split(int nch, int I, int n) {
  if (nch <= 4 && long(I) * n <= 8192) return {0, (I + 2 * kB1Waves - 1) / (2 * kB1Waves)};
  const int rpw = int(std::max(1l, (long(I) * n + 6143) / 6144));
  return {rpw, (I + kB1Waves * rpw - 1) / (kB1Waves * rpw)};
}

// Workgroups that route in the joint batch-one launch: kJointSplit wavefronts share a router row.
constexpr int kJointSplit = 2;
inline int joint_routing_workgroups(int E) {
  constexpr int rows = kRouteWaves / kJointSplit;
  return (E + rows - 1) / rows;
}

// How the gate/up rows are dealt to wavefronts beside the routing.  The routing is a chain of dependent memory accesses
// (9 us alone) and every one of them queues behind the weight loads in flight, above all those of its own compute unit.  Up
// to 64 MB of weights one gate/up workgroup goes on each compute unit that does not route: 128 experts of 768 x 2048 (50 MB,
// 64 routing workgroups) 3.9 TB/s, the prediction posted after 10.7 us, 14.5 us together; with a quarter more workgroups 13.5
// and 16.  Up to 256 MB the workgroups fill the device once, so that none is left over for a second round.  Beyond, the
// routing is short beside the stream and the split of the plain launch is as good.  Microseconds per layer step, one
// workgroup per unit / filled once, for 8 of 64 experts of 2048 columns, 2 of 8 of 4096 and 4 of 32 of 2880: at 24 MB 19.0 /
// 19.8, 22.3 / 23.7, 22.6 / 23.9; at 40 20.8 / 22.5, 25.0 / 26.7, 23.9 / 25.3; at 63 26.5 / 26.2, 26.6 / 28.3, 26.4 / 28.3;
// at 80 28.3 / 27.0, 29.2 / 31.0, 31.9 / 32.0; at 112 35.8 / 32.6, 35.4 / 35.2, 36.0 / 34.1; at 160 48.3 / 44.2, 44.8 /
// 44.4, 50.0 / 47.2; at 224 65.0 / 59.2, 59.7 / 59.7, 63.9 / 60.5.  Filled once / plain split, before the two rows per
// routing workgroup: at 256 MB 72.1 / 72.1, 72.8 / 72.6, 72.1 / 71.8; at 320, 384 MB 87.1 / 86.1, 103.9 / 106.5.
// Never fewer workgroups than a quarter of the compute units, however many of them the routing takes: with routing that
// fills the device there would be none.  Never pairs: those end at 67 MB.
inline GateupSplit beside_routing_split(int nch, int I, int H, int n, std::size_t wbytes, int n_route, int blocks_per_cu,
                                        int cus) {
  const std::size_t bytes = std::size_t(2) * I * H * n * wbytes;
  if (bytes > std::size_t(256) << 20) return gateup_b1_split(nch, I, n);
  const int places = bytes <= std::size_t(64) << 20 ? cus : blocks_per_cu * cus;
  const int wgs = std::max(1, std::max(cus / 4, places - n_route));
  const int rpw = int((long(I) * n + long(kB1Waves) * wgs - 1) / (long(kB1Waves) * wgs));
  return {rpw, (I + kB1Waves * rpw - 1) / (kB1Waves * rpw)};
}

// The same with the routing workgroups taking rows too once they have routed (all but the first, which finishes the
// prediction): the last I - first_tail rows of every expert, at most half of them, tail_rpw per wavefront, in tail_blocks
// workgroups.  They come free after about 6 us in which another workgroup streams 130 KB.  Taken where all of this holds: one
// gate/up workgroup per compute unit beside the routing (up to 64 MB of weights, see above); routing on half of the device or
// more; 320 KB and more for each of the other workgroups (the routing, 12 us, is over well before them then); rows of up to 4
// KB.  Two router rows per routing workgroup: on a whole device that is 255 and 256 experts, on a partition of it fewer.
// Microseconds per layer step, 8 of 256 experts, without / with: 1024 columns, 40 MB 27.3 / 24.7, 48 MB 30.3 / 26.4, 63 MB
// 37.5 / 32.8; 2048 columns, 40 MB 24.6 / 24.6 (again: 23.9 / 24.4), 44 MB 25.5 / 24.9, 48 MB 26.4 / 25.7, 63 MB 33.2 / 31.4;
// 1536 columns, 47 MB 29.2 / 27.4; 16 of 256 of 704 x 1016 29.2 / 26.7; 8 of 255 of 704 x 2048 25.1 / 24.8.  Not taken: fewer
// bytes, 1024 columns 36 MB 26.0 / 23.7 and 2048 columns 36 MB 24.1 / 23.8; fewer routing workgroups, 128 experts of 2048
// columns 40 MB 21.5 / 22.1, 48 MB 22.6 / 23.1, 63 MB 29.2 / 28.9 and of 1024 columns 48 MB 24.2 / 24.4, 63 MB 31.7 / 30.2,
// 200 experts of 2048 columns 44 MB 24.4 / 24.7, 63 MB 31.2 / 31.2 and of 1024 columns 48 MB 28.2 / 26.8.  So the limit on
// routing workgroups rests on rows of 4 KB, and leaves out gains of up to 8 % at rows of 2 KB; the one on bytes per workgroup
// rests on rows of 4 KB as well.  The limit on rows was drawn with one router row per workgroup (8 of 128 of 640 x 2880 370
// without, 375 us a pass with).
struct SharedSplit {
  GateupSplit stream;                          // of rows [0, first_tail)
  int first_tail, tail_rpw, tail_blocks;       // tail_blocks 0: none
};
inline SharedSplit share_with_routing(const GateupSplit &s, int I, int H, int n, std::size_t wbytes, int n_route, int cus) {
  const SharedSplit none{s, I, 0, 0};
  const std::size_t row = std::size_t(2) * H * wbytes, bytes = row * I * n;
  const int helpers = (n_route - 1) / n;       // workgroups per expert
  if (s.rpw < 1 || helpers < 1 || H * wbytes > 4096 || 2 * n_route < cus || bytes > std::size_t(64) << 20 ||
      bytes < std::size_t(320 << 10) * s.blocks * n)
    return none;
  const double lead = 130e3 / double(row), stream_wgs = double(s.blocks) * n, tail_wgs = double(helpers) * n;
  const double rows_each = (double(I) * n + tail_wgs * lead) / (stream_wgs + tail_wgs);
  const int tail_rpw = int((rows_each - lead) / kB1Waves);
  if (tail_rpw < 1) return none;
  SharedSplit out{s, I, tail_rpw, std::min(helpers, I / 2 / (kB1Waves * tail_rpw))};
  if (out.tail_blocks < 1) return none;
  out.first_tail = I - out.tail_blocks * kB1Waves * tail_rpw;
  out.stream.rpw = (out.first_tail + kB1Waves * s.blocks - 1) / (kB1Waves * s.blocks);
  out.stream.blocks = (out.first_tail + kB1Waves * out.stream.rpw - 1) / (kB1Waves * out.stream.rpw);
  return out;
}

// Workgroups per token of a routing launch beside matrix-core experts, whose rows may be dealt to any number of them:
// about one per compute unit in all (half as many: 2 % slower at 32 tokens, a quarter 16 %; twice as many 1 %), at least
// a router row for every wavefront, and two pairs of rows where the estimator's projection rides along (proj_rows, else
// 0).  Sized by the router alone, the projection is a serial chain where experts are few: a layer step of 8 experts of
// 4096 columns with a latent size of 1024 takes 236 us at 2 tokens and 293 us at 8 like that, 73 and 126 us like this.
// One pair instead of two: 4 tokens of 128 experts of 2048 columns 1 % slower, the others within 3 % either way.
inline int beside_experts_workgroups(int E, int proj_rows, int B, int cus) {
  const int rows = std::max(E, (proj_rows + 3) / 4);
  return std::max(1, std::min(cus / B, (rows + kRouteWaves - 1) / kRouteWaves));
}

// The same for a routing launch of its own: rows_per_wg router rows each, and more workgroups where the projection has
// more row pairs than those have wavefronts (one token of the layer above: 87 us sized by the router, 50 us like this).
inline int routing_workgroups(int E, int rows_per_wg, int proj_rows, int B, int cus) {
  const int for_router = (E + rows_per_wg - 1) / rows_per_wg;
  return std::max(for_router, std::min(cus / B, ((proj_rows + 1) / 2 + kRouteWaves - 1) / kRouteWaves));
}

// Workgroups of the estimator's launch.  A group of them has up to two tokens, of 4096 values together at most, and its
// workgroups wait for one another, so all groups have to be on the device together.  Four rows of the larger matrix per
// wavefront, which it multiplies with both tokens at once, or more where the groups fill the device.  With four tokens per
// group a step of this chain takes a wavefront twice as long: 4 tokens, latent size 512, feed-forward 1024, 128 experts 22.4
// us instead of 13.5.
struct EstimatorSplit {
  int tokens, groups, wgs;                     // per group, groups, workgroups per group; wgs 0: not to be launched
};
inline EstimatorSplit estimator_split(int dm, int F, int B, int cus) {
  const int longest = std::max(dm, F), tokens = std::min(std::min(2, B), 4096 / longest);
  if (tokens < 1) return {0, 0, 0};
  const int groups = (B + tokens - 1) / tokens, room = cus / groups;
  if (room < 4) return {0, 0, 0};
  return {tokens, groups, std::max(4, std::min(room, (longest + 15) / 16))};
}

// Wavefronts per 16-row tile of the matrix-core kernels.  Each sums its part of a row in a float32 chain of its own, so the
// rules of what a row's sum consists of go by the length of the reduction and the tokens of the batch or prompt alone: a
// result does not depend on how many experts a launch has, on the slots they are in or on what runs beside it.
// Gate/up, and both products of a prompt: each should still walk eight steps of 64 columns, below that the shared start-up
// (partial sums) outweighs what the extra parallelism wins; in batches of a single tile of tokens two are enough (16 experts
// of 1024 columns, 64 tokens, 1 / 2 / 4 wavefronts: 15.2 / 13.5 / 14.9 us; 12 of them, 8 tokens: 13.6 / 12.3 / 10.3).
inline int gateup_ksplit(int K, int token_tiles) {
  const int steps = (K + 63) / 64;
  if (steps >= 32 || (token_tiles == 1 && steps >= 8)) return 4;
  return steps >= 16 ? 2 : 1;
}

// Down projection of a decode batch: as many as leave each two whole steps of 128 columns.  In batches of a single tile two
// wavefronts have two chains each, so that a sum of 449 columns and more has four of them: in one chain of 456 columns it is
// 1.5 times as far from 64 bits.  With two tiles of tokens the second accumulators would cost a wavefront per SIMD.
// From 1024 columns on one wavefront takes the four parts one after another, with the same sum, if the experts have eight
// positions or more on average and there are two workgroups per compute unit without a split: then the activations weigh as
// much as the weights, and the four wavefronts of a workgroup share them if they walk the same columns.  Microseconds with 1
// / 2 / 4 wavefronts: 30 experts of 768 columns x 2048 rows at 1 position each 18.2 / 18.0 / 19.5, 48 of them at 5 27.4 / 28.2
// / 29.9, 21 of 2880 x 2880 at 1.5 60.9 / 58.1 / 54.1, 8 of 14336 x 4096 at 4 148 / 155 / 153, at 8 164 / 177 / 182, at 16 201
// / 238 / 249, 5 of them at 1.6 130 / 103 / 90.6, 16 of 2048 x 2048 at 16 31 / 35 / 37, 16 of 1024 x 1024 at 16 (256
// workgroups without a split) 10.7 / 9.1 / 9.0.
inline int down_ksplit(int K, int token_tiles, int rows, int experts, int positions, int cus) {
  if (K < 1024) return K >= 512 || (token_tiles == 1 && K > 448) ? 2 : 1;
  return positions >= 8 * experts && long(experts) * ((rows + 63) / 64) >= 2l * cus ? 1 : 4;
}

// How a request's n blocks are dealt to the two DMA queues: the second one takes `second` whole blocks and the first `cut`
// bytes of one more (0: none).  A half each, in turn, as long as the queues are equally fast.  They are not where something
// else uses the engine behind one of them: the GPU driver clears freed device memory with it, some 16 GB/s, and meanwhile a 9.4
// MB block takes 300 us on the second queue instead of 172, both queues still fill the link together, and the first one
// waits for the second at the end of every request (47 ms instead of 37 for 32 layer steps of 128 experts of 768 x 2048 with
// 16 slots, for 1.3 s after an engine of 22 GB was given back).  So the second queue's share follows how much later than the
// first it was done in an earlier request.  Left at a half until a share of less than 0.38 is indicated, so that the odd block
// of ordinary requests (0.43 of seven) moves nothing.
constexpr double kEvenShare = 0.5;
struct QueueDeal {
  int second;
  std::size_t cut;
};
inline QueueDeal deal_to_queues(int n, std::size_t block, double share) {
  if (share == kEvenShare || n < 2) return {n / 2, 0};
  const double blocks = share * n;
  QueueDeal deal{int(blocks), std::size_t((blocks - int(blocks)) * double(block)) & ~std::size_t(4095)};
  if (deal.cut < block / 8) deal.cut = 0;                 // what a transfer costs beside its bytes is some 10 us
  if (deal.cut > block - block / 8) { deal.cut = 0; deal.second += 1; }
  return deal;
}
// Of block `index` of a request's n: the bytes, from its first on, that the second queue takes (the first queue: the rest).
// The cut block is the last one, the second queue's whole ones are spread evenly over the others.
inline std::size_t second_queue_bytes(int n, std::size_t block, double share, int index) {
  if (share == kEvenShare) return index % 2 ? block : 0;
  const QueueDeal deal = deal_to_queues(n, block, share);
  const int whole = n - (deal.cut > 0);
  if (index >= whole) return deal.cut;
  return (index + 1) * deal.second / whole > index * deal.second / whole ? block : 0;
}
// taken: the part of the request's bytes that the second queue had; late_us: how much later than the first it was done.
// What is left when one queue is done travels at 30 to 55 GB/s, and some two thirds of it belong to the other queue.  Half of
// the way there each time: a request's blocks are few and their times scatter.  first_sign: the even share was indicated to
// be wrong by the request measured before as well (a single one is an accident of the link).  Never more than a half: only the
// first queue waits for the other one at a request's end, so where copies never pause the second begins each request earlier,
// by up to half a request, and is done earlier (by 0.4 to 1.2 ms of 37 to 75 MB) without being faster.  Followed upwards too,
// decode loops bound by the link left the even share time and again and lost 0.4 % (48 layers of 8 of 128 experts of
// 768 x 2048, 16 slots: 56.38 -> 56.61 ms a token; 32 tokens of them 194.5 -> 195.3).
inline double next_queue_share(double share, double taken, double late_us, double bytes, bool *first_sign) {
  const double to = std::min(kEvenShare, std::max(0.1, taken - late_us * 20e3 / bytes));
  if (share == kEvenShare) {
    const bool wrong = to < 0.38, again = *first_sign;
    *first_sign = wrong;
    return wrong && again ? to : kEvenShare;
  }
  const double next = 0.5 * (share + to);
  *first_sign = false;
  return next > 0.46 ? kEvenShare : next;
}

// Whether the copies of a step's second and further cache waves go on the compute stream although a prefetch for the next
// layer is queued on the copy stream right behind them and takes half of the link meanwhile.  They save an event there and
// back (some 15 us a wave) and the prefetch runs beside the kernels of the waves, but the last wave ends later, and nothing
// travels beside its kernels and the next routing.  Microseconds per layer step on the copy stream / on the compute stream,
// experts of 50 MB: 28 experts in 8 slots 24141 / 24030, 28 in 24 6768 / 6726, 16 in 6 13222 / 13107, but 28 in 16 19301 /
// 19616, 28 in 14 22666 / 22877, 16 in 10 10009 / 10061; of 9.4 MB the same six 4759 / 4680, 1445 / 1416, 2555 / 2532, 3975 /
// 4021, 4558 / 4569, 1969 / 1960; of 3.1 MB 1643 / 1580, 460 / 445, 1004 / 971, 1334 / 1338, 1530 / 1527, 785 / 771.
inline bool waves_in_order(int experts, int slots, std::size_t expert_bytes) {
  return experts > 2 * slots || 4 * (experts - slots) <= slots || expert_bytes <= std::size_t(4) << 20;
}

// Whether a prompt is routed by the launches of a decode step, one for each micro-batch of up to max_batch tokens, or all at
// once by the kernel for prompts, whose workgroups take 16 tokens each: with few of them most of the device is idle and the
// launch takes what one workgroup takes, by experts and columns.  Microseconds, launches of a decode step / prompt kernel:
// 128 experts, 2048 columns: 1 token in 1 launch 8 / 69, 64 in 1 12 / 73, 128 in 2 24 / 73, 200 in 4 42 / 73, 64 in 8 93 / 73,
// 600 in 10 116 / 81; 8, 1024: 64 in 1 6 / 17, 128 in 2 17 / 17, 200 in 4 31 / 16; 16, 8192: 64 in 1 20 / 82, 200 in 4 71 /
// 100, 600 in 10 184 / 102; 256, 8192: 64 in 1 201 / 443, 64 in 8 269 / 440, 128 in 2 401 / 441, 200 in 4 643 / 442.
inline bool routed_like_decode(int P, int max_batch, int E, int H) {
  const int launches = (P + max_batch - 1) / max_batch;
  return P <= 128 && (launches <= 2 || 20.0 * launches < 2e-4 * E * H);
}

// The last experts of a prompt's layer: nothing travels beside their kernels any more, so these end the call.  Whether
// the experts of the last group are run one by one as they arrive, and the last one in pieces, by what the kernels of an
// expert are estimated to take (600 TFLOP/s, what the tiled kernel reaches on a whole expert) beside its transfer (57
// GB/s): only if a copy takes longer than its kernels, otherwise the kernels are the bottleneck and whole groups fill the
// device better, and only if there is more than the overhead of a launch pair and of a transfer (some 10 us each).
struct TailSplit {
  bool by_expert, pieces;
};
inline TailSplit prefill_tail(double positions, int H, int I, int group, std::size_t expert_bytes) {
  const double kernels_us = 6.0 * positions * H * I / 600e6, copy_us = double(expert_bytes) / 57e3;
  if (kernels_us > copy_us) return {false, false};
  const bool pieces = kernels_us >= 300.0;
  return {pieces || (kernels_us >= 15.0 && kernels_us * (group - 1) >= 100.0), pieces};
}

}  // namespace moe_spec
