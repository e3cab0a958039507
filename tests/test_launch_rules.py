"""The rules that deal a launch's work to workgroups (csrc/launch_rules.h), swept on the CPU over the sizes the library
takes and over the compute-unit counts of a whole device and of its partitions."""
import os
import subprocess

from tests.helpers import SHARED_ROWS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def sweep(tmp_path, body):
    """Compiles a program around the rules and runs it: it prints the cases that break a rule and returns their number."""
    src, exe = tmp_path / "sweep.cpp", tmp_path / "sweep"
    src.write_text('#include <cstdio>\n#include "launch_rules.h"\nusing namespace moe_spec;\nint main() {\n  int bad = 0;\n'
                   + body + "\n  return bad ? 1 : 0;\n}\n")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2603_19289_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    done = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert done.returncode == 0, (done.returncode, done.stdout[-2000:])


def test_gate_up_rows_beside_the_routing_are_dealt_whatever_the_routing_takes(tmp_path):
    # every row belongs to exactly one wavefront, at least one row each (the body takes no pairs), and no workgroup is
    # left with more than its share of a quarter of the device, also where the routing takes every place
    sweep(tmp_path, r"""
  for (int cus : {32, 64, 128, 256}) for (int per_cu : {1, 2, 4, 8}) for (int E = 1; E <= 256; ++E) {
    const int n_route = joint_routing_workgroups(E);
    if (long(n_route) > long(per_cu) * cus) continue;         // refused by the launcher
    for (int H : {8, 512, 1024, 2048, 2880, 4096}) for (int I : {8, 768, 2880, 14336, 32768}) for (int k : {1, 2, 8, 16}) {
      for (int wbytes : {2, 4}) {
        const int nch = (H + 64 * (16 / wbytes) - 1) / (64 * (16 / wbytes));
        const GateupSplit s = beside_routing_split(nch, I, H, k, wbytes, n_route, per_cu, cus);
        const long wgs = long(s.blocks) * k, share = (long(I) * k + cus - 1) / cus;   // rows per wavefront of cus / 4 workgroups
        const bool ok = s.rpw >= 1 && long(s.blocks) * kB1Waves * s.rpw >= I && long(s.blocks - 1) * kB1Waves * s.rpw < I &&
                        wgs >= 1 && s.rpw <= share;
        if (!ok && ++bad <= 20)
          std::printf("cus %d per_cu %d E %d H %d I %d k %d wbytes %d: rpw %d blocks %d\n", cus, per_cu, E, H, I, k, wbytes, s.rpw, s.blocks);
      }
    }
  }""")


def test_estimator_projection_gets_workgroups_for_its_rows(tmp_path):
    # the rows of the projection are dealt in pairs to the wavefronts of a token's workgroups: one pair each (two beside
    # experts), or as many as it takes when the tokens' workgroups fill the device, whatever the number of experts; every
    # router row has a place; the launch without a projection is sized by the router alone
    sweep(tmp_path, r"""
  for (int cus : {32, 64, 128, 256}) for (int E : {1, 3, 8, 16, 32, 128, 200, 256}) for (int B = 1; B <= 64; ++B) {
    for (int rows : {0, 8, 64, 72, 256, 512, 1024, 4096, 8192}) {
      if (B > cus) continue;
      const int room = std::max(1, cus / B), pairs = (rows + 1) / 2;
      auto share = [](int n, int wgs) { return (n + kRouteWaves * wgs - 1) / (kRouteWaves * wgs); };   // per wavefront
      const int beside = beside_experts_workgroups(E, rows, B, cus);
      bool ok = beside >= 1 && beside <= room && share(pairs, beside) <= std::max(2, share(pairs, room));
      if (rows == 0) ok = ok && beside == std::max(1, std::min(cus / B, (E + 3) / 4));
      for (int per_wg : {1, 4, 16}) {
        const int router = (E + per_wg - 1) / per_wg, own = routing_workgroups(E, per_wg, rows, B, cus);
        ok = ok && own >= router && own <= std::max(router, room) && share(pairs, own) <= std::max(1, share(pairs, room));
        if (rows == 0) ok = ok && own == router;
      }
      if (!ok && ++bad <= 20) std::printf("cus %d E %d B %d rows %d: %d beside\n", cus, E, B, rows, beside);
    }
  }""")


def test_prefill_tail_is_split_only_where_copies_are_the_bottleneck(tmp_path):
    sweep(tmp_path, r"""
  for (double pos : {1.0, 100.0, 2500.0, 30000.0, 500000.0}) for (int H : {8, 1024, 4096, 8192}) for (int I : {8, 768, 14336, 32768})
    for (int group : {1, 2, 8, 128}) {
      const std::size_t bytes = std::size_t(6) * H * I;
      const TailSplit t = prefill_tail(pos, H, I, group, bytes);
      const double kernels = 6.0 * pos * H * I / 600e6;
      const bool ok = (!t.pieces || t.by_expert) && (kernels <= bytes / 57e3 || !t.by_expert) && (kernels >= 15.0 || !t.by_expert);
      if (!ok && ++bad <= 20) std::printf("pos %g H %d I %d group %d\n", pos, H, I, group);
    }""")


def test_rows_shared_with_the_routing_workgroups_are_dealt_once(tmp_path):
    # stream and tail together hold every row of an expert exactly once, no workgroup starts past its rows, and the first
    # routing workgroup is left out; the whole device and its partitions get there
    sweep(tmp_path, r"""
  for (int cus : {32, 64, 128, 256}) {
    int shared = 0;
    for (int per_cu : {1, 2, 4}) for (int E = 1; E <= 256; ++E) {
      const int n_route = joint_routing_workgroups(E);
      if (2 * n_route < E || 2 * n_route > E + 1) ++bad;      // two router rows each
      if (long(n_route) > long(per_cu) * cus) continue;
      for (int H : {8, 512, 1016, 1024, 2048, 2880}) for (int I : {8, 328, 480, 704, 768, 1600, 14336}) for (int k : {1, 2, 8, 16}) for (int wbytes : {2, 4}) {
        const int nch = (H + 64 * (16 / wbytes) - 1) / (64 * (16 / wbytes));
        const GateupSplit base = beside_routing_split(nch, I, H, k, wbytes, n_route, per_cu, cus);
        const SharedSplit s = share_with_routing(base, I, H, k, wbytes, n_route, cus);
        const long stream = long(s.stream.blocks) * kB1Waves * s.stream.rpw;
        const bool ok = s.stream.rpw >= 1 && stream >= s.first_tail && stream - kB1Waves * s.stream.rpw < s.first_tail &&
                        s.first_tail + long(s.tail_blocks) * kB1Waves * s.tail_rpw == I && s.tail_blocks * k <= n_route - 1 + (s.tail_blocks == 0);
        shared += s.tail_blocks > 0;
        if (!ok && ++bad <= 20) std::printf("cus %d E %d H %d I %d k %d wbytes %d\n", cus, E, H, I, k, wbytes);
      }
    }
    if (shared == 0) { ++bad; std::printf("cus %d: never\n", cus); }
  }""")


def test_cache_waves_stay_behind_a_prefetch_where_it_would_slow_them_down(tmp_path):
    # (experts of a step, slots, bytes of an expert): measured slower on the compute stream, and faster
    sweep(tmp_path, r"""
  const std::size_t MB = 1000000;
  const struct { int experts, slots; std::size_t bytes; bool in_order; } cases[] = {
    {28, 16, 50 * MB, false}, {28, 14, 50 * MB, false}, {16, 10, 50 * MB, false}, {28, 16, 28 * MB, false}, {28, 16, 9 * MB, false},
    {28, 8, 50 * MB, true}, {28, 24, 50 * MB, true}, {16, 6, 50 * MB, true}, {28, 8, 6 * MB, true}, {28, 14, 3 * MB, true}, {16, 10, MB, true}};
  for (const auto &c : cases)
    if (waves_in_order(c.experts, c.slots, c.bytes) != c.in_order) { ++bad; std::printf("%d %d %zu\n", c.experts, c.slots, c.bytes); }""")


def test_short_prompts_are_routed_by_the_launches_of_a_decode_step(tmp_path):
    # (tokens, largest batch, experts, columns): measured faster that way, and slower
    sweep(tmp_path, r"""
  const struct { int P, max_batch, E, H; bool decode; } cases[] = {
    {1, 64, 8, 1024, true}, {64, 64, 128, 2048, true}, {128, 64, 128, 2048, true}, {1, 1, 256, 8192, true}, {64, 8, 256, 8192, true},
    {16, 1, 256, 8192, true}, {200, 64, 256, 8192, false}, {600, 64, 128, 2048, false}, {64, 8, 128, 2048, false},
    {16, 1, 128, 2048, false}, {200, 64, 8, 1024, false}, {32768, 64, 8, 4096, false}};
  for (const auto &c : cases)
    if (routed_like_decode(c.P, c.max_batch, c.E, c.H) != c.decode) { ++bad; std::printf("%d %d %d %d\n", c.P, c.max_batch, c.E, c.H); }""")


def test_routing_workgroups_take_rows_at_the_sizes_of_the_gpu_test(tmp_path):
    # on the whole device, with the number of routing workgroups that the launch has
    sizes = ", ".join("{%d, %d, %d, %d}" % s for s in SHARED_ROWS)
    sweep(tmp_path, r"""
  const int sizes[][4] = {""" + sizes + r"""};
  for (const auto &v : sizes) for (int per_cu : {2, 3, 4}) {
    const int nch = (v[0] + 511) / 512, n_route = joint_routing_workgroups(v[2]);
    const SharedSplit s = share_with_routing(beside_routing_split(nch, v[1], v[0], v[3], 2, n_route, per_cu, 256), v[1], v[0], v[3], 2, n_route, 256);
    if (s.tail_blocks < 1) { ++bad; std::printf("%d %d %d %d\n", v[0], v[1], v[2], v[3]); }
  }""")


def test_estimator_groups_cover_the_batch_and_fit_on_the_device(tmp_path):
    sweep(tmp_path, r"""
  int taken = 0;
  for (int cus : {32, 64, 128, 256}) for (int dm : {8, 88, 512, 2048, 2056, 4096, 8192}) for (int F : {8, 176, 1024, 4096, 4104, 65536})
    for (int B = 1; B <= 64; ++B) {
      const EstimatorSplit s = estimator_split(dm, F, B, cus);
      if (s.wgs == 0) { if (std::max(dm, F) <= 4096 && B * 4 <= cus) ++bad; continue; }
      ++taken;
      const bool ok = s.tokens >= 1 && s.tokens <= 2 && s.tokens * std::max(dm, F) <= 4096 && s.groups * s.tokens >= B &&
                      (s.groups - 1) * s.tokens < B && s.wgs >= 4 && s.wgs * s.groups <= cus;
      if (!ok && ++bad <= 20) std::printf("cus %d dm %d F %d B %d: %d %d %d\n", cus, dm, F, B, s.tokens, s.groups, s.wgs);
    }
  if (!taken) ++bad;""")


def test_blocks_are_dealt_to_the_copy_queues_once_and_their_shares_settle(tmp_path):
    # every byte of a request goes to one queue; two queues of unequal speeds come to be done together, whatever the number of
    # blocks, and go back to even shares when the speeds are equal again; equal queues are left alone, odd blocks or not
    sweep(tmp_path, r"""
  for (int n = 1; n <= 256; ++n) for (std::size_t block : {std::size_t(3) * 8 * 8 * 2, std::size_t(9437184), std::size_t(352321536)})
    for (double share : {0.1, 0.29, 0.37, 0.5, 0.61, 0.9}) {
      const QueueDeal d = deal_to_queues(n, block, share);
      const bool ok = d.second >= 0 && d.second + (d.cut > 0) <= n && d.cut < block &&
                      (n < 2 || share == kEvenShare || block < 65536 || std::abs(d.second + double(d.cut) / block - share * n) <= 0.126);
      if (!ok && ++bad <= 20) std::printf("n %d block %zu share %g: %d %zu\n", n, block, share, d.second, d.cut);
    }
  for (int n = 1; n <= 256; ++n) for (std::size_t block : {std::size_t(3) * 8 * 8 * 2, std::size_t(316800), std::size_t(9437184)})
    for (int percent = 10; percent <= 90; ++percent) {
      const double share = percent / 100.0;                  // 0.5: even
      const QueueDeal d = deal_to_queues(n, block, share);
      std::size_t second = 0;
      int cuts = 0;
      bool ok = true;
      for (int i = 0; i < n; ++i) {
        const std::size_t b = second_queue_bytes(n, block, share, i);
        ok = ok && b <= block && (b == 0 || b == block || (b == d.cut && b % 4096 == 0 && i == n - 1));
        cuts += b != 0 && b != block;
        second += b;
      }
      ok = ok && second == d.second * block + d.cut && cuts == (d.cut > 0);
      if (!ok && ++bad <= 20) std::printf("n %d block %zu share %g: %zu of %d + %zu\n", n, block, share, second, d.second, d.cut);
    }
  const double block = 9437184, link = 57e3;               // bytes per us
  // lead: the second queue begins a request earlier, as it does where copies never pause (only the first waits at a request's
  // end): being done earlier then says nothing about its speed; a slow first queue cannot be told from that and is left alone
  for (double slow : {1.0, 0.55, 0.7}) for (int which : {0, 1}) for (int n : {2, 3, 7, 8, 16}) for (double lead : {0.0, 150.0, 600.0, 1200.0}) {
    if (slow != 1.0 && which == 1 && lead > 0.0) continue;   // a queue that lags does not lead
    double share = kEvenShare, late = 0, length = 0;
    bool sign = false;
    for (int step = 0; step < 60; ++step) {
      const double factor = step < 40 ? slow : 1.0;
      const QueueDeal d = deal_to_queues(n, std::size_t(block), share);
      double left[2] = {n * block - (d.second * block + d.cut), d.second * block + d.cut};
      const double taken = left[1] / (n * block), own[2] = {55e3 * (which == 0 ? factor : 1.0), 55e3 * (which == 1 ? factor : 1.0)};
      double at[2] = {0, 0}, t = -lead;                      // both: the link shared by speed; one: its own speed
      while (left[0] > 1 || left[1] > 1) {
        const bool runs[2] = {left[0] > 1 && t >= 0, left[1] > 1};
        double v[2], go = t < 0 ? -t : 1e30;
        for (int q = 0; q < 2; ++q) v[q] = runs[0] && runs[1] ? std::min(own[q], link * own[q] / (own[0] + own[1])) : own[q];
        for (int q = 0; q < 2; ++q) if (runs[q]) go = std::min(go, left[q] / v[q]);
        t += go;
        for (int q = 0; q < 2; ++q) if (runs[q]) { left[q] -= v[q] * go; if (left[q] <= 1) at[q] = t; }
      }
      late = at[1] - at[0]; length = t;
      share = next_queue_share(share, taken, late, n * block, &sign);
      if ((slow == 1.0 || which == 0) && share != kEvenShare) { ++bad; std::printf("even n %d slow %g lead %g: %g\n", n, slow, lead, share); break; }
      if (step == 39 && slow < 0.6 && which == 1 && n >= 7 && std::abs(late) > 0.25 * length) { ++bad; std::printf("slow %g n %d: %g of %g\n", slow, n, late, length); }
    }
    if (share != kEvenShare) { ++bad; std::printf("not even again: slow %g queue %d n %d lead %g: %g\n", slow, which, n, lead, share); }
  }
  // requests of seven and of eight blocks measured in a decode loop bound by the link, no queue slow
  const double seen[][3] = {{0.429, -1134.4, 66.1e6}, {0.429, -1120.2, 66.1e6}, {0.5, -989.5, 75.5e6}, {0.5, -392.9, 37.7e6}, {0.4, -875.8, 47.2e6}};
  bool sign = false;
  for (int step = 0; step < 20; ++step) if (next_queue_share(kEvenShare, seen[step % 5][0], seen[step % 5][1], seen[step % 5][2], &sign) != kEvenShare) ++bad;
""")
