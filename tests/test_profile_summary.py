"""Attribution of a profiler's dispatch list to the legs of bench.py (paper_2603_19289_amd/profile_summary.py)."""
import os
import random
import re
import subprocess

import bench
from paper_2603_19289_amd import profile_summary as P

NS = "void moe_spec::(anonymous namespace)::"
ROUTE, GATEUP, DOWN = NS + "route_pair_kernel<unsigned short, 4, 1, 1, false>", NS + "gateup_b1_pair_kernel<unsigned short, 4>", \
    NS + "down_combine_b1_kernel<unsigned short, 2, 6>"
JOINT, JOINT_MFMA = NS + "route_gateup_b1_kernel<unsigned short, 4>", NS + "route_gateup_mfma_kernel<1, 4, false>"
MFMA_GU, MFMA_DOWN, TILE_DOWN = NS + "expert_mfma_kernel<true, 1, 4>", NS + "expert_mfma_kernel<false, 1, 4>", NS + "expert_tile_kernel<false>"


def test_bench_counts_by_the_names_the_summary_cuts_at():
    assert {bench.ROUTE_SYM, bench.MFMA_GU_SYM, bench.MFMA_DOWN_SYM, "gateup_b1", "down_combine_b1", "advance_kernel"} <= set(P.COUNTED)
    assert {sym for _, sym in bench.KERNEL_NAMES.values()} <= set(P.COUNTED)


def test_joint_launches_have_a_row_of_their_own_and_count_as_routing_and_gate_up():
    # two tokens of two layers at batch one, the second joint in its second layer, then a batch of two with one joint
    # layer, then the plain gate/up by itself: plain rows hold plain launches only, and the cuts stay in step
    dispatches = [(ROUTE, 11.0), (GATEUP, 9.0), (DOWN, 6.0), (ROUTE, 12.0), (GATEUP, 10.0), (DOWN, 6.0),
                  (ROUTE, 13.0), (GATEUP, 9.5), (DOWN, 6.0), (JOINT, 18.0), (DOWN, 6.5),
                  (ROUTE, 16.0), (MFMA_GU, 47.0), (MFMA_DOWN, 27.0), (JOINT_MFMA, 53.0), (TILE_DOWN, 28.0),
                  (GATEUP, 8.0), (GATEUP, 8.1)]
    legs = [{"leg": "a/speculative/rep0", "counts": {bench.ROUTE_SYM: 4, "gateup_b1": 4, "down_combine_b1": 4}},
            {"leg": "b/speculative/rep0", "counts": {bench.ROUTE_SYM: 2, bench.MFMA_GU_SYM: 2, bench.MFMA_DOWN_SYM: 2}},
            {"leg": "a/isolated/expert_gateup_gemv", "counts": {"gateup_b1": 2}}]
    got = P.attribute(dispatches, legs)
    assert got == {
        ("a/speculative/rep0", "route_pair_kernel"): [11.0, 12.0, 13.0], ("a/speculative/rep0", "route_gateup_b1"): [18.0],
        ("a/speculative/rep0", "gateup_b1"): [9.0, 10.0, 9.5], ("a/speculative/rep0", "down_combine_b1"): [6.0, 6.0, 6.0, 6.5],
        ("b/speculative/rep0", "route_pair_kernel"): [16.0], ("b/speculative/rep0", "route_gateup_mfma"): [53.0],
        ("b/speculative/rep0", "expert_mfma_kernel<true"): [47.0], ("b/speculative/rep0", "expert_mfma_kernel<false"): [27.0],
        ("b/speculative/rep0", "expert_tile_kernel<false"): [28.0], ("a/isolated/expert_gateup_gemv", "gateup_b1"): [8.0, 8.1]}


def test_a_prompt_s_launches_stay_in_its_leg():
    # a prompt between two workloads, under the names its kernels have: position lists, tiles and its own routing
    lists = [NS + f"expert_mfma_lists_kernel<{b}, 4, 2>" for b in ("true", "false")]
    tiles = [NS + f"expert_tile_kernel<{b}>" for b in ("true", "false")]
    decode = [NS + "expert_mfma_kernel<true, 1, 4, 1, true>", NS + "expert_mfma_kernel<false, 1, 1, 4, true>"]
    route = NS + "route_prompt_kernel<unsigned short, 8>"
    dispatches = [(ROUTE, 11.0), (GATEUP, 9.0), (DOWN, 6.0), (route, 70.0), (lists[0], 20.0), (lists[1], 10.0), (tiles[0], 30.0),
                  (tiles[1], 15.0), (ROUTE, 16.0), (decode[0], 47.0), (decode[1], 27.0)]
    legs = [{"leg": "a/speculative/rep0", "counts": {bench.ROUTE_SYM: 1, "gateup_b1": 1, "down_combine_b1": 1}},
            {"leg": "a/prefill", "counts": {bench.ROUTE_SYM: 0, bench.ROUTE_PROMPT_SYM: 1, bench.MFMA_GU_SYM: 2, bench.MFMA_DOWN_SYM: 2}},
            {"leg": "b/speculative/rep0", "counts": {bench.ROUTE_SYM: 1}, "uncounted": [bench.MFMA_GU_SYM, bench.MFMA_DOWN_SYM]}]
    got = P.attribute(dispatches, legs)
    assert got == {
        ("a/speculative/rep0", "route_pair_kernel"): [11.0], ("a/speculative/rep0", "gateup_b1"): [9.0],
        ("a/speculative/rep0", "down_combine_b1"): [6.0], ("a/prefill", "route_prompt_kernel"): [70.0],
        ("a/prefill", "expert_mfma_lists_kernel<true"): [20.0], ("a/prefill", "expert_mfma_lists_kernel<false"): [10.0],
        ("a/prefill", "expert_tile_kernel<true"): [30.0], ("a/prefill", "expert_tile_kernel<false"): [15.0],
        ("b/speculative/rep0", "route_pair_kernel"): [16.0], ("b/speculative/rep0", "expert_mfma_kernel<true"): [47.0],
        ("b/speculative/rep0", "expert_mfma_kernel<false"): [27.0]}


def test_every_expert_kernel_of_the_library_is_counted():
    # a kernel that is renamed, or added, would be missing from the summaries or taken for another leg's
    csrc = os.path.join(os.path.dirname(os.path.abspath(P.__file__)), "csrc")
    names = set()
    for name in os.listdir(csrc):
        with open(os.path.join(csrc, name)) as f:
            names |= set(re.findall(r"\bvoid\s+(\w+_kernel)\s*\(", f.read()))
    names = {n for n in names if n.startswith(("expert_", "route_", "gateup_b1", "down_combine_b1"))}
    assert {"expert_mfma_kernel", "expert_mfma_lists_kernel", "expert_tile_kernel", "route_prompt_kernel"} <= names
    # the general kernels' lists and the one-routing kernel make launches that no leg counts
    for n in names - {"expert_lists_kernel", "route_kernel"}:
        assert any(P.named(f"{n}<{b}, ", symbol) for symbol in P.COUNTED for b in ("true", "false")), n


def test_launches_of_a_prompt_are_those_of_the_launch_rules(tmp_path):
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text(r"""
#include <cstdio>
#include "launch_rules.h"
using namespace moe_spec;
int main() {
  int P, mb, E, k, H, I, S, bf16, dma;
  while (std::scanf("%d %d %d %d %d %d %d %d %d", &P, &mb, &E, &k, &H, &I, &S, &bf16, &dma) == 9) {
    const int group = std::min(std::max(S / 2, 1), E), last = (E - 1) % group + 1;
    const TailSplit t = bf16 && dma ? prefill_tail(double(P) * k / E, H, I, last, std::size_t(6) * H * I) : TailSplit{false, false};
    int pairs = 0;
    for (int e0 = 0; e0 < E; e0 += group) pairs += t.by_expert && e0 + group >= E ? std::min(group, E - e0) + t.pieces : 1;
    std::printf("%d %d\n", routed_like_decode(P, mb, E, H) ? (P + mb - 1) / mb : 0, pairs);
  }
}""")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(os.path.dirname(os.path.abspath(P.__file__)), "csrc"), str(src),
                    "-o", str(exe)], check=True)
    rng = random.Random(8)
    cases = [[round(2 ** rng.uniform(0, 15)), rng.choice([1, 8, 64]), rng.randint(4, 256), rng.randint(1, 4), 8 * rng.randint(1, 1024),
              8 * rng.randint(1, 2000), rng.randint(4, 256), rng.randint(0, 1), rng.randint(0, 1)] for _ in range(3000)]
    done = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, c)) for c in cases), capture_output=True, text=True, timeout=60)
    want = [tuple(map(int, line.split())) for line in done.stdout.splitlines()]
    got = [tuple(map(int, P.prompt_launches(*c[:7], c[7] == 1, c[8] == 1))) for c in cases]
    assert got == want and any(w[0] for w in want) and not all(w[0] for w in want)


def test_launches_queued_in_vain_are_not_counted():
    gateup, down = GATEUP.replace("4>", "4, {}>"), DOWN[:-1] + ", {}>"
    step = [(ROUTE, 6.0)]
    queued, again = [(gateup.format("true"), 10.0), (down.format("true"), 6.0)], [(gateup.format("false"), 10.5), (down.format("false"), 6.5)]
    void = [(n, 1.5) for n, _ in queued]
    assert P.without_void(step + queued + step + void + again + step + again) == step + queued + step + again + step + again
    signature = [(n + "(moe_spec::ExpertArgs)", v) for n, v in step + void + again]
    assert P.without_void(signature) == [signature[0]] + signature[3:]
