"""Attribution of a profiler's dispatch list to the legs of bench.py (paper_2603_19289_amd/profile_summary.py)."""
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
