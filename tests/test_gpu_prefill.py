"""GPU parity of the prefill step (Sec. 5.2, prefill phase): all prompt tokens of a layer at once, every
expert streamed through the layer's slots, true routing executed.  Against the CPU checker on the same
seeded inputs: ids equal, gates to float32 rounding, outputs within 1e-5 (float32) / 2e-2 (bf16), and
the transfer counters equal (E expert blocks per layer)."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from paper_2603_19289_amd import moe_spec as M
from paper_2603_19289_amd import workload as W
from tests.helpers import build, check_output, kernels_launched, launches, make_advance, oracle_model, small_workload

pytestmark = pytest.mark.gpu

def prompt_of(wl, P):
    """[P,H] first-layer residuals and [L,P,H] noise for the layer-to-layer update, from the seeded generators."""
    x0, eps = W.make_inputs(dataclasses.replace(wl, batch=P), tokens=1)
    return x0[0], eps[0]


def run_prefill(wl, P, max_batch, label, prebuilt=None, load=None, **engine_kw):
    from paper_2603_19289_amd.engine import engine_for
    print(f"[case] prefill {label} L={wl.n_layers} H={wl.hidden} E={wl.n_experts} k={wl.top_k} I={wl.inter} "
          f"P={P} micro-batch={max_batch} S={wl.slots} {wl.dtype} {engine_kw}", flush=True)
    if prebuilt is None:
        res, ex, model = build(wl, "random")
    else:
        res, model, ex = prebuilt
    r_np, eps = prompt_of(wl, P)
    orc = O.MoEOracle(model, O.MODE_SPECULATIVE, wl.slots)
    eng = engine_for(wl, O.MODE_SPECULATIVE, res, ex, max_batch=max_batch, max_prefill_tokens=P + 3, **engine_kw)
    worst = worst_elem = 0.0
    try:
        for l in range(wl.n_layers):
            want = orc.prefill_layer_step(l, r_np)
            if load is not None:
                load[:] = np.bincount(want.true_ids.ravel(), minlength=wl.n_experts)
            r = torch.from_numpy(r_np.astype(np.float32)).to("cuda")
            out, ids, gates = eng.prefill_layer_step(l, r, want_ids=True)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(ids.cpu().numpy(), want.true_ids, err_msg=f"layer {l}")
            np.testing.assert_allclose(gates.cpu().numpy(), want.true_gates, atol=2e-7, rtol=1e-6, err_msg=f"layer {l}")
            l2, elem = check_output(out.cpu().numpy(), want.out, wl.dtype, f"layer {l}", terms=wl.top_k * wl.inter)
            worst, worst_elem = max(worst, l2), max(worst_elem, elem)
            r_np = W.advance_residual(wl, r_np, want.out, eps[l])
        st = eng.stats()
        for name in ("layer_steps", "cache_hits", "cache_misses", "h2d_bytes", "predictions"):
            assert st[name] == getattr(orc.stats, name), (name, st[name], getattr(orc.stats, name))
        assert st["prefill_tokens"] == P * wl.n_layers
    finally:
        eng.close()
    print(f"[ok] worst relative L2 error {worst:.3e}, worst element error {worst_elem:.3e} of the row RMS", flush=True)


@pytest.mark.parametrize("copy_engine", [M.COPY_DMA, M.COPY_KERNEL, M.COPY_DMA2])
def test_prefill_fp32_ragged_micro_batches(copy_engine):
    wl = small_workload(n_layers=2, dtype="f32", slots=4)           # groups of 2 experts, 4 groups per layer
    run_prefill(wl, P=37, max_batch=16, label="f32", copy_engine=copy_engine)


def test_prefill_bf16_matrix_core_and_generic_tail():
    wl = small_workload(n_layers=2, hidden=128, n_experts=16, top_k=4, inter=96, dtype="bf16", slots=5)
    run_prefill(wl, P=100, max_batch=32, label="bf16 odd S", copy_engine=M.COPY_DMA2)   # 32+32+32+4 tokens


def test_prefill_bf16_small_micro_batch():
    wl = small_workload(n_layers=1, hidden=128, n_experts=16, top_k=4, inter=96, dtype="bf16", slots=8)
    run_prefill(wl, P=19, max_batch=8, label="bf16 generic", copy_engine=M.COPY_DMA)


def test_prefill_single_slot_and_single_token():
    wl = small_workload(n_layers=2, top_k=1, slots=1, dtype="f32")  # one slot: copy and compute alternate
    run_prefill(wl, P=5, max_batch=4, label="S=1", copy_engine=M.COPY_DMA2)
    run_prefill(small_workload(n_layers=1, dtype="f32"), P=1, max_batch=1, label="P=1", copy_engine=M.COPY_DMA)


def test_prefill_pool_larger_than_expert_count():
    wl = small_workload(n_layers=1, dtype="bf16", slots=40)         # both halves hold all 8 experts: one group
    run_prefill(wl, P=21, max_batch=16, label="S>2E", copy_engine=M.COPY_KERNEL)


@pytest.mark.parametrize("hidden,inter,experts,top_k,P", [
    (72, 136, 4, 2, 4300),        # one chain of sums, a reduction that ends inside a step, rows past the matrix
    (520, 264, 6, 3, 2900),       # two chains of sums, two and three row tiles
    (64, 1032, 3, 1, 8300),       # the down projection's reduction ends inside its third chain
    (128, 128, 64, 1, 9000),      # whole tiles of rows; many experts with about one tile of positions each
])
def test_prefill_tiled_matrix_product(hidden, inter, experts, top_k, P):
    """Prompts long enough for the tiled kernel in the gate/up and the down launch: positions per expert
    around its 128-position tile, remainders of its 64-column steps and of its row tiles."""
    wl = small_workload(n_layers=1, hidden=hidden, n_experts=experts, top_k=top_k, inter=inter, dtype="bf16", slots=2 * experts)
    counts = kernels_launched(lambda: run_prefill(wl, P=P, max_batch=64, label="tiles", copy_engine=M.COPY_DMA2),
                              {"expert_lists": 1, "combine": 1})
    assert (launches(counts, "expert_tile_kernel<true>"), launches(counts, "expert_tile_kernel<false>")) == (1, 1), counts


@pytest.mark.parametrize("hidden,inter,top_k,P,slots,groups", [(520, 264, 1, 9000, 4, 3), (264, 520, 2, 5000, 6, 2),
                                                               (520, 264, 1, 9000, 12, 1)])
def test_prefill_tiled_matrix_product_uneven_experts(hidden, inter, top_k, P, slots, groups):
    """The same kernel with several groups of experts (launch pairs), experts of very different load in a launch and, with
    top-1 routing, one without a position: expert 5 has expert 0's router row, and of equal logits the lower index wins."""
    wl = small_workload(n_layers=1, hidden=hidden, n_experts=6, top_k=top_k, inter=inter, dtype="bf16", slots=slots)
    res, ex, _ = build(wl, "random")
    row = res["router_w"][0]
    w = O.decode_weights(row)
    row[1] = W.to_storage(3 * w[1], "bf16")                # chosen often
    row[2] = W.to_storage(0.6 * w[0] + 0.6 * w[4], "bf16")  # between two others: seldom the largest logit
    row[3] = W.to_storage(0.51 * w[0] + 1.53 * w[1], "bf16")
    row[5] = row[0]
    model = oracle_model(wl, res, ex)
    load = np.zeros(6, dtype=int)
    counts = kernels_launched(lambda: run_prefill(wl, P=P, max_batch=64, label="uneven tiles", prebuilt=(res, model, ex),
                                                  copy_engine=M.COPY_DMA2, load=load), {"expert_lists": 1, "combine": 1})
    print("[case] positions per expert", load.tolist(), flush=True)
    assert top_k > 1 or (load.max() > 10 * load[2] > 10 * load[3] > 0 and load[5] == 0), load
    assert (launches(counts, "expert_tile_kernel<true>"), launches(counts, "expert_tile_kernel<false>")) == (groups, groups), counts


@pytest.mark.parametrize("name,P,layers", [("c2_qwen3_30b_a3b", 150, 2), ("c3_gpt_oss_20b", 70, 1)])
def test_prefill_at_full_layer_shape(name, P, layers):
    """The benchmark's layer shape and slot count, micro-batches of 64 tokens plus a ragged tail."""
    from tests.test_gpu_full_shapes import prebuilt
    wl = W.CONFIGS[name].with_(n_layers=layers, tokens=1)
    run_prefill(wl, P=P, max_batch=64, label=name, prebuilt=prebuilt(wl), copy_engine=M.COPY_DMA2)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_default_vectors_calibrated_by_prefill(dtype):
    """Offline calibration (Sec. 3.1): two prompts through the prefill step with accumulation on; the
    per-expert mean outputs and execution counts equal the checker's."""
    from paper_2603_19289_amd.engine import engine_for
    wl = small_workload(n_layers=2, hidden=136, n_experts=12, top_k=3, inter=104, dtype=dtype, slots=6, seed=23)
    res, ex, model = build(wl, "random")
    orc = O.MoEOracle(model, O.MODE_ON_DEMAND, wl.slots)
    eng = engine_for(wl, O.MODE_ON_DEMAND, res, ex, max_batch=16, max_prefill_tokens=64, accumulate_defaults=1,
                     copy_engine=M.COPY_DMA)
    try:
        for P, seed in ((41, 23), (18, 24)):
            r_np, eps = prompt_of(dataclasses.replace(wl, seed=seed), P)
            for l in range(wl.n_layers):
                want = orc.prefill_layer_step(l, r_np)
                out, _, _ = eng.prefill_layer_step(l, torch.from_numpy(r_np.astype(np.float32)).to("cuda"))
                torch.cuda.synchronize()
                check_output(out.cpu().numpy(), want.out, dtype, f"prompt of {P}, layer {l}")
                r_np = W.advance_residual(wl, r_np, want.out, eps[l])
        for l in range(wl.n_layers):
            mean, counts = eng.read_default_vectors(l)
            assert counts == orc.dacc_cnt[l].tolist()
            got, want = mean.cpu().numpy().astype(np.float64), orc.default_vectors(l)
            for e in range(wl.n_experts):
                if counts[e]:
                    check_output(got[e], want[e], dtype, f"default vector of layer {l}, expert {e}")
                else:
                    assert not got[e].any()
    finally:
        eng.close()


@pytest.mark.parametrize("mode", [O.MODE_SPECULATIVE, O.MODE_ON_DEMAND])
def test_decode_after_prefill_starts_from_an_empty_cache(mode):
    """Prefill over every layer, then decode steps: ids, outputs and cache counters follow the checker,
    whose pools are empty after its prefill."""
    from paper_2603_19289_amd.engine import engine_for
    wl = small_workload(n_layers=3, dtype="bf16", batch=2, tokens=3, slots=4)
    res, ex, model = build(wl, "random")
    P = 11
    r_np, eps_p = prompt_of(wl, P)
    x0, eps = W.make_inputs(wl)
    orc = O.MoEOracle(model, mode, wl.slots)
    eng = engine_for(wl, mode, res, ex, max_batch=4, max_prefill_tokens=P, copy_engine=M.COPY_DMA2)
    try:
        # a few decode steps first so that the pools hold something the prefill must drop
        warm = O.run_tokens(orc, x0[:1], make_advance(wl, eps))
        eng.begin_token()
        for l in range(wl.n_layers):
            eng.layer_step(l, torch.from_numpy(warm[0][l][0].astype(np.float32)).to("cuda"))
        for l in range(wl.n_layers):
            want = orc.prefill_layer_step(l, r_np)
            out, _, _ = eng.prefill_layer_step(l, torch.from_numpy(r_np.astype(np.float32)).to("cuda"))
            torch.cuda.synchronize()
            check_output(out.cpu().numpy(), want.out, "bf16", f"prefill layer {l}")
            r_np = W.advance_residual(wl, r_np, want.out, eps_p[l])
        trace = O.run_tokens(orc, x0[1:], lambda t, l, r, out: W.advance_residual(wl, r, out, eps[t + 1, l]))
        for t in range(len(trace)):
            eng.begin_token()
            for l in range(wl.n_layers):
                r_l, want = trace[t][l]
                out, ids = eng.layer_step(l, torch.from_numpy(r_l.astype(np.float32)).to("cuda"), want_ids=True)
                torch.cuda.synchronize()
                np.testing.assert_array_equal(ids["exec_ids"].cpu().numpy(), want.exec_ids)
                check_output(out.cpu().numpy(), want.out, "bf16", f"decode token {t} layer {l}")
        st = eng.stats()
        for name in ("tokens", "layer_steps", "predictions", "hits", "cache_hits", "cache_misses", "h2d_bytes"):
            assert st[name] == getattr(orc.stats, name), (name, st[name], getattr(orc.stats, name))
    finally:
        eng.close()


def test_prefill_argument_and_state_errors():
    from paper_2603_19289_amd.engine import engine_for
    wl = small_workload(n_layers=2, dtype="f32")
    res, ex, _ = build(wl)
    r = torch.zeros((4, wl.hidden), dtype=torch.float32, device="cuda")
    eng = engine_for(wl, O.MODE_SPECULATIVE, res, ex, max_batch=2, max_prefill_tokens=3)
    try:
        with pytest.raises(M.MoeSpecError) as ei:
            eng.prefill_layer_step(0, r)                        # 4 tokens > 3
        assert ei.value.code == M.EINVAL
        with pytest.raises(M.MoeSpecError) as ei:
            eng.prefill_layer_step(2, r[:2].contiguous())       # no such layer
        assert ei.value.code == M.EINVAL
        eng.begin_token()
        with pytest.raises(M.MoeSpecError) as ei:
            eng.prefill_layer_step(0, r[:2].contiguous())       # inside a decode step
        assert ei.value.code == M.ESTATE
    finally:
        eng.close()
    eng = engine_for(wl, O.MODE_SPECULATIVE, res, ex, max_batch=2)
    try:
        with pytest.raises(M.MoeSpecError) as ei:
            eng.prefill_layer_step(0, r[:2].contiguous())       # created without a prefill path
        assert ei.value.code == M.ESTATE
    finally:
        eng.close()


def test_prefill_randomised_configurations():
    """Eighty seeded draws of layer sizes, expert counts, pool sizes, prompt lengths, micro-batches, dtypes and copy
    engines within the documented limits, each against the checker."""
    rng = np.random.default_rng(21)
    hiddens = [8, 16, 24, 40, 64, 72, 136, 256, 520, 1000]
    inters = [8, 16, 40, 48, 104, 256]
    for case in range(80):
        H, I = int(rng.choice(hiddens)), int(rng.choice(inters))
        E = int(rng.integers(1, 49)) if rng.random() < 0.9 else int(rng.integers(49, 200))
        k = int(rng.integers(1, min(E, 16) + 1))
        S = int(rng.integers(k, E + 3))
        P = int(rng.choice([1, 2, 3, 7, 16, 17, 33, 64, 65, 100, 130, 257]))
        micro = int(rng.choice([1, 2, 3, 8, 16, 31, 64]))
        dtype = "bf16" if rng.random() < 0.7 else "f32"
        L = int(rng.integers(1, 4))
        while L * E * 3 * H * I > 1.0e8:             # the pool is drawn on the CPU
            if I > 48:
                I = 48
            elif H > 136:
                H = 136
            else:
                E = max(k, E // 2)
                S = max(k, min(S, E + 2))
        while P * k * L * 3 * H * I > 1.5e9 and P > 1:   # the checker's work
            P = max(1, P // 2)
        wl = small_workload(name=f"pdraw{case}", n_layers=L, hidden=H, n_experts=E, top_k=k, inter=I, dtype=dtype,
                            batch=1, tokens=1, slots=S, seed=5000 + case)
        run_prefill(wl, P=P, max_batch=micro, label=f"draw {case}", copy_engine=int(rng.integers(0, 3)))


def test_prefill_after_decode_starts_its_copies_beside_the_routing():
    """The experts of a prompt travel while its tokens are routed, also into a pool that the decode step just before has
    read: the copies wait for that step's kernels, not for the prompt's routing.  The layer is shaped so that routing
    (128 launches of 64 tokens, 256 experts) takes longer than issuing it and than the copies; behind the routing the
    copies lengthen the call by a third (7.1 against 5.3 ms).  Compared with the same call after another prefill, which
    finds the kernels before it ended, whatever hardware queues the process's streams share."""
    from paper_2603_19289_amd.engine import engine_for
    P = 8192
    wl = small_workload(name="decode_then_prefill", n_layers=1, hidden=4096, n_experts=256, top_k=1, inter=8, dtype="bf16",
                        slots=512, seed=43)
    res, ex, _ = build(wl)
    eng = engine_for(wl, M.MODE_SPECULATIVE, res, ex, max_batch=64, max_prefill_tokens=P, copy_engine=M.COPY_DMA2)
    r = torch.randn((P, wl.hidden), generator=torch.Generator(device="cuda").manual_seed(9), device="cuda")
    took = {"prefill": [], "decode": []}
    try:
        eng.prefill_layer_step(0, r)
        for before in ("prefill", "decode") * 5:
            if before == "decode":
                eng.begin_token()
                eng.layer_step(0, r[:1])
            torch.cuda.synchronize()
            start, done = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record(eng.compute)
            eng.prefill_layer_step(0, r)
            done.record(eng.compute)
            torch.cuda.synchronize()
            took[before].append(start.elapsed_time(done))
    finally:
        eng.close()
    print("[case] prefill after " + ", after ".join(f"{k}: {min(v):.2f} ms" for k, v in took.items()), flush=True)
    assert min(took["decode"]) < 1.15 * min(took["prefill"]), took


@pytest.mark.parametrize("dtype,hidden,experts,top_k,P", [
    ("bf16", 8, 1, 1, 1), ("bf16", 40, 16, 16, 15), ("f32", 72, 17, 4, 16), ("bf16", 136, 33, 8, 17), ("f32", 1032, 64, 16, 33),
    ("bf16", 264, 65, 3, 31), ("f32", 40, 129, 16, 20), ("bf16", 2056, 128, 8, 18), ("bf16", 72, 256, 16, 47), ("bf16", 8192, 9, 2, 16)])
def test_prefill_routing_at_the_edges_of_its_tiles(dtype, hidden, experts, top_k, P):
    """The routing of a prompt at every number of router tiles, with row counts around 16, reductions that end inside
    a 32-column step, and token counts around its 16-token tile; two experts with the same router row, of whose equal logits
    the lower index wins."""
    wl = small_workload(n_layers=1, hidden=hidden, n_experts=experts, top_k=top_k, inter=8, dtype=dtype, slots=experts)
    res, ex, _ = build(wl, "random")
    if experts > 1:
        res["router_w"][0][experts - 1] = res["router_w"][0][0]
    run_prefill(wl, P=P, max_batch=16, label="routing", prebuilt=(res, oracle_model(wl, res, ex), ex))


@pytest.mark.parametrize("dtype,hidden,experts,top_k,P,max_batch,launches_like_decode", [
    ("bf16", 40, 16, 16, 15, 4, 0), ("f32", 72, 17, 4, 16, 4, 0), ("bf16", 136, 33, 8, 17, 4, 0), ("f32", 1032, 64, 16, 33, 16, 0),
    ("bf16", 264, 65, 3, 31, 8, 0), ("f32", 40, 129, 16, 20, 1, 0), ("bf16", 2056, 128, 8, 18, 4, 0), ("bf16", 72, 256, 16, 47, 16, 0),
    ("bf16", 8192, 9, 2, 16, 4, 0), ("bf16", 2056, 128, 8, 18, 18, 1), ("f32", 264, 12, 3, 40, 39, 2), ("bf16", 264, 12, 3, 128, 64, 2),
    ("f32", 264, 12, 3, 129, 64, 0), ("bf16", 8192, 64, 2, 10, 4, 3)])
def test_prefill_routing_by_the_prompt_kernel_and_by_decode_launches(dtype, hidden, experts, top_k, P, max_batch, launches_like_decode):
    """Prompts of up to two micro-batches, and of more where the routers are large, are routed by the launches of a decode
    step, all others by the kernel for prompts; both against the checker, at the edges of the latter's tiles."""
    wl = small_workload(n_layers=1, hidden=hidden, n_experts=experts, top_k=top_k, inter=8, dtype=dtype, slots=experts)
    counts = kernels_launched(lambda: run_prefill(wl, P=P, max_batch=max_batch, label="routing"), {"combine": 1})
    assert launches(counts, "route_pair_kernel") == launches_like_decode, counts
    assert launches(counts, "route_prompt_kernel") == (launches_like_decode == 0), counts


@pytest.mark.parametrize("dtype,P,max_batch,passes", [("f32", 37, 16, 3), ("f32", 16, 16, 1), ("bf16", 37, 16, 1)])
def test_prefill_counts_the_weight_bytes_its_kernels_read(dtype, P, max_batch, passes):
    """float32 experts are launched, and read, once for each micro-batch; bf16 experts and the router once per prompt."""
    from paper_2603_19289_amd.engine import engine_for
    wl = small_workload(n_layers=1, hidden=72, n_experts=6, top_k=2, inter=40, dtype=dtype, slots=4)
    eng = engine_for(wl, M.MODE_ON_DEMAND, *build(wl, "random")[:2], max_batch=max_batch, max_prefill_tokens=P)
    try:
        eng.prefill_layer_step(0, torch.from_numpy(prompt_of(wl, P)[0]).cuda())
        size = 4 if dtype == "f32" else 2
        assert eng.stats()["hbm_bytes_algorithmic"] == 6 * 72 * size + passes * 6 * 3 * 72 * 40 * size
    finally:
        eng.close()


@pytest.mark.parametrize("experts", [9, 70])
def test_prefill_non_finite_inputs_keep_expert_ids_in_range(experts):
    from paper_2603_19289_amd.engine import engine_for
    wl = small_workload(n_layers=1, hidden=128, n_experts=experts, top_k=4, inter=64, dtype="bf16", slots=8)
    res, ex, _ = build(wl, "random")
    eng = engine_for(wl, M.MODE_ON_DEMAND, res, ex, max_batch=16, max_prefill_tokens=20)
    try:
        r = torch.from_numpy(prompt_of(wl, 20)[0]).cuda()
        clean, clean_ids, _ = eng.prefill_layer_step(0, r, want_ids=True)
        bad = r.clone()
        bad[3, 5], bad[17, 0] = float("nan"), float("inf")
        out, ids, gates = eng.prefill_layer_step(0, bad, want_ids=True)
        torch.cuda.synchronize()
        assert ((ids >= 0) & (ids < experts)).all() and all(len(set(row)) == wl.top_k for row in ids.tolist())
        rest = [b for b in range(20) if b not in (3, 17)]
        assert torch.isnan(out[[3, 17]]).all() and torch.isnan(gates[[3, 17]]).all()
        assert torch.equal(ids[rest], clean_ids[rest]) and torch.equal(out[rest], clean[rest])
    finally:
        eng.close()


@pytest.mark.parametrize("slots,engine,pairs", [(6, M.COPY_DMA2, 4), (4, M.COPY_DMA, 3)])
def test_prefill_tail_in_pieces_equals_whole_groups(slots, engine, pairs):
    """Kernels of 0.3 ms per expert: the last group runs expert by expert and the last expert in halves of its rows, which
    end inside a tile.  Bit for bit what the copy kernel's whole groups give: a tile's sums do not depend on its launch."""
    from paper_2603_19289_amd.engine import engine_for
    P = 7400
    wl = small_workload(n_layers=1, hidden=2056, n_experts=3, top_k=1, inter=6008, dtype="bf16", slots=slots)
    g = torch.Generator(device="cuda").manual_seed(5)
    pool = torch.empty((1, 3, 3 * wl.hidden * wl.inter), dtype=torch.bfloat16, pin_memory=True)
    pool.copy_(0.02 * torch.randn(pool.shape, generator=g, device="cuda"))
    r = torch.randn((P, wl.hidden), generator=g, device="cuda")
    got = []
    for e in (engine, M.COPY_KERNEL):
        eng = engine_for(wl, M.MODE_ON_DEMAND, W.make_resident(wl), pool, max_batch=64, max_prefill_tokens=P, copy_engine=e)
        try:
            counts = kernels_launched(lambda: got.append(eng.prefill_layer_step(0, r)[0]), {"expert_lists": 1, "combine": 1})
            assert torch.isfinite(got[-1]).all() and got[-1].square().mean() > 0.01
        finally:
            eng.close()
        whole = (3 + slots // 2 - 1) // (slots // 2)
        expected = pairs if e == engine else whole
        assert [launches(counts, f"expert_tile_kernel<{b}>") for b in ("true", "false")] == [expected] * 2, counts
    assert torch.equal(got[0], got[-1])


def tail_inputs(hidden, inter, experts, top_k, P):
    """A layer of `experts` random experts and a prompt, everything from one seed: (workload, pool, residuals)."""
    wl = small_workload(n_layers=1, hidden=hidden, n_experts=experts, top_k=top_k, inter=inter, dtype="bf16", slots=2 * experts)
    g = torch.Generator(device="cuda").manual_seed(9)
    pool = torch.empty((1, experts, 3 * hidden * inter), dtype=torch.bfloat16, pin_memory=True)
    pool.copy_(0.02 * torch.randn(pool.shape, generator=g, device="cuda"))
    return wl, pool, torch.randn((P, hidden), generator=g, device="cuda")


@pytest.mark.parametrize("hidden,inter,experts,top_k,P", [(2056, 6008, 3, 1, 7400), (520, 1032, 8, 2, 16000)])
def test_prefill_profile_separates_the_tail_s_kernels_from_their_waits(hidden, inter, experts, top_k, P):
    """The last group's experts one by one, with and without the last one in pieces: every wait for a transfer is a stall (the
    only group here, so there is no other) and apart from the kernels: the spans of a stream cannot add up to more than the
    call, but for the resolution of the events."""
    from paper_2603_19289_amd.engine import engine_for
    wl, pool, r = tail_inputs(hidden, inter, experts, top_k, P)
    eng = engine_for(wl, M.MODE_ON_DEMAND, W.make_resident(wl), pool, max_batch=64, max_prefill_tokens=P, copy_engine=M.COPY_DMA2,
                     profile=1)
    try:
        eng.prefill_layer_step(0, r)
        eng.reset()
        start, done = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record(eng.compute)
        eng.prefill_layer_step(0, r)
        done.record(eng.compute)
        st = eng.stats()
        took = start.elapsed_time(done)
        print(f"[case] profile of the tail: {took:.2f} ms, copies {st['copy_ms']:.2f}, kernels {st['compute_ms']:.2f}, "
              f"stalls {st['stall_ms']:.2f}", flush=True)
        assert st["stall_ms"] > 0 and st["compute_ms"] > 0 and st["compute_ms"] + st["stall_ms"] < 1.05 * took
    finally:
        eng.close()


@pytest.mark.parametrize("hidden,inter,experts,top_k,P,kernels", [
    (520, 1032, 8, 2, 16000, {"expert_tile_kernel<true>": 8, "expert_tile_kernel<false>": 8}),
    # one expert by itself has too few row tiles for the tiled kernel, the whole group has enough
    (2048, 512, 8, 2, 6000, {"expert_mfma_lists_kernel<true": 8, "expert_tile_kernel<false>": 8}),
    (2056, 6008, 3, 1, 7400, {"expert_tile_kernel<true>": 4, "expert_tile_kernel<false>": 4})])
def test_prefill_tail_expert_by_expert_equals_whole_groups(hidden, inter, experts, top_k, P, kernels):
    """The last group's experts one by one as they arrive, the last one whole or in pieces, against the copy kernel's whole
    group: outputs, and the running means of every expert's outputs, which the tail adds up one expert at a time."""
    from paper_2603_19289_amd.engine import engine_for
    wl, pool, r = tail_inputs(hidden, inter, experts, top_k, P)
    got = []
    for e, expected in ((M.COPY_DMA2, kernels), (M.COPY_KERNEL, {"expert_tile_kernel<true>": 1, "expert_tile_kernel<false>": 1})):
        eng = engine_for(wl, M.MODE_ON_DEMAND, W.make_resident(wl), pool, max_batch=64, max_prefill_tokens=P, copy_engine=e,
                         accumulate_defaults=1)
        try:
            out = torch.zeros_like(r)

            def prompt():                              # again where the profiler missed a launch: from empty sums
                eng.reset()
                eng.prefill_layer_step(0, r, out)
            counts = kernels_launched(prompt, {"expert_lists": 1, "combine": 1})
            assert all(launches(counts, name) == n for name, n in expected.items()), counts
            mean, n = eng.read_default_vectors(0)
            got.append((out.cpu().numpy(), mean.cpu().numpy(), n))
        finally:
            eng.close()
    (out, mean, n), (want, want_mean, want_n) = got
    assert n == want_n and sum(n) == P * top_k and min(n) > 0
    check_output(out, want, "bf16", "outputs", terms=top_k * inter)
    check_output(mean, want_mean, "bf16", "means")
