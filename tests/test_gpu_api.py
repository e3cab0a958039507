"""GPU-side checks of the C ABI's state machine and error returns, of reset/repeatability, of the
two copy engines agreeing, and free-running parity with a margin audit."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import moe_oracle as O
from paper_2603_19289_amd import moe_spec as M
from paper_2603_19289_amd import workload as W
from tests.helpers import SHARED_ROWS, build, check_output, kernels_launched, launches, make_advance, small_workload

pytestmark = pytest.mark.gpu


def _engine(wl, mode, res, ex, **kw):
    from paper_2603_19289_amd.engine import engine_for
    return engine_for(wl, mode, res, ex, **kw)


def test_state_machine_errors():
    wl = small_workload(n_layers=3, tokens=1)
    res, ex, _ = build(wl)
    eng = _engine(wl, M.MODE_SPECULATIVE, res, ex)
    r = torch.randn(1, wl.hidden, device="cuda")
    out = torch.empty_like(r)
    lib = M.lib()
    step = lambda layer, batch=1: lib.moe_spec_layer_step(eng.ctx, layer, r.data_ptr(), batch, out.data_ptr(), None)
    assert step(0) == M.ESTATE                                   # before begin_token
    assert b"begin_token" in lib.moe_spec_last_error(eng.ctx)
    eng.begin_token()
    assert step(1) == M.ESTATE                                   # out of order
    assert step(0, batch=2) == M.EINVAL                          # beyond max_batch
    assert lib.moe_spec_layer_step(eng.ctx, 0, None, 1, out.data_ptr(), None) == M.EINVAL
    assert step(0) == M.OK
    assert step(0) == M.ESTATE                                   # layer 0 twice
    assert step(1) == M.OK and step(2) == M.OK
    assert step(3) == M.ESTATE                                   # past the last layer: token is closed
    torch.cuda.synchronize()
    # registration errors
    assert lib.moe_spec_set_layer_resident(eng.ctx, 9, 1, 1, 1) == M.EINVAL
    assert lib.moe_spec_load_host_experts(eng.ctx, 0, 0, wl.n_experts + 1, eng.pool.data_ptr(), 0) == M.EINVAL
    assert lib.moe_spec_load_host_experts(eng.ctx, 0, 0, 1, eng.pool.data_ptr(), 7) == M.EINVAL          # wrong size
    pageable = np.zeros(eng.expert_bytes, dtype=np.uint8)
    assert lib.moe_spec_load_host_experts(eng.ctx, 0, 0, 1, pageable.ctypes.data, eng.expert_bytes) == M.EINVAL
    assert b"pinned" in lib.moe_spec_last_error(eng.ctx)
    eng.close()


def test_stepping_a_layer_whose_tables_or_experts_are_missing():
    wl = small_workload(n_layers=2, tokens=1)
    cfg = M.Config(n_layers=2, hidden=wl.hidden, n_experts=wl.n_experts, top_k=wl.top_k, inter=wl.inter, max_batch=1,
                   slots_per_layer=wl.slots, dtype=M.BF16, mode=M.MODE_ON_DEMAND, rms_eps=1e-6, copy_engine=M.COPY_KERNEL)
    arena = torch.empty(M.moe_spec_arena_bytes(cfg), dtype=torch.uint8, device="cuda")
    cs, ks = torch.cuda.Stream(), torch.cuda.Stream()
    cfg.device_arena, cfg.device_arena_bytes = arena.data_ptr(), arena.numel()
    cfg.compute_stream, cfg.copy_stream = cs.cuda_stream, ks.cuda_stream
    ctx = M.moe_spec_create(cfg)
    r = torch.randn(1, wl.hidden, device="cuda"); out = torch.empty_like(r)
    torch.cuda.synchronize()
    lib = M.lib()
    M.moe_spec_begin_token(ctx)
    assert lib.moe_spec_layer_step(ctx, 0, r.data_ptr(), 1, out.data_ptr(), None) == M.ESTATE    # no tables
    res, ex, _ = build(wl)
    from paper_2603_19289_amd.engine import _np_to_torch_storage
    rw = _np_to_torch_storage(res["router_w"]).cuda(); dv = _np_to_torch_storage(res["dvecs"]).cuda()
    gn = torch.from_numpy(res["rms_gain"]).cuda()
    for l in range(2):
        M.moe_spec_set_layer_resident(ctx, l, rw[l].data_ptr(), gn[l].data_ptr(), dv[l].data_ptr())
    torch.cuda.synchronize()
    assert lib.moe_spec_layer_step(ctx, 0, r.data_ptr(), 1, out.data_ptr(), None) == M.ESTATE    # no experts registered
    assert b"never registered" in lib.moe_spec_last_error(ctx)
    M.moe_spec_destroy(ctx)


def _run_free(eng, wl, x0, eps):
    """GPU runs free: its own outputs feed the synthetic residual driver."""
    dev_x0, dev_eps = torch.from_numpy(x0).cuda(), torch.from_numpy(eps).cuda()
    ids_log, outs = [], []
    for t in range(x0.shape[0]):
        eng.begin_token()
        r = dev_x0[t].clone()
        for l in range(wl.n_layers):
            out, ids = eng.layer_step(l, r, want_ids=True)
            ids_log.append({k: v for k, v in ids.items()})
            outs.append(out)
            if l + 1 < wl.n_layers:
                with torch.cuda.stream(eng.compute):
                    r = eng.advance(r, out, dev_eps[t, l], wl.res_a, wl.res_b)
    torch.cuda.synchronize()
    return ids_log, outs


@pytest.mark.parametrize("mode", [M.MODE_ON_DEMAND, M.MODE_SPECULATIVE])
def test_free_running_c1_matches_the_checker_with_margin_audit(mode):
    # The GPU computes its own residual trajectory in float32.  Expert sets must still match the
    # checker's unless the deciding logit margin is at rounding level; any mismatch with a
    # comfortable margin is a bug.
    wl = W.CONFIGS["c1_tiny"]
    res, ex, model = build(wl, gains="ones")
    x0, eps = W.make_inputs(wl)
    orc = O.MoEOracle(model, mode, wl.slots)
    trace = O.run_tokens(orc, x0, make_advance(wl, eps))
    eng = _engine(wl, mode, res, ex)
    ids_log, outs = _run_free(eng, wl, x0, eps)
    mismatches = 0
    i = 0
    for t in range(wl.tokens):
        for l in range(wl.n_layers):
            want = trace[t][l][1]
            got = ids_log[i]["true_ids"].cpu().numpy()
            if not np.array_equal(np.sort(got), np.sort(want.true_ids)):
                mismatches += 1
                assert want.true_margin.min() < 1e-4, (t, l, got, want.true_ids, want.true_margin)
            i += 1
    st = eng.stats()
    eng.close()
    if mismatches == 0:
        assert st["hits"] == orc.stats.hits and st["cache_misses"] == orc.stats.cache_misses
        err = np.linalg.norm(outs[-1].cpu().numpy() - trace[-1][-1][1].out) / np.linalg.norm(trace[-1][-1][1].out)
        assert err < 1e-4
    print(f"[free-running] mode={mode} mismatching layer steps: {mismatches}", flush=True)


def test_reset_makes_runs_repeatable_and_copy_engines_agree():
    wl = small_workload(n_layers=4, hidden=264, n_experts=12, top_k=3, inter=200, tokens=6, slots=4, seed=21)
    res, ex, _ = build(wl)
    x0, eps = W.make_inputs(wl)
    results = []
    for engine_kind in (M.COPY_KERNEL, M.COPY_DMA, M.COPY_DMA2):
        eng = _engine(wl, M.MODE_SPECULATIVE, res, ex, copy_engine=engine_kind)
        for rep in range(2):
            eng.reset()
            ids_log, outs = _run_free(eng, wl, x0, eps)
            st = eng.stats()
            results.append((torch.stack(outs).cpu().numpy(), torch.stack([d["exec_ids"] for d in ids_log]).cpu().numpy(),
                            {k: st[k] for k in ("hits", "predictions", "cache_hits", "cache_misses", "h2d_bytes", "tokens")}))
        eng.close()
    for other in results[1:]:
        np.testing.assert_array_equal(other[0], results[0][0])          # bit-identical outputs
        np.testing.assert_array_equal(other[1], results[0][1])
        assert other[2] == results[0][2]


def test_smallest_pool_reuses_every_slot_without_corruption():
    # S = k: every token overwrites every slot of every layer; with repeated inputs the outputs must
    # repeat exactly, which fails if a copy ever lands in a slot that is still being read
    wl = small_workload(n_layers=3, hidden=264, n_experts=12, top_k=3, inter=200, tokens=8, slots=3, seed=33)
    res, ex, _ = build(wl)
    x0, eps = W.make_inputs(wl)
    x0[4:] = x0[:4]
    eps[4:] = eps[:4]
    eng = _engine(wl, M.MODE_SPECULATIVE, res, ex)
    _, outs = _run_free(eng, wl, x0, eps)
    eng.close()
    o = torch.stack(outs).cpu().numpy().reshape(8, wl.n_layers, -1)
    np.testing.assert_array_equal(o[:4], o[4:])


@pytest.mark.parametrize("signal", [0, 1])
@pytest.mark.parametrize("dtype,B", [("bf16", 1), ("f32", 3), ("bf16", 20)])
def test_per_layer_diagnostics_match_the_checker(signal, dtype, B):
    # recall, per-rank agreement and cosine similarity per layer, for the quasi-hidden state and for
    # the baseline signal s_l; teacher-forced so that both sides see the same inputs
    wl = small_workload(n_layers=5, hidden=264, n_experts=12, top_k=3, inter=200, dtype=dtype, batch=B,
                        tokens=4, slots=12, seed=41)
    res, ex, model = build(wl, gains="random")
    x0, eps = W.make_inputs(wl)
    orc = O.MoEOracle(model, O.MODE_SPECULATIVE, wl.slots, predict_signal=signal)
    trace = O.run_tokens(orc, x0, make_advance(wl, eps))
    eng = _engine(wl, M.MODE_SPECULATIVE, res, ex, predict_signal=signal, diagnostics=1)
    for t in range(wl.tokens):
        eng.begin_token()
        for l in range(wl.n_layers):
            r = torch.from_numpy(trace[t][l][0].astype(np.float32)).cuda()
            _, ids = eng.layer_step(l, r, want_ids=True)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(ids["exec_ids"].cpu().numpy(), trace[t][l][1].exec_ids)
    for l in range(wl.n_layers):
        got, want = eng.layer_diagnostics(l), orc.diag[l]
        assert got["predictions"] == want.predictions and got["hits"] == want.hits, l
        assert got["rank_match"][:wl.top_k] == want.rank_match, l
        assert got["cos_count"] == want.cos_count
        assert abs(got["cos_sum"] - want.cos_sum) <= 1e-6 * max(1, want.cos_count), (l, got["cos_sum"], want.cos_sum)
    st = eng.stats()
    assert st["hits"] == orc.stats.hits and st["predictions"] == orc.stats.predictions
    eng.close()


@pytest.mark.parametrize("dtype,B,mode", [("f32", 1, M.MODE_ON_DEMAND), ("bf16", 1, M.MODE_SPECULATIVE), ("f32", 3, M.MODE_ON_DEMAND),
                                           ("bf16", 3, M.MODE_SPECULATIVE), ("bf16", 20, M.MODE_ON_DEMAND)])
def test_accumulated_default_vectors_match_the_checker(dtype, B, mode):
    # the offline statistic behind d_{l,e}: mean un-gated output per executed expert, with counts
    wl = small_workload(n_layers=3, hidden=264, n_experts=12, top_k=3, inter=200, dtype=dtype, batch=B,
                        tokens=5, slots=5, seed=61)
    res, ex, model = build(wl, gains="random")
    x0, eps = W.make_inputs(wl)
    orc = O.MoEOracle(model, mode, wl.slots)
    trace = O.run_tokens(orc, x0, make_advance(wl, eps))
    eng = _engine(wl, mode, res, ex, accumulate_defaults=1)
    for t in range(wl.tokens):
        eng.begin_token()
        for l in range(wl.n_layers):
            out, _ = eng.layer_step(l, torch.from_numpy(trace[t][l][0].astype(np.float32)).cuda())
            torch.cuda.synchronize()
            check_output(out.cpu().numpy(), trace[t][l][1].out, dtype, f"token {t} layer {l}")
    for l in range(wl.n_layers):
        mean, counts = eng.read_default_vectors(l)
        assert counts == orc.dacc_cnt[l].tolist()
        got, want = mean.cpu().numpy().astype(np.float64), orc.default_vectors(l)
        for e in range(wl.n_experts):
            if counts[e]:
                check_output(got[e], want[e], dtype, f"default vector of layer {l}, expert {e}")
            else:
                assert not got[e].any()
    eng.close()
    # a context without the flag refuses
    eng = _engine(wl, mode, res, ex)
    buf = torch.empty((wl.n_experts, wl.hidden), device="cuda")
    assert M.lib().moe_spec_read_default_vectors(eng.ctx, 0, buf.data_ptr(), None) == M.ESTATE
    eng.close()


def test_time_kernel_modes_and_their_byte_counts():
    # the measurement aid: every mode runs, reports the weight bytes of its launch, and refuses what it cannot do
    wl = small_workload(n_layers=3, hidden=128, n_experts=12, top_k=3, inter=96, dtype="bf16", batch=20, slots=5)
    res, ex, _ = build(wl)
    eng = _engine(wl, M.MODE_SPECULATIVE, res, ex)
    w = 2
    want = {0: wl.top_k * 2 * wl.inter * wl.hidden * w, 1: wl.top_k * wl.inter * wl.hidden * w,
            2: wl.n_experts * wl.hidden * w, 3: wl.top_k * 2 * wl.inter * wl.hidden * w,
            4: 5 * 2 * wl.inter * wl.hidden * w, 5: 5 * wl.inter * wl.hidden * w,     # 5 = min(S, E, B*k) slots
            6: wl.n_experts * wl.hidden * w, 7: (2 * wl.n_experts + wl.batch * wl.top_k) * wl.hidden * w,
            9: wl.top_k * wl.inter * wl.hidden * w}
    for which, nbytes in want.items():
        ms, got = eng.time_kernel(which, 6)
        assert ms > 0 and got == nbytes, (which, ms, got, nbytes)
    with pytest.raises(M.MoeSpecError):
        eng.time_kernel(10, 1)
    eng.begin_token()
    with pytest.raises(M.MoeSpecError) as ei:
        eng.time_kernel(0, 1)                    # not inside a decode step
    assert ei.value.code == M.ESTATE
    eng.close()
    wl32 = small_workload(dtype="f32")
    res, ex, _ = build(wl32)
    eng = _engine(wl32, M.MODE_ON_DEMAND, res, ex)
    with pytest.raises(M.MoeSpecError) as ei:
        eng.time_kernel(4, 1)                    # matrix-core kernels are bf16 only
    assert ei.value.code == M.ESTATE
    eng.close()


@pytest.mark.parametrize("dtype,B", [("f32", 1), ("bf16", 1), ("bf16", 6)])
def test_non_finite_inputs_keep_expert_ids_in_range(dtype, B):
    # NaN or infinite activations give NaN logits; the ranking must still hand out k distinct ids inside
    # [0, E) (they index weight rows and host tables), outputs are NaN, and the context stays usable
    wl = small_workload(n_layers=3, hidden=128, n_experts=70, top_k=4, inter=64, dtype=dtype, batch=B, slots=8, tokens=2)
    res, ex, model = build(wl, "random")
    x0, eps = W.make_inputs(wl)
    for mode in (M.MODE_SPECULATIVE, M.MODE_ON_DEMAND):
        eng = _engine(wl, mode, res, ex)
        try:
            for bad in (float("nan"), float("inf")):
                eng.begin_token()
                r = torch.from_numpy(x0[0]).cuda()
                r[0, 5] = bad
                for l in range(wl.n_layers):
                    out, ids = eng.layer_step(l, r, want_ids=True)
                    torch.cuda.synchronize()
                    for key in ("true_ids", "exec_ids") + (("next_ids",) if l + 1 < wl.n_layers else ()):
                        got = ids[key].cpu().numpy()
                        assert ((got >= 0) & (got < wl.n_experts)).all(), (key, got)
                        assert all(len(set(row)) == wl.top_k for row in got.tolist()), (key, got)
                    assert torch.isnan(out[0]).all()
                    r = r + out
            # a clean token afterwards matches the checker again
            eng.reset()
            orc = O.MoEOracle(model, mode, wl.slots)
            trace = O.run_tokens(orc, x0[:1], make_advance(wl, eps))
            eng.begin_token()
            for l in range(wl.n_layers):
                r_np, want = trace[0][l]
                out, ids = eng.layer_step(l, torch.from_numpy(r_np.astype(np.float32)).cuda(), want_ids=True)
                torch.cuda.synchronize()
                np.testing.assert_array_equal(ids["exec_ids"].cpu().numpy(), want.exec_ids)
        finally:
            eng.close()


@pytest.mark.parametrize("batch", [1, 3])
def test_a_wait_of_the_estimator_that_runs_out_is_reported(batch):
    # as below for the launch that carries the estimator on (three waits in a row): with one poll allowed every kernel still
    # runs to its end and ids stay in range; whether a waiter gave up is up to timing, and if one did, a call says so
    wl = small_workload(n_layers=3, hidden=512, n_experts=24, top_k=4, inter=64, dtype="bf16", slots=24, tokens=3, batch=batch, seed=79)
    res, ex, _ = build(wl, "random")
    x0, eps = W.make_inputs(wl)
    eng = _engine(wl, M.MODE_SPECULATIVE, res, ex, wait_spin_limit=1, estimator=W.make_estimator(wl, m=2, n=2))
    try:
        try:
            for t in range(wl.tokens):
                eng.begin_token()
                for l in range(wl.n_layers):
                    _, ids = eng.layer_step(l, torch.from_numpy(x0[t] + 0.3 * eps[t, l]).cuda(), want_ids=True)
                    torch.cuda.synchronize()
                    got = ids["exec_ids"].cpu().numpy()
                    assert ((got >= 0) & (got < wl.n_experts)).all()
            eng.stats()
        except M.MoeSpecError as err:
            assert err.code == M.EHIP and "bounded wait" in str(err)
        eng.reset()
        assert eng.stats()["tokens"] == 0
    finally:
        eng.close()


def test_a_wait_that_runs_out_is_reported_and_reset_recovers():
    # The fused kernels wait, boundedly, for results of other workgroups of the same launch.  With the bound
    # forced down to one poll from the host, waiters give up early: every kernel still runs to its end, ids
    # stay inside [0, E), the next call (or moe_spec_stats) reports the failure, and moe_spec_reset brings
    # the context back.  With the default bound the same inputs match the checker.
    wl = small_workload(n_layers=3, hidden=512, n_experts=64, top_k=4, inter=256, dtype="bf16", slots=8, tokens=3, seed=77)
    res, ex, model = build(wl, "random")
    x0, eps = W.make_inputs(wl)
    orc = O.MoEOracle(model, O.MODE_SPECULATIVE, wl.slots)
    trace = O.run_tokens(orc, x0, make_advance(wl, eps))
    eng = _engine(wl, M.MODE_SPECULATIVE, res, ex, wait_spin_limit=1)
    gave_up = False
    try:
        for t in range(wl.tokens):
            try:
                eng.begin_token()
                for l in range(wl.n_layers):
                    _, ids = eng.layer_step(l, torch.from_numpy(trace[t][l][0].astype(np.float32)).cuda(), want_ids=True)
                    torch.cuda.synchronize()
                    got = ids["exec_ids"].cpu().numpy()
                    assert ((got >= 0) & (got < wl.n_experts)).all()
            except M.MoeSpecError as err:
                assert err.code == M.EHIP and "bounded wait" in str(err)
                gave_up = True
                break
        if not gave_up:
            try:
                eng.stats()
            except M.MoeSpecError as err:
                assert err.code == M.EHIP and "bounded wait" in str(err)
                gave_up = True
        print(f"[bounded wait] one poll allowed: waiters gave up = {gave_up}", flush=True)
        eng.reset()
        assert eng.stats()["tokens"] == 0                        # the context answers again
    finally:
        eng.close()
    eng = _engine(wl, M.MODE_SPECULATIVE, res, ex)
    try:
        for t in range(wl.tokens):
            eng.begin_token()
            for l in range(wl.n_layers):
                _, ids = eng.layer_step(l, torch.from_numpy(trace[t][l][0].astype(np.float32)).cuda(), want_ids=True)
                torch.cuda.synchronize()
                np.testing.assert_array_equal(ids["exec_ids"].cpu().numpy(), trace[t][l][1].exec_ids)
        assert eng.stats()["hits"] == orc.stats.hits
    finally:
        eng.close()


def test_random_call_sequences_leave_a_working_context():
    """Forty seeded contexts, each put through 10 to 60 random calls, valid and invalid (steps in and out of order,
    oversized batches, null pointers, resets and statistics in the middle of a token, timing and prefill calls at the
    wrong moment, both entry points of the layer step): invalid calls must be refused with EINVAL / ESTATE, and
    afterwards a clean token through the context must equal, bit for bit, the same token through a context that saw
    none of it."""
    rng = np.random.default_rng(61)
    modes = [M.MODE_ON_DEMAND, M.MODE_SPECULATIVE, M.MODE_PREFETCH_HINT]

    def clean_token(eng, wl, x, static):
        eng.reset()
        eng.begin_token()
        outs, r = [], x
        for l in range(wl.n_layers):
            out, _ = eng.layer_step(l, r, static_scratch=static)
            torch.cuda.synchronize()
            outs.append(out.clone())
            r = (r + out).contiguous()
        return outs

    for case in range(40):
        L, E = int(rng.integers(2, 6)), int(rng.integers(2, 24))
        k = int(rng.integers(1, min(E, 6) + 1))
        S, Bmax = int(rng.integers(k, E + 1)), int(rng.choice([1, 2, 5, 16]))
        mode = modes[int(rng.integers(0, 3))]
        wl = small_workload(name=f"calls{case}", n_layers=L, hidden=int(rng.choice([16, 64, 264])), n_experts=E, top_k=k,
                            inter=int(rng.choice([8, 40, 104])), dtype="bf16" if rng.random() < 0.6 else "f32",
                            batch=Bmax, tokens=1, slots=S, seed=6100 + case)
        look = 2 if (mode != M.MODE_ON_DEMAND and L >= 3 and rng.random() < 0.3) else 0
        kw = dict(copy_engine=int(rng.integers(0, 3)), lookahead=look, max_prefill_tokens=int(rng.choice([0, 0, 32])))
        res, ex, _ = build(wl, "random")
        eng, ref = _engine(wl, mode, res, ex, **kw), _engine(wl, mode, res, ex, **kw)
        g = torch.Generator(device="cuda").manual_seed(case)
        is_open, nxt, batch = False, 0, 0
        try:
            for _ in range(int(rng.integers(10, 60))):
                op = rng.choice(["begin", "step", "step", "step", "wrong_layer", "bad_batch", "reset", "stats", "time",
                                 "prefill", "null"])
                must_fail = must_pass = False
                try:
                    if op == "begin":
                        must_pass = True
                        eng.begin_token()
                        is_open, nxt = True, 0
                    elif op == "step":
                        B = int(rng.integers(1, Bmax + 1)) if nxt == 0 else batch
                        must_pass, must_fail = is_open, not is_open
                        r = torch.randn((B, wl.hidden), generator=g, device="cuda")
                        eng.layer_step(nxt if is_open else 0, r, static_scratch=bool(rng.random() < 0.5))
                        batch, nxt = B, nxt + 1
                        is_open = nxt < L
                    elif op == "wrong_layer":
                        must_fail = True
                        r = torch.randn((max(batch, 1), wl.hidden), generator=g, device="cuda")
                        eng.layer_step(nxt + 1, r)
                    elif op == "bad_batch":
                        must_fail = True
                        eng.layer_step(nxt, torch.randn((Bmax + 1, wl.hidden), generator=g, device="cuda"))
                    elif op == "reset":
                        must_pass = True
                        eng.reset()
                        is_open, nxt = False, 0
                    elif op == "stats":
                        must_pass = True
                        eng.stats()
                    elif op == "time":
                        must_fail = is_open
                        eng.time_kernel(int(rng.choice([0, 1, 2, 3, 9])), 3)
                    elif op == "prefill":
                        must_fail = kw["max_prefill_tokens"] == 0 or is_open
                        must_pass = not must_fail
                        r = torch.randn((int(rng.integers(1, 33)), wl.hidden), generator=g, device="cuda")
                        for l in range(L):
                            eng.prefill_layer_step(l, r)
                    else:
                        must_fail = True
                        M.moe_spec_layer_step(eng.ctx, nxt, 0, 1, 0)
                    assert not must_fail, (case, op)
                except M.MoeSpecError as e:
                    assert e.code in (M.EINVAL, M.ESTATE), (case, op, e)
                    assert not must_pass, (case, op, e)
            torch.cuda.synchronize()
            x = torch.randn((Bmax, wl.hidden), generator=torch.Generator(device="cuda").manual_seed(999), device="cuda")
            for static in (False, True):
                a, b = clean_token(eng, wl, x, static), clean_token(ref, wl, x, static)
                for l in range(L):
                    assert torch.equal(a[l].view(torch.int32), b[l].view(torch.int32)), (case, static, l)
        finally:
            eng.close()
            ref.close()


def beside_and_separate(wl, kernel, joint_layers, **engine_kw):
    """Decodes the same token again and again with profile = 0 and with profile = 1, where routing and experts are always
    separate launches: equal ids, gates, output bits and counters.  From the second token on all experts are in their
    slots; there the first engine is to make joint_layers[0] joint launches, joint_layers[1] of them of `kernel`, the
    other one none."""
    from paper_2603_19289_amd.engine import engine_for
    res, ex, _ = build(wl, "random")
    x0, eps = W.make_inputs(wl)
    got, joint = [], []
    for profile in (0, 1):
        eng = engine_for(wl, M.MODE_SPECULATIVE, res, ex, profile=profile, **engine_kw)

        def token():
            log = []
            eng.begin_token()
            for l in range(wl.n_layers):
                r = torch.from_numpy(x0[0] + 0.3 * eps[0, l]).cuda()
                out, ids = eng.layer_step(l, r, want_ids=True)
                torch.cuda.synchronize()
                log.append([out.cpu()] + [t.cpu() for _, t in sorted(ids.items())])
            return log
        try:
            log = token() + token()
            stats = {n: eng.stats()[n] for n in ("hits", "predictions", "cache_hits", "cache_misses", "hbm_bytes_algorithmic")}
            counts = kernels_launched(token, {"_kernel<false" if wl.dtype == "bf16" and wl.batch > 1 else "down_": wl.n_layers})
        finally:
            eng.close()
        got.append((log, stats))
        joint.append((launches(counts, "route_gateup"), launches(counts, kernel)))
    assert joint == [joint_layers, (0, 0)], (joint, counts)
    assert got[0][1] == got[1][1]
    for step, (a, b) in enumerate(zip(got[0][0], got[1][0])):
        for x, y in zip(a, b):
            assert torch.equal(x.view(torch.int32), y.view(torch.int32)), step


@pytest.mark.parametrize("dtype,hidden,inter,experts,top_k,batch,kernel", [
    ("bf16", 8, 8, 1, 1, 1, "route_gateup_b1"), ("f32", 264, 72, 6, 2, 1, "route_gateup_b1"),
    ("bf16", 520, 200, 9, 3, 1, "route_gateup_b1"), ("bf16", 2048, 1056, 9, 8, 1, "route_gateup_b1"),
    ("bf16", 2056, 40, 200, 16, 1, "route_gateup_b1"), ("f32", 2048, 24, 70, 5, 1, "route_gateup_b1"),
    ("bf16", 4096, 16, 256, 4, 1, "route_gateup_b1"), ("bf16", 4104, 16, 12, 3, 1, None),
    ("bf16", 8, 8, 1, 1, 2, "route_gateup_mfma"), ("bf16", 264, 72, 6, 2, 3, "route_gateup_mfma"),
    ("bf16", 1032, 200, 9, 3, 17, "route_gateup_mfma"), ("bf16", 2056, 40, 70, 5, 40, "route_gateup_mfma"),
    ("bf16", 4096, 16, 256, 16, 64, "route_gateup_mfma"), ("bf16", 4104, 16, 12, 3, 5, None), ("f32", 264, 72, 6, 2, 3, None)])
def test_gate_up_beside_the_routing_equals_separate_launches(dtype, hidden, inter, experts, top_k, batch, kernel):
    """Predicted experts that needed no copy share a launch with the routing, at every chunk count of the rows and every
    count of token tiles; kernel None: sizes beyond what the shared launches take."""
    wl = small_workload(name="beside", n_layers=3, hidden=hidden, n_experts=experts, top_k=top_k, inter=inter, dtype=dtype,
                        batch=batch, tokens=2, slots=experts, seed=41)
    print(f"[case] beside routing H={hidden} I={inter} E={experts} k={top_k} B={batch} {dtype}", flush=True)
    n = wl.n_layers - 1 if kernel else 0                     # layer 0 has no prediction to execute
    beside_and_separate(wl, kernel or "route_gateup", (n, n))


@pytest.mark.parametrize("hidden,inter,experts,top_k", SHARED_ROWS + [(1024, 344, 200, 16), (1016, 352, 256, 16)])
def test_rows_taken_by_the_routing_workgroups_equal_separate_launches(hidden, inter, experts, top_k):
    """Batch one with so many experts that their routing workgroups take gate/up rows afterwards: bit for bit the launches of
    their own (profile = 1), over two tokens of resident experts.  The last two sizes fall short of what that takes."""
    from paper_2603_19289_amd.engine import engine_for
    wl = small_workload(name="shared_rows", n_layers=3, hidden=hidden, n_experts=experts, top_k=top_k, inter=inter, dtype="bf16",
                        batch=1, tokens=1, slots=experts)
    g = torch.Generator(device="cuda").manual_seed(3)
    pool = torch.empty((experts, 3 * hidden * inter), dtype=torch.bfloat16, pin_memory=True)
    pool.copy_(0.02 * torch.randn(pool.shape, generator=g, device="cuda"))
    r = torch.randn((2, wl.n_layers, 1, hidden), generator=g, device="cuda")
    got = []
    for profile in (0, 1):
        eng = engine_for(wl, M.MODE_SPECULATIVE, W.make_resident(wl), [pool] * wl.n_layers, profile=profile)

        def tokens(log):
            for t in range(2):
                eng.begin_token()
                for l in range(wl.n_layers):
                    log.append(eng.layer_step(l, r[t, l])[0])
        try:
            tokens([])
            log = []
            counts = kernels_launched(lambda: (log.clear(), tokens(log)), {"down_": 2 * wl.n_layers})
            assert launches(counts, "route_gateup_b1") == (0 if profile else 2 * (wl.n_layers - 1)), counts
            got.append(log)
        finally:
            eng.close()
    assert all(torch.equal(a, b) for a, b in zip(*got)) and all(torch.isfinite(a).all() and a.abs().max() > 0 for a in got[0])


@pytest.mark.parametrize("mode", ["ON_DEMAND", "PREFETCH_HINT"])
@pytest.mark.parametrize("engine,dtype,like", [("KERNEL", "bf16", 0.0), ("DMA", "f32", 0.9), ("DMA2", "bf16", 0.9), ("DMA2", "f32", 0.0)])
def test_experts_queued_behind_the_routing_in_vain(mode, engine, dtype, like):
    """Batch one, true experts, as many slots as experts of a step, residuals that change every fourth token: after two steps that
    found their experts in their slots they are queued behind the routing, which wins at the fourth token of a run and is in
    vain at the first of the next one, where all experts (or, with like residuals, some) are absent.  Then they are copied and
    launched again: bit for bit the launches that waited for the ids (profile = 1)."""
    wl = small_workload(name="in_vain", n_layers=2, hidden=264, n_experts=40, top_k=4, inter=200, dtype=dtype, batch=1, tokens=12,
                        slots=4, seed=29)
    res, ex, _ = build(wl)
    g = torch.Generator(device="cuda").manual_seed(5)
    r = torch.randn((2, wl.n_layers, 1, wl.hidden), generator=g, device="cuda")
    r[1] = like * r[0] + (1.0 - like * like) ** 0.5 * r[1]
    runs = []
    for profile in (0, 1):
        log = []

        def tokens():
            log.clear()
            eng = _engine(wl, getattr(M, "MODE_" + mode), res, ex, profile=profile, copy_engine=getattr(M, "COPY_" + engine))
            try:
                for t in range(wl.tokens):
                    eng.begin_token()
                    for l in range(wl.n_layers):
                        out, ids = eng.layer_step(l, r[t // 4 % 2, l], want_ids=True)
                        log.append((out.clone(), ids["exec_ids"].clone(), ids["exec_gates"].clone()))
                torch.cuda.synchronize()
            finally:
                eng.close()
        counts = kernels_launched(tokens, {"route_": wl.tokens * wl.n_layers})
        down = {kind: sum(n for name, n in counts.items() if name.startswith("down_combine_b1_kernel") and name.endswith(kind + ">"))
                for kind in ("true", "false")}
        runs.append((log, down))
    (got, queued), (want, plain) = runs
    steps = wl.tokens * wl.n_layers
    assert plain == {"true": 0, "false": steps}
    if mode == "ON_DEMAND":                       # per layer: three won, two in vain
        assert queued == {"true": 5 * wl.n_layers, "false": 9 * wl.n_layers}, queued
    else:                                         # layer 0 so; layer 1's slots also change with the prefetches
        assert queued["true"] >= 5 and queued["true"] + queued["false"] >= steps + 2, queued
    for a, b in zip(got, want):
        assert all(torch.equal(x, y) for x, y in zip(a, b))
    before, after = (set(got[i][1].flatten().tolist()) for i in (3 * wl.n_layers, 4 * wl.n_layers))
    assert before != after and (like == 0.0 or before & after)


@pytest.mark.parametrize("hidden,experts,m,batch,kernel", [
    (520, 3, 1, 2, "<1, 4, true>"),          # one token tile, four wavefronts per 16 rows; more projection rows than router rows
    (72, 40, 9, 16, "<1, 1, true>"),         # latent size 8: most wavefronts have no row of it
    (264, 9, 3, 17, "<2, 1, true>"), (1032, 5, 3, 20, "<2, 2, true>"), (2056, 128, 1, 32, "<2, 4, true>"),
    (264, 200, 3, 48, "<3, 1, true>"), (1032, 8, 1, 33, "<3, 2, true>"), (2056, 2, 1, 40, "<3, 4, true>"),
    (72, 256, 9, 64, "<4, 1, true>"), (1096, 16, 1, 64, "<4, 2, true>"), (4096, 9, 4, 49, "<4, 4, true>")])
def test_estimator_projection_and_gate_up_beside_the_routing_equal_separate_launches(hidden, experts, m, batch, kernel):
    """The same with the estimator at every layer: its projection rides in the shared launch too (layers 1 and 2; the last
    layer predicts nothing)."""
    wl = small_workload(name="beside_est", n_layers=4, hidden=hidden, n_experts=experts, top_k=2, inter=40, dtype="bf16",
                        batch=batch, tokens=2, slots=experts, seed=47)
    print(f"[case] estimator beside routing H={hidden} E={experts} m={m} B={batch}", flush=True)
    beside_and_separate(wl, f"route_gateup_mfma_kernel{kernel}", (3, 2), estimator=W.make_estimator(wl, m=m, n=2))


@pytest.mark.parametrize("dtype,batch,slots", [("bf16", 1, 8), ("f32", 1, 3), ("bf16", 5, 3), ("bf16", 3, 8), ("f32", 3, 4)])
@pytest.mark.parametrize("mode", ["MODE_SPECULATIVE", "MODE_PREFETCH_HINT"])
def test_a_step_that_failed_for_an_unregistered_expert_can_be_called_again(dtype, batch, slots, mode, monkeypatch):
    """The prefetch for the next layer fails when its experts are not registered yet.  Registered afterwards, the same
    step is called again and executes what it would have executed, with every expert in its slots, with copies and with
    several cache waves."""
    from paper_2603_19289_amd.engine import engine_for
    wl = small_workload(name="again", n_layers=4, hidden=264, n_experts=8, top_k=2, inter=72, dtype=dtype, batch=batch,
                        tokens=1, slots=slots, seed=61)
    res, ex, _ = build(wl, "random")
    x0, eps = W.make_inputs(wl)
    r = [torch.from_numpy(x0[0] + 0.3 * eps[0, l]).cuda() for l in range(wl.n_layers)]
    register = M.moe_spec_load_host_experts
    held_back = []

    def later(ctx, layer, *rest):
        if layer == 0:
            register(ctx, layer, *rest)
        else:
            held_back.append((ctx, layer) + rest)

    def token(eng):
        log = []
        eng.begin_token()
        for l in range(wl.n_layers):
            if held_back:
                with pytest.raises(M.MoeSpecError) as ei:
                    eng.layer_step(l, r[l])
                assert ei.value.code == M.ESTATE and "never registered" in str(ei.value)
                register(*held_back.pop(0))
            out, ids = eng.layer_step(l, r[l], want_ids=True)
            torch.cuda.synchronize()
            log.append([out.cpu()] + [t.cpu() for _, t in sorted(ids.items())])
        return log

    plain = engine_for(wl, getattr(M, mode), res, ex)
    with monkeypatch.context() as m:
        m.setattr(M, "moe_spec_load_host_experts", later)
        eng = engine_for(wl, getattr(M, mode), res, ex)
    try:
        assert len(held_back) == wl.n_layers - 1
        for _ in range(2):
            for step, (a, b) in enumerate(zip(token(eng), token(plain))):
                for x, y in zip(a, b):
                    assert torch.equal(x.view(torch.int32), y.view(torch.int32)), step
    finally:
        eng.close()
        plain.close()


@pytest.mark.parametrize("mode,lookahead,batch,slots,dtype", [
    ("MODE_ON_DEMAND", 0, 1, 2, "f32"), ("MODE_ON_DEMAND", 0, 3, 4, "bf16"), ("MODE_SPECULATIVE", 0, 3, 2, "f32"),
    ("MODE_SPECULATIVE", 0, 8, 5, "bf16"), ("MODE_PREFETCH_HINT", 0, 1, 3, "bf16"), ("MODE_PREFETCH_HINT", 0, 8, 3, "bf16"),
    ("MODE_PREFETCH_HINT", 2, 3, 5, "bf16"), ("MODE_SPECULATIVE", 2, 5, 3, "bf16")])
def test_copies_in_order_with_the_kernels_and_beside_them_give_the_same_outputs(mode, lookahead, batch, slots, dtype):
    """Copies that the next kernels wait for run on the compute stream, unless earlier ones into that pool still travel on the
    copy stream, and prefetches follow them there: slots given away again while copies and their readers are under way.  The
    same steps with every copy on the copy stream (profile = 1) and with two DMA queues are bit for bit the same; experts of
    2 to 4 MB travel longer than the kernels of a layer take."""
    from paper_2603_19289_amd.engine import engine_for
    wl = small_workload(name="in_order", n_layers=4, hidden=264, n_experts=8, top_k=2, inter=2568, dtype=dtype, batch=batch, tokens=6,
                        slots=slots, seed=53)
    res, ex, _ = build(wl, "random")
    x0, eps = W.make_inputs(wl)
    r = [[torch.from_numpy(x0[t] + 0.3 * eps[t, l]).cuda() for l in range(wl.n_layers)] for t in range(wl.tokens)]
    got = []
    for kw in (dict(copy_engine=M.COPY_KERNEL), dict(copy_engine=M.COPY_KERNEL, profile=1), dict(copy_engine=M.COPY_DMA2)):
        eng = engine_for(wl, getattr(M, mode), res, ex, predict_in_on_demand=0, lookahead=lookahead, **kw)
        outs = [[torch.zeros_like(v) for v in row] for row in r]
        try:
            for t in range(wl.tokens):                 # no wait for the GPU in between
                eng.begin_token()
                for l in range(wl.n_layers):
                    eng.layer_step(l, r[t][l], outs[t][l])
            assert eng.stats()["cache_misses"] > wl.n_layers * wl.top_k * 2
            got.append(torch.stack([torch.stack(row) for row in outs]).cpu())
        finally:
            eng.close()
    assert torch.isfinite(got[0]).all() and (got[0].abs().amax(dim=(2, 3)) > 0).all()
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])
