"""GPU parity: the HIP path (called through the C ABI) against the fp64 oracle
on the same seeded inputs.  Tolerances: max-abs 1e-5 (fp32) / 2e-2 (bf16) on
outputs, 1e-5 / 1e-2 on log-sum-exps; caches bit-exact."""
import numpy as np
import pytest
import torch

import paper_2411_17116_amd as sa
import workloads
from tests import parity_harness as ph

pytestmark = pytest.mark.gpu


def _report(rep):
    print(f"\n[{rep.name}] {rep.detail}", flush=True)
    assert rep.ok, rep.detail


def test_config1_fp32_every_row():
    """Config 1 in full: every row, head and decode step.  Its log-sum-exps stay
    below the magnitude floor of the fp32 LSE bound, so the configuration the
    north star names is held to the plain 1e-5 on every statistic."""
    rep = ph.run_parity(workloads.CONFIGS["C1"], all_rows=True, verbose=True)
    _report(rep)
    assert rep.lse_range < ph.LSE_MAGNITUDE_FLOOR["fp32"], rep.lse_range
    assert rep.info["phase1_LSE_unscaled"] <= 1e-5, rep.info


@pytest.mark.parametrize("L,b,a,lq,nd", [
    (1000, 256, 256, 5, 3),      # ragged last block
    (777, 200, 37, 70, 2),       # nothing tile-aligned, anchor < block, two row tiles
    (300, 512, 512, 3, 1),       # single block: full causal attention
    (640, 128, 0, 9, 2),         # no anchor
])
def test_fp32_odd_shapes(L, b, a, lq, nd):
    cfg = workloads.StarConfig("f32odd", "fp32", 2, 4, 2, 64, L, b, a, lq, nd, seed=L + b)
    _report(ph.run_parity(cfg, all_rows=True))


def test_fp32_head_dim_128():
    cfg = workloads.StarConfig("f32d128", "fp32", 1, 2, 1, 128, 500, 128, 64, 33, 2, seed=9)
    _report(ph.run_parity(cfg, all_rows=True))


def test_fp32_hundreds_of_one_token_blocks():
    """Block size 1 without an anchor: 513 context parts of one token each, so
    the merge of a query row is 514 sequential additions per accumulator -- the
    case that needs the compensated part fold to stay within the fp32
    tolerance (an uncompensated fp32 fold of these pairs is off by ~1e-5)."""
    cfg = workloads.StarConfig("f32b1", "fp32", 1, 4, 1, 128, 513, 1, 0, 70, 3, seed=5200023,
                               n_planted=2)
    _report(ph.run_parity(cfg, all_rows=True))


@pytest.mark.parametrize("Hq,Hkv,L,b,a,lq,nd", [
    (4, 1, 2048, 512, 512, 40, 3),     # G = 4: four heads per workgroup
    (8, 1, 1500, 400, 100, 130, 2),    # G = 8, ragged everything, anchor < block
    (2, 2, 1024, 256, 256, 64, 2),     # G = 1: one head per workgroup
    (6, 2, 700, 256, 129, 20, 2),      # G = 3: odd group, one head per workgroup
    (6, 3, 900, 300, 0, 17, 2),        # G = 2, no anchor
    (4, 1, 700, 1024, 1024, 5, 4),     # single block (block > context)
])
def test_bf16_small_every_row(Hq, Hkv, L, b, a, lq, nd):
    """Small bf16 shapes compared on every row: several row tiles, several key
    tiles, ragged tails, every GQA packing."""
    cfg = workloads.StarConfig("bf16small", "bf16", 2, Hq, Hkv, 128, L, b, a, lq, nd,
                               seed=Hq * 1000 + L, n_planted=4)
    _report(ph.run_parity(cfg, all_rows=True))


def test_bf16_extreme_scores_take_the_exact_softmax_path():
    """Planted rows with gamma = 6 put one logit ~65 nats above everything a row
    saw in its first keys: the fast key loop's fixed reference maximum is no
    longer safe and the workgroup must redo its rows with the exact online
    softmax.  Rows without such a key share workgroups with rows that have one."""
    cfg = workloads.StarConfig("bf16peaky", "bf16", 1, 8, 2, 128, 3072, 1024, 512, 96, 3,
                               seed=77, n_planted=16, gamma=6.0)
    _report(ph.run_parity(cfg, all_rows=True))


def test_config2_bf16_sampled():
    rep = ph.run_parity(workloads.CONFIGS["C2"], verbose=True)
    _report(rep)
    # K + V = 134 MB stay in the last-level cache: flat plan, ordinary loads (label 1)
    assert set(rep.flat_plans.values()) == {(1, 1, 0, 1)}, rep.flat_plans
    assert "decode_flat_O" in rep.checks


def _assert_streaming_decode_was_checked(rep):
    """The decode steps compared as `decode_flat_O` ran the set-up a serving loop
    (and the benchmark) runs at this size: the flat comb plan on the non-temporal
    kernel (label 2)."""
    assert rep.flat_plans and set(rep.flat_plans.values()) == {(1, 1, 1, 2)}, rep.flat_plans
    assert rep.checks["decode_flat_O"] <= 2e-2


def test_config3_bf16_sampled():
    rep = ph.run_parity(workloads.CONFIGS["C3"], verbose=True)
    _report(rep)
    _assert_streaming_decode_was_checked(rep)


def test_config5_bf16_sampled():
    rep = ph.run_parity(workloads.CONFIGS["C5"], n_random=128, decode_samples=3, verbose=True)
    _report(rep)
    _assert_streaming_decode_was_checked(rep)


def test_config4_bf16_sampled():
    rep = ph.run_parity(workloads.CONFIGS["C4"], n_random=96, decode_samples=2, verbose=True)
    _report(rep)
    _assert_streaming_decode_was_checked(rep)


def test_run_to_run_determinism():
    """Same inputs, same bits (no floating-point atomics anywhere)."""
    cfg = workloads.StarConfig("det", "bf16", 1, 8, 2, 128, 4096, 1024, 1024, 48, 2, seed=3)
    inp = workloads.make_inputs(cfg, "cuda")
    outs = []
    for _ in range(2):
        run = ph.HipRun(cfg, inp)
        run.phase1()
        O, Op, Lp = run.phase2(inp.Qq, inp.Kq, inp.Vq)
        O1, _, _ = run.phase2(inp.Qd[:, :1].contiguous(), inp.Kd[:, :1].contiguous(),
                              inp.Vd[:, :1].contiguous(), want_parts=False)
        torch.cuda.synchronize()
        outs.append((run.O_ctx.clone(), run.LSE_ctx.clone(), O, Op, Lp, O1))
    for x, y in zip(*outs):
        assert torch.equal(x, y)


def test_phase1_work_queues_in_caller_workspaces_many_launches_in_flight():
    """The bf16 phase-1 kernel draws its row tiles from eight counters in the
    call's workspace.  200 launches with workspaces of their own, spread over four
    streams and never synchronised in between -- far more in flight than the
    library has counter sets of its own -- must all give the first launch's bits."""
    cfg = workloads.StarConfig("queues", "bf16", 1, 8, 2, 128, 3000, 512, 200, 1, 0, seed=17)
    inp = workloads.make_inputs(cfg, "cuda")
    ref = ph.HipRun(cfg, inp)
    ref.phase1()
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(4)]
    runs = [ph.HipRun(cfg, inp) for _ in range(8)]          # two output sets per stream
    wss = [torch.empty(256, dtype=torch.uint8, device="cuda") for _ in range(200)]
    for s in streams:
        s.wait_stream(torch.cuda.current_stream())
    for i in range(200):
        r = runs[i % 8]
        sa.phase1(r.shape, inp.Q, inp.K, inp.V, r.O_ctx, r.Kc, r.Vc, LSE_ctx=r.LSE_ctx,
                  workspace=wss[i], stream=streams[i % 4])
    torch.cuda.synchronize()
    for r in runs:
        assert torch.equal(r.O_ctx, ref.O_ctx) and torch.equal(r.LSE_ctx, ref.LSE_ctx)
        assert torch.equal(r.Kc, ref.Kc) and torch.equal(r.Vc, ref.Vc)


def test_phase1_without_workspace_never_shares_a_counter_set():
    """Without a workspace a launch takes one of the library's 64 static counter
    sets; a set is handed out again only once its launch has finished.  200
    unsynchronised launches over four streams either run (first launch's bits) or
    are refused with STAR_ATTN_ERR_BUSY before anything is enqueued -- never a
    silently mis-scheduled launch.  After a synchronise every set is free again."""
    cfg = workloads.StarConfig("queues0", "bf16", 1, 8, 2, 128, 3000, 512, 200, 1, 0, seed=17)
    inp = workloads.make_inputs(cfg, "cuda")
    ref = ph.HipRun(cfg, inp)
    ref.phase1()
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(4)]
    runs = [ph.HipRun(cfg, inp) for _ in range(8)]
    for s in streams:
        s.wait_stream(torch.cuda.current_stream())
    ran, busy = 0, 0
    for i in range(200):
        r = runs[i % 8]
        try:
            r.phase1(own_workspace=False, stream=streams[i % 4])
            ran += 1
        except sa.StarAttnError as e:
            assert e.code == -11, e                       # STAR_ATTN_ERR_BUSY
            busy += 1
    torch.cuda.synchronize()
    print(f"\n[static counter sets] {ran} launches ran, {busy} refused as busy", flush=True)
    assert ran >= 64
    for r in runs:
        assert torch.equal(r.O_ctx, ref.O_ctx) and torch.equal(r.LSE_ctx, ref.LSE_ctx)
        assert torch.equal(r.Kc, ref.Kc) and torch.equal(r.Vc, ref.Vc)
    for r in runs:                                        # all sets are free again
        r.O_ctx.zero_()
        r.phase1(own_workspace=False)
    torch.cuda.synchronize()
    assert all(torch.equal(r.O_ctx, ref.O_ctx) for r in runs)


def test_phase1_static_counter_sets_taken_from_several_host_threads():
    """Four host threads, each launching on a stream of its own without a
    workspace (ctypes drops the interpreter lock during the call, so the calls
    really overlap): a counter set that one thread has taken but not yet launched
    on must not be handed to another.  Every launch that ran gives the first
    launch's bits; the rest are refused as busy."""
    import threading
    cfg = workloads.StarConfig("queues_mt", "bf16", 1, 8, 2, 128, 3000, 512, 200, 1, 0, seed=17)
    inp = workloads.make_inputs(cfg, "cuda")
    ref = ph.HipRun(cfg, inp)
    ref.phase1()
    torch.cuda.synchronize()
    n_threads = 4
    streams = [torch.cuda.Stream() for _ in range(n_threads)]
    runs = [[ph.HipRun(cfg, inp) for _ in range(2)] for _ in range(n_threads)]
    for s in streams:
        s.wait_stream(torch.cuda.current_stream())
    counts = [[0, 0] for _ in range(n_threads)]
    errors = []

    def worker(k):
        try:
            for i in range(40):
                try:
                    runs[k][i % 2].phase1(own_workspace=False, stream=streams[k])
                    counts[k][0] += 1
                except sa.StarAttnError as e:
                    if e.code != -11:                      # STAR_ATTN_ERR_BUSY
                        raise
                    counts[k][1] += 1
        except Exception as e:                             # noqa: BLE001 - reported below
            errors.append((k, repr(e)))

    threads = [threading.Thread(target=worker, args=(k,)) for k in range(n_threads)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    print(f"\n[static counter sets, {n_threads} threads] (ran, busy) per thread: {counts}", flush=True)
    assert not errors, errors
    assert sum(c[0] for c in counts) >= 64
    for k in range(n_threads):
        for r in runs[k]:
            assert torch.equal(r.O_ctx, ref.O_ctx) and torch.equal(r.LSE_ctx, ref.LSE_ctx)
            assert torch.equal(r.Kc, ref.Kc) and torch.equal(r.Vc, ref.Vc)


@pytest.mark.parametrize("Hq,Hkv,lq", [(4, 1, 4), (4, 2, 5), (8, 1, 2), (6, 2, 3), (1, 1, 16)])
def test_decode_sized_calls_with_several_new_tokens(Hq, Hkv, lq):
    """G * q_len <= 16 rows per KV head take the streaming split-KV kernel even
    when the call brings more than one token (speculative / chunked decoding):
    the new tokens attend causally among themselves.  With and without per-part
    outputs (block-aligned and flat split plans)."""
    cfg = workloads.StarConfig("multitok", "bf16", 2, Hq, Hkv, 128, 3000, 1024, 300, lq, 3,
                               seed=Hq * 10 + lq, n_planted=4)
    rep = ph.run_parity(cfg, all_rows=True)          # query call and decode steps, per-part outputs
    _report(rep)
    # the same query call without per-part outputs (flat plan) must give the same O
    inp = workloads.make_inputs(cfg, "cuda")
    r1, r2 = ph.HipRun(cfg, inp, "cuda"), ph.HipRun(cfg, inp, "cuda")
    r1.phase1()
    r2.phase1()
    O1, _, _ = r1.phase2(inp.Qq, inp.Kq, inp.Vq, want_parts=True)
    O2, _, _ = r2.phase2(inp.Qq, inp.Kq, inp.Vq, want_parts=False)
    torch.cuda.synchronize()
    assert (O1.float() - O2.float()).abs().max().item() <= 2e-2
    assert torch.equal(r1.Kc, r2.Kc) and torch.equal(r1.Vc, r2.Vc)
