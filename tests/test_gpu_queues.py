"""The work queues of long bf16 prefills: many launches in flight, the library's own counter sets
handed out between streams and host threads, and capture into a graph, at a size that takes
them (shorter prefills, which the other tests of these rules use, read no counters)."""
import threading

import pytest
import torch

import paper_2411_17116_amd as sa
import workloads
from tests import parity_harness as ph

pytestmark = pytest.mark.gpu

CFG = workloads.StarConfig("queues", "bf16", 1, 32, 8, 128, 17003, 5000, 5000, 1, 0, seed=19)
BUSY = -11


@pytest.fixture(scope="module")
def first():
    """Inputs, and the first launch's results."""
    inp = workloads.make_inputs(CFG, "cuda")
    run = ph.HipRun(CFG, inp)
    assert sa.phase1_plan(run.shape).queued == 1
    run.phase1()
    torch.cuda.synchronize()
    return inp, run


def _same(run, ref):
    return (torch.equal(run.O_ctx, ref.O_ctx) and torch.equal(run.LSE_ctx, ref.LSE_ctx)
            and torch.equal(run.Kc, ref.Kc) and torch.equal(run.Vc, ref.Vc))


def _streams(n):
    streams = [torch.cuda.Stream() for _ in range(n)]
    for s in streams:
        s.wait_stream(torch.cuda.current_stream())
    return streams


def test_many_launches_in_flight_with_counters_of_their_own(first):
    inp, ref = first
    runs, wss = [ph.HipRun(CFG, inp) for _ in range(4)], [torch.full((256,), 255, dtype=torch.uint8, device="cuda")
                                                          for _ in range(80)]
    streams = _streams(4)
    for i, ws in enumerate(wss):
        r = runs[i % 4]
        sa.phase1(r.shape, inp.Q, inp.K, inp.V, r.O_ctx, r.Kc, r.Vc, LSE_ctx=r.LSE_ctx, workspace=ws, stream=streams[i % 4])
    torch.cuda.synchronize()
    assert all(_same(r, ref) for r in runs)


def test_the_library_s_own_counter_sets_from_several_threads(first):
    """Four host threads with a stream each: every launch gives the first one's bits or is refused
    as busy, and afterwards every set is free again."""
    inp, ref = first
    runs, streams = [ph.HipRun(CFG, inp) for _ in range(4)], _streams(4)
    ran, errors = [0] * 4, []

    def worker(k):
        try:
            for _ in range(40):
                try:
                    runs[k].phase1(own_workspace=False, stream=streams[k])
                    ran[k] += 1
                except sa.StarAttnError as e:
                    if e.code != BUSY:
                        raise
        except Exception as e:                             # noqa: BLE001 - reported below
            errors.append((k, repr(e)))

    threads = [threading.Thread(target=worker, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    print(f"launches that ran, of 40 per thread: {ran}", flush=True)
    assert not errors and sum(ran) >= 64
    assert all(_same(r, ref) for n, r in zip(ran, runs) if n)
    for r in runs:
        r.O_ctx.zero_()
        r.phase1(own_workspace=False)
    torch.cuda.synchronize()
    assert all(_same(r, ref) for r in runs)


@pytest.mark.parametrize("rope", [False, True])
def test_capture_with_a_workspace_and_refusal_without(first, rope):
    """Replayed with eager work in between; with unrotated projections the kernel that rotates
    them clears the counters of the launch behind it."""
    inp, ref = first
    run = ph.HipRun(CFG, inp)
    Q = inp.Q.clone()

    def call(workspace):
        if rope:
            sa.phase1_rope(run.shape, 500000.0, Q, inp.K, inp.V, run.O_ctx, run.Kc, run.Vc, LSE_ctx=run.LSE_ctx,
                           workspace=workspace)
        else:
            sa.phase1(run.shape, Q, inp.K, inp.V, run.O_ctx, run.Kc, run.Vc, LSE_ctx=run.LSE_ctx, workspace=workspace)

    call(run.ws1)
    torch.cuda.synchronize()
    want = [x.clone() for x in (run.O_ctx, run.LSE_ctx, run.Kc, run.Vc)]
    if not rope:
        assert _same(run, ref)
    side, graph, refused = torch.cuda.Stream(), torch.cuda.CUDAGraph(), None
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        Q.copy_(inp.Q)
        call(run.ws1)
    side.synchronize()
    with torch.cuda.graph(graph, stream=side):
        try:
            call(None)
        except sa.StarAttnError as e:
            refused = e.code
        call(run.ws1)
    assert refused == BUSY
    for rep in range(3):
        print(f"replay {rep}", flush=True)
        run.O_ctx.fill_(7.0)
        run.LSE_ctx.fill_(7.0)
        run.Kc.zero_()                                   # (rows past the context stay zero)
        run.Vc.zero_()
        run.ws1.fill_(255)
        Q.copy_(inp.Q)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(x, w) for x, w in zip((run.O_ctx, run.LSE_ctx, run.Kc, run.Vc), want)), rep
