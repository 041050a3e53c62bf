"""The bf16 row-tiled phase-2 kernel at the edges of its tiling: rows packed over tokens and
heads (groups that do and do not divide a tile), tiles of 128 rows whose workgroup halves
share the keys (odd and even numbers of key tiles, a half without any) and tiles of 256,
splits of equal runs and of parts, new tokens read from the call's tensors and appended by
the kernel, and the exact fallback of the softmax in both halves."""
import math

import pytest
import torch

import paper_2411_17116_amd as sa
import workloads
from tests import parity_harness as ph

pytestmark = pytest.mark.gpu


# tiles: rows of the tile with per-part outputs and without; a split of no more than 64 keys (every
# tail here up to 64 tokens long) leaves the second half of a 128-row tile without any
@pytest.mark.parametrize("B,Hq,Hkv,L,b,a,lq,gamma,tiles", [
    (1, 1, 1, 40, 64, 64, 17, 1.5, (256, 256)),        # one ragged tile, 57 keys in all
    (1, 1, 1, 64, 64, 64, 65, 1.5, (256, 256)),        # cached and new rows in key tiles of their own
    (2, 3, 1, 700, 300, 100, 21, 1.5, (128, 128)),     # G = 3: 63 rows, tokens straddle row blocks
    (1, 5, 1, 1000, 256, 0, 51, 1.5, (128, 128)),      # 255 rows: a whole tile and a ragged one
    (1, 4, 2, 1300, 400, 64, 32, 1.5, (128, 128)),     # 64 rows: half a tile
    (1, 4, 2, 1300, 400, 64, 33, 1.5, (128, 128)),     # 66 rows: into the next row block
    (1, 8, 2, 1300, 1300, 64, 65, 1.5, (128, 128)),    # 260 rows: three tiles
    (1, 8, 2, 900, 100, 100, 97, 1.5, (128, 128)),     # 388 rows: four tiles
    (1, 40, 2, 600, 200, 7, 3, 1.5, (128, 128)),       # G = 20
    (1, 8, 2, 6000, 1500, 64, 21, 6.0, (128, 128)),    # scores far above the reference: the exact loop
    (1, 4, 2, 3000, 800, 64, 60, 6.0, (128, 128)),     # the same, another number of tiles per half
    (2, 32, 8, 2000, 1000, 100, 150, 1.5, (256, 128)),     # 600 rows: three tiles, the last ragged
    (1, 32, 8, 9000, 9000, 64, 300, 6.0, (256, 256)),      # 1200 rows: five tiles, the exact loop
    (1, 32, 8, 12000, 12000, 0, 400, 1.5, (128, 256)),     # seven tiles of 256 rows
])
def test_row_tile_edges(B, Hq, Hkv, L, b, a, lq, gamma, tiles):
    cfg = workloads.StarConfig("rows", "bf16", B, Hq, Hkv, 128, L, b, a, lq, 1, seed=L + lq, n_planted=8,
                               gamma=gamma)
    print(f"[{cfg}]", flush=True)
    assert tuple(sa.phase2_plan(ph.shape_of(cfg), L, lq, parts).tile_rows for parts in (True, False)) == tiles
    rep = ph.run_parity(cfg, all_rows=L < 1500)      # the query call with per-part outputs
    assert rep.ok, rep.detail
    # the same call as a serving program makes it, without per-part outputs
    inp = workloads.make_inputs(cfg, "cuda")
    run = ph.HipRun(cfg, inp, "cuda")
    run.phase1()
    O, _, _ = run.phase2(inp.Qq, inp.Kq, inp.Vq, want_parts=False)
    torch.cuda.synchronize()
    heads = list(range(Hq)) if Hq <= 8 else [0, 1, Hq // 2 - 1, Hq // 2, Hq - 1]
    res = ph.check_phase2(run, inp.Qq, ([inp.Kq], [inp.Vq]), L, O, None, None, heads, tag="flat")
    assert res["flat_O"] <= ph.TOL["bf16"]["o"], res
    for g in range(Hkv):
        assert torch.equal(run.Kc[:, g, L:L + lq], inp.Kq[:, :, g])
        assert torch.equal(run.Vc[:, g, L:L + lq], inp.Vq[:, :, g])
        assert not run.Kc[:, g, L + lq:].any()


@pytest.mark.parametrize("B,Hq,Hkv,L,b,lq", [
    (1, 8, 2, 1024, 256, 64),       # a split per block and one behind
    (1, 8, 2, 750, 256, 47),        # the last block short
    (1, 8, 2, 4096, 1024, 84),      # four splits per block
    (2, 16, 16, 1024, 512, 40),
    (1, 12, 4, 1024, 1024, 30),
])
def test_splits_along_blocks_without_per_part_outputs(B, Hq, Hkv, L, b, lq):
    """Splits that follow the blocks are merged at once where no per-part outputs are asked for; the result is that
    of the call which writes them."""
    gen = torch.Generator(device="cuda").manual_seed(L + lq)
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda", dtype=torch.bfloat16)
    cap = L + lq
    shape = sa.StarShape.make("bf16", B, Hq, Hkv, 128, L, b, 0, cap)
    assert sa.phase2_plan(shape, L, lq).flat == 0
    Kc, Vc, Q, K, V = rnd(B, Hkv, cap, 128), rnd(B, Hkv, cap, 128), rnd(B, lq, Hq, 128), rnd(B, lq, Hkv, 128), rnd(B, lq, Hkv, 128)
    ws, got, want = sa.alloc_workspace(shape, lq), torch.empty_like(Q), torch.empty_like(Q)
    parts = -(-L // b) + 1
    O_part, LSE_part = torch.empty((B, parts, Hq, lq, 128), device="cuda"), torch.empty((B, parts, Hq, lq), device="cuda")
    sa.phase2(shape, L, Q, K, V, Kc, Vc, got, ws)
    sa.phase2(shape, L, Q, K, V, Kc, Vc, want, ws, O_part=O_part, LSE_part=LSE_part)
    torch.cuda.synchronize()
    # fp32 folds in another order before one rounding to bf16: no more than neighbouring values
    torch.testing.assert_close(got.float(), want.float(), rtol=2.0 ** -7, atol=1e-4)


def test_workspace_covers_every_shorter_call():
    """Whatever a call of at most max_q tokens on a cache of any length plans fits what
    star_attn_workspace_bytes asked for."""
    for Hq, Hkv, B in ((4, 1, 1), (3, 1, 2), (20, 1, 1), (64, 8, 2), (12, 4, 1)):
        shape = sa.StarShape.make("bf16", B, Hq, Hkv, 128, 30000, 7000, 100, 30000 + 5000)
        for max_q in (7, 75, 300):
            have = sa.workspace_bytes(shape, max_q)
            for q in range(1, max_q + 1):
                for parts in (False, True):
                    for cached in (30000, 33333, 35000 - q):
                        assert sa.phase2_plan(shape, cached, q, parts).workspace_bytes <= have, (Hq, q, parts)


@pytest.mark.parametrize("dtype,Hq,Hkv,d,q,lengths", [
    ("bf16", 32, 8, 128, 32, (1000, 8000, 20000)),     # 2.6 MB on 1000 keys, 16.9 MB on 8000
    ("bf16", 20, 1, 128, 1, (64, 700, 20000)),         # G = 20
    ("fp32", 8, 2, 128, 1, (200, 1500, 9000)),         # one split, then many
    ("fp32", 8, 2, 64, 33, (300, 4000, 9000)),
])
def test_workspace_of_the_first_call_serves_a_growing_cache(dtype, Hq, Hkv, d, q, lengths):
    """A program that sizes its workspace by the plan of its first call and lets the cache grow
    is not refused later; its results are those of any workspace."""
    cap = lengths[-1] + q
    shape = sa.StarShape.make(dtype, 1, Hq, Hkv, d, lengths[0], lengths[0], 0, cap)
    gen = torch.Generator(device="cuda").manual_seed(q)
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda").to(dt)
    Kc, Vc = rnd(1, Hkv, cap, d), rnd(1, Hkv, cap, d)
    Q, K, V = rnd(1, q, Hq, d), rnd(1, q, Hkv, d), rnd(1, q, Hkv, d)
    need = [sa.phase2_plan(shape, n, q).workspace_bytes for n in lengths]
    assert need[0] < need[-1], need
    first, full = torch.empty(need[0], dtype=torch.uint8, device="cuda"), sa.alloc_workspace(shape, q)
    guard = torch.full((need[0] + 4096,), 171, dtype=torch.uint8, device="cuda")
    for n in lengths:
        print(f"{dtype} {Hq}/{Hkv} q={q} cache={n}: {need[0]} bytes of {need}", flush=True)
        got, want = torch.empty_like(Q), torch.empty_like(Q)
        sa.phase2(shape, n, Q, K, V, Kc, Vc, got, guard[:need[0]])
        sa.phase2(shape, n, Q, K, V, Kc, Vc, want, full)
        torch.cuda.synchronize()
        tol = 2 * ph.TOL[dtype]["o"]          # other splits: each within the bound of the exact result
        assert (got.float() - want.float()).abs().max().item() <= tol
        assert (guard[need[0]:] == 171).all()
    with pytest.raises(sa.StarAttnError) as e:            # not even one split fits
        sa.phase2(shape, lengths[0], Q, K, V, Kc, Vc, got, first[:Hq * q * 4])
    assert e.value.code == -7


@pytest.mark.parametrize("Hq,Hkv,L,lq", [(8, 2, 16384, 21), (2, 1, 32768, 40), (4, 1, 16384, 80)])
def test_sums_over_many_parts_lose_nothing(Hq, Hkv, L, lq):
    """A host's pair whose splits follow the blocks: every split's output is a whole number of 24 bits and its weight
    one, so that only the merge rounds.  Sums held to more than 32 bits leave two roundings, of the sum and of
    the quotient: 2^-23.  Plain fp32 sums of 64 and 128 splits miss that."""
    b, d, cap, n = 256, 128, L + lq, L // 256
    shape = sa.StarShape.make("bf16", 1, Hq, Hkv, d, L, b, 0, cap)
    plan = sa.phase2_plan(shape, L, lq)
    assert plan.flat == 0 and plan.split_len == b
    gen = torch.Generator(device="cuda").manual_seed(L)
    whole = torch.randint(1 << 23, 1 << 24, (Hkv, n, d), generator=gen, device="cuda")
    Kc, Vc = (torch.zeros((1, Hkv, cap, d), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    rows = Vc[0, :, :L].view(Hkv, n, b, d)                     # three bytes of it, at keys of their own; the rest are zero
    for key, shift in ((0, 16), (64, 8), (128, 0)):
        rows[:, :, key] = (((whole >> shift) & 255) << shift).bfloat16()
    Q = torch.zeros((1, lq, Hq, d), dtype=torch.bfloat16, device="cuda")
    K = torch.zeros((1, lq, Hkv, d), dtype=torch.bfloat16, device="cuda")
    Q[..., 0], K[..., 0] = 1.0, -30000.0                       # equal logits in the context; the new tokens weigh nothing
    A, lse = torch.empty((1, Hq, lq, d), device="cuda"), torch.empty((1, Hq, lq), device="cuda")
    sa.phase2_partial(shape, L, Q, Kc, Vc, A, lse, sa.alloc_workspace(shape, lq), Kq=K, Vq=torch.zeros_like(K))
    torch.cuda.synchronize()
    want = (whole.double().sum(dim=1) / (n * b)).repeat_interleave(Hq // Hkv, dim=0)[:, None]
    assert ((A[0].double() - want) / want).abs().max().item() <= 2.0 ** -23
    assert (lse.double() - math.log(L)).abs().max().item() <= 2.0 ** -20       # ulp near 10
