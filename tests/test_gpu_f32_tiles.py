"""The fp32 kernels at the edges of their tiling: 16- and 32-row tiles packed over the
heads of a KV group (groups that do and do not divide a tile), 16-key units dealt to
the wavefronts of a workgroup (fewer units than wavefronts, ragged last units), calls
of one workgroup per row tile that write their results themselves and calls whose
splits are merged, with and without per-part outputs."""
import math

import pytest
import torch

import paper_2411_17116_amd as sa
import workloads
from tests import parity_harness as ph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv,d,L,b,a,lq,nd", [
    (1, 1, 1, 64, 15, 16, 16, 1, 2),        # one ragged unit, one row tile
    (1, 3, 1, 128, 129, 17, 9, 11, 2),      # G = 3: tokens straddle row tiles; 33 rows: two tiles
    (2, 5, 1, 64, 257, 64, 33, 13, 2),      # G = 5
    (1, 40, 2, 64, 100, 50, 25, 2, 1),      # G = 20: one token's heads in two tiles
    (1, 2, 2, 128, 239, 100, 16, 17, 2),    # query call: 256 KiB of K and V, one workgroup per row tile
    (1, 2, 2, 128, 240, 100, 16, 17, 2),    # beyond that: splits and a merge
    (1, 4, 2, 64, 2500, 700, 1, 33, 2),     # 16-row and 32-row tiles, several splits
    (2, 3, 1, 128, 333, 7, 0, 5, 1),        # one unit per block: a wavefront per tile
    (1, 4, 2, 64, 500, 16, 16, 3, 1),       # two units
    (1, 5, 5, 64, 300, 17, 0, 3, 1),        # the second of one key
    (1, 8, 2, 64, 280, 20, 5, 300, 1),      # per-part splits of up to four units: a wavefront per 32-row tile
    (1, 6, 3, 128, 250, 60, 60, 260, 1),
])
def test_fp32_tile_edges(B, Hq, Hkv, d, L, b, a, lq, nd):
    cfg = workloads.StarConfig("f32tiles", "fp32", B, Hq, Hkv, d, L, b, a, lq, nd, seed=L + Hq, n_planted=2)
    print(f"[{cfg}]", flush=True)
    rep = ph.run_parity(cfg, all_rows=True)
    assert rep.ok, rep.detail
    # the same query call without per-part outputs: other splits (or none), each within
    # the fp32 bound of the oracle, so within twice the bound of each other
    inp = workloads.make_inputs(cfg, "cuda")
    one, two = ph.HipRun(cfg, inp, "cuda"), ph.HipRun(cfg, inp, "cuda")
    one.phase1()
    two.phase1()
    want, _, _ = one.phase2(inp.Qq, inp.Kq, inp.Vq, want_parts=True)
    got, _, _ = two.phase2(inp.Qq, inp.Kq, inp.Vq, want_parts=False)
    torch.cuda.synchronize()
    assert (want - got).abs().max().item() <= 2 * ph.TOL["fp32"]["o"]
    assert torch.equal(one.Kc, two.Kc) and torch.equal(one.Vc, two.Vc)


@pytest.mark.parametrize("B,Hq,Hkv,d,L,b,a", [
    (2, 6, 2, 128, 3001, 500, 301),         # 32-row tiles, all blocks in one group
    (1, 4, 1, 64, 13000, 3000, 99),         # 32-row tiles, block by block
    (1, 4, 2, 128, 1100, 256, 256),         # 16-row tiles, four wavefronts
])
def test_fp32_many_rows(B, Hq, Hkv, d, L, b, a):
    """Enough rows for the kernel set-ups of longer prefills."""
    cfg = workloads.StarConfig("f32many", "fp32", B, Hq, Hkv, d, L, b, a, 100, 1, seed=5, n_planted=2)
    rep = ph.run_parity(cfg)
    assert rep.ok, rep.detail
    # the query call (100 tokens: 32-row tiles of phase 2 on the longer contexts) in equal runs of keys
    inp = workloads.make_inputs(cfg, "cuda")
    one, two = ph.HipRun(cfg, inp, "cuda"), ph.HipRun(cfg, inp, "cuda")
    one.phase1()
    two.phase1()
    want, _, _ = one.phase2(inp.Qq, inp.Kq, inp.Vq, want_parts=True)
    got, _, _ = two.phase2(inp.Qq, inp.Kq, inp.Vq, want_parts=False)
    torch.cuda.synchronize()
    assert (want - got).abs().max().item() <= 2 * ph.TOL["fp32"]["o"]
    assert torch.equal(one.Kc, two.Kc) and torch.equal(one.Vc, two.Vc)


@pytest.mark.parametrize("B,Hq,Hkv,d,L,b,a", [
    (1, 2, 2, 64, 130, 64, 64),             # the last block of two keys
    (2, 6, 3, 64, 351, 100, 30),            # its tiles end below, the first block's above those behind an anchor
    (1, 4, 1, 128, 260, 90, 1),             # an anchor of less than half a tile: one class with the first block
    (1, 4, 2, 64, 390, 128, 64),            # two blocks of each kind in a class
    (1, 8, 2, 64, 1200, 400, 0),            # no anchor: all blocks alike
    (3, 2, 1, 64, 700, 690, 690),           # one full block, and the last short
    (1, 8, 2, 64, 1060, 265, 265),          # 16-row tiles, 268 of them: the lighter ones in reverse
    (1, 8, 2, 64, 2050, 512, 512),          # 16-row tiles, 514: beyond two per CU
    (1, 4, 4, 64, 2000, 2000, 2000),        # one block: 500 in reverse
])
def test_fp32_tile_order(B, Hq, Hkv, d, L, b, a):
    """Every tile of every block once, whatever order a call's blocks give them (every row is
    compared, and every cache row)."""
    cfg = workloads.StarConfig("f32order", "fp32", B, Hq, Hkv, d, L, b, a, 2, 1, seed=L, n_planted=2)
    print(f"[{cfg}]", flush=True)
    rep = ph.run_parity(cfg, all_rows=True)
    assert rep.ok, rep.detail


def test_fp32_workspace_covers_every_shorter_call():
    """Whatever a query call of at most max_q tokens plans must fit what
    star_attn_workspace_bytes asked for (tiles hold 32 / G tokens: not a whole number)."""
    for Hq, Hkv in ((4, 1), (3, 1), (20, 1), (8, 8)):
        shape = sa.StarShape.make("fp32", 1, Hq, Hkv, 64, 3000, 700, 100, 3400)
        for max_q in (75, 130, 400):
            have = sa.workspace_bytes(shape, max_q)
            for q in range(1, max_q + 1):
                for parts in (False, True):
                    for cached in (3000, 3400 - q):
                        assert sa.phase2_plan(shape, cached, q, parts).workspace_bytes <= have, (Hq, q, parts)


@pytest.mark.parametrize("d,G", [(64, 1), (128, 4)])
@pytest.mark.parametrize("run", [16, 64, 128])           # keys of a step: one unit of one, of four and of eight wavefronts
@pytest.mark.parametrize("step", [7.9, 8.1])             # log2 units: within the softmax's headroom, and beyond it
def test_scores_that_climb_over_large_values(step, run, d, G):
    """Rows whose scores rise in steps, over values whose weighted sums are within fp32 as long as no weight is above
    one (128 keys of up to 1e36 at the top step) and beyond it with weights of 2^7.9."""
    L, q, big = 512, 20, 1e36
    shape = sa.StarShape.make("fp32", 1, G, 1, d, L, L, 0, L + q, softmax_scale=1.0)
    gen = torch.Generator(device="cuda").manual_seed(run)
    V = big * (0.5 + 0.5 * torch.rand((1, L + q, 1, d), generator=gen, device="cuda"))
    K = torch.zeros_like(V)
    K[0, :, 0, 0] = torch.arange(L + q, device="cuda") // run * (step * math.log(2.0))
    Q = torch.zeros((1, L + q, G, d), device="cuda")
    Q[..., 0] = 1.0
    O, lse = torch.empty((1, L, G, d), device="cuda"), torch.empty((1, G, L), device="cuda")
    Kc, Vc = sa.alloc_cache(shape)
    sa.phase1(shape, Q[:, :L].contiguous(), K[:, :L].contiguous(), V[:, :L].contiguous(), O, Kc, Vc, LSE_ctx=lse)
    s = K[0, :, 0, 0].double().repeat(L + q, 1).masked_fill(torch.ones((L + q, L + q), device="cuda").triu(1).bool(), -math.inf)
    want, want_lse = torch.softmax(s, 1) @ (V[0, :, 0].double() / big), torch.logsumexp(s, 1)
    tol = ph.TOL["fp32"]["o"]
    torch.cuda.synchronize()
    for h in range(G):
        assert (O[0, :, h].double() / big - want[:L]).abs().max().item() <= tol
        assert ((lse[0, h].double() - want_lse[:L]).abs() <= 2.0 ** -22 * want_lse[:L].abs() + 1e-6).all()
    cached = L
    for n in (1, q - 1):                                 # one token, then several
        Oq, ws = torch.empty((1, n, G, d), device="cuda"), sa.alloc_workspace(shape, n)
        part = slice(cached, cached + n)
        sa.phase2(shape, cached, Q[:, part].contiguous(), K[:, part].contiguous(), V[:, part].contiguous(), Kc, Vc, Oq, ws)
        torch.cuda.synchronize()
        assert (Oq[0].double() / big - want[part][:, None]).abs().max().item() <= tol
        cached += n


# tiles: of phase 1, and of phase 2 if that is one split.  Up to 64 share quarters of d, up to 128 halves (which the plans do not say).
@pytest.mark.parametrize("B,Hq,Hkv,d,L,b,a,lq,tiles", [
    (1, 1, 1, 64, 1024, 256, 256, 1, (64, None)),       # quarters of d
    (1, 3, 3, 128, 337, 100, 33, 70, (72, None)),       # short last blocks: halves
    (2, 5, 1, 128, 200, 200, 0, 3, (126, 2)),           # tiles that end between tokens: halves; 203 keys: quarters
    (1, 2, 2, 64, 1025, 1025, 0, 40, (130, None)),      # whole
    (1, 33, 1, 128, 31, 31, 16, 33, (64, 69)),          # quarters; 64 keys: halves
    (1, 16, 4, 64, 64, 64, 7, 64, (64, 64)),
    (1, 4, 2, 64, 1001, 250, 43, 2, (258, None)),       # whole, short ranges
    (1, 1, 1, 64, 2501, 625, 625, 5, (161, None)),      # whole, long ranges
    (1, 1, 1, 128, 2099, 300, 300, 5, (133, None)),     # whole
])
def test_fp32_columns_shared_by_workgroups(B, Hq, Hkv, d, L, b, a, lq, tiles):
    """Calls of few tiles, whose columns of d are computed by two or four workgroups."""
    shape = sa.StarShape.make("fp32", B, Hq, Hkv, d, L, b, a, L + lq)
    one, two = sa.phase1_plan(shape), sa.phase2_plan(shape, L, lq)
    assert one.tile_rows == 16 and one.wavefronts == 8 and one.n_tiles == tiles[0]
    assert two.tile_rows == 16 and (two.n_splits == 1) == (tiles[1] is not None)
    assert tiles[1] in (None, B * Hkv * -(-(Hq // Hkv) * lq // 16))
    cfg = workloads.StarConfig("f32pieces", "fp32", B, Hq, Hkv, d, L, b, a, lq, 1, seed=L, n_planted=2)
    print(f"[{cfg}]", flush=True)
    rep = ph.run_parity(cfg, all_rows=True)
    assert rep.ok, rep.detail
    inp = workloads.make_inputs(cfg, "cuda")
    parts, whole = ph.HipRun(cfg, inp, "cuda"), ph.HipRun(cfg, inp, "cuda")
    parts.phase1()
    whole.phase1()
    want, _, _ = parts.phase2(inp.Qq, inp.Kq, inp.Vq, want_parts=True)
    got, _, _ = whole.phase2(inp.Qq, inp.Kq, inp.Vq, want_parts=False)      # (one workgroup per tile and piece)
    torch.cuda.synchronize()
    assert (want - got).abs().max().item() <= 2 * ph.TOL["fp32"]["o"]
    assert torch.equal(parts.Kc, whole.Kc) and torch.equal(parts.Vc, whole.Vc)
