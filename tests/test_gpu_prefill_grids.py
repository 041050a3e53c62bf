"""The plain launches of short bf16 prefills: 128-row items of four wavefronts, items whose
keys the halves of a workgroup share (odd and even numbers of key tiles, a half without
any), tiles taken block by block and interleaved with the light half turned round, head
groups that exceed a workgroup, ragged last blocks, every kind of anchor, the exact
fallback of the softmax; and the queues that longer prefills take, at ragged sizes, odd head
groups and several head sub-groups.  star_attn_phase1_plan says which of them a call takes."""
import pytest
import torch

import paper_2411_17116_amd as sa
import workloads
from tests import parity_harness as ph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv,L,b,a,gamma", [
    (1, 1, 1, 1, 1, 0, 1.5),               # one row
    (1, 2, 2, 130, 130, 130, 1.5),         # one block, two items per head, a ragged tile
    (1, 8, 1, 600, 600, 0, 1.5),           # ten key tiles at most: halves share the keys
    (1, 4, 1, 1300, 650, 65, 1.5),         # the same with an anchor, odd numbers of tiles
    (1, 16, 1, 900, 300, 300, 1.5),        # G = 16: two head sub-groups
    (1, 3, 1, 1400, 700, 700, 1.5),        # G = 3: one head per item
    (2, 8, 4, 1700, 425, 425, 1.5),        # more items than CUs: pairs of heavy and light
    (1, 64, 8, 1100, 275, 100, 1.5),       # several rounds, block by block
    (1, 8, 2, 1500, 500, 200, 6.0),        # scores far above the reference: the exact loop, halves
    (1, 32, 8, 1000, 250, 250, 6.0),       # and without them
    (1, 3, 3, 14000, 500, 200, 1.5),       # heads no multiple of 8: groups of sixteen blocks, a ragged one
    (1, 3, 3, 14000, 3500, 700, 1.5),      # blocks too long for that: runs of eight items turned on
    (2, 6, 2, 9001, 1500, 0, 1.5),         # the same over two batches, no anchors: one section
    (8, 5, 5, 7001, 3500, 100, 1.5),       # forty blocks at once in every XCD: block by block
])
def test_plain_grids(B, Hq, Hkv, L, b, a, gamma):
    cfg = workloads.StarConfig("plain", "bf16", B, Hq, Hkv, 128, L, b, a, 1, 0, seed=L + Hq, n_planted=8 if L > 64 else 0,
                               gamma=gamma)
    print(f"[{cfg}]", flush=True)
    plan = sa.phase1_plan(ph.shape_of(cfg))
    assert plan.queued == 0 and plan.tile_rows == 128
    assert plan.wavefronts == (8 if plan.n_tiles <= 256 and -(-a // 64) + -(-min(b, L) // 64) > 8 else 4)
    rep = ph.run_parity(cfg, all_rows=B * Hq * L <= 12000, n_random=2048)
    assert rep.ok, rep.detail


@pytest.mark.parametrize("B,Hq,Hkv,L,b,a,gamma", [
    (2, 12, 4, 15001, 7001, 7001, 1.5),    # G = 3, two sequences, a ragged last block and last tile
    (1, 48, 3, 12007, 6007, 6007, 1.5),    # G = 16: two head sub-groups, heads no multiple of 8
    (1, 40, 8, 12007, 6007, 6007, 6.0),    # G = 5; scores far above the reference: the exact loop
    (1, 32, 8, 19999, 19999, 0, 1.5),      # one block
])
def test_work_queues(B, Hq, Hkv, L, b, a, gamma):
    cfg = workloads.StarConfig("queues", "bf16", B, Hq, Hkv, 128, L, b, a, 1, 0, seed=L + Hq, n_planted=8, gamma=gamma)
    print(f"[{cfg}]", flush=True)
    assert sa.phase1_plan(ph.shape_of(cfg)).queued == 1
    rep = ph.run_parity(cfg, n_random=512)
    assert rep.ok, rep.detail


@pytest.mark.parametrize("mode", [sa.ANCHOR_PREVIOUS, sa.ANCHOR_PER_BLOCK, sa.ANCHOR_ALL_BLOCKS])
@pytest.mark.parametrize("Hq,Hkv,L,b,a", [(4, 2, 1900, 600, 77), (32, 8, 1500, 300, 150)])
def test_plain_grids_give_what_each_row_gives_alone(mode, Hq, Hkv, L, b, a):
    """Anchor variants: a block encoded in a call of its own, as one block whose anchor is
    handed in, must give the same rows within the storage rounding of the two splits."""
    gen = torch.Generator(device="cuda").manual_seed(L + mode)
    n = -(-L // b)
    rnd = lambda *s: torch.randn(s, generator=gen, device="cuda").to(torch.bfloat16)
    Q, K, V = rnd(1, L, Hq, 128), rnd(1, L, Hkv, 128), rnd(1, L, Hkv, 128)
    anchors = n if mode == sa.ANCHOR_PER_BLOCK else 1
    Ka, Va = rnd(1, anchors * a, Hkv, 128), rnd(1, anchors * a, Hkv, 128)
    shape = sa.StarShape.make("bf16", 1, Hq, Hkv, 128, L, b, a, L)
    Kc, Vc = sa.alloc_cache(shape)
    O = torch.empty_like(Q)
    print(f"mode {mode} {Hq}/{Hkv} L={L} b={b} a={a}", flush=True)
    sa.phase1_anchor(shape, mode, Q, K, V, O, Kc, Vc, K_anchor=Ka, V_anchor=Va)
    for i in range(n):
        s, e = i * b, min(L, (i + 1) * b)
        if mode == sa.ANCHOR_PREVIOUS:
            ka, va = K[:, s - a:s], V[:, s - a:s]
        elif mode == sa.ANCHOR_PER_BLOCK:
            ka, va = Ka[:, i * a:(i + 1) * a], Va[:, i * a:(i + 1) * a]
        else:
            ka, va = Ka, Va
        plain = i == 0 and mode != sa.ANCHOR_ALL_BLOCKS
        own = sa.StarShape.make("bf16", 1, Hq, Hkv, 128, e - s, max(e - s, a), 0 if plain else a, e - s)
        k1, v1 = sa.alloc_cache(own)
        o1 = torch.empty_like(Q[:, s:e])
        sa.phase1_anchor(own, sa.ANCHOR_ALL_BLOCKS, Q[:, s:e].contiguous(), K[:, s:e].contiguous(),
                         V[:, s:e].contiguous(), o1, k1, v1, K_anchor=ka.contiguous(), V_anchor=va.contiguous())
        torch.cuda.synchronize()
        # both within 2e-2 of the exact result (two roundings of P and one of O each)
        diff, ref = o1.float() - O[:, s:e].float(), o1.float()
        assert diff.abs().max().item() <= 2e-2, i
        # relative: four roundings to 8 bits of mantissa, rms 2^-9 / sqrt(3) each, is 2.3e-3
        assert diff.norm().item() <= 6e-3 * ref.norm().item(), i
        assert torch.equal(k1, Kc[:, :, s:e]) and torch.equal(v1, Vc[:, :, s:e])
