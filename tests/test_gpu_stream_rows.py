"""Phase-2 calls that stream the cache through the decode kernel with more than one 16-row block of columns, or
with several wavefronts to a split: at the edges of the row blocks, of the 32-key steps and of the rules that choose
the set-up, against plain fp64 attention."""
import math

import pytest
import torch

import paper_2411_17116_amd as sa
from tests import parity_harness as ph

pytestmark = pytest.mark.gpu


# decode: 1 where the call streams; splits: per KV head.  Caches beyond 192 MiB of K + V: 49152 keys of eight heads.
@pytest.mark.parametrize("B,Hq,Hkv,L,q,decode,splits", [
    (1, 17, 1, 63, 1, 0, None),        # 64 keys, one key tile: row-tiled
    (1, 17, 1, 64, 1, 1, 2),           # 17 rows, three steps shared by two wavefronts of two splits
    (2, 8, 2, 90, 8, 1, 2),            # 32 rows, the new tokens in two steps
    (1, 33, 1, 700, 1, 0, None),       # 33 rows of a resident cache: row-tiled
    (1, 32, 1, 2047, 1, 1, 32),        # 2048 keys: the last with two wavefronts to a split
    (1, 32, 1, 2048, 1, 1, 17),        # and the first with four, the last split with one step
    (1, 12, 4, 5000, 9, 1, 40),        # 27 rows, tokens straddle the row blocks
    (33, 64, 8, 300, 3, 1, 1),         # a split per KV head
    (6, 32, 8, 796, 8, 1, 4),          # 48 KV heads: as few splits as two steps for each of four wavefronts ask for
    (4, 32, 8, 2000, 5, 1, 8),         # 32
    (32, 32, 8, 2000, 5, 1, 1),        # 256, beyond the last-level cache: four wavefronts and non-temporal loads
    (33, 8, 4, 2600, 9, 0, None),      # 132 keep half the CUs busy: row-tiled beyond 2560 keys
    (1, 32, 8, 4096, 4, 1, 33),        # 16 rows: 65 splits become 33 of four wavefronts
    (1, 32, 8, 8158, 4, 1, 64),        # new tokens in the last step and one of their own
    (1, 32, 8, 8190, 4, 1, 86),        # a step more than the wavefronts of 64 splits: one to a split again
    (1, 4, 1, 9000, 1, 1, 71),         # few KV heads
    (1, 32, 1, 400000, 1, 1, 256),     # beyond the last-level cache: 32 rows
    (1, 33, 1, 400000, 1, 1, 256),     # 33, 48, 49 and 64 rows
    (1, 24, 2, 200000, 4, 1, 128),
    (1, 49, 1, 400031, 1, 1, 256),
    (1, 32, 4, 98333, 8, 1, 64),
    (1, 65, 1, 400000, 1, 0, None),
])
def test_streamed_rows(B, Hq, Hkv, L, q, decode, splits):
    gen = torch.Generator(device="cuda").manual_seed(L + q)
    new = lambda *s: torch.randn(s, generator=gen, device="cuda", dtype=torch.bfloat16)
    cap, G, d = L + q + 40, Hq // Hkv, 128
    shape = sa.StarShape.make("bf16", B, Hq, Hkv, d, L, max(1, L // 4), 0, cap)
    plan = sa.phase2_plan(shape, L, q)
    print(f"[{B} {Hq}/{Hkv} L={L} q={q}] splits {plan.n_splits}", flush=True)
    assert plan.decode == decode and (splits is None or plan.n_splits == splits)
    Kc, Vc = new(B, Hkv, cap, d), new(B, Hkv, cap, d)
    Q, K, V = new(B, q, Hq, d), new(B, q, Hkv, d), new(B, q, Hkv, d)
    Q[:, 0] = (1.5 * Kc[:, :, L // 2].float()).bfloat16().repeat_interleave(G, dim=1)      # a row that points at one key
    behind = Kc[:, :, L + q:].clone(), Vc[:, :, L + q:].clone()
    O, ws = torch.empty_like(Q), sa.alloc_workspace(shape, q)
    sa.phase2(shape, L, Q, K, V, Kc, Vc, O, ws)
    # a host's share of the same call: nothing appended, every token sees the L + q rows
    A, lse = torch.empty((B, Hq, q, d), device="cuda"), torch.empty((B, Hq, q), device="cuda")
    sa.phase2_partial(shape, L + q, Q, Kc, Vc, A, lse, ws)
    torch.cuda.synchronize()
    assert torch.equal(Kc[:, :, L:L + q], K.transpose(1, 2)) and torch.equal(Vc[:, :, L:L + q], V.transpose(1, 2))
    assert torch.equal(Kc[:, :, L + q:], behind[0]) and torch.equal(Vc[:, :, L + q:], behind[1])
    tol = ph.TOL["bf16"]
    for beta in sorted({0, B - 1}):
        for g in sorted({0, Hkv - 1}):
            hs = slice(g * G, (g + 1) * G)
            k, v = Kc[beta, g, :L + q].double(), Vc[beta, g, :L + q].double()
            s = Q[beta, :, hs].double().reshape(q * G, d) @ k.T / math.sqrt(d)
            assert (lse[beta, hs].T.reshape(-1) - torch.logsumexp(s, 1)).abs().max().item() <= tol["lse"]
            want = (torch.softmax(s, 1) @ v).view(q, G, d).transpose(0, 1)
            assert (A[beta, hs].double() - want).abs().max().item() <= tol["o"]
            bound = L + 1 + torch.arange(q, device="cuda").repeat_interleave(G)
            s.masked_fill_(torch.arange(L + q, device="cuda")[None] >= bound[:, None], -math.inf)
            want = (torch.softmax(s, 1) @ v).view(q, G, d)
            assert (O[beta, :, hs].double() - want).abs().max().item() <= tol["o"]


def test_workspace_covers_streamed_calls():
    """Whatever a streamed call plans, on a cache of any length, fits what star_attn_workspace_bytes asked for; and a
    call that brings room for fewer splits makes do with them."""
    for Hq, Hkv, B, cap in ((8, 2, 1, 700), (32, 8, 1, 9000), (64, 8, 4, 30000), (33, 1, 1, 420000), (20, 1, 2, 2500)):
        for L in (1, 33, 64, 600, 2047, 2048, 8191, cap - 64):
            if L > cap - 64:
                continue
            shape = sa.StarShape.make("bf16", B, Hq, Hkv, 128, L, L, 0, cap)
            for q in range(1, 64 * Hkv // Hq + 1):
                have = sa.workspace_bytes(shape, q)
                for cached in (L, (L + cap) // 2, cap - q):
                    assert sa.phase2_plan(shape, cached, q).workspace_bytes <= have, (Hq, Hkv, B, L, q, cached)


def test_streamed_call_with_room_for_fewer_splits():
    B, Hq, Hkv, L, q, d = 1, 32, 8, 5000, 8, 128
    gen = torch.Generator(device="cuda").manual_seed(3)
    new = lambda *s: torch.randn(s, generator=gen, device="cuda", dtype=torch.bfloat16)
    shape = sa.StarShape.make("bf16", B, Hq, Hkv, d, L, L, 0, L + q)
    Kc, Vc, Q, K, V = new(B, Hkv, L + q, d), new(B, Hkv, L + q, d), new(B, q, Hq, d), new(B, q, Hkv, d), new(B, q, Hkv, d)
    one = B * Hq * q * (d + 1) * 4
    full, want = sa.alloc_workspace(shape, q), torch.empty_like(Q)
    sa.phase2(shape, L, Q, K, V, Kc, Vc, want, full)
    for splits in (1, 2, 7):
        room = (splits * one + 255) // 256 * 256
        guard = torch.full((room + 4096,), 171, dtype=torch.uint8, device="cuda")
        got = torch.empty_like(Q)
        sa.phase2(shape, L, Q, K, V, Kc, Vc, got, guard[:room])
        torch.cuda.synchronize()
        assert (guard[room:] == 171).all()
        assert (got.float() - want.float()).abs().max().item() <= 2 * ph.TOL["bf16"]["o"]
    with pytest.raises(sa.StarAttnError) as e:
        sa.phase2(shape, L, Q, K, V, Kc, Vc, got, full[:one // 2])
    assert e.value.code == -7
