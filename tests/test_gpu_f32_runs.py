"""fp32 phase-2 calls whose rows are one 16-row tile per KV head, cut into equal runs of 64 keys and more: at the edges
of the units, of the tile and of the rule, against plain fp64 attention."""
import math

import pytest
import torch

import paper_2411_17116_amd as sa
from tests import parity_harness as ph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv,d,L,q,splits", [
    (1, 1, 1, 64, 511, 1, 1),          # 256 KiB of K + V: one workgroup
    (1, 1, 1, 64, 512, 1, 9),          # a run of one key at the end
    (2, 6, 2, 64, 1000, 5, 16),        # 15 rows
    (1, 16, 1, 128, 575, 1, 9),        # a whole tile; 64 keys to every run
    (1, 17, 1, 128, 575, 1, 5),        # 17 rows: runs of 128 keys
    (1, 2, 2, 128, 8150, 2, 128),      # 8152 keys: as many runs as are worth merging, all that start at once
    (1, 3, 3, 128, 8150, 2, 64),       # more than that: runs of 128 keys
    (1, 4, 1, 64, 40959, 1, 128),      # one KV head: five units for each of four wavefronts
    (1, 4, 1, 64, 40960, 1, 214),      # beyond that eight wavefronts on all CUs
    (1, 2, 2, 64, 50000, 1, 121),      # two: as many runs as start at once at any length
])
def test_short_runs(B, Hq, Hkv, d, L, q, splits):
    gen = torch.Generator(device="cuda").manual_seed(L)
    new = lambda *s: torch.randn(s, generator=gen, device="cuda")
    cap, G = L + q + 30, Hq // Hkv
    shape = sa.StarShape.make("fp32", B, Hq, Hkv, d, L, max(1, L // 4), 0, cap)
    print(f"[{B} {Hq}/{Hkv} d={d} L={L} q={q}]", flush=True)
    assert sa.phase2_plan(shape, L, q).n_splits == splits
    Kc, Vc = new(B, Hkv, cap, d), new(B, Hkv, cap, d)
    Q, K, V = new(B, q, Hq, d), new(B, q, Hkv, d), new(B, q, Hkv, d)
    O, ws = torch.empty_like(Q), sa.alloc_workspace(shape, q)
    A, lse = torch.empty((B, Hq, q, d), device="cuda"), torch.empty((B, Hq, q), device="cuda")
    sa.phase2(shape, L, Q, K, V, Kc, Vc, O, ws)
    sa.phase2_partial(shape, L + q, Q, Kc, Vc, A, lse, ws)      # a host's share: all L + q rows visible
    torch.cuda.synchronize()
    assert torch.equal(Kc[:, :, L:L + q], K.transpose(1, 2)) and torch.equal(Vc[:, :, L:L + q], V.transpose(1, 2))
    tol = ph.TOL["fp32"]["o"]
    for beta in range(B):
        for g in range(Hkv):
            hs = slice(g * G, (g + 1) * G)
            k, v = Kc[beta, g, :L + q].double(), Vc[beta, g, :L + q].double()
            s = Q[beta, :, hs].double().reshape(q * G, d) @ k.T / math.sqrt(d)
            # (natural logarithms near log(L): a few ulp of 5e-7)
            assert (lse[beta, hs].T.reshape(-1) - torch.logsumexp(s, 1)).abs().max().item() <= 1e-5
            assert (A[beta, hs].double() - (torch.softmax(s, 1) @ v).view(q, G, d).transpose(0, 1)).abs().max().item() <= tol
            bound = L + 1 + torch.arange(q, device="cuda").repeat_interleave(G)
            s.masked_fill_(torch.arange(L + q, device="cuda")[None] >= bound[:, None], -math.inf)
            assert (O[beta, :, hs].double() - (torch.softmax(s, 1) @ v).view(q, G, d)).abs().max().item() <= tol


@pytest.mark.parametrize("dtype,B,Hq,Hkv,d,L,q", [
    ("fp32", 1, 65535, 1, 64, 700, 1),          # the largest group and number of KV heads a launch's arguments hold
    ("fp32", 1, 65535, 65535, 64, 40, 2),
    ("bf16", 1, 65535, 65535, 128, 40, 1),
    ("fp32", 3, 255, 85, 64, 600, 7),
])
def test_many_heads(dtype, B, Hq, Hkv, d, L, q):
    gen = torch.Generator(device="cuda").manual_seed(L)
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    new = lambda *s: torch.randn(s, generator=gen, device="cuda").to(dt)
    shape = sa.StarShape.make(dtype, B, Hq, Hkv, d, L, L, 0, L + q)
    Kc, Vc = new(B, Hkv, L + q, d), new(B, Hkv, L + q, d)
    Q, K, V = new(B, q, Hq, d), new(B, q, Hkv, d), new(B, q, Hkv, d)
    O = torch.empty_like(Q)
    print(f"[{dtype} {B} {Hq}/{Hkv} d={d} L={L} q={q}]", flush=True)
    sa.phase2(shape, L, Q, K, V, Kc, Vc, O, sa.alloc_workspace(shape, q))
    torch.cuda.synchronize()
    assert torch.equal(Kc[:, :, L:], K.transpose(1, 2)) and torch.equal(Vc[:, :, L:], V.transpose(1, 2))
    for h in sorted({0, 1, Hq // 2, Hq - 2, Hq - 1}):
        k, v = Kc[:, h * Hkv // Hq].double(), Vc[:, h * Hkv // Hq].double()
        s = (Q[:, :, h].double().unsqueeze(2) * k.unsqueeze(1)).sum(-1) / d ** 0.5
        seen = torch.arange(L + q, device="cuda") <= L + torch.arange(q, device="cuda")[:, None]
        w = torch.softmax(s.masked_fill(~seen, -float("inf")), dim=-1)
        want = (w.unsqueeze(-1) * v.unsqueeze(1)).sum(2)
        assert (O[:, :, h].double() - want).abs().max().item() <= (1e-5 if dtype == "fp32" else 2e-2), h
