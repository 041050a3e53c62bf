"""The streaming decode kernel's last steps: where the call's tokens begin and end among the 32-key steps, with as many whole
steps in front as none, one or several, several last steps to a wavefront, and two tiles of rows (whose registers hold one step)."""
import pytest
import torch

import paper_2411_17116_amd as sa
from tests import parity_harness as ph

pytestmark = pytest.mark.gpu


def _call(B, Hq, Hkv, L, q, seed):
    gen = torch.Generator().manual_seed(seed)
    x = lambda *s: torch.randn(s, generator=gen).bfloat16().cuda()
    shape = sa.StarShape.make("bf16", B, Hq, Hkv, 128, L, L, 0, L + q + 3)
    return shape, x(B, q, Hq, 128), x(B, q, Hkv, 128), x(B, q, Hkv, 128), x(B, Hkv, L + q + 3, 128), x(B, Hkv, L + q + 3, 128)


def _exact(Q, K, V, q):
    """K, V: the caches in 64 bits, the call's rows in them."""
    G, L = Q.shape[2] // K.shape[1], K.shape[2] - q
    s = torch.einsum("bqhd,bhkd->bhqk", Q, K.repeat_interleave(G, dim=1)) / 128 ** 0.5
    s.masked_fill_(torch.arange(L + q)[None, :] > L + torch.arange(q)[:, None], float("-inf"))
    return torch.einsum("bhqk,bhkd->bqhd", s.softmax(-1), V.repeat_interleave(G, dim=1))


@pytest.mark.parametrize("B,Hq,Hkv,L,q", [
    (1, 8, 2, 31, 1), (1, 8, 2, 32, 1), (1, 8, 2, 1, 4),          # a step ends with the token, begins with it; one step in all
    (1, 8, 2, 2047, 1), (1, 8, 2, 2048, 4), (1, 8, 2, 2077, 4),   # a last step alone; across two wavefronts
    (64, 8, 8, 30, 16), (64, 8, 8, 90, 16), (64, 8, 8, 64, 15),   # one wavefront to a head: two last steps behind none, two; one behind two
    (1, 4, 4, 1009, 32), (1, 32, 8, 2041, 8), (64, 8, 8, 90, 31), # two tiles of rows
    (1, 32, 8, 8191, 1), (1, 32, 8, 8192, 4),                     # four wavefronts to a split: one last step, whole steps in front
])
def test_last_steps(B, Hq, Hkv, L, q):
    shape, Q, Kn, Vn, Kc, Vc = _call(B, Hq, Hkv, L, q, L + q)
    print(f"{B} {Hq}/{Hkv} {L} {q}", flush=True)
    K, V = Kc.clone(), Vc.clone()
    K[:, :, L:L + q], V[:, :, L:L + q] = Kn.transpose(1, 2), Vn.transpose(1, 2)
    O = torch.empty_like(Q)
    sa.phase2(shape, L, Q, Kn, Vn, Kc, Vc, O, sa.alloc_workspace(shape, q))
    torch.cuda.synchronize()
    assert torch.equal(Kc, K) and torch.equal(Vc, V)
    want = _exact(Q.double().cpu(), K[:, :, :L + q].double().cpu(), V[:, :, :L + q].double().cpu(), q)
    assert (O.double().cpu() - want).abs().max().item() <= ph.TOL["bf16"]["o"]


@pytest.mark.parametrize("B,Hq,Hkv,L,q", [(1, 8, 2, 2046, 4), (64, 8, 8, 30, 8), (64, 8, 8, 92, 8), (1, 32, 8, 8191, 1), (1, 8, 2, 32, 1)])
def test_last_steps_unrotated(B, Hq, Hkv, L, q):
    """Turned on the way, against rotation first and the call on what it leaves: the same bits."""
    shape, Q, Kn, Vn, Kc, Vc = _call(B, Hq, Hkv, L, q, L)
    print(f"{B} {Hq}/{Hkv} {L} {q}", flush=True)
    tokens = lambda H: sa.StarShape.make("bf16", B, H, H, 128, q, q, 0, q)
    Qr, Kr, K, V, want, O = torch.empty_like(Q), torch.empty_like(Kn), Kc.clone(), Vc.clone(), torch.empty_like(Q), torch.empty_like(Q)
    sa.rope(tokens(Hq), Q, Qr, 500000.0, pos0=L + 7)
    sa.rope(tokens(Hkv), Kn, Kr, 500000.0, pos0=L + 7)
    sa.phase2(shape, L, Qr, Kr, Vn, K, V, want, sa.alloc_workspace(shape, q))
    sa.phase2_rope(shape, 500000.0, L, Q, Kn, Vn, Kc, Vc, O, sa.alloc_workspace(shape, q), pos0=7)
    torch.cuda.synchronize()
    assert torch.equal(Kc, K) and torch.equal(Vc, V) and torch.equal(Q, Qr) and torch.equal(O, want)


# Caches read from HBM: every step is requested while the one before it is worked on, the last ones among them
HBM = [
    (512, 8, 8, 90, 16),          # one wavefront to a head: two last steps behind two whole ones
    (1100, 8, 8, 30, 16),         # two behind none
    (1300, 8, 8, 31, 9),          # the second of eight keys
    (512, 8, 8, 96, 8),           # one, which begins with the tokens, behind three
    (200, 16, 8, 260, 8),         # G = 2
]


def _from_hbm(B, Hq, Hkv, L, q, rope):
    shape, Q, Kn, Vn, Kc, Vc = _call(B, Hq, Hkv, L, q, L + q)
    plan = sa.phase2_plan(shape, L, q)
    assert plan.decode == 1 and plan.non_temporal == 1 and plan.flat == 1 and plan.n_splits == 1
    print(f"{B} {Hq}/{Hkv} {L} {q} rope={rope}", flush=True)
    O, ws = torch.empty_like(Q), sa.alloc_workspace(shape, q)
    return shape, Q, Kn, Vn, Kc, Vc, O, ws


@pytest.mark.parametrize("B,Hq,Hkv,L,q", HBM)
def test_last_steps_of_caches_from_hbm(B, Hq, Hkv, L, q):
    shape, Q, Kn, Vn, Kc, Vc, O, ws = _from_hbm(B, Hq, Hkv, L, q, False)
    K, V = Kc.clone(), Vc.clone()
    K[:, :, L:L + q], V[:, :, L:L + q] = Kn.transpose(1, 2), Vn.transpose(1, 2)
    sa.phase2(shape, L, Q, Kn, Vn, Kc, Vc, O, ws)
    torch.cuda.synchronize()
    assert torch.equal(Kc, K) and torch.equal(Vc, V)
    some = [0, 1, B // 2, B - 1]
    want = _exact(Q[some].double().cpu(), K[some, :, :L + q].double().cpu(), V[some, :, :L + q].double().cpu(), q)
    assert (O[some].double().cpu() - want).abs().max().item() <= ph.TOL["bf16"]["o"]


@pytest.mark.parametrize("B,Hq,Hkv,L,q", [(1400, 8, 8, 28, 8), (512, 8, 8, 92, 8), (1100, 16, 8, 40, 8)])
def test_last_steps_of_caches_from_hbm_unrotated(B, Hq, Hkv, L, q):
    shape, Q, Kn, Vn, Kc, Vc, O, ws = _from_hbm(B, Hq, Hkv, L, q, True)
    tokens = lambda H: sa.StarShape.make("bf16", B, H, H, 128, q, q, 0, q)
    Qr, Kr, K, V, want = torch.empty_like(Q), torch.empty_like(Kn), Kc.clone(), Vc.clone(), torch.empty_like(Q)
    sa.rope(tokens(Hq), Q, Qr, 500000.0, pos0=L + 7)
    sa.rope(tokens(Hkv), Kn, Kr, 500000.0, pos0=L + 7)
    sa.phase2(shape, L, Qr, Kr, Vn, K, V, want, ws)
    sa.phase2_rope(shape, 500000.0, L, Q, Kn, Vn, Kc, Vc, O, ws, pos0=7)
    torch.cuda.synchronize()
    assert torch.equal(Kc, K) and torch.equal(Vc, V) and torch.equal(Q, Qr) and torch.equal(O, want)
