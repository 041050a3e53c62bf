"""What lies in memory a call must not use -- NaN in cache rows behind the visible ones and in caches
about to be filled -- leaves no trace in its results, on every kernel; and a logit of minus
infinity takes its key out of the softmax."""
import pytest
import torch

import paper_2411_17116_amd as sa

pytestmark = pytest.mark.gpu


def _tensors(dtype, seed, *sizes):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    return [torch.randn(s, generator=gen, device="cuda").to(dt) for s in sizes]


# dtype, heads, KV heads, d, cached, new tokens: streaming decode, 128-row and 256-row tiles, fp32 in one
# workgroup per tile, 16-row and 32-row tiles; streamed calls of two wavefronts to a split, of four with one and two
# blocks of rows, and of a cache beyond the last-level cache with four
CALLS = [("bf16", 8, 2, 128, 1001, 1), ("bf16", 8, 2, 128, 1001, 33), ("bf16", 32, 8, 128, 9001, 300),
         ("fp32", 4, 2, 64, 203, 3), ("fp32", 4, 2, 64, 3001, 3), ("fp32", 8, 2, 128, 5001, 100),
         ("bf16", 8, 2, 128, 1001, 5), ("bf16", 32, 8, 128, 8190, 1), ("bf16", 8, 2, 128, 4001, 7), ("bf16", 32, 8, 128, 50001, 15)]


@pytest.mark.parametrize("parts", [False, True])
@pytest.mark.parametrize("dtype,Hq,Hkv,d,L,q", CALLS)
def test_rows_behind_the_visible_ones(dtype, Hq, Hkv, d, L, q, parts):
    cap, b = L + q + 130, L // 2 + 1
    shape = sa.StarShape.make(dtype, 1, Hq, Hkv, d, L, b, 0, cap)
    Q, K, V, Kc, Vc = _tensors(dtype, L + q, (1, q, Hq, d), (1, q, Hkv, d), (1, q, Hkv, d), (1, Hkv, cap, d), (1, Hkv, cap, d))
    n = -(-L // b) + 1
    out = []
    for fill in (0.0, float("nan")):
        kc, vc, O = Kc.clone(), Vc.clone(), torch.empty_like(Q)
        kc[:, :, L:], vc[:, :, L:] = fill, fill
        Op = torch.empty((1, n, Hq, q, d), device="cuda") if parts else None
        Lp = torch.empty((1, n, Hq, q), device="cuda") if parts else None
        print(f"{dtype} {Hq}/{Hkv} L={L} q={q} parts={parts} fill={fill}", flush=True)
        sa.phase2(shape, L, Q, K, V, kc, vc, O, sa.alloc_workspace(shape, q), O_part=Op, LSE_part=Lp)
        torch.cuda.synchronize()
        out.append((O, kc[:, :, :L + q], vc[:, :, :L + q]) + ((Op, Lp) if parts else ()))
    assert torch.isfinite(out[1][0].float()).all()
    assert all(torch.equal(x, y) for x, y in zip(*out))


@pytest.mark.parametrize("dtype,Hq,Hkv,d,L,b,a", [
    ("bf16", 8, 2, 128, 777, 200, 70), ("bf16", 32, 8, 128, 1500, 500, 500), ("bf16", 32, 8, 128, 13003, 13003, 0),
    ("bf16", 40, 8, 128, 12007, 6007, 6007), ("fp32", 4, 2, 64, 500, 15, 0), ("fp32", 4, 2, 64, 777, 200, 70),
    ("fp32", 8, 2, 128, 4500, 1500, 99)])
def test_caches_about_to_be_filled(dtype, Hq, Hkv, d, L, b, a):
    shape = sa.StarShape.make(dtype, 1, Hq, Hkv, d, L, b, a, L + 70)
    Q, K, V = _tensors(dtype, L, (1, L, Hq, d), (1, L, Hkv, d), (1, L, Hkv, d))
    out = []
    for fill in (0.0, float("nan")):
        Kc, Vc = sa.alloc_cache(shape)
        Kc.fill_(fill)
        Vc.fill_(fill)
        O, LSE = torch.empty_like(Q), torch.empty((1, Hq, L), device="cuda")
        print(f"{dtype} {Hq}/{Hkv} L={L} fill={fill}", flush=True)
        sa.phase1(shape, Q, K, V, O, Kc, Vc, LSE_ctx=LSE)
        torch.cuda.synchronize()
        assert Kc[:, :, L:].isnan().all() if fill else not Kc[:, :, L:].any()
        out.append((O, LSE, Kc[:, :, :L], Vc[:, :, :L]))
    assert torch.isfinite(out[1][0].float()).all() and torch.isfinite(out[1][1]).all()
    assert all(torch.equal(x, y) for x, y in zip(*out))


@pytest.mark.parametrize("key", [0, 40, -1])
@pytest.mark.parametrize("dtype,Hq,Hkv,d,L,q", CALLS)
def test_a_logit_of_minus_infinity(dtype, Hq, Hkv, d, L, q, key):
    """The call with one key far enough down that its products overflow, against 64 bits without it."""
    shape = sa.StarShape.make(dtype, 1, Hq, Hkv, d, L, L, 0, L + q)
    Q, K, V, Kc, Vc = _tensors(dtype, L + q, (1, q, Hq, d), (1, q, Hkv, d), (1, q, Hkv, d), (1, Hkv, L + q, d), (1, Hkv, L + q, d))
    Q = Q.abs() + 0.5                                  # every product of the key has the same sign
    Kc[:, :, L - 1 if key < 0 else key] = -3e38
    O = torch.empty_like(Q)
    print(f"{dtype} {Hq}/{Hkv} L={L} q={q} key={key}", flush=True)
    sa.phase2(shape, L, Q, K, V, Kc, Vc, O, sa.alloc_workspace(shape, q))
    torch.cuda.synchronize()
    keep = torch.ones(L + q, dtype=torch.bool, device="cuda")
    keep[L - 1 if key < 0 else key] = False
    for h in range(0, Hq, max(1, Hq // 4)):
        s = Q[0, :, h].double() @ Kc[0, h // (Hq // Hkv), keep].double().T / d ** 0.5
        seen = (torch.arange(L + q, device="cuda")[keep] <= L + torch.arange(q, device="cuda")[:, None])
        w = torch.softmax(s.masked_fill(~seen, -float("inf")), dim=1)
        want = w @ Vc[0, h // (Hq // Hkv), keep].double()
        assert (O[0, :, h].double() - want).abs().max().item() <= (1e-5 if dtype == "fp32" else 2e-2), h
