"""fp32 calls of many rows, whose products are taken in bf16 parts: every row against 64 bits, at ragged units and
tiles, and with values that the parts do not hold (which are taken in fp32 products instead)."""
import pytest
import torch

import paper_2411_17116_amd as sa

pytestmark = pytest.mark.gpu

# 1e-5 is what the fp32 path is held to (1.5e-7 of it are roundings of sums of a few hundred terms, see test_gpu_f32_tiles.py)
TOL = 1e-5


def _values(kind, Q, K, V):
    """The kinds of values; returns the size that an error is measured by."""
    if kind == "huge":                     # beyond the largest bf16 number, 3.39e38
        V *= 1e35                          # (few enough that sums of weighted values stay finite)
        V[:, 7, :, ::5] = 3.4e38
        return 3.4e38
    if kind == "tiny":                     # parts below the smallest normal number
        V *= 1e-34
        return 1e-34
    if kind == "far":                      # a key whose logits are minus infinity, and one that cannot be split
        Q.abs_().add_(0.5)
        K[:, 3] = -3e38
        K[:, 5] = -3.4e38
    return 1.0


def _attend(Q, K, V, lim):
    s = Q @ K.T / Q.shape[1] ** 0.5
    s = s.masked_fill(torch.arange(K.shape[0], device="cuda") >= lim[:, None], -float("inf"))
    return torch.softmax(s, dim=1) @ V, torch.logsumexp(s, dim=1)


@pytest.mark.parametrize("kind", ["normal", "huge", "tiny", "far"])
@pytest.mark.parametrize("B,Hq,Hkv,d,L,b,a", [
    (1, 32, 2, 128, 481, 481, 0),      # units of 32 keys, the last of one
    (1, 32, 2, 128, 440, 220, 137),    # ragged anchor, wavefronts without a unit
    (4, 6, 2, 128, 715, 143, 143),     # tiles that end between tokens (three heads), a last tile of two rows
    (1, 40, 4, 64, 700, 689, 1),       # anchor of one key, a short last block
    (1, 32, 1, 64, 480, 240, 225),
])
def test_prefill(B, Hq, Hkv, d, L, b, a, kind):
    gen = torch.Generator(device="cuda").manual_seed(L)
    new = lambda *s: torch.randn(s, generator=gen, device="cuda")
    Q, K, V = new(B, L, Hq, d), new(B, L, Hkv, d), new(B, L, Hkv, d)
    size, G = _values(kind, Q, K, V), Hq // Hkv
    shape = sa.StarShape.make("fp32", B, Hq, Hkv, d, L, b, a, L)
    assert sa.phase1_plan(shape, sa.ANCHOR_FIRST).tile_rows == 32
    Kc, Vc = sa.alloc_cache(shape)
    O, LSE = torch.empty_like(Q), torch.empty((B, Hq, L), device="cuda")
    print(f"{Hq}/{Hkv} d={d} L={L} {kind}", flush=True)
    sa.phase1(shape, Q, K, V, O, Kc, Vc, LSE_ctx=LSE)
    torch.cuda.synchronize()
    for beta in range(B):
        for h in range(Hq):
            k, v = K[beta, :, h // G].double(), V[beta, :, h // G].double()
            for s in range(0, L, b):
                e, n = min(L, s + b), a if s else 0
                lim = n + torch.arange(1, e - s + 1, device="cuda")
                o, x = _attend(Q[beta, s:e, h].double(), torch.cat([k[:n], k[s:e]]), torch.cat([v[:n], v[s:e]]), lim)
                seen = torch.isfinite(x)               # ("far": the first rows of a block may see nothing else)
                assert ((O[beta, s:e, h].double() - o)[seen].abs().max() <= TOL * size), (h, s)
                if kind != "far":
                    assert ((LSE[beta, h, s:e].double() - x).abs() <= TOL * (x.abs() / 8).clamp(min=1)).all(), (h, s)


@pytest.mark.parametrize("kind", ["normal", "huge", "tiny", "far"])
@pytest.mark.parametrize("parts", [False, True])
@pytest.mark.parametrize("Hq,Hkv,d,L,q", [(8, 2, 128, 4003, 60), (12, 4, 128, 4500, 45), (4, 2, 64, 30001, 100)])
def test_query(Hq, Hkv, d, L, q, parts, kind):
    gen = torch.Generator(device="cuda").manual_seed(L)
    new = lambda *s: torch.randn(s, generator=gen, device="cuda")
    Q, K, V = new(1, q, Hq, d), new(1, L + q, Hkv, d), new(1, L + q, Hkv, d)
    size, G = _values(kind, Q, K, V), Hq // Hkv
    shape = sa.StarShape.make("fp32", 1, Hq, Hkv, d, L, L // 3, 0, L + q)
    assert sa.phase2_plan(shape, L, q, want_parts=parts).tile_rows == 32
    Kc, Vc = K.transpose(1, 2).contiguous(), V.transpose(1, 2).contiguous()
    Kc[:, :, L:], Vc[:, :, L:] = 0, 0
    O, n = torch.empty_like(Q), -(-L // (L // 3)) + 1
    Op = torch.empty((1, n, Hq, q, d), device="cuda") if parts else None
    Lp = torch.empty((1, n, Hq, q), device="cuda") if parts else None
    print(f"{Hq}/{Hkv} d={d} L={L} q={q} parts={parts} {kind}", flush=True)
    sa.phase2(shape, L, Q, K[:, L:].contiguous(), V[:, L:].contiguous(), Kc, Vc, O, sa.alloc_workspace(shape, q), O_part=Op, LSE_part=Lp)
    torch.cuda.synchronize()
    assert torch.equal(Kc[0], K[0].transpose(0, 1)) and torch.equal(Vc[0], V[0].transpose(0, 1))
    for h in range(Hq):
        o, _ = _attend(Q[0, :, h].double(), K[0, :, h // G].double(), V[0, :, h // G].double(), L + torch.arange(1, q + 1, device="cuda"))
        assert ((O[0, :, h].double() - o).abs().max() <= TOL * size), h


# Two factors of a product whose sizes make up for each other: what the parts lose of the smaller one shows in results of ordinary size.
FAR = 82.0        # nats from a heavy key to the others, whose weights are then about 2^-118


def _uneven(kind, Q, K, V):
    h = Q.shape[-1] // 2
    if kind == "small queries":
        Q[..., :h] *= 2.0 ** -122
        K[..., :h] *= 2.0 ** 122
    if kind == "small keys":
        Q[..., h:] *= 2.0 ** 122
        K[..., h:] *= 2.0 ** -122
    if kind == "small weights":          # every sixteenth key outweighs the others; every 32nd has values, as much larger
        Q[..., 0], K[..., 0] = 32.0, 0.0
        K[:, ::16] = 0.0
        V[:, torch.arange(V.shape[1], device="cuda") % 32 != 1] = 0.0
        K[:, ::16, :, 0] = FAR * Q.shape[-1] ** 0.5 / 32
        V *= 2.0 ** 96
    if kind == "a small column":
        V[..., 1] *= 2.0 ** -115
    if kind == "a huge value":           # of a late key
        V[:, 5 * V.shape[1] // 6, :, 6] = 3.4e38


def _close(got, q, k, v, lim, kind):
    want, _ = _attend(q, k, v, lim)
    size = _attend(q, k, v.abs(), lim)[0].amax(1, keepdim=True) if kind == "small weights" else torch.ones_like(want)
    if kind == "a small column":
        size[:, 1] = 2.0 ** -115
    if kind == "a huge value":
        size[:, 6] = 3.4e38
    # scores FAR below their reference (log2 units: 1.45 FAR): the query's scaling, the product and the difference round by 2^-24
    # of it each
    tol = TOL + (3 * 1.45 * FAR * 2.0 ** -24 if kind == "small weights" else 0.0)
    return ((got.double() - want).abs() <= tol * size).all()


KINDS = ["small queries", "small keys", "small weights", "a small column", "a huge value"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("Hq,Hkv,d,L,b,a", [(32, 2, 128, 440, 220, 137), (40, 4, 64, 700, 689, 1)])
def test_prefill_of_uneven_factors(Hq, Hkv, d, L, b, a, kind):
    gen = torch.Generator(device="cuda").manual_seed(L)
    new = lambda *s: torch.randn(s, generator=gen, device="cuda")
    Q, K, V = new(1, L, Hq, d), new(1, L, Hkv, d), new(1, L, Hkv, d)
    _uneven(kind, Q, K, V)
    shape = sa.StarShape.make("fp32", 1, Hq, Hkv, d, L, b, a, L)
    assert sa.phase1_plan(shape, sa.ANCHOR_FIRST).tile_rows == 32
    O = torch.empty_like(Q)
    print(f"{Hq}/{Hkv} d={d} L={L} {kind}", flush=True)
    sa.phase1(shape, Q, K, V, O, *sa.alloc_cache(shape))
    torch.cuda.synchronize()
    for h in range(Hq):
        k, v = K[0, :, h * Hkv // Hq].double(), V[0, :, h * Hkv // Hq].double()
        for s in range(0, L, b):
            e, n = min(L, s + b), a if s else 0
            lim = n + torch.arange(1, e - s + 1, device="cuda")
            assert _close(O[0, s:e, h], Q[0, s:e, h].double(), torch.cat([k[:n], k[s:e]]), torch.cat([v[:n], v[s:e]]), lim, kind), (h, s)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("Hq,Hkv,d,L,q", [(8, 2, 128, 4003, 60), (4, 2, 64, 30001, 100)])
def test_query_of_uneven_factors(Hq, Hkv, d, L, q, kind):
    gen = torch.Generator(device="cuda").manual_seed(L)
    new = lambda *s: torch.randn(s, generator=gen, device="cuda")
    Q, K, V = new(1, q, Hq, d), new(1, L + q, Hkv, d), new(1, L + q, Hkv, d)
    _uneven(kind, Q, K, V)
    shape = sa.StarShape.make("fp32", 1, Hq, Hkv, d, L, L // 3, 0, L + q)
    assert sa.phase2_plan(shape, L, q).tile_rows == 32
    O = torch.empty_like(Q)
    print(f"{Hq}/{Hkv} d={d} L={L} q={q} {kind}", flush=True)
    sa.phase2(shape, L, Q, K[:, L:].contiguous(), V[:, L:].contiguous(), K.transpose(1, 2).contiguous(), V.transpose(1, 2).contiguous(), O,
              sa.alloc_workspace(shape, q))
    torch.cuda.synchronize()
    for h in range(Hq):
        k, v = K[0, :, h * Hkv // Hq].double(), V[0, :, h * Hkv // Hq].double()
        assert _close(O[0, :, h], Q[0, :, h].double(), k, v, L + torch.arange(1, q + 1, device="cuda"), kind), h


@pytest.mark.parametrize("Hq,Hkv,L,b,a,seed", [(8, 2, 1100, 1100, 0, 4), (8, 2, 2099, 1024, 512, 2), (8, 2, 2099, 1024, 512, 5), (16, 1, 700, 350, 300, 5)])
def test_prefill_of_large_logits(Hq, Hkv, L, b, a, seed):
    """Logits of some 8 times N(0, 1), d = 128: what the sums over 128 products round shows in every weight.  fp32 products stay within
    9.7e-6 of 64 bits over eight seeds each, sums of large products in one chain came to 1.27e-5, in two to 7.4e-6."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    new = lambda *s: torch.randn(s, generator=gen, device="cuda")
    shape = sa.StarShape.make("fp32", 1, Hq, Hkv, 128, L, b, a, L)
    assert sa.phase1_plan(shape, sa.ANCHOR_FIRST).tile_rows == 32
    Q, K, V = new(1, L, Hq, 128) * 8, new(1, L, Hkv, 128), new(1, L, Hkv, 128)
    O, LSE = torch.empty_like(Q), torch.empty((1, Hq, L), device="cuda")
    print(f"{Hq}/{Hkv} L={L} seed={seed}", flush=True)
    sa.phase1(shape, Q, K, V, O, *sa.alloc_cache(shape), LSE_ctx=LSE)
    torch.cuda.synchronize()
    worst, square = 0.0, 0.0
    for h in range(Hq):
        k, v = K[0, :, h * Hkv // Hq].double(), V[0, :, h * Hkv // Hq].double()
        for s in range(0, L, b):
            e, n = min(L, s + b), a if s else 0
            lim = n + torch.arange(1, e - s + 1, device="cuda")
            o, x = _attend(Q[0, s:e, h].double(), torch.cat([k[:n], k[s:e]]), torch.cat([v[:n], v[s:e]]), lim)
            worst = max(worst, (O[0, s:e, h].double() - o).abs().max().item())
            square += (LSE[0, h, s:e].double() - x).pow(2).sum().item()
    assert worst <= TOL
    assert (square / (Hq * L)) ** 0.5 <= 1.39e-6      # the least that fp32 products have over the same seeds
