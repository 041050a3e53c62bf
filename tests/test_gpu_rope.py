"""GPU parity of the entry points that take unrotated projections
(star_attn_rope, star_attn_phase1_rope, star_attn_phase2_rope) against the fp64
oracle, through the C-ABI."""
import numpy as np
import pytest
import torch

import paper_2411_17116_amd as sa
import workloads
from oracle import star_oracle as so
from tests import parity_harness as ph

pytestmark = pytest.mark.gpu


def _storage_close(got: torch.Tensor, want64: np.ndarray, dtype: str):
    """Rotated values as stored: fp32 within 2e-6 relative to the row scale;
    bf16 within one rounding step of the exact value (2^-8 relative, with slack
    for values that sit on a rounding boundary, plus the fp32 arithmetic error of
    the rotation, which dominates where a pair cancels to almost nothing)."""
    g = got.float().cpu().numpy().astype(np.float64)
    err = np.abs(g - want64)
    if dtype == "fp32":
        return float((err / (1.0 + np.abs(want64))).max()) <= 2e-6
    return bool((err <= 2.0 ** -7 * np.abs(want64) + 2e-6).all())


@pytest.mark.parametrize("dtype,d", [("fp32", 64), ("fp32", 128), ("bf16", 128)])
@pytest.mark.parametrize("pos0,theta", [(0, 10000.0), (1_000_000, 500000.0)])
def test_rotation_alone(dtype, d, pos0, theta):
    B, T, H = 2, 300, 3
    tdt = torch.float32 if dtype == "fp32" else torch.bfloat16
    gen = torch.Generator().manual_seed(d + pos0 % 97)
    X = torch.randn((B, T, H, d), generator=gen).to(tdt).cuda()
    shape = sa.StarShape.make(dtype, B, H, H, d, T, T, T, T)
    want = so.rope_rotate(X.float().cpu().numpy(), pos0 + np.arange(T), theta)
    Y = torch.empty_like(X)
    print(f"rope {dtype} d={d} pos0={pos0}", flush=True)
    sa.rope(shape, X, Y, theta, pos0=pos0)
    torch.cuda.synchronize()
    assert _storage_close(Y, want, dtype)
    X2 = X.clone()
    sa.rope(shape, X2, X2, theta, pos0=pos0)               # in place
    torch.cuda.synchronize()
    assert torch.equal(X2, Y)


def _stored(dtype):
    """The storage rounding of the operator's rotated tensors (it hands rotated Q
    back and keeps rotated K in the cache in the configuration's dtype; attention
    is defined on what is stored)."""
    if dtype == "fp32":
        return lambda x: np.asarray(x, np.float32).astype(np.float64)
    return lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(torch.bfloat16).double().numpy()


def _rope_path(cfg, theta, pos0, triples=None, heads=None, decode_steps=None):
    """Whole hot path on unrotated inputs against the oracle."""
    stored = _stored(cfg.dtype)
    inp = workloads.make_inputs(cfg, "cuda")
    run = ph.HipRun(cfg, inp, "cuda")
    tol = ph.TOL[cfg.dtype]
    # the oracle's view: rotate the stored (pre-rotation) values in float64
    Q0 = inp.Q.clone()
    print(f"[{cfg.name}] phase1_rope L={cfg.L} b={cfg.b} a={cfg.a} theta={theta} pos0={pos0}", flush=True)
    sa.phase1_rope(run.shape, theta, inp.Q, inp.K, inp.V, run.O_ctx, run.Kc, run.Vc, pos0=pos0,
                   LSE_ctx=run.LSE_ctx)
    torch.cuda.synchronize()
    if triples is None:
        triples = [(beta, h, p) for beta in range(cfg.B) for h in range(cfg.Hq) for p in range(cfg.L)]
    O_ref, L_ref = so.phase1_rope_rows(ph.LazyTensor(Q0), ph.LazyTensor(inp.K), ph.LazyTensor(inp.V),
                                       triples, cfg.b, cfg.a, theta, pos0=pos0, storage=stored)
    idx = torch.tensor(triples, dtype=torch.long, device="cuda")
    bi, hi, ri = idx.unbind(1)
    eo = np.abs(run.O_ctx[bi, ri, hi].float().cpu().numpy() - O_ref).max()
    el = np.abs(run.LSE_ctx[bi, hi, ri].cpu().numpy() - L_ref).max()
    print(f"   phase 1: max|dO|={eo:.3g} max|dLSE|={el:.3g}", flush=True)
    assert eo <= tol["o"] and el <= tol["lse"]
    # For the record (not asserted): the same rows against the oracle WITHOUT the
    # storage rounding of the rotated q and k, i.e. attention on the exact fp64
    # rotation.  The difference to the figures above is what rounding the rotated
    # tensors to the storage dtype costs -- input quantisation, not compute error.
    sub = triples if len(triples) <= 4096 else triples[:: len(triples) // 4096 + 1]
    O_u, L_u = so.phase1_rope_rows(ph.LazyTensor(Q0), ph.LazyTensor(inp.K), ph.LazyTensor(inp.V),
                                   sub, cfg.b, cfg.a, theta, pos0=pos0, storage=None)
    si = torch.tensor(sub, dtype=torch.long, device="cuda")
    sb, sh, sr = si.unbind(1)
    eo_u = np.abs(run.O_ctx[sb, sr, sh].float().cpu().numpy() - O_u).max()
    el_u = np.abs(run.LSE_ctx[sb, sh, sr].cpu().numpy() - L_u).max()
    print(f"   phase 1 against the unrounded fp64 rotation ({len(sub)} rows, not asserted): "
          f"max|dO|={eo_u:.3g} max|dLSE|={el_u:.3g}", flush=True)
    # Q was rotated in place; the cache holds rotated K and plain V (sampled heads)
    rows = sorted({p for _, _, p in triples})[:64]
    pos = pos0 + np.asarray(rows)
    for beta, g in [(0, 0), (cfg.B - 1, cfg.Hkv - 1)]:
        wantK = so.rope_rotate(inp.K[beta, rows, g].float().cpu().numpy()[:, None, :], pos, theta)[:, 0]
        assert _storage_close(run.Kc[beta, g, rows], wantK, cfg.dtype)
        assert torch.equal(run.Vc[beta, g, :cfg.L], inp.V[beta, :, g])
    wantQ = so.rope_rotate(Q0[0, rows].float().cpu().numpy(), pos, theta)
    assert _storage_close(inp.Q[0, rows], wantQ, cfg.dtype)

    # phase 2: the oracle rotates every appended tensor at its own positions and
    # then runs its ordinary definition on the rotated values
    heads = list(range(cfg.Hq)) if heads is None else heads
    def rot(t, start):
        n = t.shape[1]
        return torch.from_numpy(stored(so.rope_rotate(t.float().cpu().numpy(),
                                                      pos0 + start + np.arange(n), theta))).float()

    class RotatedContext:
        """Context keys rotated on demand (large contexts are not rotated whole)."""
        def __init__(self, K):
            self.K = K
            self.shape = K.shape
        def head(self, beta, g):
            return rot(self.K[beta:beta + 1, :, g:g + 1], 0)[0, :, 0]

    Qq0, Qd0 = inp.Qq.clone(), inp.Qd.clone()
    print("   phase 2: query call", flush=True)
    cl = run.cache_len
    O = torch.empty_like(inp.Qq)
    P = cfg.n_blocks + 1
    Op = torch.empty((cfg.B, P, cfg.Hq, cfg.lq, cfg.d), dtype=torch.float32, device="cuda")
    Lp = torch.empty((cfg.B, P, cfg.Hq, cfg.lq), dtype=torch.float32, device="cuda")
    sa.phase2_rope(run.shape, theta, cl, inp.Qq, inp.Kq, inp.Vq, run.Kc, run.Vc, O, run.ws, pos0=pos0,
                   O_part=Op, LSE_part=Lp)
    torch.cuda.synchronize()
    Kq_r, Kd_r = rot(inp.Kq, cfg.L), rot(inp.Kd, cfg.L + cfg.lq)
    Qq_r, Qd_r = rot(Qq0, cfg.L), rot(Qd0, cfg.L + cfg.lq)

    class Cache:
        """[B, Hkv, rows, d] view of rotated context + rotated appended keys."""
        def __init__(self, parts_fn, rows):
            self.parts_fn = parts_fn
            self.shape = (cfg.B, cfg.Hkv, rows, cfg.d)
        def __getitem__(self, idx):
            beta, g, sl = idx
            return self.parts_fn(beta, g)[sl].numpy()

    ctx = RotatedContext(inp.K)
    memo = {}
    def kparts(beta, g):
        if (beta, g) not in memo:
            memo.clear()
            memo[(beta, g)] = torch.cat([ctx.head(beta, g), Kq_r[beta, :, g], Kd_r[beta, :, g]], dim=0)
        return memo[(beta, g)]
    def vparts(beta, g):
        return torch.cat([inp.V[beta, :, g], inp.Vq[beta, :, g], inp.Vd[beta, :, g]], dim=0).float().cpu()
    total_rows = cfg.L + cfg.lq + cfg.nd
    Kc_o, Vc_o = Cache(kparts, total_rows), Cache(vparts, total_rows)

    ref = so.phase2_rows(Qq_r.numpy(), Kc_o, Vc_o, cfg.L, cfg.b, cl, heads=heads)
    hs = torch.tensor(heads, device="cuda")
    eo = np.abs(O[:, :, hs].float().cpu().numpy() - ref["O"]).max()
    exists = ~np.isneginf(ref["LSE_part"])
    ep = np.abs(Op[:, :, hs].cpu().numpy()[exists] - ref["O_part"][exists]).max()
    elp = np.abs(Lp[:, :, hs].cpu().numpy()[exists] - ref["LSE_part"][exists]).max()
    print(f"   query: max|dO|={eo:.3g} max|dO_part|={ep:.3g} max|dLSE_part|={elp:.3g}", flush=True)
    assert eo <= tol["o"] and ep <= tol["o"] and elp <= tol["lse"]
    run.cache_len += cfg.lq

    steps = list(range(cfg.nd)) if decode_steps is None else decode_steps
    outs = []
    for t in range(cfg.nd):
        O1 = torch.empty_like(inp.Qd[:, :1])
        q1 = inp.Qd[:, t:t + 1].contiguous()
        sa.phase2_rope(run.shape, theta, run.cache_len, q1, inp.Kd[:, t:t + 1].contiguous(),
                       inp.Vd[:, t:t + 1].contiguous(), run.Kc, run.Vc, O1, run.ws, pos0=pos0)
        run.cache_len += 1
        outs.append(O1)
    torch.cuda.synchronize()
    O_dec = torch.cat(outs, dim=1)
    ref = so.phase2_rows(Qd_r.numpy(), Kc_o, Vc_o, cfg.L, cfg.b, cfg.L + cfg.lq, heads=heads, rows=steps)
    got = O_dec[:, torch.tensor(steps, device="cuda")][:, :, hs].float().cpu().numpy()
    eo = np.abs(got - ref["O"]).max()
    print(f"   decode steps {steps}: max|dO|={eo:.3g}", flush=True)
    assert eo <= tol["o"]
    # appended keys are rotated in the cache, values are plain
    tail = slice(cfg.L, cfg.L + cfg.lq + cfg.nd)
    wantK = torch.cat([Kq_r[0, :, 0], Kd_r[0, :, 0]], dim=0).numpy().astype(np.float64)
    assert _storage_close(run.Kc[0, 0, tail], wantK, cfg.dtype)
    assert torch.equal(run.Vc[0, 0, tail], torch.cat([inp.Vq[0, :, 0], inp.Vd[0, :, 0]], dim=0))


@pytest.mark.parametrize("L,b,a,pos0", [(1000, 256, 256, 0), (777, 200, 37, 123456)])
def test_fp32_unrotated_inputs_every_row(L, b, a, pos0):
    cfg = workloads.StarConfig("f32rope", "fp32", 2, 4, 2, 64, L, b, a, 9, 3, seed=L)
    _rope_path(cfg, 10000.0, pos0)


@pytest.mark.parametrize("Hq,Hkv,L,b,a,lq,nd,pos0", [
    (4, 1, 2048, 512, 512, 40, 3, 0),
    (8, 2, 1500, 400, 100, 130, 2, 900_000),
    (2, 2, 1024, 256, 0, 3, 4, 7),          # q_len 3: decode-sized call with several new tokens
])
def test_bf16_unrotated_inputs_every_row(Hq, Hkv, L, b, a, lq, nd, pos0):
    cfg = workloads.StarConfig("bf16rope", "bf16", 2, Hq, Hkv, 128, L, b, a, lq, nd,
                               seed=Hq + L, n_planted=4)
    _rope_path(cfg, 500000.0, pos0)


def test_config2_shape_unrotated_inputs_sampled():
    cfg = workloads.CONFIGS["C2"]
    inp = workloads.make_inputs(cfg, "cuda")
    triples = workloads.phase1_sample(cfg, inp.planted_ctx, n_random=64)
    del inp
    _rope_path(cfg, 500000.0, 0, triples=triples, heads=[0, 3, 31], decode_steps=[0, cfg.nd - 1])


@pytest.mark.parametrize("dtype,d,B,T,H", [
    ("bf16", 128, 2, 513, 3),        # few rows, few tokens
    ("bf16", 128, 1, 4099, 2),       # few rows, many tokens, not a multiple of a workgroup's
    ("bf16", 128, 3, 1367, 7),       # tokens of two sequences in one workgroup
    ("bf16", 128, 1, 1030, 33),      # many rows
    ("fp32", 64, 2, 2051, 1),
    ("fp32", 128, 1, 1027, 9),
])
def test_rotation_workgroup_shapes(dtype, d, B, T, H):
    """Every tokens-per-workgroup set-up of the rotation, ragged."""
    gen = torch.Generator().manual_seed(T + H)
    X = torch.randn((B, T, H, d), generator=gen).to(torch.float32 if dtype == "fp32" else torch.bfloat16).cuda()
    shape = sa.StarShape.make(dtype, B, H, H, d, T, T, T, T)
    want = so.rope_rotate(X.float().cpu().numpy(), 77 + np.arange(T), 500000.0)
    sa.rope(shape, X, X, 500000.0, pos0=77)
    torch.cuda.synchronize()
    assert _storage_close(X, want, dtype)


@pytest.mark.parametrize("B,Hq,Hkv,L,q", [
    (1, 32, 8, 1000, 1),
    (1, 16, 16, 5, 1),          # one split of one step
    (1, 16, 16, 31, 1),         # the new token ends a 32-key step
    (1, 16, 16, 32, 1),         # and begins one
    (2, 16, 16, 61, 8),         # eight tokens in two steps, of two splits
    (1, 12, 4, 3000, 5),        # 15 of 16 rows
    (1, 16, 1, 700, 1),
    (5, 64, 32, 500, 2),        # few splits of many rows: merged by rows
    (3, 32, 16, 90000, 1),      # beyond the last-level cache
    (1, 16, 16, 600, 9),        # more tokens than the decode kernel turns
    (1, 32, 8, 8158, 4),        # four wavefronts to a split, the tokens in steps of two
    (1, 32, 8, 8190, 4),        # one again
])
def test_decode_on_unrotated_projections_is_decode_on_rotated_ones(B, Hq, Hkv, L, q):
    """A decode call that turns its tokens on the way gives the bits of star_attn_rope followed by
    star_attn_phase2: outputs, queries in place and appended rows."""
    gen = torch.Generator(device="cuda").manual_seed(L + q)
    new = lambda *s: torch.randn(s, generator=gen, device="cuda", dtype=torch.bfloat16)
    shape = sa.StarShape.make("bf16", B, Hq, Hkv, 128, L, max(1, L // 4), 0, L + q)
    assert sa.phase2_plan(shape, L, q).decode == 1
    Kc, Vc = new(B, Hkv, L + q, 128), new(B, Hkv, L + q, 128)
    Q, K, V = new(B, q, Hq, 128), new(B, q, Hkv, 128), new(B, q, Hkv, 128)
    ws = sa.alloc_workspace(shape, q)
    pos0, theta = 54321, 500000.0
    Qr, Kr, Kc2, Vc2, O, O2 = Q.clone(), torch.empty_like(K), Kc.clone(), Vc.clone(), torch.empty_like(Q), torch.empty_like(Q)
    sa.rope(shape, Qr, Qr, theta, pos0=pos0 + L)
    sa.rope(shape, K, Kr, theta, pos0=pos0 + L)
    sa.phase2(shape, L, Qr, Kr, V, Kc2, Vc2, O2, ws)
    print(f"[{B} {Hq}/{Hkv} L={L} q={q}]", flush=True)
    sa.phase2_rope(shape, theta, L, Q, K, V, Kc, Vc, O, ws, pos0=pos0)
    torch.cuda.synchronize()
    assert torch.equal(O, O2)
    assert torch.equal(Q, Qr)
    assert torch.equal(Kc, Kc2) and torch.equal(Vc, Vc2)


@pytest.mark.parametrize("B,Hq,Hkv,L,q", [
    (1, 16, 1, 700, 1),
    (1, 2, 1, 61, 8),           # eight tokens in two 32-key steps
    (1, 4, 1, 9000, 4),         # four wavefronts to a split
    (5, 64, 32, 500, 2),        # merged by rows
])
def test_decode_on_unrotated_projections_in_shared_buffers(B, Hq, Hkv, L, q):
    """O stored over Qq, and new keys and values that are their own cache rows already, give the bits of buffers
    of their own."""
    gen = torch.Generator(device="cuda").manual_seed(L + q)
    new = lambda *s: torch.randn(s, generator=gen, device="cuda", dtype=torch.bfloat16)
    shape = sa.StarShape.make("bf16", B, Hq, Hkv, 128, L, max(1, L // 4), 0, L + q)
    assert sa.phase2_plan(shape, L, q).decode == 1
    Kc, Vc = new(B, Hkv, L + q, 128), new(B, Hkv, L + q, 128)
    Q, K, V = new(B, q, Hq, 128), new(B, q, Hkv, 128), new(B, q, Hkv, 128)
    ws, theta = sa.alloc_workspace(shape, q), 500000.0
    Q1, Kc1, Vc1, O = Q.clone(), Kc.clone(), Vc.clone(), torch.empty_like(Q)
    sa.phase2_rope(shape, theta, L, Q1, K, V, Kc1, Vc1, O, ws)
    print(f"[{B} {Hq}/{Hkv} L={L} q={q}]", flush=True)
    Q2, Kc2, Vc2 = Q.clone(), Kc.clone(), Vc.clone()
    sa.phase2_rope(shape, theta, L, Q2, K, V, Kc2, Vc2, Q2, ws)
    torch.cuda.synchronize()
    assert torch.equal(Q2, O) and torch.equal(Kc2, Kc1) and torch.equal(Vc2, Vc1)
    if B * Hkv > 1:                       # elsewhere a call's tokens do not lie as the cache's rows do
        return
    Q3, Kc3, Vc3 = Q.clone(), Kc.clone(), Vc.clone()
    Kc3[0, 0, L:], Vc3[0, 0, L:] = K[0, :, 0], V[0, :, 0]
    O3 = torch.empty_like(Q)
    sa.phase2_rope(shape, theta, L, Q3, Kc3[0, 0, L:].view(1, q, 1, 128), Vc3[0, 0, L:].view(1, q, 1, 128), Kc3, Vc3, O3, ws)
    torch.cuda.synchronize()
    assert torch.equal(O3, O) and torch.equal(Q3, Q1) and torch.equal(Kc3, Kc1) and torch.equal(Vc3, Vc1)


@pytest.mark.parametrize("rotated", [False, True])
@pytest.mark.parametrize("B,Hq,Hkv,d,L,q,squeezed", [
    (1, 4, 2, 64, 300, 3, False),         # one split, few row tiles: four workgroups would share one
    (1, 64, 64, 64, 200, 1, False),       # 64 tiles
    (1, 6, 2, 128, 250, 5, False),
    (2, 33, 33, 128, 200, 5, False),      # 66 tiles: two
    (1, 40, 8, 64, 400, 50, False),       # 128 tiles
    (1, 2, 1, 64, 3000, 9, True),         # a workspace that holds one split
    (3, 30, 30, 128, 2000, 2, True),
])
def test_fp32_results_over_their_queries(B, Hq, Hkv, d, L, q, squeezed, rotated):
    """fp32 calls of one split: O stored over Qq (A, where its rows lie as the queries' do) gives the bits of buffers of
    their own.  Each workgroup of a tile reads all of its query rows."""
    gen = torch.Generator(device="cuda").manual_seed(L + q)
    new = lambda *s: torch.randn(s, generator=gen, device="cuda")
    shape = sa.StarShape.make("fp32", B, Hq, Hkv, d, L, max(1, L // 4), 0, L + q)
    one = -(-B * Hq * q * (d + 1) * 4 // 256) * 256
    ws = torch.empty(one, dtype=torch.uint8, device="cuda") if squeezed else sa.alloc_workspace(shape, q)
    assert squeezed or sa.phase2_plan(shape, L, q).n_splits == 1
    Kc, Vc = new(B, Hkv, L + q, d), new(B, Hkv, L + q, d)
    Q, K, V = new(B, q, Hq, d), new(B, q, Hkv, d), new(B, q, Hkv, d)
    print(f"[{B} {Hq}/{Hkv} d={d} L={L} q={q}]", flush=True)

    def call(Qx, Kx, Vx, Ox):
        if rotated:
            sa.phase2_rope(shape, 500000.0, L, Qx, K, V, Kx, Vx, Ox, ws)
        else:
            sa.phase2(shape, L, Qx, K, V, Kx, Vx, Ox, ws)
    Q1, K1, V1, O = Q.clone(), Kc.clone(), Vc.clone(), torch.empty_like(Q)
    call(Q1, K1, V1, O)
    Q2, K2, V2 = Q.clone(), Kc.clone(), Vc.clone()
    call(Q2, K2, V2, Q2)
    torch.cuda.synchronize()
    assert torch.equal(Q2, O) and torch.equal(K2, K1) and torch.equal(V2, V1)
    if q > 1 or rotated:
        return
    A, LSE, lse = torch.empty((B, Hq, 1, d), device="cuda"), torch.empty((B, Hq, 1), device="cuda"), torch.empty((B, Hq, 1), device="cuda")
    sa.phase2_partial(shape, L, Q, Kc.clone(), Vc.clone(), A, LSE, ws, Kq=K, Vq=V)
    Q3 = Q.clone()
    sa.phase2_partial(shape, L, Q3, Kc.clone(), Vc.clone(), Q3.view(B, Hq, 1, d), lse, ws, Kq=K, Vq=V)
    torch.cuda.synchronize()
    assert torch.equal(Q3.view_as(A), A) and torch.equal(lse, LSE)


@pytest.mark.parametrize("rotated", [False, True])
@pytest.mark.parametrize("B,Hq,Hkv,d,L,b,a", [
    (1, 1, 1, 64, 1024, 256, 256),        # 64 tiles: four workgroups would share one
    (1, 4, 2, 128, 300, 100, 33),
    (1, 2, 2, 128, 600, 150, 75),         # 80 tiles: two
    (2, 2, 1, 64, 900, 900, 0),           # 114 tiles, a range of more than 512 keys
    (1, 8, 2, 128, 1300, 300, 200),       # 32-row tiles
])
def test_fp32_context_results_over_their_queries(B, Hq, Hkv, d, L, b, a, rotated):
    gen = torch.Generator(device="cuda").manual_seed(L)
    new = lambda *s: torch.randn(s, generator=gen, device="cuda")
    shape = sa.StarShape.make("fp32", B, Hq, Hkv, d, L, b, a, L)
    Q, K, V = new(B, L, Hq, d), new(B, L, Hkv, d), new(B, L, Hkv, d)
    print(f"[{B} {Hq}/{Hkv} d={d} L={L}]", flush=True)

    def call(Qx, Ox):
        caches, lse = sa.alloc_cache(shape), torch.empty((B, Hq, L), device="cuda")
        if rotated:
            sa.phase1_rope(shape, 500000.0, Qx, K, V, Ox, *caches, LSE_ctx=lse)
        else:
            sa.phase1(shape, Qx, K, V, Ox, *caches, LSE_ctx=lse)
        return [Ox, lse, *caches]
    want, Q2 = call(Q.clone(), torch.empty_like(Q)), Q.clone()
    got = call(Q2, Q2)
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(got, want))
