"""Calls whose launches exceed the 2^32 work-items a grid can hold (very many short blocks,
sequences or tokens): every part of the result must be there, not what 32 bits keep of the
grid.  The inputs are chosen so that the whole result, or samples of both ends and of the
middle, can be checked without an oracle pass over tens of gigabytes."""
import pytest
import torch

import paper_2411_17116_amd as sa

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def give_memory_back():
    yield
    torch.cuda.empty_cache()


def _normal(*size, dtype):
    return torch.empty(size, dtype=dtype, device="cuda").normal_()


def _prefill_of_one_token_blocks(dtype, d, L, H):
    """A block of one token without an anchor sees itself: O = V, LSE = scale q.k."""
    Q, K, V = (_normal(1, L, H, d, dtype=dtype) for _ in range(3))
    shape = sa.StarShape.make(dtype, 1, H, H, d, L, 1, 0, L)
    Kc, Vc = sa.alloc_cache(shape)
    O = torch.zeros_like(Q)
    n = sa.phase1_workspace_bytes(shape, sa.ANCHOR_FIRST)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda") if n else None
    print(f"{dtype} L={L} heads={H}", flush=True)
    sa.phase1(shape, Q, K, V, O, Kc, Vc, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(O, V)
    for h in range(H):
        assert torch.equal(Kc[0, h], K[0, :, h]) and torch.equal(Vc[0, h], V[0, :, h])


def test_fp32_prefill():
    # 8 x 8389608 row tiles of one wavefront: 2^32 work-items and 8000 workgroups more
    _prefill_of_one_token_blocks(torch.float32, 64, 8389608, 8)


def test_fp32_decode_step():
    """65535 sequences of 129 heads on four cached tokens: 8454015 workgroups of 512."""
    B, H, d, L = 65535, 129, 64, 4
    shape = sa.StarShape.make("fp32", B, H, H, d, L, L, 0, L + 1)
    Kc, Vc = _normal(B, H, L + 1, d, dtype=torch.float32), _normal(B, H, L + 1, d, dtype=torch.float32)
    q, k, v = (_normal(B, 1, H, d, dtype=torch.float32) for _ in range(3))
    O = torch.zeros_like(q)
    print("fp32 decode", flush=True)
    sa.phase2(shape, L, q, k, v, Kc, Vc, O, sa.alloc_workspace(shape, 1))
    torch.cuda.synchronize()
    assert torch.equal(Kc[:, :, L], k[:, 0]) and torch.equal(Vc[:, :, L], v[:, 0])
    for s in range(0, B, 4096):
        s = slice(s, s + 4096)
        w = torch.softmax((Kc[s].double() * q[s, 0, :, None].double()).sum(-1) * d ** -0.5, dim=2)
        want = (w[..., None] * Vc[s].double()).sum(2)
        assert (O[s, 0].double() - want).abs().max().item() <= 1e-5


def test_bf16_prefill():
    # the plain grid: 8 x 2098000 items of four wavefronts
    _prefill_of_one_token_blocks(torch.bfloat16, 128, 2098000, 8)


def test_rope():
    """Tokens of 16 heads are rotated by a workgroup each, here 2^24 + 1000 of them in place;
    windows of the result against the rotation of the window alone."""
    T, H = (1 << 24) + 1000, 16
    X = torch.empty((1, T, H, 128), dtype=torch.bfloat16, device="cuda")
    for t in range(0, T, 1 << 20):
        X[:, t:t + (1 << 20)].normal_()
    windows = [(0, 64), (1000, 64), (T // 2 - 7, 64), ((1 << 24) - 32, 64), (T - 64, 64)]
    before = [X[:, s:s + n].clone() for s, n in windows]
    print("rope", flush=True)
    sa.rope(sa.StarShape.make("bf16", 1, H, H, 128, T, T, 0, T), X, X, 500000.0)
    for (s, n), x in zip(windows, before):
        y = torch.empty_like(x)
        sa.rope(sa.StarShape.make("bf16", 1, H, H, 128, n, n, 0, n), x, y, 500000.0, pos0=s)
        torch.cuda.synchronize()
        assert torch.equal(X[:, s:s + n], y), s


def test_merge_of_single_pairs():
    """2^27 and some rows of one pair each, 32 lanes to a row: the output is the pair's own."""
    H, q, d = 129, 1 << 20, 128
    A = torch.empty((1, 1, H, q, d), device="cuda")
    for h in range(H):
        A[0, 0, h].normal_()
    LSE = torch.zeros((1, 1, H, q), device="cuda")
    O = torch.zeros((1, q, H, d), dtype=torch.bfloat16, device="cuda")
    print("merge", flush=True)
    sa.merge(sa.StarShape.make("bf16", 1, H, H, d, q, q, 0, q), A, LSE, O=O)
    torch.cuda.synchronize()
    for h in range(H):
        assert torch.equal(O[0, :, h], A[0, 0, h].to(torch.bfloat16)), h
