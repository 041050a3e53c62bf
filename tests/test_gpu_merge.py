"""star_attn_merge (the kernels behind every call of one part) over numbers of pairs and rows
at the edges of its set-ups, against Eq. 3-4 in float64: pieces of a row, whole rows, several
rows per workgroup; empty pairs whose slabs hold NaN; rows that saw nothing at all."""
import numpy as np
import pytest
import torch

import paper_2411_17116_amd as sa

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("fp32", 64), ("fp32", 128)])
@pytest.mark.parametrize("B,H,q,n_parts", [
    (1, 1, 1, 1), (1, 3, 1, 7), (2, 4, 8, 8), (1, 8, 8, 9), (3, 5, 1, 64), (1, 4, 1, 65), (1, 2, 1, 128),
    (1, 2, 2, 129), (1, 1, 1, 700), (2, 8, 16, 33), (1, 16, 17, 64), (1, 32, 9, 66),
])
def test_merge_against_float64(dtype, d, B, H, q, n_parts):
    gen = torch.Generator().manual_seed(n_parts * 100 + q)
    A = torch.randn((n_parts, B, H, q, d), generator=gen)
    LSE = 3.0 * torch.randn((n_parts, B, H, q), generator=gen) + 9.0
    empty = torch.rand((n_parts, B, H, q), generator=gen) < 0.2
    empty[:, 0, 0, 0] = True                                  # a row without any key
    LSE[empty] = -float("inf")
    w = torch.softmax(LSE.double(), dim=0).nan_to_num(0.0)
    want = (w[..., None] * A.double()).sum(dim=0)
    want_lse = torch.logsumexp(LSE.double(), dim=0)
    A[empty] = float("nan")                                   # never read for its value
    shape = sa.StarShape.make(dtype, B, H, H, d, 64, 64, 64, 64 + q)
    O = torch.empty((B, q, H, d), dtype=torch.float32 if dtype == "fp32" else torch.bfloat16, device="cuda")
    Am, Lm = torch.empty((B, H, q, d), device="cuda"), torch.empty((B, H, q), device="cuda")
    print(f"merge {dtype} d={d} B={B} H={H} q={q} parts={n_parts}", flush=True)
    sa.merge(shape, A.cuda(), LSE.cuda(), O=O, A=Am, LSE=Lm)
    torch.cuda.synchronize()
    # fp32 sums of up to 700 weighted values of size 1, weights that sum to 1: 700 roundings of
    # at most 2^-24 each in the worst order, far fewer in the tree: 2e-6 is eight of them
    assert (Am.cpu().double() - want).abs().max().item() <= 2e-6
    seen = torch.isfinite(want_lse)
    # the log-sum-exps are near 20 (an fp32 step there is 1.9e-6): two steps
    assert not seen.any() or (Lm.cpu().double() - want_lse)[seen].abs().max().item() <= 4e-6
    assert torch.isneginf(Lm.cpu()[~seen]).all()
    got = O.float().cpu().double().transpose(1, 2)
    step = 2.0 ** -24 if dtype == "fp32" else 2.0 ** -8
    assert ((got - want).abs() <= want.abs() * step + 2e-6).all()


def _fp32_merge_rms(A, LSE, want):
    """rms error of Eq. 3-4 in fp32 where every step is rounded once: weights against the common
    maximum, sums in index order by fused multiply-adds, one division."""
    m = LSE.max(axis=0)
    w = np.exp((LSE - m).astype(np.float64)).astype(np.float32)
    total = np.zeros_like(m)
    acc = np.zeros_like(A[0])
    for k in range(len(A)):
        total += w[k]
        acc = (acc.astype(np.float64) + A[k].astype(np.float64) * w[k][..., None]).astype(np.float32)
    return np.sqrt(np.mean(((acc / total[..., None]).astype(np.float64) - want) ** 2))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n_parts", [2, 3, 4, 8])
def test_fp32_merge_of_few_pairs_is_as_exact_as_its_roundings(n_parts, d):
    H, q = 16, 160
    gen = torch.Generator().manual_seed(n_parts)
    A = torch.randn((n_parts, 1, H, q, d), generator=gen)
    LSE = 2.0 * torch.randn((n_parts, 1, H, q), generator=gen) + 9.0
    want = (torch.softmax(LSE.double(), dim=0)[..., None] * A.double()).sum(dim=0).numpy()
    model = _fp32_merge_rms(A.numpy(), LSE.numpy(), want)
    got = torch.empty((1, H, q, d), device="cuda")
    sa.merge(sa.StarShape.make("fp32", 1, H, H, d, 64, 64, 64, 64 + q), A.cuda(), LSE.cuda(), A=got)
    rms = np.sqrt(np.mean((got.cpu().numpy().astype(np.float64) - want) ** 2))
    print(f"{n_parts} pairs, d={d}: rms error {rms:.3e}, every step rounded once {model:.3e}", flush=True)
    # 2560 independent rows give the rms to about 1 %; an exponential that is off by an ulp now
    # and then adds less than another.  A weight from a rounded product and a rounded reciprocal
    # would add 6 (eight pairs) to 11 % (two)
    assert rms <= 1.03 * model


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,q,n_parts,slab", [(1, 1, 2, 0), (8, 1, 9, 0), (4, 3, 64, 63), (2, 1, 130, 7), (8, 1, 500, 0),
                                              (8, 40, 20, 1), (4, 64, 70, 0), (16, 8, 4, 2)])
def test_merge_into_one_of_its_own_slabs(H, q, n_parts, slab, d):
    """Merging in stages: the pair may replace one of the gathered ones (few rows of many pairs
    are spread over workgroups, which all read the row's log-sum-exps)."""
    gen = torch.Generator(device="cuda").manual_seed(n_parts)
    A = torch.randn((n_parts, 1, H, q, d), generator=gen, device="cuda")
    LSE = 3.0 * torch.randn((n_parts, 1, H, q), generator=gen, device="cuda") + 9.0
    shape = sa.StarShape.make("fp32", 1, H, H, d, 64, 64, 64, 64 + q)
    want_A, want_L = torch.empty_like(A[0]), torch.empty_like(LSE[0])
    sa.merge(shape, A, LSE, A=want_A, LSE=want_L)
    print(f"d={d} H={H} q={q} parts={n_parts} slab={slab}", flush=True)
    for _ in range(5):
        A2, L2 = A.clone(), LSE.clone()
        sa.merge(shape, A2, L2, A=A2[slab], LSE=L2[slab])
        torch.cuda.synchronize()
        # a row may be cut in another way than out of place: other groups of splits, so each
        # result within 2e-6 (4e-6 for values near 20) of the exact one
        assert (A2[slab] - want_A).abs().max().item() <= 4e-6
        assert (L2[slab] - want_L).abs().max().item() <= 8e-6
