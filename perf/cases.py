"""The work a user of this library has it do, as cases that can be timed and compared.

A case is one of three kinds:
  "phase1"  context encoding (star_attn_phase1 / _rope / _anchor), prefill;
  "phase2"  a query call of `lq` tokens (none if 0) followed by `nd` single-token decode
            steps over a context of L cached tokens (star_attn_phase2 / _rope);
  "host"    one step of the query host when the cache is spread over `hosts` devices:
            its own share by star_attn_phase2_partial, then star_attn_merge of the
            gathered pairs.
Inputs are N(0, 1) with a few query rows per head that point at one key (gamma 1.5), as a
retrieval prompt does.  Calls use what a serving program keeps: caches and a workspace.
"""
import math

import torch

import paper_2411_17116_amd as sa

GAMMA = 1.5
THETA = 500000.0


def _p1(name, dtype, B, Hq, Hkv, d, L, b, a, mode="first", rope=False, lse=False):
    return {"name": name, "kind": "phase1", "dtype": dtype, "B": B, "Hq": Hq, "Hkv": Hkv, "d": d,
            "L": L, "b": b, "a": a, "mode": mode, "rope": rope, "lse": lse}


def _p2(name, dtype, B, Hq, Hkv, d, L, b, lq, nd, rope=False):
    return {"name": name, "kind": "phase2", "dtype": dtype, "B": B, "Hq": Hq, "Hkv": Hkv, "d": d,
            "L": L, "b": b, "lq": lq, "nd": nd, "rope": rope}


def _host(name, dtype, B, Hq, Hkv, d, L, b, q, hosts):
    return {"name": name, "kind": "host", "dtype": dtype, "B": B, "Hq": Hq, "Hkv": Hkv, "d": d,
            "L": L, "b": b, "q": q, "hosts": hosts}


def listed():
    return [
        # prefill of a 128K prompt on the Llama-3.1-8B shape: the headline configuration
        _p1("prefill-8b-128k", "bf16", 1, 32, 8, 128, 131072, 16384, 16384),
        # prefill of an ordinary 32K prompt, log-sum-exps kept
        _p1("prefill-8b-32k", "bf16", 1, 32, 8, 128, 32768, 4096, 4096, lse=True),
        # a context host's run of blocks on the 70B shape: reduced anchor, ragged, two sequences
        _p1("prefill-70b-host", "bf16", 2, 64, 8, 128, 12289, 4096, 1024, mode="all_blocks"),
        # a short prompt of odd length whose projections arrive unrotated
        _p1("prefill-8b-8k-rope", "bf16", 1, 32, 8, 128, 8191, 2048, 2048, rope=True),
        # the fp32 reference configuration, one head: the smallest prefill
        _p1("prefill-f32-1k", "fp32", 1, 1, 1, 64, 1024, 256, 256),
        # fp32 prefill with grouped heads, reduced anchor and a ragged last block
        _p1("prefill-f32-gqa", "fp32", 1, 8, 2, 128, 4099, 1024, 512, lse=True),
        # query encoding against a 128K cache
        _p2("query-8b-128k", "bf16", 1, 32, 8, 128, 131072, 16384, 256, 0),
        # a short query on a cache spread over eight hosts of 16K tokens each
        _host("query-8b-host", "bf16", 1, 32, 8, 128, 16384, 16384, 21, 8),
        # one decode step against a 128K cache: the headline decode
        _p2("decode-8b-128k", "bf16", 1, 32, 8, 128, 131072, 16384, 0, 1),
        # one decode step of a short conversation, projections unrotated: latency
        _p2("decode-8b-8k-rope", "bf16", 1, 32, 8, 128, 8191, 2048, 0, 1, rope=True),
        # one decode step of a batch of four on the 70B shape
        _p2("decode-70b-b4-32k", "bf16", 4, 64, 8, 128, 32768, 8192, 0, 1),
        # the fp32 reference configuration's phase 2: 32 query tokens, eight decode steps
        _p2("serve-f32-1k", "fp32", 1, 1, 1, 64, 1024, 256, 32, 8),
    ]


def _logu(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_HEADS_BF16 = [(32, 8), (32, 8), (64, 8), (8, 2), (16, 16), (12, 4)]
_HEADS_F32 = [(1, 1), (4, 2), (8, 2)]


def draw(rng):
    what = rng.choice(["p1", "p1", "p1f", "query", "decode", "decode", "host", "p2f"])
    while True:
        if what == "p1":
            Hq, Hkv = rng.choice(_HEADS_BF16)
            B, L = rng.choice([1, 1, 2, 4]), _logu(rng, 256, 131072)
            b = max(32, int(L / rng.choice([1, 2, 4, 4, 8, 8, 16])) + rng.choice([0, 0, 1, -3]))
            a = rng.choice([b, b, b // 4, b // 2, 0])
            mode = rng.choice(["first", "first", "all_blocks"])
            c = _p1("", "bf16", B, Hq, Hkv, 128, L, b, a, mode, mode == "first" and rng.random() < 0.4,
                    rng.random() < 0.4)
            fits = work(c)["flops"] <= 4.0e13 and B * L <= 131072
        elif what == "p1f":
            Hq, Hkv = rng.choice(_HEADS_F32)
            B, L = rng.choice([1, 1, 2]), _logu(rng, 128, 8192)
            b = max(16, int(L / rng.choice([1, 2, 4, 4, 8])) + rng.choice([0, 0, 1, -3]))
            a = rng.choice([b, b, b // 4, b // 2, 0])
            mode = rng.choice(["first", "first", "all_blocks"])
            c = _p1("", "fp32", B, Hq, Hkv, rng.choice([64, 128]), L, b, a, mode,
                    mode == "first" and rng.random() < 0.3, rng.random() < 0.5)
            fits = work(c)["flops"] <= 4.0e10
        elif what in ("query", "decode"):
            Hq, Hkv = rng.choice(_HEADS_BF16)
            B, L = rng.choice([1, 1, 2, 4]), _logu(rng, 512, 524288)
            b = max(256, int(L / rng.choice([4, 4, 8, 16])))
            lq, nd = (_logu(rng, 2, 300), rng.choice([0, 0, 1])) if what == "query" else (0, rng.choice([1, 1, 4]))
            c = _p2("", "bf16", B, Hq, Hkv, 128, L, b, lq, nd, rng.random() < 0.3)
            fits = B * L * Hkv <= 131072 * 8 and work(c)["flops"] <= 2.0e12
        elif what == "host":
            Hq, Hkv = rng.choice(_HEADS_BF16)
            L = _logu(rng, 512, 65536)
            c = _host("", "bf16", rng.choice([1, 1, 2]), Hq, Hkv, 128, L, max(256, L // rng.choice([1, 2, 4])),
                      rng.choice([1, 1, _logu(rng, 2, 128)]), rng.choice([2, 4, 8, 11]))
            fits = True
        else:
            Hq, Hkv = rng.choice(_HEADS_F32)
            L = _logu(rng, 128, 16384)
            c = _p2("", "fp32", rng.choice([1, 1, 2]), Hq, Hkv, rng.choice([64, 128]), L,
                    max(64, int(L / rng.choice([1, 4, 8]))), rng.choice([0, _logu(rng, 2, 100)]),
                    rng.choice([1, 2, 8]), rng.random() < 0.3)
            fits = work(c)["flops"] <= 2.0e10
        if fits:
            del c["name"]
            return c


# ------------------------------------------------------------------ inputs


def _dt(case):
    return torch.float32 if case["dtype"] == "fp32" else torch.bfloat16


def _gen(case, seed, device="cuda"):
    g = torch.Generator(device=device)
    g.manual_seed(int(seed))
    return g


def _normal(shape, gen, dtype):
    return torch.randn(shape, generator=gen, device="cuda", dtype=dtype)


def _point(Q, K, rows, keys, G):
    """Rows `rows` of every head of Q [B, T, Hq, d] become gamma times keys `keys` of K [B, S, Hkv, d]."""
    Q[:, rows] = (GAMMA * K[:, keys].float()).to(Q.dtype).repeat_interleave(G, dim=2)


def _inputs(case, seed):
    """The tensors of a case, the same for every implementation."""
    gen, dt = _gen(case, seed), _dt(case)
    B, Hq, Hkv, d, L, b = (case[k] for k in ("B", "Hq", "Hkv", "d", "L", "b"))
    G = Hq // Hkv
    host = torch.Generator().manual_seed(int(seed) + 1)
    t = {"K": _normal((B, L, Hkv, d), gen, dt), "V": _normal((B, L, Hkv, d), gen, dt)}
    if case["kind"] == "phase1":
        t["Q"] = _normal((B, L, Hq, d), gen, dt)
        rows = torch.randperm(L, generator=host)[:min(16, L)]
        start = rows // b * b                               # half point into their own block, half at
        own = start + (torch.rand(len(rows), generator=host) * (rows - start + 1)).long()
        first = (torch.rand(len(rows), generator=host) * max(1, case["a"])).long()   # the anchor's rows
        keys = torch.where(torch.arange(len(rows)) % 2 == 0, own, first)
        _point(t["Q"], t["K"], rows.cuda(), keys.cuda(), G)
        if case["mode"] == "all_blocks" and case["a"] > 0:
            t["Ka"] = _normal((B, case["a"], Hkv, d), gen, dt)
            t["Va"] = _normal((B, case["a"], Hkv, d), gen, dt)
        return t
    new = [case["q"]] if case["kind"] == "host" else ([case["lq"]] if case["lq"] else []) + [1] * case["nd"]
    t["new"] = []
    for n in new:
        q, k, v = _normal((B, n, Hq, d), gen, dt), _normal((B, n, Hkv, d), gen, dt), _normal((B, n, Hkv, d), gen, dt)
        rows = torch.arange(0, n, 4)
        keys = torch.randint(0, L, (len(rows),), generator=host)
        _point(q, t["K"], rows.cuda(), keys.cuda(), G)
        t["new"].append((q, k, v))
    if case["kind"] == "host":                              # what the other hosts sent
        rows = (B, Hq, case["q"])
        t["A"] = torch.randn((case["hosts"] - 1,) + rows + (d,), generator=gen, device="cuda") / math.sqrt(L)
        t["LSE"] = math.log(L) + 0.5 + 0.3 * torch.randn((case["hosts"] - 1,) + rows, generator=gen, device="cuda")
    return t


def prepare(case, seed):
    t = _inputs(case, seed)
    n_new = sum(x[0].shape[1] for x in t.get("new", []))
    cap = case["L"] + (n_new if n_new else 0)
    shape = sa.StarShape.make(_dt(case), case["B"], case["Hq"], case["Hkv"], case["d"], case["L"], case["b"],
                              case.get("a", 0), cap)
    s = {"case": dict(case), "shape": shape, "t": t}
    s["Kc"], s["Vc"] = sa.alloc_cache(shape)
    if case["kind"] == "phase1":
        mode = sa.ANCHOR_ALL_BLOCKS if case["mode"] == "all_blocks" else sa.ANCHOR_FIRST
        n = sa.phase1_workspace_bytes(shape, mode)
        s["ws"] = torch.empty(n, dtype=torch.uint8, device="cuda") if n else None
        s["O"] = torch.empty_like(t["Q"])
        s["lse"] = torch.empty((case["B"], case["Hq"], case["L"]), device="cuda") if case["lse"] else None
        return s
    s["Kc"][:, :, :case["L"]] = t.pop("K").transpose(1, 2)  # what phase 1 left in the caches
    s["Vc"][:, :, :case["L"]] = t.pop("V").transpose(1, 2)
    s["ws"] = sa.alloc_workspace(shape, max(x[0].shape[1] for x in t["new"]))
    s["O"] = [torch.empty_like(x[0]) for x in t["new"]]
    if case["kind"] == "host":                              # the gather buffer; slot 0 is this host's
        A, LSE = t.pop("A"), t.pop("LSE")
        s["A"] = torch.cat([torch.zeros_like(A[:1]), A])
        s["LSE"] = torch.cat([torch.zeros_like(LSE[:1]), LSE])
    return s


# ------------------------------------------------------------------ one pass


def run(s):
    case, shape, t = s["case"], s["shape"], s["t"]
    if case["kind"] == "phase1":
        if case["rope"]:                                    # rotates Q in place, as the call is defined
            sa.phase1_rope(shape, THETA, t["Q"], t["K"], t["V"], s["O"], s["Kc"], s["Vc"], LSE_ctx=s["lse"],
                           workspace=s["ws"])
        elif case["mode"] == "all_blocks":
            sa.phase1_anchor(shape, sa.ANCHOR_ALL_BLOCKS, t["Q"], t["K"], t["V"], s["O"], s["Kc"], s["Vc"],
                             K_anchor=t.get("Ka"), V_anchor=t.get("Va"), LSE_ctx=s["lse"], workspace=s["ws"])
        else:
            sa.phase1(shape, t["Q"], t["K"], t["V"], s["O"], s["Kc"], s["Vc"], LSE_ctx=s["lse"], workspace=s["ws"])
        return {"O": s["O"], "lse": s["lse"], "K_cache": s["Kc"], "V_cache": s["Vc"]}
    if case["kind"] == "host":
        q, k, v = t["new"][0]
        sa.phase2_partial(shape, case["L"], q, s["Kc"], s["Vc"], s["A"][0], s["LSE"][0], s["ws"], Kq=k, Vq=v)
        sa.merge(shape, s["A"], s["LSE"], O=s["O"][0])
        return {"A": s["A"], "LSE": s["LSE"], "O": s["O"], "K_cache": s["Kc"], "V_cache": s["Vc"]}
    cached = case["L"]
    for (q, k, v), o in zip(t["new"], s["O"]):
        if case["rope"]:                                    # rotates q in place, as the call is defined
            sa.phase2_rope(shape, THETA, cached, q, k, v, s["Kc"], s["Vc"], o, s["ws"])
        else:
            sa.phase2(shape, cached, q, k, v, s["Kc"], s["Vc"], o, s["ws"])
        cached += q.shape[1]
    return {"O": s["O"], "K_cache": s["Kc"], "V_cache": s["Vc"]}


# ------------------------------------------------------------------ what a pass cannot do without


def _blocks(case):
    """(start, end, anchored) of the context blocks."""
    L, b = case["L"], case["b"]
    for i in range(-(-L // b)):
        yield i * b, min(L, (i + 1) * b), case["a"] > 0 and (i > 0 or case["mode"] == "all_blocks")


def work(case):
    es = 4 if case["dtype"] == "fp32" else 2
    B, Hq, Hkv, d, L = (case[k] for k in ("B", "Hq", "Hkv", "d", "L"))
    if case["kind"] == "phase1":
        pairs = sum((e - s) * (case["a"] if anchored else 0) + (e - s) * (e - s + 1) // 2
                    for s, e, anchored in _blocks(case))
        nbytes = B * L * d * es * (2 * Hq + 4 * Hkv) + (4 * B * L * Hq if case["lse"] else 0)
        if case["mode"] == "all_blocks":
            nbytes += 2 * B * case["a"] * Hkv * d * es
        return {"bytes": nbytes, "flops": 4 * d * B * Hq * pairs}
    new = [case["q"]] if case["kind"] == "host" else ([case["lq"]] if case["lq"] else []) + [1] * case["nd"]
    nbytes, flops, cached = 0, 0, L
    for n in new:
        nbytes += B * d * es * (2 * Hkv * cached + 2 * Hq * n + 4 * Hkv * n)
        flops += 4 * d * B * Hq * sum(cached + j + 1 for j in range(n))
        cached += n
    if case["kind"] == "host":
        nbytes += 4 * B * Hq * case["q"] * (d + 1) * (case["hosts"] + 1)
        flops += 2 * B * Hq * case["q"] * d * case["hosts"]
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # fp32: sums of up to thousands of terms in another order.  bf16: outputs and softmax weights
    # are rounded to 8 bits of mantissa, and another split rounds other values.
    if case["dtype"] == "fp32":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1e-2, "max": 0.2}


# ------------------------------------------------------------------ the same in 64 bits


def _attend(q, K, V, lim=None):
    """Attention of rows q [R, d] over K, V [T, d]; row r sees keys below lim[r] (all if None)."""
    s = (q * (1.0 / math.sqrt(q.shape[1]))) @ K.T
    if lim is not None:
        s.masked_fill_(torch.arange(K.shape[0], device=s.device)[None, :] >= lim[:, None], -math.inf)
    m = s.amax(dim=1, keepdim=True)
    p = s.sub_(m).exp_()
    l = p.sum(dim=1, keepdim=True)
    return (p @ V) / l, (m + l.log())[:, 0]


def _rotate(X, pos0):
    """Rotary embedding in 64 bits: X [B, T, H, d], token t at pos0 + t."""
    X = X.double()
    half = X.shape[3] // 2
    freq = THETA ** (-torch.arange(half, device=X.device, dtype=torch.float64) * 2 / X.shape[3])
    ang = (pos0 + torch.arange(X.shape[1], device=X.device, dtype=torch.float64))[:, None] * freq[None, :]
    c, s = ang.cos()[None, :, None, :], ang.sin()[None, :, None, :]
    lo, hi = X[..., :half], X[..., half:]
    return torch.cat([lo * c - hi * s, hi * c + lo * s], dim=3)


def exact(case, seed):
    if work(case)["flops"] > 5.0e13:                        # beyond some 20 seconds in 64 bits
        return None
    t = _inputs(case, seed)
    B, Hq, Hkv, d, L = (case[k] for k in ("B", "Hq", "Hkv", "d", "L"))
    G = Hq // Hkv
    f64 = {"device": "cuda", "dtype": torch.float64}
    if case["kind"] == "phase1":
        if case["rope"]:
            t["Q"], t["K"] = _rotate(t["Q"], 0), _rotate(t["K"], 0)
        O = torch.empty((B, L, Hq, d), **f64)
        lse = torch.empty((B, Hq, L), **f64)
        for beta in range(B):
            for g in range(Hkv):
                hs = slice(g * G, (g + 1) * G)
                K, V = t["K"][beta, :, g].double(), t["V"][beta, :, g].double()
                if "Ka" in t:
                    Ka, Va = t["Ka"][beta, :, g].double(), t["Va"][beta, :, g].double()
                else:
                    Ka, Va = K[:case["a"]], V[:case["a"]]
                for s, e, anchored in _blocks(case):
                    a = case["a"] if anchored else 0
                    step = max(16, (1 << 26) // ((a + e - s) * G))
                    for r0 in range(s, e, step):
                        r1 = min(e, r0 + step)
                        lim = a + torch.arange(r0 - s + 1, r1 - s + 1, device="cuda").repeat_interleave(G)
                        o, x = _attend(t["Q"][beta, r0:r1, hs].double().reshape(-1, d), torch.cat([Ka[:a], K[s:r1]]),
                                       torch.cat([Va[:a], V[s:r1]]), lim)
                        O[beta, r0:r1, hs] = o.view(-1, G, d)
                        lse[beta, hs, r0:r1] = x.view(-1, G).T
        return {"O": O, "lse": lse if case["lse"] else None, "K_cache": t["K"].double().transpose(1, 2).contiguous(),
                "V_cache": t["V"].double().transpose(1, 2).contiguous()}
    rope = case.get("rope", False)
    Kc, Vc, outs, pairs, cached = t["K"].transpose(1, 2).double(), t["V"].transpose(1, 2).double(), [], [], L
    for q, k, v in t["new"]:
        n = q.shape[1]
        q, k = (_rotate(q, cached), _rotate(k, cached)) if rope else (q.double(), k.double())
        Kc, Vc = torch.cat([Kc, k.transpose(1, 2)], dim=2), torch.cat([Vc, v.double().transpose(1, 2)], dim=2)
        o, x = torch.empty((B, n, Hq, d), **f64), torch.empty((B, Hq, n), **f64)
        step = max(1, (1 << 26) // (G * (cached + n)))
        for beta in range(B):
            for g in range(Hkv):
                for j0 in range(0, n, step):
                    j1 = min(n, j0 + step)
                    lim = cached + torch.arange(j0 + 1, j1 + 1, device="cuda").repeat_interleave(G)
                    y, z = _attend(q[beta, j0:j1, g * G:(g + 1) * G].reshape(-1, d), Kc[beta, g], Vc[beta, g], lim)
                    o[beta, j0:j1, g * G:(g + 1) * G] = y.view(-1, G, d)
                    x[beta, g * G:(g + 1) * G, j0:j1] = z.view(-1, G).T
        outs.append(o)
        pairs.append((o.transpose(1, 2), x))
        cached += n
    if case["kind"] == "host":
        A = torch.cat([pairs[0][0][None], t["A"].double()])
        LSE = torch.cat([pairs[0][1][None], t["LSE"].double()])
        w = torch.softmax(LSE, dim=0)[..., None]
        return {"A": A, "LSE": LSE, "O": [(w * A).sum(dim=0).transpose(1, 2).contiguous()], "K_cache": Kc, "V_cache": Vc}
    return {"O": outs, "K_cache": Kc, "V_cache": Vc}
