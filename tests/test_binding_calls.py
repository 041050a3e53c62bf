"""The calls of the binding (csrc/marshal.cpp, and by ctypes alone) on the CPU: every argument of every entry point
arrives at its place, and what was refused in Python is refused."""
import ctypes

import pytest
import torch

import paper_2411_17116_amd as sa
from paper_2411_17116_amd import binding

NAMES = ("phase1", "phase1_anchor", "phase1_rope", "phase2", "phase2_rope", "phase2_static", "phase2_partial", "merge", "rope")


class Stream:
    cuda_stream = 0x7700


@pytest.fixture(params=["extension", "ctypes"])
def seen(request, monkeypatch):
    """Entry points that note what they are called with and answer `status`."""
    lib = sa.load_library()
    log = {"status": 0}

    class Fake:
        pass

    fake, keep = Fake(), []
    for name in NAMES:
        real = getattr(lib, "star_attn_" + name)

        def call(*args, name=name):
            shape = ctypes.cast(args[0], ctypes.POINTER(sa.StarShape)).contents
            log[name] = (shape.ctx_len,) + args[1:]
            return log["status"]

        kinds = [ctypes.c_void_p if k is real.argtypes[0] else k for k in real.argtypes]
        fn = ctypes.CFUNCTYPE(ctypes.c_int, *kinds)(call)
        keep.append(fn)
        setattr(fake, "star_attn_" + name, fn)
    if request.param == "ctypes":
        monkeypatch.setattr(binding, "_MARSHAL", binding._CtypesCalls(fake))
        yield log
        return
    binding._bind(fake)
    yield log
    binding._bind(lib)


def _t(*dims):
    return torch.zeros(dims or (8,), dtype=torch.bfloat16)


SHAPE = sa.StarShape.make("bf16", 1, 2, 1, 128, 4321, 256, 0, 5000)


def test_every_argument_at_its_place(seen):
    Q, K, V, O, L, Kc, Vc, Ka, Va, Op, Lp, A = (_t(2, 3, 4, 5) for _ in range(12))
    ws = torch.zeros(24, dtype=torch.int16)
    p = lambda *ts: tuple(t.data_ptr() for t in ts)
    st = Stream()
    sa.phase1(SHAPE, Q, K, V, O, Kc, Vc, LSE_ctx=L, workspace=ws, stream=st)
    assert seen["phase1"] == (4321, *p(Q, K, V, O, L, Kc, Vc, ws), 48, 0x7700)
    sa.phase1(SHAPE, Q, K, V, O, Kc, Vc, stream=st)
    assert seen["phase1"] == (4321, *p(Q, K, V, O), None, *p(Kc, Vc), None, 0, 0x7700)
    sa.phase1_anchor(SHAPE, 3, Q, K, V, O, Kc, Vc, K_anchor=Ka, V_anchor=Va, LSE_ctx=L, workspace=ws, stream=st)
    assert seen["phase1_anchor"] == (4321, 3, *p(Q, K, V, Ka, Va, O, L, Kc, Vc, ws), 48, 0x7700)
    sa.phase1_rope(SHAPE, 10000, Q, K, V, O, Kc, Vc, pos0=9, LSE_ctx=L, workspace=ws, stream=st)
    assert seen["phase1_rope"] == (4321, 10000.0, 9, *p(Q, K, V, O, L, Kc, Vc, ws), 48, 0x7700)
    sa.phase2(SHAPE, 4400, Q, K, V, Kc, Vc, O, ws, O_part=Op, LSE_part=Lp, stream=st)
    assert seen["phase2"] == (4321, 4400, 3, *p(Q, K, V, Kc, Vc, Op, Lp, O, ws), 48, 0x7700)
    sa.phase2_rope(SHAPE, 5e5, 4400, Q, K, V, Kc, Vc, O, ws, pos0=-1, O_part=Op, LSE_part=Lp, stream=st)
    assert seen["phase2_rope"] == (4321, 5e5, -1, 4400, 3, *p(Q, K, V, Kc, Vc, Op, Lp, O, ws), 48, 0x7700)
    sa.phase2_static(SHAPE, 4400, Q, K, V, Kc, Vc, O, stream=st)
    assert seen["phase2_static"] == (4321, 4400, 3, *p(Q, K, V, Kc, Vc, O), 0x7700)
    sa.phase2_partial(SHAPE, 4400, Q, Kc, Vc, A, L, ws, Kq=K, Vq=V, stream=st)
    assert seen["phase2_partial"] == (4321, 4400, 3, *p(Q, K, V, Kc, Vc, A, L, ws), 48, 0x7700)
    sa.merge(SHAPE, Op, Lp, O=O, A=A, LSE=L, stream=st)
    assert seen["merge"] == (4321, 2, 5, *p(Op, Lp, O, A, L), 0x7700)
    sa.rope(SHAPE, Q, Ka, 7.5, pos0=11, stream=st)
    assert seen["rope"] == (4321, 4, 3, 11, 7.5, *p(Q, Ka), 0x7700)


def test_what_is_refused_and_what_is_asked_through_python(seen):
    t, st = _t(2, 3, 4, 5), Stream()
    with pytest.raises(ValueError, match="contiguous"):
        sa.rope(SHAPE, t, t.transpose(0, 1), 7.5, stream=st)
    with pytest.raises(TypeError):
        sa.rope(None, t, t, 7.5, stream=st)
    with pytest.raises(AttributeError):
        sa.rope(SHAPE, t, 5, 7.5, stream=st)
    with pytest.raises(AttributeError):
        sa.phase2(SHAPE, 4400, None, t, t, t, t, t, t, stream=st)
    with pytest.raises(IndexError):
        sa.phase2(SHAPE, 4400, _t(), t, t, t, t, t, t, stream=st)
    seen["status"] = -3
    with pytest.raises(sa.StarAttnError) as e:
        sa.rope(SHAPE, t, t, 7.5, stream=st)
    assert e.value.code == -3
    seen["status"] = 0

    class Sub(torch.Tensor):
        pass

    sub, param = t.as_subclass(Sub), torch.nn.Parameter(t, requires_grad=True)
    sa.rope(SHAPE, sub, param, 7.5, stream=st)
    assert seen["rope"][-3:-1] == (t.data_ptr(), t.data_ptr()) and seen["rope"][1:3] == (4, 3)
    sa.phase2(SHAPE, 4400, sub, t, t, t, t, t, sub, stream=st)
    assert seen["phase2"][2] == 3 and seen["phase2"][-2] == 2 * t.numel()


def test_without_the_extension(monkeypatch):
    """A library without its extension module, or with one that this torch does not load, answers queries and takes
    calls; with it, calls go through it."""
    assert type(binding._calls()).__name__ == "module"

    def refuse(lib):
        raise ImportError("undefined symbol")

    monkeypatch.setattr(binding, "_MARSHAL", None)
    monkeypatch.setattr(binding, "_LIB", None)
    monkeypatch.setattr(binding, "_bind", refuse)
    assert sa.workspace_bytes(SHAPE, 1) > 0 and sa.phase2_plan(SHAPE, 4400, 1).decode == 1
    t = _t(1, 1, 2, 128)
    with pytest.warns(UserWarning, match="ctypes"), pytest.raises(sa.StarAttnError) as e:
        sa.phase2(SHAPE, 4400, t, None, None, t, t, t, t, stream=Stream())       # refused by the library itself
    assert e.value.code == -2
