"""The binding's native fast paths against the Python code that they stand in
for: over the forms a call can take, both give the same bits, shapes, strides
and types, or the same error."""
import numpy as np
import pytest
import torch

import paper_1806_06698_amd as s3
from paper_1806_06698_amd import _lib, gen

pytestmark = pytest.mark.gpu


class _NoFastPath:
    @staticmethod
    def solve(*a):
        return None

    @staticmethod
    def segments(*a):
        return None


def _call(monkeypatch, native, fn):
    """(values, None) or (None, error) of fn(), with or without the native
    paths; values: every returned tensor's shape, strides and content."""
    with monkeypatch.context() as m:
        if not native:
            m.setattr(_lib, "_binding", _NoFastPath)
        try:
            r = fn()
        except Exception as e:
            return None, (type(e), str(e))
    torch.cuda.synchronize()
    return [(t.shape, t.stride(), t.dtype, t.clone()) if t is not None else None for t in r], None


def _same(monkeypatch, fn):
    a, ea = _call(monkeypatch, True, fn)
    b, eb = _call(monkeypatch, False, fn)
    assert ea == eb, (ea, eb)
    if ea is None:
        assert len(a) == len(b)
        for x, y in zip(a, b):
            assert (x is None) == (y is None)
            assert x is None or (x[:3] == y[:3] and torch.equal(x[3], y[3]))
    return ea


def _inputs():
    A = gen.normal(100, 90, "cuda")
    wide = torch.empty(6, 300, dtype=A.dtype, device="cuda")
    wide[:, 7:107] = A
    full = gen.to_full(A).contiguous()
    yield "soa", A
    yield "soa", A[:, :1]
    yield "soa", wide[:, 7:107]
    yield "soa", A[:, ::2]                       # columns not of unit stride
    yield "soa", A[:, :1].expand(6, 5)           # overlapping planes
    yield "soa", A[:, :0]
    yield "soa", A[:5]
    yield "soa", A.t()
    yield "soa", A.cpu()
    yield "soa", A.half()
    yield "soa", A.clone().requires_grad_()
    yield "soa", torch.nn.Parameter(A.clone(), requires_grad=False)
    yield "aos", gen.to_aos(A)
    yield "aos", gen.to_aos(A)[::2]
    yield "aos", gen.to_aos(A)[:1]
    yield "aos", A
    yield "aos9", full
    yield "aos9", full.reshape(-1, 9)
    yield "aos9", full[::2]                      # reshaped through a copy
    yield "aos9", full.transpose(1, 2)
    yield "aos9", full[:, :2]
    yield "aos9", full[:0]
    yield "nope", A
    yield 3, A


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_inputs(monkeypatch, dtype):
    errors = 0
    for layout, A in _inputs():
        if A.dtype == torch.float64 and dtype == torch.float32:
            A = A.to(dtype) if A.stride(-1) == 0 or not A.is_cuda else \
                torch.empty_strided(A.shape, A.stride(), dtype=dtype, device="cuda").copy_(A)
        for kw in (dict(), dict(vectors=False), dict(refine=False), dict(flags=s3.FLAG_NO_SCALE),
                   dict(flags=64), dict(flags=-1), dict(flags=np.int64(0)),
                   dict(stream=torch.cuda.current_stream())):
            errors += _same(monkeypatch, lambda: s3.syev3(A, layout=layout, **kw)) is not None
    assert errors > 20


def test_outputs(monkeypatch):
    A = gen.normal(64, 91, "cuda")
    e = lambda *s, **k: torch.zeros(*s, dtype=k.get("dtype", torch.float64), device="cuda")
    alias = A[:3]  # of the input, which is refused (the others get a copy of it)
    outs = [(e(3, 64), e(9, 64)), [e(3, 64), e(9, 64)], (e(3, 70)[:, :64], e(9, 65)[:, 1:]),
            (e(3, 64), None), (None, e(9, 64)), (e(3, 65), e(9, 64)), (e(3, 64), e(9, 64).t()),
            (e(64, 3).t(), e(9, 64)), (e(3, 64, dtype=torch.float32), e(9, 64)),
            (alias, e(9, 64)), (e(3, 64), A.new_zeros(9, 64).cpu()),
            (e(1, 64).expand(3, 64), e(9, 64)), (e(3, 64),), "xy"]
    for out in outs:
        for v in (True, False):
            _same(monkeypatch, lambda: s3.syev3(A if out[0] is alias else A.clone(), out=out,
                                                vectors=v))
    l, V = e(3, 64), e(9, 64)
    got = s3.syev3(A, out=(l, V))
    assert got[0] is l and got[1] is V
    Aa, one = gen.to_aos(A), gen.to_aos(A)[:1].contiguous()
    for out in ((e(64, 3), e(64, 3, 3)), (e(64, 3), e(64, 9)), (e(3, 64).t(), e(64, 3, 3)),
                (e(64, 4)[:, :3], e(64, 3, 3))):
        _same(monkeypatch, lambda: s3.syev3(Aa, layout="aos", out=out))
    for out in ((e(1, 3), e(1, 3, 3)), (e(3, 1).t(), e(1, 3, 3)), (e(1, 6)[:, ::2], e(1, 3, 3))):
        _same(monkeypatch, lambda: s3.syev3(one, layout="aos", out=out))


def test_segments(monkeypatch):
    A = gen.normal(100, 92, "cuda")
    F = A.float()
    e = lambda *s, **k: torch.zeros(*s, dtype=k.get("dtype", torch.float64), device="cuda")
    f = lambda *s: e(*s, dtype=torch.float32)
    good = (A[:, :40], e(3, 40), e(9, 40))
    lists = [[good], (good,), [list(good)], [good, (F[:, 5:30], f(3, 25), None)], [],
             [good + (s3.FLAG_NO_SCALE,)], [good + (64,)], [good + (-1,)], [good[:2]],
             [(A[:, :0], e(3, 0), e(9, 0)), good], [(A[:, ::2], e(3, 50), None)],
             [(A.cpu(), e(3, 100), None)], [(A, e(3, 100, dtype=torch.float32), None)],
             [(A, e(3, 99), None)], [(A, e(3, 101)[:, :100], None)], [(A, A[:3], None)],
             [good, (A, good[1], None)], [good] * 1025, [(A, e(3, 100), e(9, 100).cpu())],
             [(A[:, :1], e(3, 2)[:, :1], None)], iter([good])]
    st = torch.cuda.Stream()
    for segs in lists:
        for kw in (dict(), dict(stream=st)):
            torch.cuda.synchronize()

            def fn():
                s3.syev3_solve_segments_noalloc(segs, **kw)
                torch.cuda.synchronize()
                return [t for q in (segs if isinstance(segs, (list, tuple)) else [])
                        for t in q[1:3]][:4]
            _same(monkeypatch, fn)
    lam, V = s3.syev3(A[:, :40].contiguous())
    assert torch.equal(good[1], lam) and torch.equal(good[2], V)


def test_modes_and_subclasses_take_the_python_path(monkeypatch):
    """A function mode and a tensor subclass see what they saw before: the
    calls that the Python code makes."""
    A = gen.normal(16, 93, "cuda")
    seen = []

    class Mode(torch.overrides.TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            seen.append(getattr(func, "__name__", str(func)))
            return func(*args, **(kwargs or {}))

    with Mode():
        lam, V = s3.syev3(A)
    assert "empty" in seen
    ref = s3.syev3(A)
    assert torch.equal(lam, ref[0]) and torch.equal(V, ref[1])

    class Sub(torch.Tensor):
        pass

    _same(monkeypatch, lambda: s3.syev3(A.as_subclass(Sub)))
