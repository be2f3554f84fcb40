"""Host-staged requests on pinned memory, which the tick's kernel reads and
writes in place, and the ones that have to be copied all the same: every
result equals, bit for bit, the batched solver's."""
import ctypes

import pytest
import torch

import paper_1806_06698_amd as s3
from paper_1806_06698_amd import gen, serve

pytestmark = pytest.mark.gpu

FORMS = {torch.float64: s3.F64, torch.float32: s3.F32_REFINE}


@pytest.fixture(scope="module")
def source():
    A, _ = gen.stress_mix(1 << 18, 90, "cuda")
    A[:, 5] = float("nan")
    return {torch.float64: A, torch.float32: A.float().contiguous()}


def _submit(srv, r, hA, hl, hV):
    """The C entry point: unlike the binding it takes a NULL host_V from a
    request with vectors, and any address."""
    rc = srv.L.syev3_server_submit_host(srv.h, r.id, ctypes.c_void_p(hA), ctypes.c_void_p(hl),
                                        ctypes.c_void_p(hV))
    assert rc == 0


def _same(x, y):
    x, y = x.cpu(), y.cpu()
    bits = torch.int64 if x.dtype == torch.float64 else torch.int32
    return torch.equal(x.contiguous().view(bits), y.contiguous().view(bits))


@pytest.mark.parametrize("graphs", [True, False])
@pytest.mark.parametrize("requests", [1, 40, 41, 90])
def test_pinned(source, requests, graphs):
    """Around the size of one launch's table (40 requests), with requests on
    the device and in pageable memory among them."""
    g = torch.Generator().manual_seed(requests)
    sizes = torch.randint(1, 1200, (requests,), generator=g).tolist()
    sizes[0] = 70_001  # more tiles than workgroups
    with serve.Server(hbm_budget_bytes=1 << 28, use_graphs=graphs) as srv:
        for rep in range(2):
            got = []
            for i, n in enumerate(sizes):
                dt = (torch.float64, torch.float32)[(i + rep) % 2]
                a = source[dt][:, 100 * i:100 * i + n].contiguous()
                vecs = i % 5 != 4
                r = srv.acquire(n, FORMS[dt], vectors=vecs)
                hl = hV = None
                if i % 7 == 3:
                    r.A.copy_(a)
                    torch.cuda.synchronize()
                    srv.submit(r)
                else:
                    pin = i % 7 != 5
                    hA = a.cpu()
                    hA = hA.pin_memory() if pin else hA
                    hl = torch.zeros((3, n), dtype=dt, pin_memory=pin)
                    hV = torch.zeros((9, n), dtype=dt, pin_memory=pin)
                    srv.submit_host(r, hA, hl, hV if vecs else None)
                got.append((r, a, hl, hV))
            for i, (r, a, hl, hV) in enumerate(got):
                srv.wait(r, 60.0)
                lam, V = s3.syev3(a, vectors=r.V is not None)
                assert _same(r.lam, lam), i
                assert r.V is None or _same(r.V, V), i
                if hl is not None:
                    assert _same(hl, lam), i
                    assert _same(r.A, a), i
                    assert _same(hV, V) if r.V is not None else not hV.any(), i
                srv.release(r)


@pytest.mark.parametrize("dt", [torch.float64, torch.float32])
def test_buffers_used_again(source, dt):
    """The same pinned buffers with new contents every time."""
    n = 3000
    hA = torch.empty((6, n), dtype=dt, pin_memory=True)
    hl = torch.empty((3, n), dtype=dt, pin_memory=True)
    hV = torch.empty((9, n), dtype=dt, pin_memory=True)
    src = source[dt].cpu()
    lam, V = s3.syev3(source[dt])
    lam, V = lam.cpu(), V.cpu()
    with serve.Server(hbm_budget_bytes=1 << 26) as srv:
        for rep in range(80):
            hA.copy_(src[:, rep * n:(rep + 1) * n])
            hl.zero_()
            hV.zero_()
            r = srv.acquire(n, FORMS[dt])
            srv.submit_host(r, hA, hl, hV)
            srv.wait(r, 60.0)
            srv.release(r)
            assert _same(hl, lam[:, rep * n:(rep + 1) * n]), rep
            assert _same(hV, V[:, rep * n:(rep + 1) * n]), rep


@pytest.mark.parametrize("layout", ["side by side", "no host vectors", "results over the input",
                                    "vectors over the eigenvalues", "odd addresses"])
def test_where_the_buffers_lie(source, layout):
    n, dt = 2000, torch.float64
    a = source[dt][:, :n].contiguous()
    lam, V = (t.cpu() for t in s3.syev3(a))
    pool = torch.zeros(20 * n + 64, dtype=dt, pin_memory=True)
    raw = pool.view(torch.uint8).numpy()
    base = pool.data_ptr()
    # byte offsets of the input, the eigenvalues and the vectors
    oA, ol, oV = {"side by side": (8, 8 + 48 * n, 8 + 72 * n),
                  "no host vectors": (8, 8 + 48 * n, None),
                  "results over the input": (0, 24 * n, 48 * n),
                  "vectors over the eigenvalues": (0, 48 * n, 64 * n),
                  "odd addresses": (4, 4 + 48 * n, 4 + 72 * n)}[layout]
    raw[oA:oA + 48 * n] = a.cpu().view(torch.uint8).numpy().reshape(-1)
    want = raw.copy()
    want[ol:ol + 24 * n] = lam.contiguous().view(torch.uint8).numpy().reshape(-1)
    if oV is not None:
        want[oV:oV + 72 * n] = V.contiguous().view(torch.uint8).numpy().reshape(-1)
    with serve.Server(hbm_budget_bytes=1 << 26) as srv:
        r = srv.acquire(n, s3.F64)
        _submit(srv, r, base + oA, base + ol, None if oV is None else base + oV)
        srv.wait(r, 60.0)
        assert (raw == want).all()
        assert _same(r.A, a) and _same(r.lam, lam) and _same(r.V, V)
        srv.release(r)
