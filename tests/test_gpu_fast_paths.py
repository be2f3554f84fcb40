"""The fast paths whose results are the slow ones' bit for bit are the ones
that run: the kernel on pinned host memory, by the server's count of its
requests, and the native binding, by what it returns."""
import ctypes

import pytest
import torch

import paper_1806_06698_amd as s3
from paper_1806_06698_amd import _lib, gen, serve

pytestmark = pytest.mark.gpu

FORMS = {torch.float64: s3.F64, torch.float32: s3.F32_REFINE}


def _in_place(srv):
    f = srv.L.syev3_server_solved_in_place
    f.argtypes, f.restype = [ctypes.c_void_p], ctypes.c_int64
    return f(srv.h)


def _hip():
    path = next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64.so" in l)
    return ctypes.CDLL(path)


@pytest.mark.parametrize("graphs", [True, False])
def test_pinned_requests_are_solved_in_place(graphs):
    """Pinned buffers, each its own or side by side in one, in both types,
    with and without vectors; 90 of them, so that a tick takes several
    launches.  Requests on the device and in pageable memory are not."""
    A, _ = gen.stress_mix(1 << 16, 95, "cuda")
    src = {torch.float64: A.cpu(), torch.float32: A.float().cpu()}
    with serve.Server(hbm_budget_bytes=1 << 28, use_graphs=graphs) as srv:
        reqs, want = [], 0
        for i in range(90):
            n, dt = 50 + 37 * i, (torch.float64, torch.float32)[i % 2]
            vecs, how = i % 5 != 4, i % 6
            r = srv.acquire(n, FORMS[dt], vectors=vecs)
            if how == 5:
                r.A.copy_(src[dt][:, :n])
                torch.cuda.synchronize()
                srv.submit(r)
            else:
                pool = torch.empty(18 * n, dtype=dt, pin_memory=how != 4)
                hA, hl, hV = pool[:6 * n], pool[6 * n:9 * n], pool[9 * n:]
                if how < 2:
                    hl, hV = torch.empty_like(hl).pin_memory(), torch.empty_like(hV).pin_memory()
                hA.copy_(src[dt][:, :n].reshape(-1))
                srv.submit_host(r, hA, hl, hV if vecs else None)
                want += how != 4
            reqs.append(r)
        for r in reqs:
            srv.wait(r, 60.0)
            srv.release(r)
        assert _in_place(srv) == want == 60
        assert srv.stats()["completed"] == 90


@pytest.mark.parametrize("flags,direct", [(0, 1), (0x80000000, 0)],
                         ids=["coherent", "hipHostMallocNonCoherent"])
def test_kinds_of_pinned_memory(flags, direct):
    n = 5000
    A, _ = gen.stress_mix(n, 96, "cuda")
    lam, V = (t.cpu() for t in s3.syev3(A))
    hip, p = _hip(), ctypes.c_void_p()
    assert hip.hipHostMalloc(ctypes.byref(p), ctypes.c_size_t(18 * n * 8),
                             ctypes.c_uint(flags)) == 0
    try:
        buf = torch.frombuffer((ctypes.c_double * (18 * n)).from_address(p.value),
                               dtype=torch.float64)
        hA, hl, hV = buf[:6 * n], buf[6 * n:9 * n], buf[9 * n:]
        with serve.Server(hbm_budget_bytes=1 << 26) as srv:
            for rep in range(3):
                hA.copy_(A.cpu().reshape(-1))
                buf[6 * n:].fill_(-1.0)
                r = srv.acquire(n)
                srv.submit_host(r, hA, hl, hV)
                srv.wait(r, 60.0)
                srv.release(r)
                assert torch.equal(hl.view(3, n), lam) and torch.equal(hV.view(9, n), V)
            assert _in_place(srv) == 3 * direct
    finally:
        assert hip.hipHostFree(p) == 0


def test_grid_blocks_limits_the_kernel_on_host_memory():
    """A grid of one workgroup strides over every tile."""
    n = 3000
    A, _ = gen.stress_mix(n, 97, "cuda")
    lam, V = (t.cpu() for t in s3.syev3(A))
    hA = A.cpu().pin_memory()
    hl, hV = torch.empty(3, n, dtype=A.dtype).pin_memory(), torch.empty(9, n, dtype=A.dtype).pin_memory()
    with serve.Server(hbm_budget_bytes=1 << 26, grid_blocks=1) as srv:
        r = srv.acquire(n)
        srv.submit_host(r, hA, hl, hV)
        srv.wait(r, 60.0)
        srv.release(r)
        assert _in_place(srv) == 1
    assert torch.equal(hl, lam) and torch.equal(hV, V)


def test_the_native_binding_takes_plain_calls():
    native = _lib.binding()
    A = gen.normal(100, 98, "cuda")
    e = lambda *s: torch.empty(*s, dtype=torch.float64, device="cuda")
    codes = {"soa": s3.SOA, "aos": s3.AOS, "aos9": s3.AOS9}
    full = gen.to_full(A).contiguous()
    plain = [("soa", A, None), ("soa", A[:, 3:50], None), ("soa", A.float(), None),
             ("soa", A, (e(3, 100), e(9, 100))), ("soa", A, (e(3, 101)[:, :100], e(9, 100))),
             ("aos", gen.to_aos(A).contiguous(), None), ("aos9", full, None),
             ("aos9", full.reshape(100, 9), (e(100, 3), e(100, 3, 3)))]
    for layout, a, out in plain:
        for vectors in (True, False):
            assert native.solve(a, codes[layout], vectors, 0, True, out) is not None
    refused = [(A[:5], 0, True, 0, True, None), (A[:, ::2], 0, True, 0, True, None),
               (A.cpu(), 0, True, 0, True, None), (A.half(), 0, True, 0, True, None),
               (A, 3, True, 0, True, None), (A, -1, True, 0, True, None),
               (A, 0, True, 64, True, None), (A, 0, True, -1, True, None),
               (A[:, :0], 0, True, 0, True, None), (A, 0, True, 0, True, (e(3, 100), None)),
               (A, 0, True, 0, True, (e(3, 99), e(9, 100))), (A.t(), 1, True, 0, True, None)]
    for args in refused:
        assert native.solve(*args) is None
    good = (A, e(3, 100), e(9, 100))
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    assert native.segments([good], None, None) is True
    assert native.segments((good + (s3.FLAG_NO_SCALE,),), st.device.index, st.cuda_stream) is True
    for segs in ([], [good[:2]], [good, good], [(A.cpu(), e(3, 100), None)], iter([good])):
        assert native.segments(segs, None, None) is None
    torch.cuda.synchronize()


FLAGS = [0, s3.FLAG_SIMPLIFIED_DEFLATION, s3.FLAG_NO_H_GUARD, s3.FLAG_NEWTON, s3.FLAG_PAPER_BG,
         s3.FLAG_NO_SCALE, s3.FLAG_NO_SCALE | s3.FLAG_NO_H_GUARD | s3.FLAG_SIMPLIFIED_DEFLATION,
         s3.FLAG_NEWTON | s3.FLAG_NO_SCALE]
FLAGS32 = [0, s3.FLAG_SIMPLIFIED_DEFLATION, s3.FLAG_NO_H_GUARD, s3.FLAG_REFINE_CONVERGE,
           s3.FLAG_NO_SCALE, s3.FLAG_REFINE_CONVERGE | s3.FLAG_NO_H_GUARD]


def test_flags_per_request():
    """Every flag that a request may carry, each in a request of its own in one
    launch: the shared solve takes each as the batched solver does."""
    A, _ = gen.stress_mix(3000, 99, "cuda")
    segs, want = [], []
    for a, flags in ((A, FLAGS), (A.float().contiguous(), FLAGS32)):
        for f in flags:
            segs.append((a, torch.empty(3, 3000, dtype=a.dtype, device="cuda"),
                         torch.empty(9, 3000, dtype=a.dtype, device="cuda"), f))
            want.append(s3.syev3(a, flags=f))
    s3.syev3_solve_segments_noalloc(segs)
    for (a, lam, V, f), (l, v) in zip(segs, want):
        assert torch.equal(lam, l) and torch.equal(V, v), (a.dtype, f)
