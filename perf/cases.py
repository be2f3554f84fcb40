"""The calls whose speed this library is held to: batches of every size from a
single lane to 2^26 matrices in every layout and storage type, several
requests in one launch, and requests served from host memory.

Eigenvectors of matrices with (nearly) equal eigenvalues are not determined to
working accuracy, and two correct solvers may return quite different ones.  So
FP64 cases that return vectors draw matrices with separated eigenvalues (the
paper's random entries, or the stress mix without its near-degenerate pairs);
the condition-1e8 blocks and the whole stress mix are drawn for
eigenvalues and for FP32 storage, whose rounding separates the pairs.
"""
import random

import torch

import paper_1806_06698_amd as s3
from paper_1806_06698_amd import gen, serve

# Matrices per call: one wavefront's worth and less, up to the largest batch
# that the benchmark solves with vectors.
MAX_N = 1 << 26


def listed():
    return [
        # one element's or a few material points' tensors, solved in a time
        # loop: launch and call overhead
        {"name": "soa_f64_vecs_33", "kind": "batch", "layout": "soa", "dtype": "f64",
         "vectors": True, "data": "normal", "n": 33, "out": False},
        # the small configuration of the tests and the benchmark
        {"name": "soa_f64_vecs_4k", "kind": "batch", "layout": "soa", "dtype": "f64",
         "vectors": True, "data": "normal", "n": 4096, "out": False},
        # full matrices as torch.linalg.eigh takes them: a mesh's or an
        # image slice's symmetric tensors
        {"name": "aos9_f32_vecs_200k", "kind": "batch", "layout": "aos9", "dtype": "f32",
         "vectors": True, "data": "normal", "n": 200_003, "out": False},
        # an ordinary batch with a ragged last tile (a volume's tensors)
        {"name": "soa_f64_vecs_1m", "kind": "batch", "layout": "soa", "dtype": "f64",
         "vectors": True, "data": "uniform", "n": 1_000_003, "out": False},
        # principal values alone (yield criteria, vesselness filters)
        {"name": "soa_f32_vals_4m", "kind": "batch", "layout": "soa", "dtype": "f32",
         "vectors": False, "data": "chi2", "n": (1 << 22) + 5, "out": True},
        # the stress mix at the benchmark's size: every branch in a wavefront
        {"name": "soa_f64_vals_16m", "kind": "batch", "layout": "soa", "dtype": "f64",
         "vectors": False, "data": "stress_mix", "n": 1 << 24, "out": True},
        # packed rows as most programs store symmetric tensors
        {"name": "aos_f64_vecs_16m", "kind": "batch", "layout": "aos", "dtype": "f64",
         "vectors": True, "data": "separated_mix", "n": (1 << 24) + 77, "out": True},
        # finite-element blocks of condition up to 1e8 in FP32 storage
        {"name": "soa_f32_vecs_64m", "kind": "batch", "layout": "soa", "dtype": "f32",
         "vectors": True, "data": "spd_fe", "n": 1 << 26, "out": True},
        # the largest batch, in the layout and type that the headline times
        {"name": "soa_f64_vecs_64m", "kind": "batch", "layout": "soa", "dtype": "f64",
         "vectors": True, "data": "normal", "n": 1 << 26, "out": True},
        # a scheduler's tick of many small requests in one launch
        {"name": "segments_40_small", "kind": "segments", "requests": 40, "max_log2": 12,
         "vectors": True, "sizes": 1},
        # a tick at saturation: the benchmark's serving mix, about 2^24 matrices
        {"name": "segments_200_large", "kind": "segments", "requests": 200, "max_log2": 20,
         "vectors": True, "sizes": 2},
        # requests whose input and results live in host memory
        {"name": "server_host_12", "kind": "server", "requests": 12, "max_log2": 19,
         "vectors": True, "sizes": 3},
    ]


def draw(rng):
    kind = rng.choices(["batch", "segments", "server"], [9, 2, 1])[0]
    if kind == "batch":
        dtype = rng.choice(["f64", "f32"])
        vectors = rng.random() < 0.7
        layout = rng.choice(["soa", "soa", "aos", "aos9"])
        if dtype == "f64" and vectors:
            data = rng.choice(["normal", "uniform", "chi2", "separated_mix"])
        else:
            data = rng.choice(["normal", "uniform", "chi2", "spd_fe", "stress_mix"])
        # full matrices hold half as much again: a quarter of the largest batch
        n = int((MAX_N if layout != "aos9" else MAX_N / 4) ** rng.random())
        return {"kind": "batch", "layout": layout, "dtype": dtype, "vectors": vectors,
                "data": data, "n": max(1, n), "out": n >= 1 << 21}
    if kind == "segments":
        return {"kind": "segments", "requests": int(1024 ** rng.random()),
                "max_log2": rng.randint(4, 20), "vectors": rng.random() < 0.8,
                "sizes": rng.randrange(1 << 20)}
    return {"kind": "server", "requests": rng.randint(1, 16), "max_log2": rng.randint(8, 19),
            "vectors": rng.random() < 0.8, "sizes": rng.randrange(1 << 20)}


def _draw_soa(data, n, seed):
    """(6, n) float64 on the GPU."""
    if data == "separated_mix":
        A, cat = gen.stress_mix(n, seed, "cuda")
        near = cat == gen.CAT_NEAR_DEGENERATE
        return torch.where(near.unsqueeze(0), gen.normal(n, seed + 1, "cuda"), A)
    return gen.make(data, n, seed, "cuda")[0]


def _inputs(case, seed):
    """A batch's input in its layout and storage type."""
    A = _draw_soa(case["data"], case["n"], seed)
    if case["dtype"] == "f32":
        A = A.float()
    if case["layout"] == "aos":
        return gen.to_aos(A)
    if case["layout"] == "aos9":
        return gen.to_full(A).contiguous()
    return A.contiguous()


def _requests(case):
    """(n, is_f32) of every request: floor(2^U(0, max_log2)) matrices each,
    FP64 and FP32 storage in turn, 2^24 matrices together at most."""
    rng = random.Random(case["sizes"])
    got, left = [], 1 << 24
    for k in range(case["requests"]):
        n = min(int(2 ** rng.uniform(0, case["max_log2"])), left)
        if n < 1:
            break
        got.append((n, k % 2 == 1))
        left -= n
    return got


def _pools(case, seed):
    """The requests' matrices, (6, n) each, side by side in one (6, total)
    tensor per storage type: FP64 from the separated mix, FP32 from the whole
    stress mix.  Returns {is_f32: tensor}."""
    reqs = _requests(case)
    pools = {}
    for f32 in (False, True):
        total = sum(n for n, f in reqs if f == f32)
        A = _draw_soa("stress_mix" if f32 else "separated_mix", max(total, 1),
                      2 * seed + f32)
        pools[f32] = (A.float() if f32 else A).contiguous()
    return reqs, pools


def _slices(reqs):
    """(is_f32, first, last) of every request in its pool."""
    at = {False: 0, True: 0}
    for n, f32 in reqs:
        yield f32, at[f32], at[f32] + n
        at[f32] += n


def prepare(case, seed):
    if case["kind"] == "batch":
        A = _inputs(case, seed)
        n, out = case["n"], None
        if case["out"]:
            soa = case["layout"] == "soa"
            lam = torch.empty((3, n) if soa else (n, 3), dtype=A.dtype, device="cuda")
            V = None
            if case["vectors"]:
                V = torch.empty((9, n) if soa else (n, 3, 3), dtype=A.dtype, device="cuda")
            out = (lam, V)
        return {"case": case, "A": A, "out": out}

    reqs, pools = _pools(case, seed)
    if case["kind"] == "segments":
        segs, outs = [], {}
        for f32, A in pools.items():
            # the requests' outputs, one after another in one buffer per type
            outs[f32] = (torch.empty(3 * A.shape[1], dtype=A.dtype, device="cuda"),
                         torch.empty(9 * A.shape[1], dtype=A.dtype, device="cuda")
                         if case["vectors"] else None)
        for f32, a, b in _slices(reqs):
            lam, V = outs[f32]
            segs.append((pools[f32][:, a:b], lam[3 * a:3 * b].view(3, b - a),
                         V[9 * a:9 * b].view(9, b - a) if case["vectors"] else None))
        used = sorted({f32 for _, f32 in reqs})
        return {"case": case, "segs": segs, "pools": pools,
                "outs": [t for f32 in used for t in outs[f32] if t is not None]}

    # host-staged serving: pinned buffers in and out, and the server's handle
    bufs = []
    for f32, a, b in _slices(reqs):
        host = [torch.empty((k, b - a), dtype=pools[f32].dtype, pin_memory=True)
                for k in ((6, 3, 9) if case["vectors"] else (6, 3))]
        host[0].copy_(pools[f32][:, a:b])
        bufs.append((s3.F32_REFINE if f32 else s3.F64, host[0], host[1],
                     host[2] if case["vectors"] else None))
    return {"case": case, "bufs": bufs, "server": serve.Server(hbm_budget_bytes=1 << 32)}


def run(state):
    case = state["case"]
    if case["kind"] == "batch":
        lam, V = s3.syev3(state["A"], vectors=case["vectors"], layout=case["layout"],
                          out=state["out"])
        return (lam, V) if case["vectors"] else lam
    if case["kind"] == "segments":
        s3.syev3_solve_segments_noalloc(state["segs"])
        return state["outs"]
    srv, reqs = state["server"], []
    for dtype, A, lam, V in state["bufs"]:
        r = srv.acquire(A.shape[1], dtype, vectors=V is not None)
        srv.submit_host(r, A, lam, V)
        reqs.append(r)
    for r in reqs:
        srv.wait(r)
        srv.release(r)
    return [t for _, _, lam, V in state["bufs"] for t in (lam, V) if t is not None]


def work(case):
    # per matrix: 6 entries (9 of a full matrix) in, 3 eigenvalues and 9
    # vector entries out; about 200 operations for the eigenvalues and 80
    # more for the vectors
    if case["kind"] == "batch":
        batches = [(case["n"], case["dtype"] == "f32")]
        entries = 9 if case["layout"] == "aos9" else 6
    else:
        batches, entries = _requests(case), 6
    values = entries + (12 if case["vectors"] else 3)
    return {"bytes": sum(n * values * (4 if f32 else 8) for n, f32 in batches),
            "flops": sum(n for n, _ in batches) * (280 if case["vectors"] else 200)}


def _eigenvalues(A):
    """Ascending eigenvalues (3, n) of (6, n) float64 entries: cyclic Jacobi
    rotations on the whole batch, each matrix scaled to unit size."""
    scale = A.abs().amax(0)
    scale = torch.where(scale > 0, scale, torch.ones_like(scale))
    a, b, c, d, e, f = A / scale  # a11 a12 a13 a22 a23 a33

    def rotate(p, q, r, x, y):
        """Annihilates r between the diagonal entries p and q; x and y are
        their couplings to the third.  Returns p, q, x, y."""
        t = 0.5 * (q - p)
        t = torch.where(t < 0, -1.0, 1.0) * r / (t.abs() + torch.hypot(t, r))
        t = torch.nan_to_num(t, nan=0.0)
        co = torch.rsqrt(1 + t * t)
        si = t * co
        return p - t * r, q + t * r, co * x - si * y, si * x + co * y

    zero = torch.zeros_like(a)
    for _ in range(7):
        a, d, c, e = rotate(a, d, b, c, e)  # a12 = 0
        b = zero
        a, f, b, e = rotate(a, f, c, b, e)  # a13 = 0
        c = zero
        d, f, b, c = rotate(d, f, e, b, c)  # a23 = 0
        e = zero
    lo, hi = torch.minimum(a, d), torch.maximum(a, d)
    return torch.stack([torch.minimum(lo, f), torch.maximum(lo, torch.minimum(hi, f)),
                        torch.maximum(hi, f)]) * scale


def exact(case, seed):
    # an eigenvector's sign is free: only the eigenvalues have one value
    if case["kind"] == "batch":
        A = _inputs(case, seed)
        if case["layout"] == "aos":
            A = A.t()
        elif case["layout"] == "aos9":
            A = A.reshape(-1, 9).t()[[0, 1, 2, 4, 5, 8]]
        lam = _eigenvalues(A.double())
        lam = lam if case["layout"] == "soa" else lam.t().contiguous()
        return (lam, None) if case["vectors"] else lam
    reqs, pools = _pools(case, seed)
    lams = {f32: _eigenvalues(A.double()) for f32, A in pools.items()}
    got = [(f32, lams[f32][:, a:b].contiguous()) for f32, a, b in _slices(reqs)]
    none = [None] if case["vectors"] else []
    if case["kind"] == "server":
        return [t for _, lam in got for t in [lam.cpu()] + none]
    return [t for f32 in sorted({f for f, _ in got})
            for t in [torch.cat([lam.reshape(-1) for f, lam in got if f == f32])] + none]
