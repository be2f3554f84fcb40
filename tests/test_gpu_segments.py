"""syev3_solve_segments_noalloc around the sizes where its table changes
place (the kernel's argument up to 56 segments, device memory above) and its
search takes another round (64 or 256 segments): every request equals, bit
for bit, the batched solver's result."""
import pytest
import torch

import paper_1806_06698_amd as s3
from paper_1806_06698_amd import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nseg,big", [(1, 0), (55, 0), (56, 0), (57, 0), (256, 0), (257, 0),
                                      (1024, 0), (56, 1100000), (57, 1100000)])
def test_tables(nseg, big):
    """Requests of 1 to 600 matrices, FP64 and FP32 in turn, every third
    without vectors; `big`: one more request large enough for the chunked
    order of tiles (4096 tiles and more)."""
    g = torch.Generator().manual_seed(nseg + big)
    sizes = torch.randint(1, 601, (nseg,), generator=g).tolist()
    if big:
        sizes[nseg // 2] = big
    A, _ = gen.stress_mix(sum(sizes), 80, "cuda")
    src = (A, A.float().contiguous())
    segs, off = [], 0
    for i, n in enumerate(sizes):
        a = src[i % 2][:, off:off + n]
        off += n
        segs.append((a, torch.full((3, n), float("nan"), dtype=a.dtype, device="cuda"),
                     None if i % 3 == 2 else
                     torch.full((9, n), float("nan"), dtype=a.dtype, device="cuda")))
    s3.syev3_solve_segments_noalloc(segs)
    ref = [s3.syev3(a) for a in src]
    off = 0
    for i, (n, (_, lam, V)) in enumerate(zip(sizes, segs)):
        l, v = ref[i % 2]
        assert torch.equal(lam, l[:, off:off + n]), i
        assert V is None or torch.equal(V, v[:, off:off + n]), i
        off += n


def test_calls_on_two_streams():
    """Calls whose table is the kernel's argument share nothing: two streams
    at once, many calls each."""
    A, _ = gen.stress_mix(40_000, 81, "cuda")
    lam, V = s3.syev3(A)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    outs = []
    for rep in range(20):
        for k, st in enumerate(streams):
            segs = []
            for i in range(20):
                a = A[:, (20 * k + i) * 1000:(20 * k + i + 1) * 1000]
                segs.append((a, torch.zeros(3, 1000, dtype=a.dtype, device="cuda"),
                             torch.zeros(9, 1000, dtype=a.dtype, device="cuda")))
            torch.cuda.synchronize()
            outs.append((k, segs))
    for k, segs in outs:
        s3.syev3_solve_segments_noalloc(segs, stream=streams[k])
    torch.cuda.synchronize()
    for k, segs in outs:
        for i, (_, l, v) in enumerate(segs):
            c = (20 * k + i) * 1000
            assert torch.equal(l, lam[:, c:c + 1000]) and torch.equal(v, V[:, c:c + 1000])


def test_a_captured_call_replays_with_its_own_table():
    """56 requests captured in a graph; before each replay new inputs, the
    outputs cleared and a call on other requests."""
    A, _ = gen.stress_mix(56 * 300, 82, "cuda")

    def requests(k, n):
        return [(A[:, i * n:(i + 1) * n], torch.zeros(3, n, dtype=A.dtype, device="cuda"),
                 torch.zeros(9, n, dtype=A.dtype, device="cuda")) for i in range(k)]

    segs, other = requests(56, 300), requests(60, 10)
    s3.syev3_solve_segments_noalloc(segs)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        s3.syev3_solve_segments_noalloc(segs)
    for rep in range(4):
        A.copy_(gen.stress_mix(56 * 300, 83 + rep, "cuda")[0])
        lam, V = s3.syev3(A)
        for _, l, v in segs:
            l.zero_()
            v.zero_()
        s3.syev3_solve_segments_noalloc(other)
        graph.replay()
        torch.cuda.synchronize()
        for i, (_, l, v) in enumerate(segs):
            assert torch.equal(l, lam[:, i * 300:(i + 1) * 300]), (rep, i)
            assert torch.equal(v, V[:, i * 300:(i + 1) * 300]), (rep, i)
