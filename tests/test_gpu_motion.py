"""The dispatch of a batch's data movement (workgroup order, non-temporal or
plain accesses, workgroups per compute unit) changes no result: around each of
its limits, for aligned and unaligned planes and in every layout, a batch
equals, bit for bit, the same matrices solved in small launches, which take
none of it."""
import pytest
import torch

import paper_1806_06698_amd as s3
from paper_1806_06698_amd import gen

pytestmark = pytest.mark.gpu

BLOCK = 256
PIECE = 1000 * BLOCK  # below every limit


def _pieces(A):
    """The solution of A (6, n), contiguous pieces solved one by one."""
    outs = [s3.syev3(A[:, i:i + PIECE].contiguous()) for i in range(0, A.shape[1], PIECE)]
    return torch.cat([l for l, _ in outs], 1), torch.cat([v for _, v in outs], 1)


def _strided(rows, n, ld, first, dtype):
    """An uninitialised (rows, n) view, row stride ld, `first` elements into
    its buffer."""
    return torch.empty(rows * ld + first, dtype=dtype,
                       device="cuda")[first:].view(rows, ld)[:, :n]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("n", [1280 * BLOCK - 1, 1280 * BLOCK, 1281 * BLOCK + 5,
                               3071 * BLOCK, 3072 * BLOCK, 3072 * BLOCK + 1,
                               5000 * BLOCK + 77])
def test_limits(n, dtype):
    A, _ = gen.stress_mix(n, 60, "cuda")
    A = A.to(dtype).contiguous()
    lam, V = _pieces(A)
    got = {"default": s3.syev3(A)}
    # the planes of every array on 128-byte lines, and off them
    up = (n + 31) // 32 * 32
    for name, ld, first in (("aligned", up, 0), ("offset", up, 1), ("odd stride", up + 1, 0)):
        out = (_strided(3, n, ld, first, dtype), _strided(9, n, ld, first, dtype))
        got[name] = s3.syev3(A, out=out)
    for name, (l, v) in got.items():
        assert torch.equal(l, lam) and torch.equal(v, V), name
    assert torch.equal(s3.syev3(A, vectors=False)[0], lam)
    la, va = s3.syev3(gen.to_aos(A), layout="aos")
    assert torch.equal(la.t(), lam) and torch.equal(va.reshape(n, 9).t(), V)


def test_planes_half_a_gigabyte_apart():
    """Plane strides at and within 64 KB of 2^29 bytes (chunks of 256 tiles),
    just outside, and at 2^31 bytes (chunks of 32)."""
    n = 4100 * BLOCK + 33
    A, _ = gen.stress_mix(n, 61, "cuda")
    lam, V = _pieces(A)
    for ld in (1 << 26, (1 << 26) - (1 << 13), (1 << 26) + (1 << 13), (1 << 26) + (1 << 14),
               1 << 28):
        l, v = s3.syev3(A, out=(_strided(3, n, ld, 0, A.dtype), _strided(9, n, ld, 0, A.dtype)))
        assert torch.equal(l, lam) and torch.equal(v, V), ld
        del l, v
        torch.cuda.empty_cache()


def test_eigenvalues_alone_from_planes_half_a_gigabyte_apart():
    """The same for the input's planes, whose stride chooses the order where
    only eigenvalues are asked for."""
    n = 4100 * BLOCK + 33
    A, _ = gen.stress_mix(n, 62, "cuda")
    lam, _ = _pieces(A)
    for ld in (1 << 26, (1 << 26) - (1 << 13), (1 << 26) + (1 << 14)):
        B = _strided(6, n, ld, 0, A.dtype)
        B.copy_(A)
        assert torch.equal(s3.syev3(B, vectors=False)[0], lam), ld
        del B
        torch.cuda.empty_cache()


@pytest.mark.parametrize("n", [2047 * BLOCK + 1, 2047 * BLOCK - 1])
def test_unaligned_fp32_planes(n):
    """Around the size from which FP32 storage with planes off 128-byte lines
    takes plain accesses and the chunked order."""
    A, _ = gen.stress_mix(n, 63, "cuda")
    A = A.float().contiguous()
    lam, V = _pieces(A)
    l, v = s3.syev3(A)
    assert torch.equal(l, lam) and torch.equal(v, V)


@pytest.mark.parametrize("blocks", [2559, 2560, 3640, 3641, 5461, 5462, 16383, 16384])
def test_packed_rows(blocks):
    """AoS FP64 around the limits of its workgroup caps (2560 and 16384 blocks)
    and of the plain loads (64 MB of input: 5461 blocks of packed rows, 3640 of full
    matrices), with a full and a short last tile; full matrices also solved
    in place, also from an address that no 16-byte load may take."""
    for n in (blocks * BLOCK, blocks * BLOCK - 100):
        A, _ = gen.stress_mix(n, 64, "cuda")
        lam, V = _pieces(A)
        full = gen.to_full(A).contiguous()
        for layout, rows in (("aos", gen.to_aos(A).contiguous()), ("aos9", full),
                             ("aos9", full.reshape(n, 9))):
            l, v = s3.syev3(rows, layout=layout)
            assert torch.equal(l.t(), lam) and torch.equal(v.reshape(n, 9).t(), V), layout
        for first in (0, 1):
            M = torch.empty(9 * n + first, dtype=A.dtype,
                            device="cuda")[first:].view(n, 3, 3).copy_(full)
            l = s3.syev3_inplace(M)
            assert torch.equal(l.t(), lam) and torch.equal(M.reshape(n, 9).t(), V), first


def test_unrefined_fp32_planes_a_quarter_gigabyte_apart():
    """The unrefined FP32 form's planes at and next to 2^28 bytes apart."""
    n = 4100 * BLOCK + 33
    A, _ = gen.stress_mix(n, 65, "cuda")
    A = A.float().contiguous()
    pieces = [s3.syev3(A[:, i:i + PIECE].contiguous(), refine=False)
              for i in range(0, n, PIECE)]
    lam, V = (torch.cat(p, 1) for p in zip(*pieces))
    for ld in (1 << 26, (1 << 26) - (1 << 14), (1 << 26) + (1 << 14), (1 << 26) + (1 << 15)):
        out = (_strided(3, n, ld, 0, A.dtype), _strided(9, n, ld, 0, A.dtype))
        l, v = s3.syev3(A, out=out, refine=False)
        assert torch.equal(l, lam) and torch.equal(v, V), ld
        del l, v, out
        torch.cuda.empty_cache()


@pytest.mark.parametrize("n", [(1 << 29) + 64, (1 << 29) + (1 << 26)])
def test_64_bit_offsets_with_aligned_planes(n):
    """Planes of more than 2^32 bytes, all on 128-byte lines: the hinted
    variants of the kernel with 64-bit offsets (an odd count takes the plain
    one), with planes a multiple of 2^31 bytes apart and one of 2^29 alone,
    which loads without the hint.  The input repeats one piece, and every
    repeat equals it."""
    piece = 1 << 20
    base, _ = gen.stress_mix(piece, 66, "cuda")
    lam, V = s3.syev3(base)
    A = torch.empty(6, n, dtype=torch.float64, device="cuda")
    for i in range(0, n, piece):
        A[:, i:i + piece] = base[:, :n - i]
    l, v = s3.syev3(A)
    del A
    for i in range(0, n, piece):
        m = min(piece, n - i)
        assert torch.equal(l[:, i:i + m], lam[:, :m]), i
        assert torch.equal(v[:, i:i + m], V[:, :m]), i
    del l, v
    torch.cuda.empty_cache()


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("n", [1023 * BLOCK, 1023 * BLOCK + 16, 1024 * BLOCK, 1024 * BLOCK + 32])
def test_hinted_stores(n, dtype):
    """FP64 around the size from which planes on 128-byte lines are stored
    with the non-temporal hint (1024 blocks), beside planes off them."""
    A, _ = gen.stress_mix(n, 67, "cuda")
    A = A.to(dtype).contiguous()
    lam, V = _pieces(A)
    for ld, first in (((n + 31) // 32 * 32, 0), (n, 0), (n + 1, 0), (n, 1)):
        out = (_strided(3, n, ld, first, dtype), _strided(9, n, ld, first, dtype))
        l, v = s3.syev3(A, out=out)
        assert torch.equal(l, lam) and torch.equal(v, V), (ld, first)
