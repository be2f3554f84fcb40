"""Matrices whose entries span many orders of magnitude, where the zero
finder's starts can be far from the zeros: every result meets the parity
tests' bars (FP64 16 eps, FP32 storage 3 eps32) in residual and
orthogonality, and in its eigenvalues against the oracle."""
import numpy as np
import pytest
import torch

import paper_1806_06698_amd as s3
from gpu_common import EPS32, EPS64, check_vs_oracle, device_measures

pytestmark = pytest.mark.gpu

N = 60_000
DIAGONAL = np.array([1, 0, 0, 1, 0, 1])


def _graded(kind, span, seed):
    """(6, n): entries N(0,1) 10^-U(0, span); "zeros": 30% of them zero;
    "arrow": large a13 and a23 over a small rest, graded each;
    "isotropic": 10^-U(0, 16) of them, beside a multiple of I."""
    g = np.random.default_rng(seed)
    A = g.standard_normal((N, 6)) * 10.0 ** (-span * g.random((N, 6)))
    if kind == "zeros":
        A[g.random((N, 6)) < 0.3] = 0
    elif kind == "arrow":
        rest = 10.0 ** (-span * g.random((N, 1))) * g.standard_normal((N, 6))
        A = A * [0, 1, 1, 0, 1, 0] + rest * DIAGONAL
    elif kind == "isotropic":
        A = A * 10.0 ** (-16 * g.random((N, 1))) + DIAGONAL * g.standard_normal((N, 1))
    return torch.from_numpy(np.ascontiguousarray(A.T))


@pytest.mark.parametrize("kind", ["all", "zeros", "arrow", "isotropic"])
def test_fp64(kind):
    for span in (20, 30, 40, 60, 100, 150, 300):
        A = _graded(kind, span, span).cuda()
        lam, V = s3.syev3(A)
        res, orth = device_measures(A, lam, V)
        bad = ~(torch.maximum(res, orth) <= 16 * EPS64)  # a NaN is bad
        assert not bad.any(), (span, int(bad.sum()), A[:, bad][:, 0].tolist())
        check_vs_oracle(A, lam, V, sample=4000, seed=span, label=f"{kind} 10^-{span}")
        assert torch.equal(s3.syev3(A, vectors=False)[0], lam)


@pytest.mark.parametrize("flags", [0, s3.FLAG_REFINE_CONVERGE])
@pytest.mark.parametrize("kind", ["all", "zeros", "arrow", "isotropic"])
def test_fp32_storage(kind, flags):
    for span in (20, 30, 40):
        A = _graded(kind, span, 1000 + span).float()
        # eigenvalues that FP32 holds to 2^-24 of the matrix
        A = A[:, A.abs().amax(0) > 1e-30].contiguous().cuda()
        lam, V = s3.syev3(A, flags=flags)
        res, orth = device_measures(A, lam, V)
        bad = ~(torch.maximum(res, orth) <= 3 * EPS32)
        assert not bad.any(), (span, int(bad.sum()), A[:, bad][:, 0].tolist())
        check_vs_oracle(A, lam, V, f32=True, sample=4000, seed=span,
                        label=f"{kind} 10^-{span} f32")
