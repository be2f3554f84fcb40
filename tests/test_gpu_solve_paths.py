"""Branches of the solve that only some matrices take, each against the path
that every matrix could take."""
import numpy as np
import pytest
import torch

import checks
import oracle
import paper_1806_06698_amd as s3

pytestmark = pytest.mark.gpu


def _arrows(n, seed):
    """Matrices with max |a_ij| in [1/2, 1) (nothing to scale), a12 = 0 and
    betas of 10^U(-12, 0): alpha beta1 beta2 on both sides of 2^-48, some
    exactly zero."""
    g = torch.Generator().manual_seed(seed)
    A = 0.98 * torch.rand((6, n), generator=g, dtype=torch.float64) - 0.49
    A[5] = torch.where(A[5] < 0, -0.75, 0.75)
    A[1] = 0
    for k in (2, 4):
        A[k] *= 10.0 ** (-12 * torch.rand(n, generator=g, dtype=torch.float64))
        A[k][torch.rand(n, generator=g) < 0.05] = 0
    return A


@pytest.mark.parametrize("flags", [0, s3.FLAG_SIMPLIFIED_DEFLATION, s3.FLAG_NO_H_GUARD])
def test_deflation_tests_skipped_or_taken(flags):
    """FLAG_NO_SCALE always takes the deflation tests; without it wavefronts
    all of whose lanes are far from deflating skip them.  On matrices that
    need no scaling both give the same bits, also where each matrix fills a
    wavefront (all lanes skip, or none)."""
    A = _arrows(6000, 71)
    A = torch.cat([A, A[:, :500].repeat_interleave(64, 1)], 1).contiguous().cuda()
    a = s3.syev3(A, flags=flags, info=True)
    b = s3.syev3(A, flags=flags | s3.FLAG_NO_SCALE, info=True)
    for x, y in zip(a, b):
        assert torch.equal(x, y)
    assert set((a[2] & 0xFF).unique().tolist()) == {2, 3, 4}


@pytest.mark.parametrize("kind", ["nearly isotropic", "tiny betas"])
def test_zeros_outside_fp32(kind):
    """Arrows whose squares leave FP32's range, so that the zero finder's FP32
    start is useless: I + 10^-k S (k to 15), and betas of 10^-10 to 10^-150
    beside an alpha of the same size.  The bars are the parity tests' 16 eps."""
    g = np.random.default_rng(72)
    n = 20_000
    A6 = g.normal(size=(n, 6))
    if kind == "nearly isotropic":
        A6 *= 10.0 ** -g.uniform(5, 15, size=(n, 1))
        A6[:, [0, 3, 5]] += 1.0
    else:
        t = 10.0 ** -g.uniform(10, 150, size=n)
        A6[:, 1] = 0
        A6[:, 2] *= t
        A6[:, 4] *= t
        A6[:, 3] = A6[:, 0] + t * g.normal(size=n)
    lam, V = s3.syev3(torch.from_numpy(np.ascontiguousarray(A6.T)).cuda())
    lam, V = lam.t().cpu().numpy(), V.t().cpu().numpy().reshape(n, 3, 3)
    lam_o, _ = oracle.solve(A6)
    worst = (checks.eig_error(A6, lam, lam_o).max(), checks.residual(A6, lam, V).max(),
             checks.orthogonality(V).max())
    print(kind, "max eigenvalue error, residual, orthogonality (eps):", worst, flush=True)
    assert max(worst) <= 16.0
