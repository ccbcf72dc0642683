"""Streaming sweeps in the forms and at the sizes that the automatic rules
leave to them beside the resident tiles."""
import numpy as np
import pytest

import oracle
from paper_1807_07382_amd import pentbatch as pb
from tests._gpu import U, colerr, d4_tol, print_case, torch_dev
from tests.test_gpu_stream import probes, rand

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return torch_dev()


def circulant_lu(stencil, n):
    """Sparse LU (pivoted) and the matrix of a row-invariant periodic stencil
    a..e, with its condition number in the infinity norm (the inverse is
    circulant too, so one column gives its norm)."""
    import scipy.sparse as sp
    import scipy.sparse.linalg as sl
    A = sum(sp.diags([v] * n, 0, shape=(n, n)).dot(sp.csr_matrix(
        (np.ones(n), (np.arange(n), (np.arange(n) + o) % n)), shape=(n, n))) for o, v in zip(range(-2, 3), stencil))
    lu = sl.splu(A.tocsc())
    e0 = np.zeros(n)
    e0[0] = 1.0
    return lu, A.tocsr(), np.sum(np.abs(stencil)) * np.sum(np.abs(lu.solve(e0)))


# an advected operator: the bottom end of the border's reach grows with the
# advection, to 16 blocks of 32 rows (as many as the workgroup has waves) at
# 9; at 10 and 20, and in the upwind step, it is longer
@pytest.mark.parametrize("stencil", [(1, -8, 11, -4, 1), (1, -13, 16, -4, 1), (1, -14, 17, -4, 1), (1, -24, 27, -4, 1),
                                     (0, -20, 21, 0, 0)])
def test_periodic_one_sided_reach(torch, stencil):
    """Solves and steps with matrices whose border reaches further up from the
    bottom than down from the top."""
    n, m = 4100, 8200
    print_case(test="periodic_reach", stencil=stencil)
    C = rand(torch, (n, m), 5)
    X = torch.empty_like(C)
    c = probes(m, 48)
    Cc = C[:, c].cpu().numpy()
    lu, A, kappa = circulant_lu(np.array(stencil, float), n)
    with pb.Cyclic.factor(*[np.full(n, float(v)) for v in stencil]) as cy:
        cy.cn_step(C, X)
        F = cy.solve_(C)
        cy.check()
    tol = 64 * U * kappa
    assert np.max(colerr(F[:, c].cpu().numpy(), lu.solve(Cc))) <= tol
    ref = lu.solve(2 * Cc - A @ Cc)
    err = np.max(np.abs(X[:, c].cpu().numpy() - ref), axis=0)
    scale = np.max(np.abs(ref), axis=0) + (2 + np.sum(np.abs(stencil))) * np.max(np.abs(Cc), axis=0)
    assert np.all(err <= tol * scale)
