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


def tail_columns(F, cols, row):
    """The columns cols of F (systems along dim 1) zero but for one row."""
    F[:, cols] = 0.0
    F[row, cols] = 1.0


def assert_tails(X, ref, sigma, rows):
    """Relative error of every stretch of rows on its own (a row adds a few
    roundings to the relative error of a tail)."""
    n = len(ref)
    for r in range(0, n, rows):
        big = np.max(np.abs(ref[r:r + rows]), axis=0)
        err = np.max(np.abs(X[r:r + rows] - ref[r:r + rows]), axis=0)
        assert np.all(err <= n * d4_tol(sigma) * big + 1e-290), r


# one to three blocks, whole and partial, rows on lines of their own and not,
# tiles of 32 to 64 systems with partial last ones; the first size past the
# rule; chains as deep as the matrix
@pytest.mark.parametrize("n,m,ld,off", [(1, 10000, 1, 0), (31, 20011, 31, 0), (32, 10000, 32, 0), (33, 10001, 48, 0),
                                        (64, 33000, 64, 0), (65, 12345, 65, 1), (95, 10050, 97, 0), (96, 40000, 96, 0),
                                        (96, 10007, 112, 1), (97, 10000, 97, 0)])
@pytest.mark.parametrize("sigma", [0.1, 1e4])
def test_system_major_few_blocks(torch, n, m, ld, off, sigma):
    """System-major solves of matrices of a few blocks: every system against
    the oracle at the edges, the gaps untouched, far tails right, non-finite
    systems alone."""
    print_case(test="t_few_blocks", n=n, m=m, ld=ld, off=off, sigma=sigma)
    buf = rand(torch, (m * ld + off,), n + m)
    F = buf[off:].view(m, ld)
    c = probes(m, 48)
    tail = np.array([2, 40, m - 3])
    tail_columns(F.t(), tail, n - 1)
    B = F.clone()
    F[5, n // 2] = float("nan")
    with pb.Plan.factor_d4(n, sigma) as p:
        p.solve_strided_(F[:, :n])
        p.check()
    assert torch.equal(F[:, n:], B[:, n:])
    dg = oracle.assemble_d4(n, sigma)
    ref = oracle.solve(dg, np.ascontiguousarray(B[c, :n].T.cpu().numpy()))
    assert np.max(colerr(F[c, :n].T.cpu().numpy(), ref)) <= d4_tol(sigma)
    ref = oracle.solve(dg, np.ascontiguousarray(B[tail, :n].T.cpu().numpy()))
    assert_tails(F[tail, :n].T.cpu().numpy(), ref, sigma, 16)
    assert not bool(torch.isfinite(F[5, :n]).any()) and bool(torch.isfinite(F[[4, 6], :n]).all())


@pytest.mark.parametrize("n,m,sigma", [(640, 10050, 5.0), (1537, 10007, 1.0), (2048, 12000, 50.0), (2113, 10003, 5.0)])
def test_system_major_far_tails(torch, n, m, sigma):
    print_case(test="t_tails", n=n, m=m, sigma=sigma)
    F = rand(torch, (m, n), n)
    c = np.array([0, 17, 63, 64, m - 1])
    tail_columns(F.t(), c, n - 1)
    tail_columns(F.t(), c[1:2], n // 2)
    ref = oracle.solve(oracle.assemble_d4(n, sigma), np.ascontiguousarray(F[c].T.cpu().numpy()))
    with pb.Plan.factor_d4(n, sigma) as p:
        p.solve_strided_(F)
        p.check()
    assert_tails(F[c].T.cpu().numpy(), ref, sigma, 128)


# x rows of one to three blocks and of resident tiles; instances that end
# inside a tile; an odd row length
@pytest.mark.parametrize("ny,ninst,nx", [(400, 26, 64), (130, 80, 95), (1000, 11, 96), (3340, 3, 33), (10010, 1, 31),
                                         (400, 26, 600), (700, 15, 1500)])
@pytest.mark.parametrize("off", [0, 1])
def test_grid_step_with_many_rows(torch, ny, ninst, nx, off):
    """A 2-D step whose x sweeps have at least 10000 systems: the explicit
    term formed in the sweeps gives the bits of the separate passes, aligned
    and not."""
    print_case(test="ch2d_many", ny=ny, ninst=ninst, nx=nx, off=off)
    sigma, h = 20.0, 1.0 / nx
    g = np.random.Generator(np.random.PCG64(ny + nx))
    dt = torch.from_numpy(sigma * h ** 4 / g.uniform(1e-3, 1e-1, ninst)).cuda()
    C = (0.1 * rand(torch, (ny * ninst * nx + off,), ny + nx))[off:].view(ny, ninst, nx)
    R = torch.empty(ny * ninst * nx + off, dtype=torch.float64, device="cuda")[off:].view(ny, ninst, nx)
    R2 = torch.empty((ny, ninst, nx), dtype=torch.float64, device="cuda")
    with pb.Plan.factor_d4(nx, sigma) as px, pb.Plan.factor_d4(ny, sigma) as py:
        pb.ch2d_rhs(C, R2, dt, h)
        px.solve_strided_(R2.view(ny * ninst, nx))
        pb.ch2d_step(px, py, C, R, dt, h)
        px.check()
        py.check()
    assert torch.equal(R, R2)
