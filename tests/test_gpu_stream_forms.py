"""Streaming sweeps in the forms and at the sizes that the automatic rules
leave to them beside the resident tiles."""
import numpy as np
import pytest

import oracle
from paper_1807_07382_amd import pentbatch as pb
from tests._gpu import U, colerr, d4_tol, print_case, torch_dev
from tests.test_gpu_stream import cyc_lu, probes, rand
from tests.test_oracle_pins import random_dd

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
    n, m = 4100, 10011
    print_case(test="periodic_reach", stencil=stencil)
    C = rand(torch, (n, m), 5)
    X = torch.empty_like(C)
    c = probes(m, 48)
    Cc = C[:, c].cpu().numpy()
    lu, A, kappa = circulant_lu(np.array(stencil, float), n)
    with pb.Cyclic.factor(*[np.full(n, float(v)) for v in stencil]) as cy:
        assert cy.form_for(m) == (pb.FORM_STREAM if stencil[1] >= -13 and stencil[0] else pb.FORM_SCHEDULE)
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
        assert p.form_for(m, True) == (pb.FORM_STREAM if n <= 96 else pb.FORM_RESIDENT)
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
        assert p.form_for(m, True) == (pb.FORM_RESIDENT if n <= 2048 else pb.FORM_SCHEDULE)
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
        assert px.form_for(ny * ninst, True) == (pb.FORM_STREAM if nx <= 96 else pb.FORM_RESIDENT)
        pb.ch2d_rhs(C, R2, dt, h)
        px.solve_strided_(R2.view(ny * ninst, nx))
        pb.ch2d_step(px, py, C, R, dt, h)
        px.check()
        py.check()
    assert torch.equal(R, R2)


def d4_extended(n, sigma, F):
    """(I + sigma D4)^{-1} F with 50 digits, rounded to the 64-bit mantissa of a
    long double: the recurrences of the factorisation row by row (no pivoting
    is needed, the matrix is symmetric positive definite).  The far tails of a
    solution have n roundings and more in them, so that a long double's own
    arithmetic would show in a relative error of one rounding of a double."""
    import decimal
    D = decimal.Decimal
    dg = oracle.assemble_d4(n, sigma)
    with decimal.localcontext() as ctx:
        ctx.prec = 50
        a, b, c, d, e = ([D(float(v)) for v in getattr(dg, k)] for k in "abcde")
        zero = D(0)
        ga, de, al, be = [zero] * (n + 2), [zero] * (n + 2), [zero] * n, [zero] * n  # ga, de from row -2 on
        for i in range(n):
            be[i] = b[i] - a[i] * ga[i]
            al[i] = 1 / (c[i] - a[i] * de[i] - be[i] * ga[i + 1])
            ga[i + 2] = (d[i] - be[i] * de[i + 1]) * al[i]
            de[i + 2] = e[i] * al[i]
        out = np.empty(F.shape, np.longdouble)
        for j in range(F.shape[1]):
            g2, g1, g = zero, zero, []
            for i in range(n):
                g2, g1 = g1, (D(float(F[i, j])) - a[i] * g2 - be[i] * g1) * al[i]
                g.append(g1)
            x1, x2 = zero, zero
            for i in range(n - 1, -1, -1):
                x1, x2 = g[i] - ga[i + 2] * x1 - de[i + 2] * x2, x1
                hi = float(x1)
                out[i, j] = np.longdouble(hi) + np.longdouble(float(x1 - D(hi)))
    return out


def refined(torch, p, F, steps, f32=False):
    assert p.form_for(F.shape[1]) == pb.FORM_STREAM
    X = torch.empty(F.shape, dtype=torch.float64, device="cuda")
    p.solve_mixed(F.float() if f32 else F, X, steps)
    p.check()
    return X


@pytest.mark.parametrize("n,m,sigma", [(2048, 5120, 100.0), (2050, 6000, 1.0), (4099, 5123, 30.0), (700, 9000, 0.1)])
@pytest.mark.parametrize("f32,steps", [(False, 1), (True, 1), (False, 2)])
def test_corrections_keep_far_tails(torch, n, m, sigma, f32, steps):
    """A corrected solve is right to rounding in every stretch of rows on its
    own, also where the solution is the far tail of a source many rows below:
    with a relative error of n d4_tol in x and in the correction of such a
    tail, what is left after it is the square of that and one rounding of x."""
    print_case(test="fix_tails", n=n, m=m, sigma=sigma, f32=f32, steps=steps)
    F = rand(torch, (n, m), n).float().double()
    c = np.array([0, 1, 17, 63, 64, m - 1])
    for col, row in zip(c[[0, 2, 3, 5]], (n - 1, n - 1, n // 2, n - 3)):
        tail_columns(F, [col], row)
    ref = d4_extended(n, sigma, F[:, c].cpu().numpy())
    with pb.Plan.factor_d4(n, sigma) as p:
        X = refined(torch, p, F, steps, f32)[:, c].cpu().numpy()
    tol = 2 * U + (n * d4_tol(sigma)) ** 2
    for r in range(0, n, 256):
        big = np.max(np.abs(ref[r:r + 256]), axis=0)
        err = np.max(np.abs(X[r:r + 256] - ref[r:r + 256]), axis=0)
        assert np.all(err <= tol * big + 1e-290), (r, err / big)


@pytest.mark.parametrize("f32", [False, True])
def test_corrections_beside_small_values(torch, f32):
    """Systems whose solution is zero in a few rows at the end of a block of
    32, and of order 1000 elsewhere: there the state that the correction's
    chain leaves out counts against x, though x falls nowhere over the rows
    that the kernel samples.  x and f are whole numbers, so the solution is
    known.  The first solve is within d4_tol, the correction within d4_tol of
    that and the compensated residual's u^2 sum |a x|, and one rounding of x."""
    n, m, sigma = 8192, 5120, 4.0
    print_case(test="fix_small_values", f32=f32)
    F = rand(torch, (n, m), 7).float().double()
    c = np.array([0, 3, 70, 71, m - 1])
    x = np.random.Generator(np.random.PCG64(3)).integers(-1000, 1000, (n, len(c))).astype(float)
    for k, at in enumerate((32, 32 * 33, 32 * 97, 32 * 130, 32 * 201)):
        x[at - 2:at + 4, k] = 0.0
    p = np.pad(x, ((2, 2), (0, 0)))
    f = 4 * p[:-4] - 16 * p[1:-3] + 25 * p[2:-2] - 16 * p[3:-1] + 4 * p[4:]
    old = F[:, c].clone()
    F[:, c] = torch.from_numpy(f).cuda()
    keep = np.setdiff1d(np.arange(m), c)
    with pb.Plan.factor_d4(n, sigma) as plan:
        X = refined(torch, plan, F, 1, f32)
        F[:, c] = old
        Y = refined(torch, plan, F, 1, f32)
    assert torch.equal(X[:, keep], Y[:, keep])  # the neighbours' bits do not depend on it
    tol = d4_tol(sigma)
    err = np.abs(X[:, c].cpu().numpy() - x)
    assert np.all(err <= U * np.abs(x) + 1000 * (tol ** 2 + 5 * 65 * U ** 2))


def test_corrections_of_many_tiles(torch):
    """More tiles to a workgroup than the streaming sweeps have slots for (32),
    some left to the other form, with partial tiles; all columns by the
    backward error, some against extended precision."""
    n, m, sigma = 70, 64 * 256 * 33 + 21, 5.0
    print_case(test="fix_many")
    F = rand(torch, (n, m), 3)
    F[:-1, 100_000:100_010] = 0.0
    F[:-1, -1] = 0.0
    eta = torch.empty(m, dtype=torch.float64, device="cuda")
    X = torch.empty_like(F)
    c = np.array([0, 99_999, 100_000, 100_009, 100_010, m - 2, m - 1])
    with pb.Plan.factor_d4(n, sigma) as p:
        assert p.form_for(m) == pb.FORM_STREAM
        p.solve_mixed(F, X, 1, eta)
        p.check()
    assert eta.max().item() <= 2 * U
    ref = d4_extended(n, sigma, F[:, c].cpu().numpy())
    assert np.max(colerr(X[:, c].cpu().numpy(), ref.astype(float))) <= 4 * U


@pytest.mark.parametrize("n,m,pad", [(777, 12000, 0), (1500, 9001, 3), (2600, 6000, 16)])
def test_general_matrix_and_bits_by_column(torch, n, m, pad):
    """Non-symmetric matrices, rows on lines of their own and not; every
    system has the same bits wherever it sits in the batch, and a system that
    is zero but for one row does not change its neighbours'."""
    print_case(test="stream_general", n=n, m=m, pad=pad)
    dg = random_dd(n, seed=n)
    B = rand(torch, (n, m + pad), 3)
    F = B[:, :m]
    perm = torch.randperm(m, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    c = probes(m, 48)
    with pb.Plan.factor(*dg) as p:
        assert p.form_for(m) == pb.FORM_STREAM
        X = p.solve_(B.clone()[:, :m])
        Y = p.solve_(F[:, perm].contiguous())
        Z = F.clone()
        tail_columns(Z, c, n - 1)
        ref_tail = oracle.solve(dg, np.ascontiguousarray(Z[:, c].cpu().numpy()))
        p.solve_(Z)
        p.check()
    assert torch.equal(X[:, perm], Y)
    keep = np.setdiff1d(np.arange(m), c)
    assert torch.equal(X[:, keep], Z[:, keep])
    ref = oracle.solve(dg, np.ascontiguousarray(F[:, c].cpu().numpy()))
    assert np.max(colerr(X[:, c].cpu().numpy(), ref)) <= 1e-13
    for r in range(0, n, 64):
        big = np.max(np.abs(ref_tail[r:r + 64]), axis=0)
        err = np.max(np.abs(Z[r:r + 64][:, c].cpu().numpy() - ref_tail[r:r + 64]), axis=0)
        assert np.all(err <= n * 1e-13 * big + 1e-290)


@pytest.mark.parametrize("f32", [False, True])
def test_more_tiles_than_slots(torch, f32):
    """More tiles to a workgroup than the 32 slots in which it notes what its
    blocks left out, some with far tails, one with a NaN, a partial last one."""
    n, m, sigma = 160, 64 * 256 * 33 + 21, 0.1
    print_case(test="stream_many", f32=f32)
    F = rand(torch, (n, m), 3).float()
    F = F if f32 else F.double()
    c = np.array([0, 63, 64 * 256 * 16, 64 * 256 * 32 + 5, m - 1])
    tail_columns(F, c, n - 1)
    F[n // 2, 200] = float("nan")
    other = np.array([1, 62, 199, 201, 64 * 256 * 32 + 6, m - 2])
    X = torch.empty((n, m), dtype=torch.float64, device="cuda")
    with pb.Plan.factor_d4(n, sigma) as p:
        assert p.form_for(m) == pb.FORM_STREAM
        p.solve_mixed(F, X, 0)
        p.check()
    dg = oracle.assemble_d4(n, sigma)
    assert not bool(torch.isfinite(X[:, 200]).any())
    ref = oracle.solve(dg, np.ascontiguousarray(F[:, other].double().cpu().numpy()))
    assert np.max(colerr(X[:, other].cpu().numpy(), ref)) <= d4_tol(sigma)
    ref = oracle.solve(dg, np.ascontiguousarray(F[:, c].double().cpu().numpy()))
    assert_tails(X[:, c].cpu().numpy(), ref, sigma, 32)


# E rows on and off block edges, one to 32 rows in the last block; few and many
# end blocks; tiles of 32 to 64 systems
@pytest.mark.parametrize("n,m,pad,sigma", [(514, 10000, 0, 0.1), (515, 16400, 3, 1.0), (1027, 10000, 16, 50.0),
                                           (1057, 10001, 0, 50.0), (2047, 12300, 0, 300.0), (4097, 10240, 0, 0.01)])
def test_periodic_edges(torch, n, m, pad, sigma):
    """Periodic solves and steps against an independent sparse LU (the bounds
    are those of the periodic streaming test)."""
    print_case(test="cyc_edges", n=n, m=m, pad=pad, sigma=sigma)
    B = rand(torch, (n, m + pad), n + 1)
    X = torch.full((n, m + pad), 7.0, dtype=torch.float64, device="cuda")
    F = B.clone()
    c = probes(m, 48)
    Bc = B[:, c].cpu().numpy()
    lu, A = cyc_lu(n, sigma)
    with pb.Cyclic.factor_d4(n, sigma) as cy:
        assert cy.form_for(m) == cy.form_for(m, True) == pb.FORM_STREAM
        cy.solve_(F[:, :m])
        cy.cn_step(B[:, :m], X[:, :m])
        cy.check()
    assert torch.equal(F[:, m:], B[:, m:]) and bool((X[:, m:] == 7.0).all())
    assert np.max(colerr(F[:, c].cpu().numpy(), lu.solve(Bc))) <= d4_tol(sigma)
    ref = lu.solve(2 * Bc - A @ Bc)
    err = np.max(np.abs(X[:, c].cpu().numpy() - ref), axis=0)
    assert np.all(err <= d4_tol(sigma) * (np.max(np.abs(ref), axis=0) + (2 + 16 * sigma) * np.max(np.abs(Bc), axis=0)))


@pytest.mark.parametrize("n,m", [(1300, 10000), (1537, 16403)])
def test_periodic_varying_rows(torch, n, m):
    """Diagonals that differ from row to row (the step reads them per row), and
    the look-back form of the same calls."""
    print_case(test="cyc_rows", n=n, m=m)
    g = np.random.Generator(np.random.PCG64(2))
    dg = [g.uniform(-1, 1, n) for _ in range(5)]
    dg[2] = 5.0 + g.uniform(0, 1, n)
    A = np.zeros((n, n))
    for o in range(-2, 3):
        for r in range(n):
            A[r, (r + o) % n] += dg[o + 2][r]
    C = rand(torch, (n, m), 6)
    X, Y = torch.empty_like(C), torch.empty_like(C)
    c = probes(m, 64)
    Cc = C[:, c].cpu().numpy()
    with pb.Cyclic.factor(*dg) as cy:
        assert cy.form_for(m) == cy.form_for(m, True) == pb.FORM_STREAM
        cy.cn_step(C, X)
        F = cy.solve_(C.clone())
        cy.set_schedule(2, 64)
        assert cy.form_for(m) == cy.form_for(m, True) == pb.FORM_SCHEDULE
        cy.cn_step(C, Y)
        cy.check()
    kappa = np.linalg.cond(A, np.inf)
    assert np.max(colerr(F[:, c].cpu().numpy(), np.linalg.solve(A, Cc))) <= 64 * U * kappa
    ref = np.linalg.solve(A, 2 * Cc - A @ Cc)
    tol = 64 * U * kappa * 12 * np.max(np.abs(Cc))
    assert np.max(np.abs(X[:, c].cpu().numpy() - ref)) <= tol
    assert float((X - Y).abs().max()) <= 2 * tol


@pytest.mark.parametrize("row", [0, 600, 1199])
def test_periodic_far_tails_and_non_finite(torch, row):
    """The tails of one non-zero row both ways round, as by the look-back form,
    in each stretch of rows; a NaN spoils its own system only."""
    n, m, sigma = 1200, 10000, 20.0
    print_case(test="cyc_tail", row=row)
    F = rand(torch, (n, m), 9)
    c = np.array([0, 17, 63, 64, m - 1])
    tail_columns(F, c, row)
    with pb.Cyclic.factor_d4(n, sigma) as cy:
        assert cy.form_for(m) == pb.FORM_STREAM
        X = cy.solve_(F.clone())
        G = F.clone()
        G[n // 2, 70] = float("nan")
        Y = cy.solve_(G)
        cy.set_schedule(2, 64)
        Z = cy.solve_(F)
        cy.check()
    assert_tails(X[:, c].cpu().numpy(), Z[:, c].cpu().numpy(), sigma, 100)
    assert not bool(torch.isfinite(Y[:, 70]).any())
    keep = [j for j in range(m) if j != 70]
    assert torch.equal(X[:, keep], Y[:, keep])


@pytest.mark.parametrize("n,m", [(2100, 6000), (4096, 16384)])
def test_forced_single_pass_is_look_back(torch, n, m):
    """A forced schedule runs its own kernels, also at sizes that the automatic
    one streams, and the automatic one gives its bits again afterwards."""
    print_case(test="forced", n=n, m=m)
    F = rand(torch, (n, m), 2)
    with pb.Plan.factor_d4(n, 5.0) as p:
        assert p.form_for(m) == pb.FORM_STREAM
        X = p.solve_(F.clone())
        p.set_schedule(4, 64)
        assert p.form_for(m) == pb.FORM_SCHEDULE and p.schedule_for(m) == (4, 64)
        Y = p.solve_(F.clone())
        p.set_schedule(0, 0)
        Z = p.solve_(F.clone())
        p.check()
    assert torch.equal(X, Z)
    assert float((X - Y).abs().max() / X.abs().max()) <= 2 * d4_tol(5.0)


# sources of one system each, at rows of their own, so that no two tiles have
# the same blocks to add to
@pytest.mark.parametrize("n,m,sigma", [(4096, 14000, 50.0), (3001, 9000, 5.0), (2100, 12001, 700.0)])
def test_tail_bits_by_place(torch, n, m, sigma):
    """A system's bits do not depend on which others share its tile, also where
    the streaming sweeps add to it afterwards."""
    print_case(test="tail_bits", n=n, m=m, sigma=sigma)
    rows = torch.arange(m, device="cuda") * 7919 % (n - 200) + 200
    F = torch.zeros((n, m), dtype=torch.float64, device="cuda")
    F[rows, torch.arange(m, device="cuda")] = 1.0
    at, k = 7, m - 3000
    part = F[:, at:at + k].contiguous()
    with pb.Plan.factor_d4(n, sigma) as p:
        assert p.form_for(m) == p.form_for(k) == pb.FORM_STREAM
        X = p.solve_(F.clone())
        assert torch.equal(X[:, at:at + k], p.solve_(part.clone()))
        nt = (m + 63) // 64
        T = torch.nn.functional.pad(F, (0, nt * 64 - m)).view(n, nt, 64).transpose(0, 1).contiguous()
        assert pb.lib().pent_solve_tiled(p.handle, T.data_ptr(), m, 64, 64 * n, torch.cuda.current_stream().cuda_stream) == pb.OK
        assert torch.equal(T.transpose(0, 1).reshape(n, nt * 64)[:, :m], X)
        p.check()
    with pb.Cyclic.factor_d4(n, sigma) as cy:
        if cy.form_for(m, True) == cy.form_for(k, True) == pb.FORM_STREAM:
            X, Y = torch.empty_like(F), torch.empty_like(part)
            cy.cn_step(F, X)
            cy.cn_step(part, Y)
            assert torch.equal(X[:, at:at + k], Y)
        cy.check()
