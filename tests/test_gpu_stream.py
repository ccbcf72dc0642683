"""Streaming sweeps (the automatic schedule of large batches): block and tile
edges, row strides and types, truncation depths, and right-hand sides for
which the truncated backward chain alone would lose values."""
import numpy as np
import pytest

import oracle
from paper_1807_07382_amd import pentbatch as pb
from tests._gpu import U, colerr, d4_tol, print_case, torch_dev
from tests.test_oracle_pins import random_dd

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return torch_dev()


def rand(torch, shape, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.rand(shape, dtype=torch.float64, device="cuda", generator=g) * 2 - 1


def probes(m, width):
    cols = {0, 1, width - 1, width, m // 2, m - 2, m - 1}
    return np.array(sorted(c for c in cols if 0 <= c < m))


# n: one block, block edges of 32 and 64 rows, a partial last block, more
# blocks than waves; m: tiles of 32, 48 and 64 systems, partial last tiles;
# sigma: depths from 1 block up to the 64-row form (1000) and past it (1e4:
# the look-back single pass)
@pytest.mark.parametrize("n,m,pad,sigma", [
    (31, 700, 0, 50.0), (32, 701, 3, 0.1), (33, 2600, 0, 1e4), (64, 5120, 16, 50.0), (65, 5123, 0, 200.0),
    (1000, 5003, 5, 1.0), (1023, 9000, 0, 50.0), (1025, 12300, 4, 50.0), (2049, 5121, 0, 300.0),
    (2113, 6000, 16, 1000.0), (4096, 16385, 0, 50.0), (4099, 5120, 1, 0.01), (1536, 5150, 0, 1e4)])
@pytest.mark.parametrize("f32", [False, True])
def test_stream_matches_oracle(torch, n, m, pad, sigma, f32):
    print_case(test="stream", n=n, m=m, pad=pad, sigma=sigma, f32=f32)
    B = rand(torch, (n, m + pad), n + m)
    if f32:
        B = B.float()
    X = torch.full((n, m + pad), 7.0, dtype=torch.float64, device="cuda")
    with pb.Plan.factor_d4(n, sigma) as p:
        p.solve_mixed(B[:, :m], X[:, :m])
        if not f32:
            F = B.clone()
            p.solve_(F[:, :m])
            assert torch.equal(F[:, :m], X[:, :m])          # in place: the same bits
            assert torch.equal(F[:, m:], B[:, m:])          # the padding is left alone
        p.check()
    assert bool((X[:, m:] == 7.0).all())
    c = probes(m, 64)
    ref = oracle.solve(oracle.assemble_d4(n, sigma), np.ascontiguousarray(B[:, c].double().cpu().numpy()))
    assert np.max(colerr(X[:, c].cpu().numpy(), ref)) <= d4_tol(sigma)


def test_stream_general_matrix_and_bits_by_column(torch):
    """A non-symmetric matrix; every system has the same bits wherever it
    sits in the batch."""
    n, m = 777, 6001
    print_case(test="stream_general", n=n, m=m)
    dg = random_dd(n, seed=5)
    F = rand(torch, (n, m), 3)
    perm = torch.randperm(m, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    with pb.Plan.factor(*dg) as p:
        X = p.solve_(F.clone())
        Y = p.solve_(F[:, perm].contiguous())
        p.check()
    assert torch.equal(X[:, perm], Y)
    c = probes(m, 48)
    ref = oracle.solve(dg, np.ascontiguousarray(F[:, c].cpu().numpy()))
    assert np.max(colerr(X[:, c].cpu().numpy(), ref)) <= 1e-13


@pytest.mark.parametrize("n,sigma", [(2050, 30.0), (2050, 700.0), (96, 0.1), (4096, 2.0)])
@pytest.mark.parametrize("where", ["top", "middle", "bottom"])
def test_stream_keeps_far_tails(torch, n, sigma, where):
    """A right-hand side that is zero but for one row: far from it the
    solution is many orders smaller, and still right in each stretch of rows
    on its own.  The neighbours in the tile are ordinary systems.  A row
    adds a few roundings (d4_tol) to the relative error of such a tail."""
    m = 5120
    print_case(test="stream_tail", n=n, sigma=sigma, where=where)
    F = rand(torch, (n, m), 9)
    c = np.array([0, 17, 63, 64, m - 1])
    row = {"top": 1, "middle": n // 2, "bottom": n - 1}[where]
    F[:, c] = 0.0
    F[row, c] = 1.0
    ref = oracle.solve(oracle.assemble_d4(n, sigma), np.ascontiguousarray(F[:, c].cpu().numpy()))
    other = np.array([1, 18, 62, 65])
    ref2 = oracle.solve(oracle.assemble_d4(n, sigma), np.ascontiguousarray(F[:, other].cpu().numpy()))
    with pb.Plan.factor_d4(n, sigma) as p:
        X = p.solve_(F)
        p.check()
    X2 = X[:, other].cpu().numpy()
    X = X[:, c].cpu().numpy()
    assert np.max(colerr(X2, ref2)) <= d4_tol(sigma)
    for r in range(0, n, 128):
        big = np.max(np.abs(ref[r:r + 128]), axis=0)
        err = np.max(np.abs(X[r:r + 128] - ref[r:r + 128]), axis=0)
        assert np.all(err <= n * d4_tol(sigma) * big + 1e-290)


@pytest.mark.parametrize("n,sigma", [(2050, 30.0), (2050, 700.0)])
def test_stream_non_finite_systems(torch, n, sigma):
    """A NaN or an infinity anywhere in a right-hand side leaves no finite
    value in that system (as in the other schedules) and the others alone."""
    m = 5120
    print_case(test="stream_nan", n=n, sigma=sigma)
    F = rand(torch, (n, m), 4)
    with pb.Plan.factor_d4(n, sigma) as p:
        clean = p.solve_(F.clone())
        bad = {3: (n - 1, np.nan), 64: (n // 2, np.inf), 65: (0, np.nan), 5119: (n - 1, -np.inf)}
        for col, (row, val) in bad.items():
            F[row, col] = val
        X = p.solve_(F)
        p.check()
    cols = list(bad)
    assert not bool(torch.isfinite(X[:, cols]).any())
    keep = [j for j in range(m) if j not in bad]
    assert torch.equal(X[:, keep], clean[:, keep])


def test_stream_tiled_layout_same_bits(torch):
    """64-system tiles stored one after the other: the bits pent_solve gives
    the same systems, and nothing written past a partial last tile's columns
    or between tiles."""
    n, m = 2100, 5150  # large enough for the single pass, which this layout wants
    print_case(test="stream_tiled", n=n, m=m)
    F = rand(torch, (n, m), 8)
    nt, ts = (m + 63) // 64, 64 * n + 32
    T = torch.full((nt, ts), 3.0, dtype=torch.float64, device="cuda")
    for t in range(nt):
        w = min(64, m - 64 * t)
        T[t, :64 * n].view(n, 64)[:, :w] = F[:, 64 * t:64 * t + w]
    with pb.Plan.factor_d4(n, 50.0) as p:
        st = pb.lib().pent_solve_tiled(p.handle, T.data_ptr(), m, 64, ts, torch.cuda.current_stream().cuda_stream)
        assert st == pb.OK
        X = p.solve_(F.clone())
        p.check()
    for t in range(nt):
        w = min(64, m - 64 * t)
        V = T[t, :64 * n].view(n, 64)
        assert torch.equal(V[:, :w], X[:, 64 * t:64 * t + w])
        assert bool((V[:, w:] == 3.0).all()) and bool((T[t, 64 * n:] == 3.0).all())


# n: partial and whole last blocks, fewer blocks than the correction's 12
# waves and more; sigma: correction depths from 1 to 8 blocks and past it
@pytest.mark.parametrize("n,m,pad,sigma", [(33, 2600, 0, 0.1), (1000, 5003, 3, 1.0), (1024, 9000, 0, 100.0),
                                           (2081, 5120, 16, 2000.0), (4100, 5125, 0, 1e4)])
@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("steps", [1, 2])
def test_stream_corrections(torch, n, m, pad, sigma, f32, steps):
    """Refined solves: within the solve's tolerance of the oracle, the
    compensated backward error at rounding level (each correction leaves at
    most one rounding of x per entry, |dx| <= u |x|, so eta <= u; 2 u covers
    the evaluation), padding untouched."""
    print_case(test="stream_fix", n=n, m=m, sigma=sigma, f32=f32, steps=steps)
    B = rand(torch, (n, m + pad), n)
    B = B.float() if f32 else B
    X = torch.full((n, m + pad), 7.0, dtype=torch.float64, device="cuda")
    eta = torch.empty(m, dtype=torch.float64, device="cuda")
    with pb.Plan.factor_d4(n, sigma) as p:
        p.solve_mixed(B[:, :m], X[:, :m], steps, eta)
        p.check()
    assert bool((X[:, m:] == 7.0).all())
    assert eta.max().item() <= 2 * U
    c = probes(m, 64)
    ref = oracle.solve(oracle.assemble_d4(n, sigma), np.ascontiguousarray(B[:, c].double().cpu().numpy()))
    assert np.max(colerr(X[:, c].cpu().numpy(), ref)) <= d4_tol(sigma)


def cyc_lu(n, sigma):
    """Sparse LU of the periodic I + sigma*D4 (scipy, with pivoting)."""
    import scipy.sparse as sp
    import scipy.sparse.linalg as sl
    rows = np.arange(n)
    A = sp.lil_matrix((n, n))
    for o, v in ((-2, sigma), (-1, -4 * sigma), (0, 1 + 6 * sigma), (1, -4 * sigma), (2, sigma)):
        for r in rows:
            A[r, (r + o) % n] += v
    return sl.splu(A.tocsc()), A.tocsr()


# n: E rows on and off block edges, with one to 32 rows in the last block;
# sigma: few and many end blocks (and, at 1e4, the look-back form)
@pytest.mark.parametrize("n,m,pad,sigma", [(514, 8192, 0, 0.1), (515, 8200, 3, 1.0), (1026, 8192, 16, 50.0),
                                           (1057, 9001, 0, 50.0), (2047, 8192, 0, 300.0), (1537, 8192, 0, 1e4)])
def test_stream_periodic(torch, n, m, pad, sigma):
    """Periodic solves and Crank-Nicolson steps of large batches against an
    independent sparse LU (kappa_2 <= 1 + 16 sigma, as for d4_tol; the step's
    right-hand side adds at most (2 + 16 sigma) of max|C|, see the stencil's
    bound in the periodic tests)."""
    print_case(test="stream_cyc", n=n, m=m, pad=pad, sigma=sigma)
    B = rand(torch, (n, m + pad), n + 1)
    X = torch.full((n, m + pad), 7.0, dtype=torch.float64, device="cuda")
    F = B.clone()
    c = probes(m, 48)
    Bc = B[:, c].cpu().numpy()
    lu, A = cyc_lu(n, sigma)
    with pb.Cyclic.factor_d4(n, sigma) as cy:
        cy.solve_(F[:, :m])
        cy.cn_step(B[:, :m], X[:, :m])
        cy.check()
    assert torch.equal(F[:, m:], B[:, m:]) and bool((X[:, m:] == 7.0).all())
    assert np.max(colerr(F[:, c].cpu().numpy(), lu.solve(Bc))) <= d4_tol(sigma)
    ref = lu.solve(2 * Bc - A @ Bc)
    err = np.max(np.abs(X[:, c].cpu().numpy() - ref), axis=0)
    assert np.all(err <= d4_tol(sigma) * (np.max(np.abs(ref), axis=0) + (2 + 16 * sigma) * np.max(np.abs(Bc), axis=0)))


def test_stream_periodic_varying_rows(torch):
    """Diagonals that differ from row to row (the step reads them per row)."""
    n, m = 700, 8192
    print_case(test="stream_cyc_rows", n=n, m=m)
    g = np.random.Generator(np.random.PCG64(2))
    dg = [g.uniform(-1, 1, n) for _ in range(5)]
    dg[2] = 5.0 + g.uniform(0, 1, n)
    A = np.zeros((n, n))
    for o in range(-2, 3):
        for r in range(n):
            A[r, (r + o) % n] += dg[o + 2][r]
    C = rand(torch, (n, m), 6)
    X = torch.empty_like(C)
    c = probes(m, 64)
    Cc = C[:, c].cpu().numpy()
    with pb.Cyclic.factor(*dg) as cy:
        cy.cn_step(C, X)
        F = cy.solve_(C.clone())
        cy.check()
    kappa = np.linalg.cond(A, np.inf)
    assert np.max(colerr(F[:, c].cpu().numpy(), np.linalg.solve(A, Cc))) <= 64 * U * kappa
    ref = np.linalg.solve(A, 2 * Cc - A @ Cc)
    assert np.max(np.abs(X[:, c].cpu().numpy() - ref)) <= 64 * U * kappa * 12 * np.max(np.abs(Cc))


@pytest.mark.parametrize("row", [0, 600, 1199])
def test_stream_periodic_far_tails_and_non_finite(torch, row):
    """A right-hand side that is zero but for one row, far tails in each
    stretch of rows (the tail unknowns are formed from the ends of the rows
    only); a system with a NaN has no finite value and spoils no other."""
    n, m, sigma = 1200, 8192, 20.0
    print_case(test="stream_cyc_tail", row=row)
    F = rand(torch, (n, m), 9)
    c = np.array([0, 17, 63, 64, m - 1])
    F[:, c] = 0.0
    F[row, c] = 1.0
    lu, A = cyc_lu(n, sigma)
    # the exact tail decays both ways round: its values by the real-space
    # Green's function of the infinite row, wrapped (the LU's own tails are
    # only normwise accurate)
    z = np.roots([sigma, -4 * sigma, 1 + 6 * sigma, -4 * sigma, sigma])
    z = z[np.abs(z) < 1]
    d = np.arange(n + 1)
    G = np.zeros(n + 1, dtype=complex)
    for r in z:  # residues of z^{d+1} / (sigma (z - r1)(z - r2)(z - 1/r1)(z - 1/r2)) inside the circle
        others = [q for q in list(z) + [1 / q for q in z] if q is not r and abs(q - r) > 1e-12]
        G += r ** (d + 1) / (sigma * np.prod([r - q for q in others]))
    G = G.real
    k = (np.arange(n) - row) % n
    ref = G[k] + G[n - k]
    assert np.max(np.abs(ref - lu.solve(F[:, :1].cpu().numpy())[:, 0])) <= 1e-12
    keep = F[:, 1].clone()
    with pb.Cyclic.factor_d4(n, sigma) as cy:
        X = cy.solve_(F.clone())
        F[n // 2, 70] = float("nan")
        Y = cy.solve_(F)
        cy.check()
    X = X[:, c].cpu().numpy()
    for r in range(0, n, 100):
        big = np.max(np.abs(ref[r:r + 100]))
        err = np.max(np.abs(X[r:r + 100] - ref[r:r + 100, None]))
        assert err <= n * d4_tol(sigma) * big
    assert not bool(torch.isfinite(Y[:, 70]).any())
    assert bool(torch.isfinite(Y[:, [69, 71]]).all())
    assert np.max(np.abs(A @ Y[:, 1].cpu().numpy() - keep.cpu().numpy())) <= 1e-11


# n: one block to many, partial last blocks of 1 to 32 rows; ld: runs on lines
# of their own, at any double, and with a gap; m: partial last tiles and slices
@pytest.mark.parametrize("n,m,ld,sigma", [(1, 3, 1, 50.0), (2, 70, 2, 0.1), (31, 64, 33, 1.0), (33, 1000, 48, 50.0),
                                          (64, 513, 64, 0.1), (257, 2100, 257, 300.0), (1021, 20011, 1021, 20.0),
                                          (1024, 999, 1040, 50.0), (2049, 10007, 2051, 50.0), (500, 333, 500, 1e4)])
def test_stream_system_major(torch, n, m, ld, sigma):
    print_case(test="stream_t", n=n, m=m, ld=ld, sigma=sigma)
    B = rand(torch, (m, ld), n + ld)
    F = B.clone()
    with pb.Plan.factor_d4(n, sigma) as p:
        p.solve_strided_(F[:, :n])
        p.check()
    assert torch.equal(F[:, n:], B[:, n:])
    c = probes(m, 48)
    ref = oracle.solve(oracle.assemble_d4(n, sigma), np.ascontiguousarray(B[c, :n].T.cpu().numpy()))
    assert np.max(colerr(F[c, :n].T.cpu().numpy(), ref)) <= d4_tol(sigma)


def test_stream_system_major_offset_and_far_tails(torch):
    """Storage that starts at an odd double; systems that are zero but for
    their last row keep their tails; one with a NaN spoils no other."""
    n, m, sigma = 900, 301, 5.0
    print_case(test="stream_t_tail", n=n, m=m)
    buf = rand(torch, (m * n + 1,), 3)
    F = buf[1:].view(m, n)
    F[::7] = 0.0
    F[::7, n - 1] = 1.0
    F[3, n // 2] = float("nan")
    ref = oracle.solve(oracle.assemble_d4(n, sigma), np.ascontiguousarray(F[[0, 1, 294, 300]].T.cpu().numpy()))
    with pb.Plan.factor_d4(n, sigma) as p:
        p.solve_strided_(F)
        p.check()
    X = F[[0, 1, 294, 300]].T.cpu().numpy()
    assert np.max(colerr(X, ref)) <= d4_tol(sigma)
    for r in range(0, n, 60):
        big = np.max(np.abs(ref[r:r + 60]), axis=0)
        assert np.all(np.max(np.abs(X[r:r + 60] - ref[r:r + 60]), axis=0) <= n * d4_tol(sigma) * big + 1e-290)
    assert not bool(torch.isfinite(F[3]).any()) and bool(torch.isfinite(F[[2, 4]]).all())
