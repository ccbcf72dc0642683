"""Whole systems resident in one workgroup (the automatic schedule of matrices
of up to 2048 rows and batches that do not fill the device): edges of blocks,
waves and tiles, types and strides, deep chains, non-finite systems, and the
periodic solve and step."""
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


# n: one row to a full workgroup; blocks of 32 rows, waves of 64 and 128, on
# and off their edges; m: tiles of 16 and (from 5000) 32, partial last tiles
SIZES = [(1, 3, 0), (2, 16, 1), (31, 17, 0), (32, 5000, 0), (33, 15, 2), (64, 5003, 1), (65, 6001, 0), (127, 100, 0),
         (128, 33, 7), (129, 33, 0), (512, 700, 0), (513, 5100, 3), (768, 1000, 0), (1000, 5003, 5), (1023, 6000, 0),
         (1024, 500, 16), (1025, 1101, 0), (1537, 2500, 1), (1920, 1200, 0), (1921, 1200, 0), (2047, 4096, 0),
         (2048, 1500, 3), (700, 7000, 0)]
# tiles of four systems: blocks of 32 rows, waves of 512, eight and sixteen waves
SIZES += [(513, 1024, 0), (1025, 1, 0), (1536, 4, 0), (1537, 5, 3), (2049, 100, 0), (2500, 390, 1), (3583, 7, 0),
          (3585, 2048, 0), (4095, 66, 2), (4096, 130, 0), (4097, 50, 0), (5000, 201, 1), (6656, 33, 0)]


@pytest.mark.parametrize("n,m,pad", SIZES)
@pytest.mark.parametrize("sigma", [0.1, 1e5])
def test_resident_matches_oracle(torch, n, m, pad, sigma):
    """In place from FP64 and out of place from FP32; nothing is written
    beside the batch."""
    print_case(test="resident", n=n, m=m, pad=pad, sigma=sigma)
    B = rand(torch, (n, m + pad), n + m).float().double()
    c = probes(m, 16)
    ref = oracle.solve(oracle.assemble_d4(n, sigma), np.ascontiguousarray(B[:, c].cpu().numpy()))
    F = B.clone()
    X = torch.full((n, m + 2 * pad), 7.0, dtype=torch.float64, device="cuda")
    with pb.Plan.factor_d4(n, sigma) as p:
        p.solve_(F[:, :m])
        p.solve_mixed(B.float()[:, :m], X[:, :m])
        p.check()
    assert torch.equal(F[:, m:], B[:, m:]) and bool((X[:, m:] == 7.0).all())
    assert np.max(colerr(F[:, c].cpu().numpy(), ref)) <= d4_tol(sigma)
    assert torch.equal(F[:, :m], X[:, :m])


@pytest.mark.parametrize("n,m", [(300, 1000), (1000, 5003), (1700, 2000), (900, 600), (3000, 300), (5000, 200)])
def test_resident_against_forced_schedule(torch, n, m):
    """A matrix of differing rows: every system against the partitioned
    schedule (both within 64 u kappa of the solution, per column), and
    non-finite right-hand sides, which leave no finite value in their system
    and the others alone."""
    print_case(test="resident_forced", n=n, m=m)
    dg = random_dd(n, seed=n)
    B = rand(torch, (n, m), n)
    with pb.Plan.factor(*(getattr(dg, k) for k in "abcde")) as p:
        X = p.solve_(B.clone())
        F = B.clone()
        bad = {3: (n - 1, np.nan), 16: (n // 2, np.inf), 17: (0, np.nan), m - 1: (n - 1, -np.inf)}
        for col, (row, val) in bad.items():
            F[row, col] = val
        Y = p.solve_(F)
        p.set_schedule(2, 64)
        ref = p.solve_(B.clone())
        p.check()
    kappa = np.linalg.cond(oracle.dense(dg), np.inf)
    err = (X - ref).abs().amax(0) / ref.abs().amax(0)
    assert float(err.max()) <= 128 * U * kappa
    assert not bool(torch.isfinite(Y[:, list(bad)]).any())
    keep = [j for j in range(m) if j not in bad]
    assert torch.equal(Y[:, keep], X[:, keep])


@pytest.mark.parametrize("n,m,pad,sigma", [(5, 7, 0, 1.0), (6, 40, 1, 0.1), (33, 16, 0, 10.0), (34, 100, 0, 10.0),
                                           (35, 100, 3, 1e4), (66, 6000, 0, 10.0), (130, 33, 0, 100.0),
                                           (131, 5003, 5, 1.0), (1026, 5100, 0, 50.0), (1027, 300, 0, 1.0),
                                           (1537, 3001, 0, 10.0), (1922, 64, 16, 1e4),
                                           (100, 20000, 0, 1.0), (500, 17000, 1, 300.0), (800, 33000, 0, 300.0),
                                           (515, 1024, 0, 1.0), (1538, 5, 1, 10.0), (2051, 1280, 0, 1.0),
                                           (3587, 90, 0, 1e4), (4098, 66, 3, 10.0), (2050, 4096, 0, 3.0)])
def test_resident_periodic(torch, n, m, pad, sigma):
    """Solves and Crank-Nicolson steps, uniform diagonals (bounds as for the
    streaming form)."""
    print_case(test="resident_cyc", n=n, m=m, pad=pad, sigma=sigma)
    B = rand(torch, (n, m + pad), n + 1)
    X = torch.full((n, m + pad), 7.0, dtype=torch.float64, device="cuda")
    F = B.clone()
    c = probes(m, 16)
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


@pytest.mark.parametrize("n,m", [(5, 20), (34, 100), (300, 5001), (1500, 2000), (700, 300), (2300, 70)])
def test_resident_periodic_varying_rows(torch, n, m):
    """Diagonals that differ from row to row (the step reads them per row)."""
    print_case(test="resident_cyc_rows", n=n, m=m)
    g = np.random.Generator(np.random.PCG64(n))
    dg = [g.uniform(-1, 1, n) for _ in range(5)]
    dg[2] = 5.0 + g.uniform(0, 1, n)
    A = np.zeros((n, n))
    for o in range(-2, 3):
        for r in range(n):
            A[r, (r + o) % n] += dg[o + 2][r]
    C = rand(torch, (n, m), 6)
    X = torch.empty_like(C)
    c = probes(m, 16)
    Cc = C[:, c].cpu().numpy()
    with pb.Cyclic.factor(*dg) as cy:
        cy.cn_step(C, X)
        F = cy.solve_(C.clone())
        C[n // 2, 4] = float("nan")
        Y = cy.solve_(C.clone())
        cy.check()
    kappa = np.linalg.cond(A, np.inf)
    assert np.max(colerr(F[:, c].cpu().numpy(), np.linalg.solve(A, Cc))) <= 64 * U * kappa
    ref = np.linalg.solve(A, 2 * Cc - A @ Cc)
    assert np.max(np.abs(X[:, c].cpu().numpy() - ref)) <= 64 * U * kappa * 12 * np.max(np.abs(Cc))
    assert not bool(torch.isfinite(Y[:, 4]).any())
    keep = [j for j in range(m) if j != 4]
    assert torch.equal(Y[:, keep], F[:, keep])


# n: waves of 128 rows, one to sixteen, full, short by one row and by nearly all
# of it; ld: runs on lines of their own, at any double, with a gap; m: partial
# last tiles of 16 systems, the last of which ends the array
@pytest.mark.parametrize("n,m,ld,sigma", [(1, 3, 1, 50.0), (2, 20, 2, 0.1), (31, 64, 33, 1.0), (97, 16, 97, 1e5),
                                          (127, 17, 127, 1.0), (128, 48, 128, 1e4), (129, 1000, 129, 50.0),
                                          (255, 33, 300, 1.0), (257, 31, 257, 1e4), (513, 5, 520, 20.0),
                                          (640, 12000, 640, 200.0), (1000, 333, 1001, 1e4), (1024, 100, 1024, 200.0),
                                          (1025, 40, 1025, 1.0), (1921, 90, 1921, 1e4), (2048, 64, 2064, 1.0)])
def test_resident_system_major(torch, n, m, ld, sigma):
    """In an array that ends with the last system's last value; nothing is
    written between the systems."""
    print_case(test="resident_t", n=n, m=m, ld=ld, sigma=sigma)
    buf = rand(torch, ((m - 1) * ld + n,), n + m)
    keep = buf.clone()
    F = buf.as_strided((m, n), (ld, 1))
    c = probes(m, 16)
    ref = oracle.solve(oracle.assemble_d4(n, sigma), np.ascontiguousarray(F.cpu().numpy()[c].T))
    with pb.Plan.factor_d4(n, sigma) as p:
        p.solve_strided_(F)
        p.check()
    assert np.max(colerr(np.ascontiguousarray(F.cpu().numpy()[c].T), ref)) <= d4_tol(sigma)
    if ld > n and m > 1:
        gap = (m - 1, ld - n)
        assert torch.equal(buf.as_strided(gap, (ld, 1), n), keep.as_strided(gap, (ld, 1), n))


@pytest.mark.parametrize("ny,nx,k", [(1, 5, 2), (16, 128, 3), (17, 127, 2), (33, 130, 1), (15, 260, 5), (40, 1000, 2),
                                     (50, 1024, 1), (18, 1500, 2)])
def test_resident_2d_x_sweep(torch, ny, nx, k):
    """The 2-D step, its explicit term formed in the x sweeps, against the
    separate passes: the same bits."""
    print_case(test="resident_ch2d", ny=ny, nx=nx, k=k)
    C = rand(torch, (ny, k, nx), ny + nx) * 0.1
    R, C2 = torch.empty_like(C), C.clone()
    h = 1.0 / nx
    dt = torch.full((k,), 200.0 * h ** 4 / 0.01, dtype=torch.float64, device="cuda")
    with pb.Plan.factor_d4(nx, 200.0) as px, pb.Plan.factor_d4(ny, 200.0) as py:
        pb.ch2d_rhs(C2, R, dt, h)
        px.solve_strided_(R.view(ny * k, nx))
        py.solve_(R.view(ny, k * nx))
        pb.ch2d_step(px, py, C, torch.empty_like(C), dt, h)
    assert bool(torch.isfinite(C).all()) and torch.equal(C, R)


@pytest.mark.parametrize("n,m", [(100, 7000), (1000, 9000), (3000, 3001)])
def test_resident_tile_schedule_any_batch(torch, n, m):
    """Forced (kind 3), past the batches that take it by themselves."""
    print_case(test="resident_kind3", n=n, m=m)
    B = rand(torch, (n, m), 3)
    c = probes(m, 16)
    ref = oracle.solve(oracle.assemble_d4(n, 10.0), np.ascontiguousarray(B[:, c].cpu().numpy()))
    with pb.Plan.factor_d4(n, 10.0) as p:
        p.set_schedule(3, 0)
        p.solve_(B)
        p.check()
    assert np.max(colerr(B[:, c].cpu().numpy(), ref)) <= d4_tol(10.0)


@pytest.mark.parametrize("n,m,gap", [(4097, 70, 0), (5000, 201, 32), (6656, 130, 1)])
def test_resident_tiled_layout_same_bits(torch, n, m, gap):
    """64-system tiles stored one after the other, at sizes where the single
    pass' schedule runs in resident tiles: the bits of pent_solve, nothing
    written past a partial tile's columns or between tiles."""
    print_case(test="resident_tiled", n=n, m=m, gap=gap)
    F = rand(torch, (n, m), 8)
    nt, ts = (m + 63) // 64, 64 * n + gap
    T = torch.full((nt, ts), 3.0, dtype=torch.float64, device="cuda")
    for t in range(nt):
        w = min(64, m - 64 * t)
        T[t, :64 * n].view(n, 64)[:, :w] = F[:, 64 * t:64 * t + w]
    with pb.Plan.factor_d4(n, 50.0) as p:
        assert p.schedule_for(m)[0] == 4 and p.form_for(m) == pb.FORM_RESIDENT
        st = pb.lib().pent_solve_tiled(p.handle, T.data_ptr(), m, 64, ts, torch.cuda.current_stream().cuda_stream)
        assert st == pb.OK
        X = p.solve_(F.clone())
        p.check()
    for t in range(nt):
        w = min(64, m - 64 * t)
        V = T[t, :64 * n].view(n, 64)
        assert torch.equal(V[:, :w], X[:, 64 * t:64 * t + w])
        assert bool((V[:, w:] == 3.0).all()) and bool((T[t, 64 * n:] == 3.0).all())
