"""The largest calls that the automatic schedule streams look at a sample of
their right-hand sides first: ordinary ones stream, ones with long tails above
their sources run by look-back (the forced single pass), bit for bit."""
import ctypes

import numpy as np
import pytest

from paper_1807_07382_amd import pentbatch as pb
from tests._gpu import print_case, torch_dev
from tests.test_gpu_stream import rand

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    return torch_dev()


def hat(torch, n, m, dtype=None):
    F = torch.zeros((n, m), dtype=dtype or torch.float64, device="cuda")
    F[n // 2:n // 2 + 40] = rand(torch, (40, m), n).to(F.dtype)
    return F


def streamed(p, F, m):
    """The bits of the first m systems as streaming sweeps (a smaller batch has
    no gate, and a system's bits do not depend on its place in the batch)."""
    assert F.shape[0] * m < 60_000_000 and p.form_for(m) == pb.FORM_STREAM
    return p.solve_(F[:, :m].contiguous())


@pytest.mark.parametrize("n,m,sigma", [(4096, 16384, 50.0), (3000, 20011, 1.0), (1100, 54546, 30.0), (2050, 40000, 700.0)])
@pytest.mark.parametrize("f32", [False, True])
def test_gate(torch, n, m, sigma, f32):
    print_case(test="gate", n=n, m=m, sigma=sigma, f32=f32)
    k = 6000
    with pb.Plan.factor_d4(n, sigma) as p:
        assert p.form_for(m) == pb.FORM_STREAM
        for data in ("random", "hat", "random"):
            F = hat(torch, n, m) if data == "hat" else rand(torch, (n, m), n)
            F = F.float().double()
            X = torch.empty_like(F)
            p.solve_mixed(F.float() if f32 else F, X)
            if data == "hat":
                p.set_schedule(4, 64)
                ref = p.solve_(F.clone())
                p.set_schedule(0, 0)
                assert torch.equal(X, ref)
            else:
                assert torch.equal(X[:, :k], streamed(p, F, k))
            p.solve_(F)
            assert torch.equal(F, X)  # in place: the same
        p.check()


def test_gate_votes(torch):
    """Eight tiles are looked at, 16 systems of each: one with a tail, or with
    nothing but zeros in its samples, is not enough, two are."""
    n, m, k = 4096, 16384, 6000
    print_case(test="gate_votes")
    at = [m // 64 * p // 8 * 64 + p % 4 * 16 + 5 for p in range(8)]
    with pb.Plan.factor_d4(n, 5.0) as p:
        for cols, row, leaves in (((at[3],), n - 1, False), ((at[3] - 64,), n - 1, False), ((at[1], at[6]), n - 1, True),
                                  ((at[0], at[7]), 1001, True), ((at[2] + 1, at[4] + 40), 2000, False)):
            F = rand(torch, (n, m), 4)
            F[:, list(cols)] = 0.0
            F[row, list(cols)] = 1.0
            other = torch.ones(k, dtype=torch.bool, device="cuda")
            other[[c for c in cols if c < k]] = False
            S = streamed(p, F, k)
            p.set_schedule(4, 64)
            L = p.solve_(F.clone())
            p.set_schedule(0, 0)
            X = p.solve_(F)
            assert not torch.equal(S, L[:, :k])
            assert torch.equal(X, L) == leaves
            assert torch.equal(X[:, :k], S) == (not leaves)
        p.check()


def test_gate_other_layout_and_no_allocation(torch):
    """The tiled layout and the allocation-free solve decide alike."""
    n, m = 4096, 16400
    print_case(test="gate_layouts")
    s = torch.cuda.current_stream().cuda_stream
    nt = (m + 63) // 64
    with pb.Plan.factor_d4(n, 50.0) as p:
        for F in (hat(torch, n, m), rand(torch, (n, m), 2)):
            T = torch.zeros((nt, n, 64), dtype=torch.float64, device="cuda")
            pad = torch.nn.functional.pad(F, (0, nt * 64 - m))
            T.copy_(pad.view(n, nt, 64).transpose(0, 1))
            assert pb.lib().pent_solve_tiled(p.handle, T.data_ptr(), m, 64, 64 * n, s) == pb.OK
            N = F.clone()
            assert pb.lib().pent_solve_noalloc(p.handle, N.data_ptr(), m, m, s) == pb.OK
            X = p.solve_(F)
            assert torch.equal(N, X)
            assert torch.equal(T.transpose(0, 1).reshape(n, nt * 64)[:, :m], X)
        p.check()


@pytest.mark.parametrize("n,m,sigma", [(4098, 16384, 50.0), (1200, 52000, 5.0)])
@pytest.mark.parametrize("varying", [False, True])
def test_gate_periodic(torch, n, m, sigma, varying):
    print_case(test="gate_cyc", n=n, m=m, varying=varying)
    k = 11000
    dg = [np.full(n, v) for v in (sigma, -4 * sigma, 1 + 6 * sigma, -4 * sigma, sigma)]
    if varying:
        dg[2] = dg[2] + np.arange(n) % 3
    with pb.Cyclic.factor(*dg) as cy:
        assert cy.form_for(m) == cy.form_for(m, True) == cy.form_for(k) == pb.FORM_STREAM and n * k < 60_000_000
        for data in ("hat", "random", "hat"):
            F = hat(torch, n, m) if data == "hat" else rand(torch, (n, m), n)
            X = torch.empty_like(F)
            cy.cn_step(F, X)
            S = cy.solve_(F.clone())
            if data == "hat":
                cy.set_schedule(2, 64)
                Y = torch.empty_like(F)
                cy.cn_step(F, Y)
                assert torch.equal(X, Y)
                assert torch.equal(S, cy.solve_(F))
                cy.set_schedule(0)
            else:
                G = F[:, :k].contiguous()
                Y = torch.empty_like(G)
                cy.cn_step(G, Y)
                assert torch.equal(X[:, :k], Y)
                assert torch.equal(S[:, :k], cy.solve_(G))
        cy.check()


def test_gate_in_a_graph(torch):
    """A captured solve decides anew at every replay."""
    n, m = 4096, 16384
    print_case(test="gate_graph")
    inputs = [rand(torch, (n, m), 1), hat(torch, n, m), rand(torch, (n, m), 3), hat(torch, n, m) * 2, rand(torch, (n, m), 5)]
    F = torch.empty((n, m), dtype=torch.float64, device="cuda")
    with pb.Plan.factor_d4(n, 50.0) as p:
        refs = [p.solve_(G.clone()) for G in inputs]
        graph = torch.cuda.CUDAGraph()
        side = torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=side):
            st = pb.lib().pent_solve_noalloc(p.handle, F.data_ptr(), m, m,
                                             ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == pb.OK
        for G, ref in zip(inputs, refs):
            F.copy_(G)
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(F, ref)
        p.check()


def test_gate_needs_scratch(torch):
    """pent_solve has nothing to allocate under capture, and streams."""
    n, m, k = 4096, 16384, 6000
    print_case(test="gate_no_scratch")
    inputs = [hat(torch, n, m), rand(torch, (n, m), 3), hat(torch, n, m) * 2]
    F = torch.empty((n, m), dtype=torch.float64, device="cuda")
    with pb.Plan.factor_d4(n, 50.0) as p:
        refs = [streamed(p, G, k) for G in inputs]
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
            st = pb.lib().pent_solve(p.handle, F.data_ptr(), m, m, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == pb.OK
        for G, ref in zip(inputs, refs):
            F.copy_(G)
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(F[:, :k], ref)
        p.check()
