"""Factorisation of host diagonals: the bits of the oracle's row-by-row
recurrence in every case, and the floating-point environment left alone."""
import numpy as np
import pytest

import oracle
from paper_1807_07382_amd import pentbatch as pb
from tests._gpu import print_case, torch_dev
from tests.test_oracle_pins import random_dd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 3, 63, 64, 65, 1025, 20011])
def test_subnormal_factors_with_flushing_on(n):
    """Off-diagonals so small that gamma and delta are subnormal, with the
    calling thread set to flush those: same bits, and still set afterwards."""
    torch = torch_dev()
    print_case(test="factor_host", n=n)
    dg = random_dd(n, seed=n)
    for x in (dg.d, dg.e):
        x[::3] *= 1e-309
    ref = oracle.factor(dg)
    tiny = torch.tensor([1e-310], dtype=torch.float64)
    assert torch.set_flush_denormal(True)
    try:
        with pb.Plan.factor(*dg) as p:
            flushed = (tiny * 0.5).item() == 0.0
            got = p.factors()
    finally:
        torch.set_flush_denormal(False)
    assert flushed
    for g, r in zip(got, ref):
        assert np.array_equal(g, r)
    if n >= 63:
        sub = np.abs(ref[3])
        assert np.any((sub > 0) & (sub < np.finfo(np.float64).tiny))
