"""Factorisation at the ends of the FP64 range."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.newmark import NewmarkOracle
from workloads.mesh import cube_mesh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("exponent", [-1030, 500])
def test_subnormal_and_large_pivots(exponent):
    # one subdomain (the interface products of more would overflow): A and b scaled
    # by 2^exponent leave x as it is.  At 2^-1030 the diagonal, 4 to 7 unscaled, and
    # every pivot are subnormal; an entry and each of up to 512 updates of it is
    # rounded to 2^-1075, 2^-47 of the diagonal.
    from paper_2204_13254_amd.solver import DDSolver
    n = 4
    c, t, _ = cube_mesh(n)
    part = np.zeros(len(t), dtype=np.int32)
    scale = float(2.0 ** exponent)
    o = NewmarkOracle(c, t, dt=1.0)
    free = np.flatnonzero(~o.d.pec)
    A = o.A.toarray()
    assert 4.0 <= np.diag(A).min() and np.diag(A).max() <= 8.0 and len(free) <= 512
    x = np.random.default_rng(0).uniform(-1, 1, len(free))
    b = np.zeros((1, o.d.n_e))
    b[0, free] = (A @ x) * scale
    s = DDSolver(c, t, part, np.full(len(t), scale), dt=float(2.0 ** (exponent // 2)), nrhs=1, precision="fp64")
    got = s.solve(torch.tensor(b, device="cuda")).cpu().numpy()[0, free]
    unit = 2.0 ** (-47 if exponent < 0 else -53)
    assert np.linalg.norm(got - x) <= 512 * unit * np.linalg.cond(A) * np.linalg.norm(x)
