"""The step's non-finite flag."""
import numpy as np
import pytest

import paper_1906_11036_amd as dg
from paper_1906_11036_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", [W.DIRICHLET, W.MIRROR])
def test_finite_state_raises_no_flag(bc):
    """The non-finite flag comes from updated cells only: finite binary64 states
    beside walls (lanes past the wall hold no cell) leave it unset."""
    for nx, ny in ((20, 5), (40, 33), (59, 9), (63, 5), (100, 33)):
        for deg in (1, 2, 3):
            for rows in (4, 32):
                p = W.random_problem(1010, nx, ny, bcx=bc, bcy=bc, bdeg=deg, ddeg=1)
                if bc == W.MIRROR:
                    p.bx, p.by = (0.0, 0.1), (0.0, 0.1)
                s = dg.Solver(p, storage="f64", launch=(rows, 1, 0, 1))
                if bc == W.DIRICHLET:
                    s.set_dirichlet(p.rings(3))
                s.set_phi(p.phi0)
                s.step(1)
                assert s.diag(check=False)["flags"] == 0
                s.step(2)
                assert s.diag(check=False)["flags"] == 0
                assert np.isfinite(s.get_f()).all()
