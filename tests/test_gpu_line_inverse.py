"""Local factorisations at the edges of the line block's inverse (one half or
two of 16 pivots, eight or sixteen in the second), in FP64 against the oracle
at the parity bar (1e-10) and in the FP32 form at its own (1e-6), over two
decades of permeability contrast per cell."""
import numpy as np
import pytest

from inputs import make_workload
from inputs.fields import gaussian_logk
from inputs.workloads import _dirichlet_x

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-10), ("fp32_refine", 1e-6)])
@pytest.mark.parametrize("nb", [1, 2, 7, 8, 9, 15, 16, 17, 23, 24, 25, 31, 32])
def test_line_block(nb, precision, tol):
    from gpu_util import gpu_solve, oracle_solve, rel
    print("case", nb, precision, flush=True)
    n = (2 * nb, 10)
    y = 2.0 * gaussian_logk(n, 1.0 / n[0], 1.0, 0.1, nb)
    types, vals = _dirichlet_x(n)
    wl = make_workload("c1").with_(
        ncell=n, h=1.0 / n[0], logk=y, source=np.zeros_like(y), bc_type=tuple(types), bc_value=vals,
        sub=(nb, 5), overlap=0, space="linear" if nb > 2 else "const", beta_mode="alpha", beta_mbf=1.0,
        beta_smooth=1.0, nsmooth=2)
    p, fl, _, _ = gpu_solve(wl, precision=precision, tol=1e-12, max_refine=30)
    rp, rf, _, _ = oracle_solve(wl)
    ep, ef = rel(p, rp), rel(fl, rf)
    print("  p %.1e flux %.1e" % (ep, ef), flush=True)
    assert ep <= tol and ef <= tol
