"""Block inverses of the interface cyclic reduction (16-pivot Gauss-Jordan
steps): every number of 16-row strips, layers that end inside a strip, and
the quarters of layers above 128 unknowns, against the oracle's direct
solution.  Bars: those of the FP64 parity tests (1e-10 in pressure and
flux, 1e-9 in the interface unknowns)."""
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


def _strip(mx, my, space, sub=4):
    n = (sub * mx, sub * my)
    y = gaussian_logk(n, 1.0 / n[0], 1.0, 0.1, 7)
    types, vals = _dirichlet_x(n)
    return make_workload("c1").with_(
        ncell=n, h=1.0 / n[0], logk=y, source=np.zeros_like(y), bc_type=tuple(types), bc_value=vals,
        sub=(sub, sub), overlap=1, space=space, beta_mode="alpha", beta_mbf=1.0, beta_smooth=1.0, nsmooth=1)


# constant spaces: an interior layer of mx subdomains has 4 mx - 2 unknowns
# (linear: twice as many); an end layer mx fewer
@pytest.mark.parametrize("mx,my,space", [
    (2, 3, "const"),     # 6 unknowns, block 32
    (4, 5, "const"),     # 14: one strip
    (5, 4, "const"),     # 18: two strips
    (8, 2, "const"),     # end layers only (22)
    (9, 5, "const"),     # 34, block 64
    (16, 3, "const"),    # 62: four strips
    (17, 4, "const"),    # 66, block 96
    (12, 3, "linear"),   # 92: six strips
    (25, 3, "const"),    # 98, block 128
    (16, 5, "linear"),   # 124: eight strips
    (33, 4, "const"),    # 130, quarters of 96
    (24, 3, "linear"),   # 188: quarters of 96
    (32, 3, "linear"),   # 252: quarters of 128
])
def test_layer_sizes(mx, my, space):
    from gpu_util import gpu_solve, oracle_solve, rel
    print("case", mx, my, space, flush=True)
    wl = _strip(mx, my, space)
    p, fl, X, st = gpu_solve(wl, solver="bcr")
    rp, rf, rX, _ = oracle_solve(wl)
    ep, ef, ex = rel(p, rp), rel(fl, rf), rel(X, rX)
    print("  n %d: p %.1e flux %.1e X %.1e residual %.1e"
          % (st["n_unknowns"], ep, ef, ex, st["interface_residual"]), flush=True)
    assert st["interface_solver"] == 2
    assert ep <= 1e-10 and ef <= 1e-10 and ex <= 1e-9
