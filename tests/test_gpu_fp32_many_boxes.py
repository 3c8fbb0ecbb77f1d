"""FP32 Steps 1-2 and 4 where the boxes are many (two waves per box, inverses
streamed) at the edges of that form: lines of 5 to 32 cells, odd and even,
boxes of 3 to 32 lines, up to 4, 8 and 14 seeds.  A batch of eight members
of 128 subdomains takes it, a member alone (four waves per box) does not:
equal bits, and the member against the oracle at the FP32 form's bar (1e-6)."""
import numpy as np
import pytest

from inputs import make_workload
from inputs.fields import gaussian_logk
from inputs.workloads import _dirichlet_x
from test_gpu_batched import solve_batch, solve_one

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("sub,overlap,space", [
    ((4, 4), 1, "const"), ((4, 4), 1, "linear"), ((3, 4), 1, "fine"), ((9, 7), 2, "const"), ((8, 8), 1, "linear"),
    ((14, 15), 1, "const"), ((5, 30), 1, "const"), ((30, 5), 1, "linear"), ((32, 3), 0, "const")])
def test_two_waves_per_box(sub, overlap, space):
    from gpu_util import oracle_solve, rel
    print("case", sub, overlap, space, flush=True)
    n = (16 * sub[0], 8 * sub[1])
    types, vals = _dirichlet_x(n)
    wls = []
    for k in range(8):
        y = gaussian_logk(n, 1.0 / n[0], 1.0, 0.1, 20 + k)
        wls.append(make_workload("c1").with_(
            ncell=n, h=1.0 / n[0], logk=y, source=np.zeros_like(y), bc_type=tuple(types), bc_value=vals,
            sub=sub, overlap=overlap, space=space, beta_mode="alpha", beta_mbf=1.0, beta_smooth=2.0, nsmooth=1))
    ps, fls, _, st = solve_batch(wls, "fp32_refine")
    assert st["n_subdomains"] == 1024
    for k in (0, 5):
        p, fl, _ = solve_one(wls[k], "fp32_refine")
        assert np.array_equal(ps[k], p) and np.array_equal(fls[k], fl)
    rp, rf, _, _ = oracle_solve(wls[5])
    ep, ef = rel(ps[5], rp), rel(fls[5], rf)
    print("  p %.1e flux %.1e" % (ep, ef), flush=True)
    assert ep <= 1e-6 and ef <= 1e-6
