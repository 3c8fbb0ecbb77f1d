"""Smoothing with a box's factors resident in LDS (every length of line at
the edges of its products-per-step forms) and streamed (boxes that do not
fit), with and without overlap and down to lines and columns one cell wide,
against the oracle at the FP64 parity bar (1e-10), and the same bits for
every number of threads per box."""
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


def _wl(sub, overlap, space="const"):
    n = (3 * sub[0], 3 * sub[1])
    y = gaussian_logk(n, 1.0 / n[0], 1.0, 0.2, 11)
    types, vals = _dirichlet_x(n)
    f = np.zeros_like(y)
    f[n[1] // 2, n[0] // 2] = 3.0
    return make_workload("c1").with_(
        ncell=n, h=1.0 / n[0], logk=y, source=f, bc_type=tuple(types), bc_value=vals, sub=sub,
        overlap=overlap, space=space, beta_mode="alpha", beta_mbf=1.0, beta_smooth=1.0, nsmooth=2)


@pytest.mark.parametrize("sub,overlap", [
    ((8, 8), 0), ((9, 7), 1), ((16, 6), 2), ((17, 5), 2), ((20, 7), 2), ((21, 4), 2), ((24, 5), 2),
    ((25, 3), 2), ((28, 6), 2), ((32, 3), 0), ((5, 1), 0), ((1, 6), 0), ((2, 2), 1),
    ((16, 76), 2),  # 80 lines of 20: streamed
])
def test_line_lengths(sub, overlap):
    import torch
    import paper_2404_13811_amd as m
    from paper_2404_13811_amd import api
    from gpu_util import oracle_solve, rel
    print("case", sub, overlap, flush=True)
    wl = _wl(sub, overlap)
    rp, rf, _, _ = oracle_solve(wl)
    out = []
    for nt in (64, 128, 256):
        ctx = m.create(2, wl.ncell, wl.h)
        api.configure(ctx, wl)
        m.set_smoothing(ctx, True, nt)
        m.build_basis(ctx)
        m.solve_interface(ctx)
        m.smooth(ctx, wl.nsmooth)
        p, fl = m.get_solution(ctx)
        torch.cuda.synchronize()
        out.append((p.cpu().numpy(), fl.cpu().numpy()))
        m.destroy(ctx)
    ep, ef = rel(out[0][0], rp), rel(out[0][1], rf)
    print("  p %.1e flux %.1e" % (ep, ef), flush=True)
    assert ep <= 1e-10 and ef <= 1e-10
    for p, fl in out[1:]:
        assert np.array_equal(p, out[0][0]) and np.array_equal(fl, out[0][1])
