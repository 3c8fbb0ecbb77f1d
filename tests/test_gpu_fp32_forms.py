"""FP32 factors with FP64 refinement at the edges of the kernel classes: line
lengths around the products-per-step forms, boxes with few and many lines
(inverses held in registers up to 33 lines, streamed beyond), constant and
linear seeds, no overlap and subdomains one or two cells thick, for every
number of threads per box, against the oracle at the FP32 form's parity bar
(1e-6, backward error 1e-12)."""
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


# linear seeds where the box with eight of them fits the FP32 form's LDS
SIZES = [((8, 8), 0), ((5, 9), 1), ((20, 21), 2), ((20, 22), 2), ((21, 6), 2), ((24, 7), 2), ((28, 29), 2),
         ((28, 30), 2), ((32, 5), 0), ((12, 40), 2), ((5, 2), 0), ((2, 6), 0), ((3, 3), 1)]


@pytest.mark.parametrize("sub,overlap,space", [
    (s, l, space) for s, l in SIZES for space in ("const", "linear")
    if space == "const" or (s[0] + 2 * l) * (s[1] + 2 * l) <= 800])
def test_fp32_classes(sub, overlap, space):
    import torch
    import paper_2404_13811_amd as m
    from paper_2404_13811_amd import api
    from gpu_util import oracle_solve, rel
    print("case", sub, overlap, space, flush=True)
    n = (3 * sub[0], 3 * sub[1])
    y = gaussian_logk(n, 1.0 / n[0], 1.0, 0.2, 11)
    types, vals = _dirichlet_x(n)
    f = np.zeros_like(y)
    f[n[1] // 2, n[0] // 2] = 3.0
    wl = make_workload("c1").with_(
        ncell=n, h=1.0 / n[0], logk=y, source=f, bc_type=tuple(types), bc_value=vals, sub=sub,
        overlap=overlap, space=space, beta_mode="alpha", beta_mbf=1.0, beta_smooth=1.0, nsmooth=2)
    rp, rf, _, _ = oracle_solve(wl)
    for nt in (64, 128, 256):
        ctx = m.create(2, wl.ncell, wl.h)
        api.configure(ctx, wl, "fp32_refine", tol=1e-12, max_refine=30)
        m.set_smoothing(ctx, True, nt)
        m.build_basis(ctx)
        m.solve_interface(ctx)
        m.smooth(ctx, wl.nsmooth)
        p, fl = m.get_solution(ctx)
        st = m.get_stats(ctx)
        torch.cuda.synchronize()
        ep, ef = rel(p.cpu().numpy(), rp), rel(fl.cpu().numpy(), rf)
        print("  %d threads: p %.1e flux %.1e backward error %.1e"
              % (nt, ep, ef, st["refine_max_resid"]), flush=True)
        m.destroy(ctx)
        assert ep <= 1e-6 and ef <= 1e-6 and st["refine_max_resid"] <= 1e-12
