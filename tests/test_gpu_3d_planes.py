"""3-D local factors (FP64) at the edges of their plane blocks: one to four
tiles of 16 cells, the last with up to eight pivots or up to sixteen, planes
down to one cell wide, two Robin parameters (Step 6's factor), scalar and
diagonal-tensor K, against the oracle at the FP64 parity bar (1e-10)."""
import numpy as np
import pytest

from inputs import make_workload
from inputs.fields import layered_logk
from inputs.workloads import _dirichlet_x

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("plane,overlap,tensor", [
    ((1, 7), 0, False), ((8, 1), 0, False), ((3, 3), 0, False), ((4, 4), 0, True), ((17, 1), 0, False),
    ((6, 4), 0, False), ((5, 5), 0, True), ((8, 4), 0, False), ((11, 3), 0, False), ((4, 4), 1, False),
    ((4, 4), 1, True), ((8, 5), 0, False), ((1, 41), 0, False), ((8, 6), 0, False), ((7, 7), 0, False),
    ((8, 7), 0, False), ((19, 3), 0, False), ((4, 4), 2, True)])
def test_plane_blocks(plane, overlap, tensor):
    from gpu_util import gpu_solve, oracle_solve, rel
    print("case", plane, overlap, tensor, flush=True)
    sub = plane + (4,)
    n = tuple(3 * s if overlap else 2 * s for s in sub)
    y = layered_logk(n, 1.0 / 64, 5.0, (0.2, 0.2, 0.02), 9, 1e6)
    types, vals = _dirichlet_x(n)
    wl = make_workload("c4", scale=8).with_(
        ncell=n, logk=y, source=np.zeros_like(y), bc_type=tuple(types), bc_value=vals, sub=sub,
        overlap=overlap, beta_mbf=0.5, beta_smooth=1.0, nsmooth=1)
    if tensor:
        rng = np.random.default_rng(5)
        wl = wl.with_tensor([rng.standard_normal(y.shape) for _ in range(3)])
    p, fl, _, _ = gpu_solve(wl)
    rp, rf, _, _ = oracle_solve(wl)
    ep, ef = rel(p, rp), rel(fl, rf)
    print("  p %.1e flux %.1e" % (ep, ef), flush=True)
    assert ep <= 1e-10 and ef <= 1e-10
