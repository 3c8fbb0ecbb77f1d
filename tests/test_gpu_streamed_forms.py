"""Forms that take over where a box's factors do not fit LDS: the reverse
smoothing phase that streams them (boxes of 32 x 32 and 21 x 64 cells, whose forward
phase holds them) against the CPU adjoint at the bars of the other reverse
cases, and the one-launch smoothing sweep that streams them (boxes of 80
lines), bit for bit the same as one launch per phase, also where a workgroup
takes several boxes of a colour."""
import numpy as np
import pytest

from inputs import make_workload
from inputs.fields import gaussian_logk
from inputs.workloads import _dirichlet_x
from test_gpu_adjoint import _gpu_grad, _oracle_grad
from test_gpu_parity import _smooth_trace

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _wl(sub, overlap):
    n = (3 * sub[0], 3 * sub[1])
    y = gaussian_logk(n, 1.0 / n[0], 1.0, 0.2, 12)
    types, vals = _dirichlet_x(n)
    return make_workload("c1").with_(
        ncell=n, h=1.0 / n[0], logk=y, source=np.zeros_like(y), bc_type=tuple(types), bc_value=vals,
        sub=sub, overlap=overlap, space="const", beta_mode="alpha", beta_mbf=1.0, beta_smooth=1.0, nsmooth=2)


@pytest.mark.parametrize("sub,overlap", [((24, 24), 4), ((32, 32), 0), ((17, 60), 2)])
def test_streamed_reverse_phase(sub, overlap):
    print("case", sub, overlap, flush=True)
    wl = _wl(sub, overlap)
    Jg, g = _gpu_grad(wl, 2)
    Jo, go = _oracle_grad(wl, 2)
    err = np.linalg.norm(g - go) / np.linalg.norm(go)
    print("  J %.12e vs %.12e  gradient rel L2 %.3e" % (Jg, Jo, err), flush=True)
    assert abs(Jg - Jo) <= 1e-10 * abs(Jo)
    assert err <= 1e-8


@pytest.mark.parametrize("sub,overlap", [((16, 76), 2), ((20, 80), 0)])
def test_streamed_persistent_sweep(sub, overlap):
    print("case", sub, overlap, flush=True)
    wl = _wl(sub, overlap)
    steps = [2, 1]
    ref, _ = _smooth_trace(wl, False, 256, steps)
    for threads, groups in [(256, 0), (128, 0), (64, 0), (256, 3), (128, 1)]:
        got, st = _smooth_trace(wl, False, threads, steps, persistent=(True, groups))
        assert st["smooth_persistent"] == 1 and st["n_smooth_launches"] == 1
        for (p, fl), (rp, rf) in zip(got, ref):
            assert np.array_equal(p, rp) and np.array_equal(fl, rf)
