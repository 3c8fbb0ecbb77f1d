"""The smoothing autotuner measures each precision form for itself: its
choice for one is dropped when the context goes over to the other, and the
results do not depend on it."""
import numpy as np
import pytest

from inputs import make_workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("name,scale", [("c2", 4), ("c4", 8)])
def test_each_precision_form_is_tuned(name, scale):
    import paper_2404_13811_amd as m
    from paper_2404_13811_amd import api
    wl = make_workload(name, scale=scale).with_(overlap=2)
    ctx = m.create(wl.dim, wl.ncell, wl.h)
    try:
        api.configure(ctx, wl)
        out = []
        for precision in ("fp64", "fp64", "fp32_refine", "fp64"):
            m.set_precision(ctx, precision, 1e-12, 30)
            before = m.get_stats(ctx)["smooth_threads"]
            m.build_basis(ctx)
            m.solve_interface(ctx)
            m.smooth(ctx, 2)
            out.append((before, m.get_stats(ctx)["smooth_threads"], m.get_pressure(ctx).cpu().numpy()))
        print(name, [o[:2] for o in out], flush=True)
    finally:
        m.destroy(ctx)
    assert [o[0] == 0 for o in out] == [True, False, True, True]
    assert all(o[1] in (64, 128, 256) for o in out)
    assert np.array_equal(out[0][2], out[1][2]) and np.array_equal(out[0][2], out[3][2])
