"""Device memory of what FP64 smoothing keeps per box: one vector (the static
right-hand side) and the coefficients of the box-side and Gamma faces, in FP64
contexts only (every other array of a plan serves both precision forms)."""
import pytest

from inputs import make_workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def test_static_smoothing_arrays():
    import torch
    import paper_2404_13811_amd as m
    from paper_2404_13811_amd import api
    wl = make_workload("c3")  # 4096 boxes of 24 x 24 cells, four seeds
    used = {}
    # the first round loads the kernels and their scratch memory
    for precision in ("fp32_refine", "fp64") * 2:
        ctx = m.create(wl.dim, wl.ncell, wl.h)
        try:
            api.configure(ctx, wl, precision)
            torch.cuda.synchronize()
            free = torch.cuda.mem_get_info()[0]
            m.build_basis(ctx)
            torch.cuda.synchronize()
            used[precision] = free - torch.cuda.mem_get_info()[0]
        finally:
            m.destroy(ctx)
    more = used["fp64"] - used["fp32_refine"]
    b0, faces = 8 * 4096 * 24 * 24, 8 * 4096 * (4 * (16 + 16 + 4 * 4) + 4 * 16)
    slack = 3 * 4 * 2**20  # granularity of three allocations
    print("FP32 form %d bytes, FP64 %d: %d more, arrays %d" % (used["fp32_refine"], used["fp64"], more, b0 + faces),
          flush=True)
    assert b0 - slack <= more <= b0 + faces + slack
