"""One seed's line is the same line whatever the call around it: which gather the
launch word names, one field or a batch, few seeds or many.  Bit for bit, over
the interpolation modes, record types, orders and steppers."""
import numpy as np
import pytest

import synth
from test_gpu_quad import _equal, _field, charges  # noqa: F401 (a fixture)

pytestmark = pytest.mark.gpu


def _seeds(n, seed):
    """Random seeds in the box, a third of them on its bottom face, some on
    other faces, outside it and not finite."""
    import torch
    s = synth.random_seeds(seed, n)
    s[::3, 2] = 0.0
    s[-4:] = [[1.0, 0.3, 0.5], [0.2, 0.1, 1.0], [2.0, 0.0, 0.5], [np.nan, 0.0, 0.5]]
    return torch.from_numpy(s).cuda()


@pytest.mark.parametrize("stepper", ["ck54", "euler"])
@pytest.mark.parametrize("storage,mode", [("f32", "interp_normalize"), ("bf16", "interp_normalize"), ("f32", "paper")])
def test_gathers_and_batches(charges, storage, mode, stepper):  # noqa: F811
    import torch

    from paper_1609_00724_amd import _abi as A
    from paper_1609_00724_amd.api import TraceBatchPlan, TracePlan, make_opts
    f = _field(charges, storage, mode)
    f.add_cells()
    f.add_bricks()
    gathers = [A.GATHER_AUTO, A.GATHER_DIRECT, A.GATHER_CACHED, A.GATHER_REGS, A.GATHER_CELLS, A.GATHER_BRICKS]
    if storage == "f32":
        f.add_cell_dirs()
        gathers.append(A.GATHER_DIRS)
    h = min(charges[2])
    s = _seeds(2500, 11)
    soa = s.t().contiguous()
    runs = {}
    for g in gathers:
        o = make_opts(1e-4, 1e-4, h_init=(0.2 if stepper == "euler" else 0.1) * h, h_max=2 * h, stepper=stepper,
                      launch=A.launch_word(2, 64, g))
        runs["gather %d" % g] = TracePlan(s.shape[0], s.device, want_steps=True).run(f, soa, o)
        if g <= A.GATHER_DIRECT:
            runs["batch, gather %d" % g] = TraceBatchPlan([(f, s[:40]), (f, s)], o, want_steps=True).run()[1]
    torch.cuda.synchronize()
    ref = runs["gather 1"]
    assert ((ref["status"] & 0xFF) <= 5).sum() > 1500
    assert [k for k, r in runs.items() if not _equal(r, ref)] == []
