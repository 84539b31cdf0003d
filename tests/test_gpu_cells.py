"""The stepping kernel's register cell cache at the workgroup sizes of the launch
word: each wave's lanes have LDS slots of their own for the cell they left, and
the brick variant parks position and length behind them.  Short steps (lanes
stay in their cell, or go back and forth over a face) and long ones (most stages
land in another cell) give the direct gather's outputs, bit for bit."""
import numpy as np
import pytest

from test_gpu_trace import _mixed_seeds, gpu_field, small_charges  # noqa: F401 (a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wg", [64, 128, 256])
@pytest.mark.parametrize("cap", [0.3, 1.5, 6.0])
def test_register_cache_by_workgroup_and_step(small_charges, wg, cap):
    import torch

    from paper_1609_00724_amd import _abi as A
    from paper_1609_00724_amd.api import TracePlan, make_opts
    c = small_charges
    h = min(c["spacing"])
    dev = torch.device("cuda:0")
    n = 1777   # the last workgroup and its last wave partly filled
    seeds = torch.from_numpy(np.ascontiguousarray(_mixed_seeds(n, 5).T)).to(dev)
    for storage in ("f32", "bf16"):
        fg = gpu_field(c["b"], c["origin"], c["spacing"], storage=storage)
        gathers = [A.GATHER_DIRECT, A.GATHER_REGS]
        if storage == "f32":
            fg.add_bricks()
            fg.add_cell_dirs()
            gathers += [A.GATHER_BRICKS, A.GATHER_DIRS]
        ref = None
        for gather in gathers:
            plan = TracePlan(n, dev, want_steps=True)
            opts = make_opts(1e-3, 1e-3, h_init=0.1 * h, h_max=cap * h, step_dtype="f32",
                             launch=A.launch_word(1, wg, gather))
            out = plan.run(fg, seeds, opts)
            torch.cuda.synchronize()
            out = {k: v.clone() for k, v in out.items() if v is not None}
            if ref is None:
                ref = out
            for k in ref:
                assert torch.equal(torch.nan_to_num(out[k], nan=-7.0), torch.nan_to_num(ref[k], nan=-7.0)), (storage, gather, k)
        assert int((ref["steps"][0] > 3).sum()) > n // 4
