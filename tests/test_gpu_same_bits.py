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


@pytest.mark.parametrize("stepper", ["ck54", "euler"])
@pytest.mark.parametrize("mode", ["paper", "interp_normalize"])
@pytest.mark.parametrize("storage,order", [("f32", "linear"), ("bf16", "linear"), ("f64", "linear"), ("f32", "quadratic"),
                                           ("f64", "quadratic"), ("f32", "cubic"), ("f64", "cubic")])
def test_ends_by_call_size(charges, storage, order, mode, stepper):  # noqa: F811
    """Landing and Q of a small call (four lanes a half-line) against the same
    seeds in a call past 2^18 seeds (one lane, an assembly of its own)."""
    import torch

    import paper_1609_00724_amd as q
    b, origin, spacing = charges
    dt = np.float64 if storage == "f64" else np.float32
    # 20 nodes along z: folded stencils at both faces and plain ones between
    b = [torch.from_numpy(np.ascontiguousarray(c[:20].astype(dt))).cuda() for c in b]
    f = q.field_init(*b, origin, spacing, storage=storage, mode=mode, order=order)
    h, n = min(spacing), 3000
    s = _seeds(n, 5)
    s[:, 2] *= 19 / 26   # into the box, the bottom and top faces kept
    pad = torch.tensor([[2.0, 0.0, 0.0]], dtype=torch.float64, device="cuda").expand((1 << 18) + 1, 3)   # outside: no work
    kw = dict(rtol=1e-4, atol=1e-4, h_init=0.2 * h, h_max=2 * h, stepper=stepper, want_steps=True)
    a = q.trace(f, s, **kw)
    r = q.trace(f, torch.cat([s, pad]), **kw)
    torch.cuda.synchronize()
    r = {k: v[..., :n] for k, v in r.items()}
    assert ((a["status"] & 0xFF) <= 5).sum() > 2000
    assert [k for k in a if not torch.equal(a[k].nan_to_num(-7.0), r[k].nan_to_num(-7.0))] == []


@pytest.mark.parametrize("storage,mode", [("f32", "paper"), ("bf16", "interp_normalize"), ("f64", "interp_normalize")])
def test_batch_ends_by_call_size(charges, storage, mode):  # noqa: F811
    """The same for a batch, whose larger calls begin past 2^20 seeds."""
    import torch

    from paper_1609_00724_amd.api import TraceBatchPlan, make_opts
    f, g = _field(charges, storage, mode), _field([[np.ascontiguousarray(c[:20]) for c in charges[0]], *charges[1:]], storage, mode)
    h, n = min(charges[2]), 2000
    s, t = _seeds(n, 6), _seeds(n, 7)
    t[:, 2] *= 19 / 26
    pad = torch.tensor([[2.0, 0.0, 0.0]], dtype=torch.float64, device="cuda").expand((1 << 20) + 1, 3)
    o = make_opts(1e-4, 1e-4, h_init=0.2 * h, h_max=2 * h)
    a = TraceBatchPlan([(f, s), (g, t)], o, want_steps=True).run()
    b = TraceBatchPlan([(f, s), (g, t), (f, pad)], o, want_steps=True).run()
    torch.cuda.synchronize()
    assert [(i, k) for i in range(2) for k in a[i] if not torch.equal(a[i][k].nan_to_num(-7.0), b[i][k].nan_to_num(-7.0))] == []


@pytest.mark.parametrize("step", ["f32", "f64"])
@pytest.mark.parametrize("parts", [False, True])
def test_spread_lists_keep_to_fewer_workgroups(step, parts):
    """A list that the device finds spread leaves the last workgroups of the
    launch unused: every line is still traced, once, with the same result, and
    so is each of a list that is not (seeds on the bottom face)."""
    import torch

    import paper_1609_00724_amd as q
    from paper_1609_00724_amd import _abi as A
    from paper_1609_00724_amd.api import TracePlan, make_opts
    n, seeds = (121, 121, 61) if step == "f64" else (97, 81, 41), 290000   # above the rules' lines (8 and 4 MB; 2^19 half-lines)
    b = synth.sample_charges(synth.point_charges(7, 4), n, dtype=np.float32)
    f = q.field_init(*(torch.from_numpy(c).cuda() for c in b), *synth.grid_geometry(n))
    h = min(f.spacing)
    gather = A.GATHER_REGS if step == "f32" else A.GATHER_DIRECT
    for bottom in (False, True):
        s = synth.random_seeds(3, seeds)
        if bottom:
            s[:, 2] = 0.0
        soa = torch.from_numpy(np.ascontiguousarray(s.T)).cuda()
        r = []
        for lanes in (0, 1):
            plan = TracePlan(seeds, soa.device, want_steps=True, want_work=True)
            r.append(plan.run(f, soa, make_opts(1e-2, 1e-2, h_init=h, h_max=8 * h, step_dtype=step,
                                                launch=A.launch_word(lanes, 256, gather, parts=parts))))
        torch.cuda.synchronize()
        assert _equal(*r)
        assert int(r[0]["work"][2]) > (1.5 if not bottom else 0.5) * seeds


@pytest.mark.parametrize("storage,step", [("f32", "f64"), ("f32", "f32"), ("f64", "f64")])
def test_volume_whose_levels_keep_to_fewer_workgroups(charges, storage, step):  # noqa: F811
    """A volume whose base list is long and whose levels' lists are short, in
    one set of workgroups or some of it: the same samples as with a named
    number of lanes, the work counted in full."""
    import torch

    import paper_1609_00724_amd as q
    from paper_1609_00724_amd import _abi as A
    from paper_1609_00724_amd.api import make_opts
    f = _field(charges, storage, "paper")
    h = min(charges[2])
    spec = q.VolumeSpec(-1.0, 1.0, -1.0, 1.0, 0.0, 1.0, 7, 1, 7, 0.3, 1)
    got = []
    for lanes in (0, 1, 2):
        plan = q.QMapPlan(spec, 2**22, "cuda", want_steps=True)
        plan.run(f, make_opts(1e-2, 1e-2, 0.1 * h, 8 * h, step_dtype=step, launch=A.launch_word(lanes, 256, 0)))
        r = plan.result()
        assert int(plan.work[0]) == int(r["steps"].sum())
        got.append({k: r[k].double() for k in ("keys", "fll", "q_perp", "status", "steps")})
    n = got[0]["keys"].shape[0]
    assert 2**21 < n < 2**21 + 2**18      # the levels' lists are short
    for other in got[1:]:
        assert _equal(got[0], other)
