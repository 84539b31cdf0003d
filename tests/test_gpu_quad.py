"""The four-lane stepping kernel (automatic gather, short work lists) against
the one-lane kernel (a named gather): the same results bit for bit, at list
lengths around its spread, its full waves and its refills."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

N = (45, 38, 27)


@pytest.fixture(scope="module")
def charges():
    n, ch = N, synth.point_charges(7, 4)
    b = synth.sample_charges(ch, n, dtype=np.float32)
    return b, *synth.grid_geometry(n)


def _field(charges, storage, mode):
    import torch

    import paper_1609_00724_amd as q
    b, origin, spacing = charges
    dt = np.float64 if storage == "f64" else np.float32
    return q.field_init(*(torch.from_numpy(c.astype(dt)).cuda() for c in b), origin, spacing, storage=storage, mode=mode)


def _equal(a, b):
    import torch
    return all(torch.equal(a[k].nan_to_num(-7.0), b[k].nan_to_num(-7.0)) for k in b)


def _runs(field, n, words, **kw):
    """Outputs of the trace per launch word: random seeds in the box, the last
    ones on its faces, outside it and not finite."""
    import torch
    from paper_1609_00724_amd.api import TracePlan, make_opts
    s = synth.random_seeds(n, n)
    if n >= 8:
        s[-4:] = [[1.0, 0.3, 0.5], [0.2, 0.1, 0.0], [2.0, 0.0, 0.5], [np.nan, 0.0, 0.5]]
    soa = torch.from_numpy(np.ascontiguousarray(s.T)).cuda()
    out = []
    for w in words:
        plan = TracePlan(n, soa.device, want_steps=True, want_work=True)
        plan.run(field, soa, make_opts(launch=w, **kw))
        torch.cuda.synchronize()
        out.append(plan.out)
    return out


@pytest.mark.parametrize("n", [1, 9, 511, 513, 8200, 36000])
def test_list_lengths(charges, n):
    from paper_1609_00724_amd import _abi as A
    h = min(charges[2])
    r = _runs(_field(charges, "f32", "paper"), n, (0, A.launch_word(2, 64, A.GATHER_REGS)), rtol=1e-4, atol=1e-4,
              h_init=0.1 * h, h_max=h)
    assert _equal(*r)


@pytest.mark.parametrize("storage,step,mode,stepper", [
    ("f32", "f32", "interp_normalize", "ck54"), ("f32", "f32", "interp_normalize", "euler"), ("bf16", "f32", "paper", "ck54"),
    ("bf16", "f64", "interp_normalize", "euler"), ("f64", "f64", "paper", "ck54"), ("f64", "f64", "interp_normalize", "ck54"),
    ("f64", "f32", "paper", "euler"), ("f32", "f64", "paper", "ck54")])
def test_types_and_modes(charges, storage, step, mode, stepper):
    from paper_1609_00724_amd import _abi as A
    h = min(charges[2])
    # the automatic choice of the one-lane kernel: the register cache for FP32
    # stepping over FP32 or BF16 records, direct loads otherwise
    gather = A.GATHER_REGS if step == "f32" and storage != "f64" else A.GATHER_DIRECT
    hi = 0.2 * h if stepper == "euler" else 0.1 * h
    r = _runs(_field(charges, storage, mode), 3001, (0, A.launch_word(2, 64, gather)), rtol=1e-5, atol=1e-5, h_init=hi,
              h_max=2 * h, step_dtype=step, stepper=stepper)
    assert _equal(*r)


@pytest.mark.parametrize("limit", [dict(max_steps=7), dict(max_length=0.05), dict(rtol=1e-17, atol=1e-17)])
def test_stops(charges, limit):
    from paper_1609_00724_amd import _abi as A
    h = min(charges[2])
    kw = dict(dict(rtol=1e-4, atol=1e-4, h_init=0.1 * h, h_max=h, step_dtype="f64"), **limit)
    a, b = _runs(_field(charges, "f32", "paper"), 700, (0, A.launch_word(2, 64, A.GATHER_DIRECT)), **kw)
    assert _equal(a, b)
    want = 7 if "max_steps" in limit else 6 if "max_length" in limit else 9
    assert ((b["status"] & 0xFF) == want).any()


@pytest.mark.parametrize("step", ["f32", "f64"])
def test_batch(step):
    import torch

    from paper_1609_00724_amd import _abi as A
    from paper_1609_00724_amd.api import TraceBatchPlan, field_init, make_opts
    sets = []
    for k, f in enumerate(synth.batch_c3(count=5, first_seed=3100, dims=((24, 24, 16), (20, 31, 18)), seeds_range=(20, 3000))):
        fld = field_init(*(torch.from_numpy(c).cuda() for c in f["b"]), f["origin"], f["spacing"])
        sets.append((fld, torch.from_numpy(f["seeds"] if k != 2 else f["seeds"][:0]).cuda()))
    res = []
    for w in (0, A.launch_word(2, 64, A.GATHER_DIRECT)):
        plan = TraceBatchPlan(sets, make_opts(1e-4, 1e-4, step_dtype=step, launch=w), want_steps=True, want_work=True)
        res.append((plan.run(), plan.work))
    torch.cuda.synchronize()
    assert torch.equal(res[0][1], res[1][1])
    assert all(_equal(a, b) for a, b in zip(res[0][0], res[1][0]))


@pytest.mark.parametrize("n", [1, 130, 20000, 45000])
def test_general_geometry_list_lengths(n):
    """A spherical trace of n seeds (spread, full waves, refills) gives every
    seed what it gets in a call of its own few."""
    import torch

    import paper_1609_00724_amd as q
    lo, hi, g = (-0.3, -0.3, 1.0), (0.3, 0.3, 1.5), (25, 21, 17)
    ch = np.array([[0.93, 0.05, 0.1, 1.0], [0.95, -0.1, -0.05, -1.0]])
    b, origin, spacing = synth.sample_charges_spherical(ch, g, lo, hi, dtype=np.float32)
    f = q.field_init(*(torch.from_numpy(np.ascontiguousarray(c)).cuda() for c in b), origin, spacing, geometry="spherical")
    s = torch.from_numpy(synth.random_seeds(n + 1, n, lo=lo, hi=hi)).cuda()
    kw = dict(rtol=1e-4, atol=1e-4, h_init=0.002, h_max=0.02, want_steps=True)
    full = q.trace(f, s, **kw)
    idx = torch.arange(0, n, max(1, n // 50), device=s.device)
    part = q.trace(f, s[idx], **kw)
    torch.cuda.synchronize()
    assert _equal({k: v[..., idx] for k, v in full.items()}, part)


@pytest.mark.parametrize("n,where", [(1, "box"), (15, "box"), (33, "bottom"), (5000, "mixed")])
@pytest.mark.parametrize("stepper,mode", [("ck54", "paper"), ("ck54", "interp_normalize"), ("euler", "paper")])
def test_small_calls_end_as_large_ones(charges, n, where, stepper, mode):
    """Landing and Q of a small call (one kernel) against the same seeds inside
    a call past 2^18 seeds (landing list, separate assembly), bit for bit."""
    import torch

    import paper_1609_00724_amd as q
    h = min(charges[2])
    f = _field(charges, "f32", mode)
    s = synth.random_seeds(n, n)
    if where != "box":
        s[:: 1 if where == "bottom" else 2, 2] = 0.0
    s = torch.from_numpy(s).cuda()
    pad = torch.tensor([[2.0, 0.0, 0.0]], dtype=torch.float64, device="cuda").expand((1 << 18) + 1, 3)   # outside: no work
    kw = dict(rtol=1e-4, atol=1e-4, h_init=0.2 * h, h_max=2 * h, stepper=stepper, want_steps=True)
    a = q.trace(f, s, **kw)
    b = q.trace(f, torch.cat([s, pad]), **kw)
    torch.cuda.synchronize()
    assert _equal({k: v[..., :n] for k, v in b.items()}, a)


@pytest.mark.parametrize("order", ["quadratic", "cubic"])
@pytest.mark.parametrize("storage,step,mode,stepper", [
    ("f32", "f32", "paper", "ck54"), ("f64", "f64", "paper", "ck54"), ("f32", "f64", "interp_normalize", "ck54"),
    ("f64", "f32", "interp_normalize", "euler")])
def test_higher_orders(charges, order, storage, step, mode, stepper):
    """Quad stencils (folded ones at every face: 4 nodes along z) against one lane's."""
    import torch

    import paper_1609_00724_amd as q
    from paper_1609_00724_amd import _abi as A
    b, origin, spacing = charges
    dt = np.float64 if storage == "f64" else np.float32
    b = [torch.from_numpy(np.ascontiguousarray(c[:4].astype(dt))).cuda() for c in b]
    f = q.field_init(*b, origin, spacing, storage=storage, mode=mode, order=order)
    h = min(spacing)
    hi = 0.2 * h if stepper == "euler" else 0.1 * h
    r = _runs(f, 1100, (0, A.launch_word(2, 64, A.GATHER_DIRECT)), rtol=1e-4, atol=1e-4, h_init=hi, h_max=2 * h,
              step_dtype=step, stepper=stepper)
    assert ((r[0]["status"] & 0xFF) <= 5).sum() > 50
    assert _equal(*r)


@pytest.mark.parametrize("n", [1, 17, 129, 20001])
@pytest.mark.parametrize("geometry", ["cartesian", "spherical"])
def test_work_counters_of_every_workgroup_arrive(charges, n, geometry):
    # a workgroup adds its waves' counts in one piece: lists of part of a
    # wave, of some waves of a workgroup, and of many workgroups
    import torch

    import paper_1609_00724_amd as q
    b, origin, spacing = charges
    if geometry == "spherical":
        origin, spacing = (-0.3, -0.3, 1.0), tuple(w / (m - 1) for w, m in zip((0.6, 0.6, 0.5), N))
    f = q.field_init(*(torch.from_numpy(c).cuda() for c in b), origin, spacing, storage="f32", geometry=geometry)
    hi = [o + s * (m - 1) for o, s, m in zip(origin, spacing, N)]
    rng = np.random.default_rng(n)
    seeds = torch.from_numpy(rng.uniform(origin, hi, (n, 3))).cuda()
    h = min(spacing)
    out = q.trace(f, seeds, rtol=1e-4, atol=1e-4, h_init=0.1 * h, h_max=2 * h, want_steps=True, want_work=True)
    steps = out["steps"]
    attempts, evals, halves, landed = out["work"].tolist()
    assert attempts == int(steps.sum()) and halves == int((steps > 0).sum())
    assert 5 * attempts < evals <= 6 * attempts and (n == 1 or landed > 0) and landed <= halves
