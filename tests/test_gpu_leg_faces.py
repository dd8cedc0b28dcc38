"""V-cycle legs at their faces: non-finite sources beside one wall, against the oracle; face values
under a memory budget, legs on a budget that holds no scratch, and the large levels' one-sweep up pass."""
import numpy as np
import pytest

import oracle
from oracle import FIXED, PERIODIC, ZERO_GRADIENT

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

KINDS = {
    "layer": [PERIODIC] * 4 + [FIXED, ZERO_GRADIENT],
    "fixed": [FIXED] * 6,
    "mixed": [FIXED, ZERO_GRADIENT, PERIODIC, PERIODIC, ZERO_GRADIENT, FIXED],
    "periodic": [PERIODIC] * 6,
}
OMEGA = 1.15


@pytest.fixture(scope="module")
def mg():
    import paper_2302_13903_amd as m
    return m


def dev(a, dt=torch.float64):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0", dt)


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy().astype(np.float64)


def homogeneous(kinds):
    return [k if k in (PERIODIC, ZERO_GRADIENT) else FIXED for k in kinds]


def sweeps(u, f, h, kinds, bext, count):
    for _ in range(count):
        u = oracle.smooth(u, f, h, OMEGA, kinds, bext)
    return u


@pytest.mark.parametrize("f32", [False, True], ids=["fp64", "fp32"])
@pytest.mark.parametrize("ns", [1, 2])
@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("n", [32, 64, 128])
def test_non_finite_source_stays_at_its_wall(mg, n, kind, ns, f32):
    """A NaN or an infinity in f beside one wall makes exactly the cells non-finite that the sweeps
    carry it to: none beside the opposite wall, unless the axis is periodic."""
    kinds = KINDS[kind]
    print(f"non-finite source n={n} {kind} ns={ns} f32={f32}", flush=True)
    rng = np.random.default_rng(n + ns)
    u, e = rng.standard_normal((n,) * 3), rng.standard_normal((n // 2,) * 3)
    f = rng.standard_normal((n,) * 3) * n * n
    f[n - 1, n // 2, n // 3] = np.nan
    f[0, n // 4, n - 1] = np.inf
    f[n // 2, n - 1, 5] = -np.inf
    f[n // 3, 7, 0] = np.nan
    none, dt, h = [None] * 6, (torch.float32 if f32 else torch.float64), 1.0 / n
    down, up = (mg.mg_op_down_f32, mg.mg_op_up_f32) if f32 else (mg.mg_op_down, mg.mg_op_up)
    ctx = mg.Context(0)
    with np.errstate(all="ignore"):
        ref = sweeps(u, f, h, kinds, none, ns)
        ref_fc = oracle.restrict(oracle.defect(ref, f, h, kinds, none))
        ref_up = sweeps(oracle.prolong_add(e, u, homogeneous(kinds)), f, h, kinds, none, ns)
    du, fc, uc = dev(u, dt), dev(e, dt), dev(e, dt)
    down(du, dev(f, dt), fc, uc, h, OMEGA, ns, kinds, none, ctx=ctx)
    assert np.array_equal(np.isfinite(host(du)), np.isfinite(ref))
    assert np.array_equal(np.isfinite(host(fc)), np.isfinite(ref_fc))
    du = dev(u, dt)
    up(du, dev(f, dt), dev(e, dt), h, OMEGA, ns, kinds, none, homogeneous(kinds), ctx=ctx)
    assert np.array_equal(np.isfinite(host(du)), np.isfinite(ref_up))


@pytest.mark.parametrize("f32", [False, True], ids=["fp64", "fp32"])
@pytest.mark.parametrize("ns", [1, 2])
@pytest.mark.parametrize("kind", ["layer", "fixed", "mixed"])
@pytest.mark.parametrize("n", [32, 64, 128, 256])
def test_face_values_need_no_more_memory(mg, n, kind, ns, f32):
    """A leg with face values takes one level array of scratch: with a budget of that much it runs the
    same kernels as without one, bitwise, and leaves f as it was.  A zero-gradient face ignores values."""
    kinds = KINDS[kind]
    print(f"valued legs n={n} {kind} ns={ns} f32={f32}", flush=True)
    gen = torch.Generator(device="cuda:0").manual_seed(n + ns)
    dt, h = (torch.float32 if f32 else torch.float64), 1.0 / n

    def rand(shape, t):
        return torch.randn(shape, generator=gen, dtype=t, device="cuda:0")

    u, f, e = rand((n,) * 3, dt), rand((n,) * 3, dt) * n * n, rand((n // 2,) * 3, dt)
    f0 = f.clone()
    bext = [rand((n + 2,) * 2, torch.float64) if k == FIXED else None for k in kinds]
    ignored = [rand((n + 2,) * 2, torch.float64) if k == ZERO_GRADIENT else b for k, b in zip(kinds, bext)]
    down, up = (mg.mg_op_down_f32, mg.mg_op_up_f32) if f32 else (mg.mg_op_down, mg.mg_op_up)
    budget = mg.mg_footprint_bytes(mg.params(2, 0.5)) + u.element_size() * n ** 3
    out = []
    for ctx, b in ((mg.Context(0), bext), (mg.Context(0, hbm_budget=budget), ignored)):
        a, fc, uc = u.clone(), torch.zeros_like(e), torch.ones_like(e)
        down(a, f, fc, uc, h, OMEGA, ns, kinds, b, ctx=ctx)
        c = u.clone()
        up(c, f, e, h, OMEGA, ns, kinds, b, homogeneous(kinds), ctx=ctx)
        out.append((a, fc, c))
    torch.cuda.synchronize()
    assert torch.equal(f, f0)
    assert all(torch.equal(x, y) for x, y in zip(*out))


@pytest.mark.parametrize("f32", [False, True], ids=["fp64", "fp32"])
@pytest.mark.parametrize("kind", ["periodic", "mixed"])
def test_one_sweep_without_scratch(mg, kind, f32):
    """One sweep at 32^3 on a budget that holds no level array runs in place, as with memory (u to the
    sums' rounding, 40 epsilons of the terms of either side); two sweeps are refused."""
    n, kinds = 32, KINDS[kind]
    print(f"legs without scratch {kind} f32={f32}", flush=True)
    rng = np.random.default_rng(4)
    dt, h = (torch.float32 if f32 else torch.float64), 1.0 / n
    u, f = dev(rng.standard_normal((n,) * 3), dt), dev(rng.standard_normal((n,) * 3) * n * n, dt)
    e = dev(rng.standard_normal((n // 2,) * 3), dt)
    bext = [dev(rng.standard_normal((n + 2,) * 2)) if k == FIXED else None for k in kinds]
    down, up = (mg.mg_op_down_f32, mg.mg_op_up_f32) if f32 else (mg.mg_op_down, mg.mg_op_up)
    tight = mg.Context(0, hbm_budget=mg.mg_footprint_bytes(mg.params(2, 0.5)))
    out = []
    for ctx in (mg.Context(0), tight):
        a, c, fc, uc = u.clone(), u.clone(), torch.zeros_like(e), torch.ones_like(e)
        down(a, f, fc, uc, h, OMEGA, 1, kinds, bext, ctx=ctx)
        up(c, f, e, h, OMEGA, 1, kinds, bext, homogeneous(kinds), ctx=ctx)
        assert float(uc.abs().max()) == 0.0
        out.append((host(a), host(fc), host(c)))
    eps = 40 * float(torch.finfo(dt).eps)
    su = 6 * max(float(u.abs().max()) + float(e.abs().max()), h * h * float(f.abs().max()),
                 2 * max([0.0] + [float(b.abs().max()) for b in bext if b is not None]))
    for x, y, scale in zip(*out, (su, float(f.abs().max()) + 12 * su / h ** 2, su)):
        assert np.abs(x - y).max() <= 2 * eps * scale
    with pytest.raises(mg.MgError, match="OOM"):
        down(u.clone(), f, torch.zeros_like(e), torch.zeros_like(e), h, OMEGA, 2, kinds, bext, ctx=tight)


@pytest.mark.parametrize("kind", ["periodic", "layer"])
def test_large_one_sweep_up_is_the_one_sweep_pass(mg, kind):
    """FP32 at 512^3, one sweep, no x or y wall: the pass that runs with the streaming legs off, bitwise."""
    n, kinds = 512, KINDS[kind]
    print(f"up 512^3 one sweep {kind}", flush=True)
    gen = torch.Generator(device="cuda:0").manual_seed(1)
    u, f, e = (torch.randn((m,) * 3, generator=gen, dtype=torch.float32, device="cuda:0") for m in (n, n, n // 2))
    out = []
    for text in ("march fp32 2\n", "march fp32 0\n"):
        ctx = mg.Context(0)
        ctx.set_tuning(text)
        a = u.clone()
        mg.mg_op_up_f32(a, f, e, 1.0 / n, OMEGA, 1, kinds, None, homogeneous(kinds), ctx=ctx)
        torch.cuda.synchronize()
        out.append(a)
        ctx.close()
    assert torch.equal(*out)
