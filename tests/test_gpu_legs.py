"""The one-launch kernels of the small levels at the sizes where they can go wrong: the region-tile
legs (32^3: regions shorter than the halo, so a wall lies in the halo of the region after next;
64^3 and 128^3) with one and two sweeps per leg, and the coarse tail (every grid <= 16^3, sweep
counts 0..4), against the oracle.

Bounds: a leg's u is 1e-13 (FP64) or 40 FP32 epsilons of the largest magnitude in its sums (the
values, the face values and h^2 f); its coarse source the same of max|f| + 12 max|u| / h^2.  Whole
solves at equal cycle counts: phi to 1e-10, as every solve check."""
import numpy as np
import pytest

import oracle
import workloads as wl
from oracle import FIXED, PERIODIC, ZERO_GRADIENT
from parity import rel

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

KINDS = {
    "periodic": [PERIODIC] * 6,
    "fixed": [FIXED] * 6,
    "layer": [PERIODIC] * 4 + [FIXED, ZERO_GRADIENT],
    "mixed": [FIXED, ZERO_GRADIENT, ZERO_GRADIENT, FIXED, PERIODIC, PERIODIC],
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


def sweeps(u, f, h, kinds, bext, count):
    for _ in range(count):
        u = oracle.smooth(u, f, h, OMEGA, kinds, bext)
    return u


@pytest.mark.parametrize("f32", [False, True], ids=["fp64", "fp32"])
@pytest.mark.parametrize("ns", [1, 2])
@pytest.mark.parametrize("n,kind", [(32, "periodic"), (32, "fixed"), (32, "layer"), (64, "layer"), (64, "mixed"),
                                    (128, "fixed")])
def test_tile_legs(mg, n, kind, ns, f32):
    kinds = KINDS[kind]
    hom = [k if k in (PERIODIC, ZERO_GRADIENT) else FIXED for k in kinds]
    print(f"tile legs n={n} {kind} ns={ns} f32={f32}", flush=True)
    rng = np.random.default_rng(n + ns)
    u, e = rng.standard_normal((n,) * 3), rng.standard_normal((n // 2,) * 3)
    f = rng.standard_normal((n,) * 3) * n * n
    bext = [rng.standard_normal((n + 2,) * 2) if k == FIXED else None for k in kinds]
    dt, h = (torch.float32 if f32 else torch.float64), 1.0 / n
    if f32:
        u, e, f = (a.astype(np.float32).astype(np.float64) for a in (u, e, f))
    dbext = [None if b is None else dev(b) for b in bext]
    ctx = mg.Context(0)
    ctx.set_tuning("march fp64 0\nmarch fp32 0\n")
    su = max(np.abs(u).max(), np.abs(e).max(), h * h * np.abs(f).max()) + 2 * max([0.0] + [np.abs(b).max() for b in bext if b is not None])
    eps = 40 * float(np.finfo(np.float32).eps) if f32 else 1e-13
    down, up = (mg.mg_op_down_f32, mg.mg_op_up_f32) if f32 else (mg.mg_op_down, mg.mg_op_up)

    ref = sweeps(u, f, h, kinds, bext, ns)
    ref_fc = oracle.restrict(oracle.defect(ref, f, h, kinds, bext))
    du, fc, uc = dev(u, dt), dev(e, dt), dev(e, dt)
    down(du, dev(f, dt), fc, uc, h, OMEGA, ns, kinds, dbext, ctx=ctx)
    assert np.abs(host(du) - ref).max() <= eps * 6 * su
    assert np.abs(host(fc) - ref_fc).max() <= eps * (np.abs(f).max() + 12 * su / h ** 2)
    assert float(uc.abs().max()) == 0.0

    ref = sweeps(oracle.prolong_add(e, u, hom), f, h, kinds, bext, ns)
    du = dev(u, dt)
    up(du, dev(f, dt), dev(e, dt), h, OMEGA, ns, kinds, dbext, hom, ctx=ctx)
    assert np.abs(host(du) - ref).max() <= eps * 12 * su


@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("n,npre,npost", [(2, 2, 2), (4, 1, 3), (8, 0, 2), (8, 4, 0), (16, 2, 2), (16, 1, 1), (16, 3, 4),
                                          (32, 1, 1), (64, 1, 2), (64, 1, 1)])
@pytest.mark.parametrize("mode", ["fmg", "mgi"])
def test_small_solves(mg, n, npre, npost, kind, mode):
    kinds = KINDS[kind]
    print(f"solve n={n} V({npre},{npost}) {kind} {mode}", flush=True)
    rng = np.random.default_rng(7 * n + npre)
    rho = rng.standard_normal((n,) * 3)
    fb = [rng.standard_normal((n, n)) if k == FIXED else None for k in kinds]
    phi0 = rng.standard_normal((n,) * 3)
    ref, hist, _ = oracle.solve(rho, 1.0 / n, kinds, fixed_b=fb, fixed_cycles=4, npre=npre, npost=npost, mode=mode,
                                phi0=phi0 if mode == "mgi" else None)
    phi = dev(phi0)
    got, ghist, _ = mg.solve(dev(rho), 1.0 / n, kinds, fixed_b=[None if b is None else dev(b) for b in fb],
                             fixed_cycles=4, npre=npre, npost=npost, mode=mode, phi=phi)
    assert rel(host(got), ref) < 1e-10
    # a defect is a difference of terms 12 max|phi| / h^2: its floor beside the history's own 1e-6
    rms_f = 4 * np.pi * np.sqrt(np.mean(rho ** 2))
    floor = 12 * np.finfo(np.float64).eps * np.abs(ref).max() * n * n / rms_f
    assert len(ghist) == len(hist)
    for a, b in zip(ghist, hist):
        assert abs(a - b) <= 1e-6 * b + 10 * floor


@pytest.mark.parametrize("npre,npost", [(1, 1), (2, 1)])
def test_blocks_one_sweep(mg, npre, npost):
    """Block levels with one sweep per leg give the dense potential."""
    n = 64
    rho = wl.gaussian_clumps(n, 3, n_clumps=6)
    a, _, _ = mg.solve(dev(rho), 1.0 / n, "fixed", fixed_cycles=4, npre=npre, npost=npost)
    b, _, _ = mg.solve(mg.to_blocks(dev(rho), 16), 1.0 / n, "fixed", fixed_cycles=4, npre=npre, npost=npost, layout="blocks")
    assert rel(host(mg.from_blocks(b, n, 16)), host(a)) < 1e-12


@pytest.mark.parametrize("f32", [False, True], ids=["fp64", "fp32"])
@pytest.mark.parametrize("n", [32, 256])
def test_legs_with_face_values_under_a_budget(mg, n, f32):
    """Face values reach a leg through a copy of the source, which a context with a memory budget
    does not take: both ways give the same leg (bounds as above, each side's error counted)."""
    kinds = KINDS["mixed"]
    rng = np.random.default_rng(n)
    dt, h = (torch.float32 if f32 else torch.float64), 1.0 / n
    u, f = dev(rng.standard_normal((n,) * 3), dt), dev(rng.standard_normal((n,) * 3) * n * n, dt)
    bext = [dev(rng.standard_normal((n + 2,) * 2)) if k == FIXED else None for k in kinds]
    size = (4 if f32 else 8) * n ** 3
    out = []
    for ctx in (mg.Context(0), mg.Context(0, hbm_budget=(64 << 20) + size + size // 2)):
        print(f"valued legs n={n} f32={f32}", flush=True)
        a, fc, uc = u.clone(), torch.empty((n // 2,) * 3, dtype=dt, device="cuda:0"), torch.empty((n // 2,) * 3, dtype=dt, device="cuda:0")
        (mg.mg_op_down_f32 if f32 else mg.mg_op_down)(a, f, fc, uc, h, OMEGA, 2, kinds, bext, ctx=ctx)
        out.append((host(a), host(fc)))
    eps = 40 * float(np.finfo(np.float32).eps) if f32 else 1e-13
    su = max(float(u.abs().max()), h * h * float(f.abs().max())) + 2 * max(float(b.abs().max()) for b in bext if b is not None)
    assert np.abs(out[0][0] - out[1][0]).max() <= 2 * eps * 6 * su
    assert np.abs(out[0][1] - out[1][1]).max() <= 2 * eps * (float(f.abs().max()) + 12 * su / h ** 2)


@pytest.mark.parametrize("f32", [False, True], ids=["fp64", "fp32"])
@pytest.mark.parametrize("n,kind", [(128, "periodic"), (256, "layer"), (256, "fixed"), (256, "mixed")])
def test_streaming_legs_of_one_sweep(mg, n, kind, f32):
    """The streaming passes with one sweep per leg (bounds as for the tile legs)."""
    kinds = KINDS[kind]
    hom = [k if k in (PERIODIC, ZERO_GRADIENT) else FIXED for k in kinds]
    print(f"streaming legs n={n} {kind} f32={f32}", flush=True)
    rng = np.random.default_rng(n)
    u, e = rng.standard_normal((n,) * 3), rng.standard_normal((n // 2,) * 3)
    f = rng.standard_normal((n,) * 3) * n * n
    bext = [rng.standard_normal((n + 2,) * 2) if k == FIXED else None for k in kinds]
    dt, h = (torch.float32 if f32 else torch.float64), 1.0 / n
    if f32:
        u, e, f = (a.astype(np.float32).astype(np.float64) for a in (u, e, f))
    dbext = [None if b is None else dev(b) for b in bext]
    ctx = mg.Context(0)
    ctx.set_tuning("fusedmin fp32 128\n")
    su = max(np.abs(u).max(), np.abs(e).max(), h * h * np.abs(f).max()) + 2 * max([0.0] + [np.abs(b).max() for b in bext if b is not None])
    eps = 40 * float(np.finfo(np.float32).eps) if f32 else 1e-13
    down, up = (mg.mg_op_down_f32, mg.mg_op_up_f32) if f32 else (mg.mg_op_down, mg.mg_op_up)

    ref = sweeps(u, f, h, kinds, bext, 1)
    ref_fc = oracle.restrict(oracle.defect(ref, f, h, kinds, bext))
    du, fc, uc = dev(u, dt), dev(e, dt), dev(e, dt)
    down(du, dev(f, dt), fc, uc, h, OMEGA, 1, kinds, dbext, ctx=ctx)
    assert np.abs(host(du) - ref).max() <= eps * 6 * su
    assert np.abs(host(fc) - ref_fc).max() <= eps * (np.abs(f).max() + 12 * su / h ** 2)
    assert float(uc.abs().max()) == 0.0

    ref = sweeps(oracle.prolong_add(e, u, hom), f, h, kinds, bext, 1)
    du = dev(u, dt)
    up(du, dev(f, dt), dev(e, dt), h, OMEGA, 1, kinds, dbext, hom, ctx=ctx)
    assert np.abs(host(du) - ref).max() <= eps * 12 * su


@pytest.mark.parametrize("kind", ["periodic", "mixed"])
def test_one_sweep_cycles_agree_across_layouts_and_schemes(mg, kind):
    """V(1,1) cycles on 256^3: the block layout gives the dense potential and history, and so does
    the Full Approximation Scheme, as every whole-solve check: phi to 1e-10."""
    n, kinds = 256, KINDS[kind]
    rho = dev(wl.gaussian_clumps(n, 5, n_clumps=6))
    a, ha, _ = mg.solve(rho, 1.0 / n, kinds, fixed_cycles=3, npre=1, npost=1)
    b, hb, _ = mg.solve(mg.to_blocks(rho, 16), 1.0 / n, kinds, fixed_cycles=3, npre=1, npost=1, layout="blocks")
    c, hc, _ = mg.solve(rho, 1.0 / n, kinds, fixed_cycles=3, npre=1, npost=1, scheme="fas")
    a = host(a)
    assert rel(host(mg.from_blocks(b, n, 16)), a) < 1e-10 and rel(host(c), a) < 1e-10
    for h in (hb, hc):
        assert len(h) == len(ha) and all(abs(x - y) <= 1e-6 * y for x, y in zip(h, ha))


@pytest.mark.parametrize("n,lb,lmax", [(8, 0, 4), (16, 0, 4), (32, 0, 3), (128, 0, 4), (256, 0, 4), (64, 3, 4), (64, 4, 2)])
def test_moments_by_columns(mg, n, lb, lmax):
    """Moments summed column by column (8, 16 and 32 cells, a whole side or a part) against the
    oracle's, and the potential of a solve in blocks against the dense one.  A moment is a sum of
    n^3 terms no larger than the mass's (the box has side 1): 1e-12 of the mass."""
    rng = np.random.default_rng(n + lb)
    rho = rng.random((n,) * 3)
    kw = dict(lmax=lmax, fixed_cycles=3)
    if lb:
        a, _, _ = mg.solve(dev(rho), 1.0 / n, "multipole", **kw)
        b, _, _ = mg.solve(mg.to_blocks(dev(rho), 1 << lb), 1.0 / n, "multipole", layout="blocks", block_n=1 << lb, **kw)
        assert rel(host(mg.from_blocks(b, n, 1 << lb)), host(a)) < 1e-12
        return
    o_ref, q_ref = oracle.multipole_moments(rho, 1.0 / n, lmax=lmax)
    o, q = mg.mg_multipole_moments(dev(rho), 1.0 / n, lmax=lmax)
    nq = (lmax + 1) ** 2
    assert np.abs(np.asarray(o) - np.asarray(o_ref)).max() < 1e-12
    assert np.abs(np.asarray(q)[:nq] - np.asarray(q_ref)[:nq]).max() < 1e-12 * abs(q_ref[0])
