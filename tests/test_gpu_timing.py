"""mg_last_timing: set-up and FMG sweep (or, from an initial guess, the first residual) are reported
apart, with and without the sweep, and add up with the cycles to no more than the call's wall time."""
import time

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("mode", ["fmg", "mgi"])
@pytest.mark.parametrize("n,kw", [
    (16, {}),                                # the tail alone
    (64, {}),                                # region tiles
    (128, {}),                               # streaming passes
    (128, dict(npre=3, npost=3)),            # head pass
    (64, dict(precision="mixed")),
    (64, dict(layout="blocks", block_n=16)),
    (64, dict(scheme="fas")),
])
def test_setup_and_start_are_apart(n, kw, mode):
    import paper_2302_13903_amd as mg
    print(f"timing n={n} {kw} {mode}", flush=True)
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    rho = torch.randn((n,) * 3, generator=gen, dtype=torch.float64, device="cuda:0")
    if kw.get("layout") == "blocks":
        rho = mg.to_blocks(rho, kw["block_n"])
    phi = torch.zeros_like(rho) if mode == "mgi" else None
    ctx = mg.Context(0)
    for _ in range(2):
        torch.cuda.synchronize()
        t = time.perf_counter()
        mg.solve(rho, 1.0 / n, "fixed", mode=mode, phi=phi, fixed_cycles=3, ctx=ctx, **kw)
        torch.cuda.synchronize()
        wall = 1e3 * (time.perf_counter() - t)
    setup, start, cycles = ctx.last_timing()
    assert setup > 0 and start > 0 and len(cycles) == 3 and min(cycles) > 0, (setup, start, cycles)
    assert setup + start + sum(cycles) <= wall, (setup, start, cycles, wall)
