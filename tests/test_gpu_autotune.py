"""The autotuner times what solves of these sweeps run: with one or two sweeps per leg from 128^3 the
streaming passes, against what would replace them."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("npre,npost", [(1, 1), (2, 1), (2, 2)])
@pytest.mark.parametrize("layout", ["dense", "blocks"])
def test_streaming_legs_are_tuned_as_they_run(layout, npre, npost, precision):
    import paper_2302_13903_amd as mg
    print(f"autotune {layout} V({npre},{npost}) {precision}", flush=True)
    n, prec = 128, "fp32" if precision == "mixed" else "fp64"
    ctx = mg.Context(0)
    p = mg.params(n, 1.0 / n, precision=precision, layout=layout, block_n=16, npre=npre, npost=npost)
    ctx.check(ctx._lib.mg_autotune(ctx.handle, ctypes.byref(p), 5), "mg_autotune")
    lines = ctx.tuning().splitlines()
    if layout == "dense":
        # (a V(1,1) cycle takes 80 us with the streaming passes and 97 with blocked sweeps)
        assert f"tb {prec} 0" in lines, lines
    else:
        assert any(line.startswith(f"blkz {prec} ") for line in lines), lines
    gen = torch.Generator(device="cuda:0").manual_seed(3)
    rho = torch.randn((n,) * 3, generator=gen, dtype=torch.float64, device="cuda:0")
    x = mg.to_blocks(rho, 16) if layout == "blocks" else rho
    kw = dict(precision=precision, layout=layout, block_n=16, npre=npre, npost=npost, fixed_cycles=4)
    a, ha, _ = mg.solve(x, 1.0 / n, "fixed", ctx=ctx, **kw)
    b, hb, _ = mg.solve(x, 1.0 / n, "fixed", **kw)
    # another schedule, the same iteration: the iterates agree far below its residual (mixed: to the
    # FP32 correction's rounding of what the last cycle changed)
    assert float((a - b).norm() / b.norm()) < (1e-9 if precision == "mixed" else 1e-12)
    assert len(ha) == len(hb)
