"""The two-stream split of the FP64 streaming passes (interior tiles and wall tiles as two concurrent
launches), at 512^3: the levels whose interior tiles are the more take it.  Against the single launch, for every kind
of wall and one and two sweeps per leg, and its timing records."""
import math
import statistics

import numpy as np
import pytest

import workloads as wl
from oracle import FIXED, PERIODIC, ZERO_GRADIENT

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N = 512
KINDS = {
    "fixed": [FIXED] * 6,
    "x and z": [FIXED, ZERO_GRADIENT, PERIODIC, PERIODIC, ZERO_GRADIENT, FIXED],
    "y": [PERIODIC, PERIODIC, ZERO_GRADIENT, FIXED, PERIODIC, PERIODIC],
}


@pytest.fixture(scope="module")
def mg():
    import paper_2302_13903_amd as m
    return m


@pytest.fixture(scope="module")
def rho():
    return torch.from_numpy(np.ascontiguousarray(wl.gaussian_clumps(N, 31, remove_mean=False))).to("cuda:0")


@pytest.mark.parametrize("kind,ns,layout", [(kind, ns, "dense") for kind in KINDS for ns in (1, 2)] +
                         [("fixed", 2, "blocks"), ("x and z", 1, "blocks")])
def test_split_passes_match_one_launch_512(mg, rho, kind, ns, layout):
    """phi agrees to rounding and the norms to 1e-12 and the round-off floor of a defect."""
    kinds = KINDS[kind]
    print(f"split 512^3 {kind} V({ns},{ns}) {layout}", flush=True)
    x = mg.to_blocks(rho, 16) if layout == "blocks" else rho
    rng = np.random.default_rng(8)
    faces = [torch.from_numpy(rng.standard_normal((N, N)) * 0.1).to("cuda:0") if k == FIXED else None for k in kinds]
    out = []
    for split in (1, 0):
        ctx = mg.Context(0)
        ctx.set_tuning(f"split fp64 {split}\n")
        phi, hist, st = mg.solve(x, 1.0 / N, kinds, fixed_b=faces, fixed_cycles=3, npre=ns, npost=ns, layout=layout,
                                 block_n=16, ctx=ctx)
        assert st == mg.MG_OK
        out.append((phi, hist))
        ctx.close()
    (a, ha), (b, hb) = out
    assert float((a - b).norm()) < 1e-13 * float(b.norm())
    assert float((a - b).abs().max()) < 1e-13 * float(b.abs().max())
    rms_f = 4 * math.pi * float((rho * rho).mean().sqrt())
    floor = 12 * np.finfo(float).eps * float(b.abs().max()) * N * N / rms_f
    assert len(ha) == len(hb) == 4
    for p, q in zip(ha, hb):
        assert abs(p - q) <= 1e-12 * q + floor, (ha, hb, floor)


@pytest.mark.parametrize("ns", [1, 2])
def test_split_is_taken_512(mg, rho, ns):
    """The norms' partial sums are grouped by workgroup, so over many cycles some of the norms differ in
    their last bit between the split and the single launch; all equal would mean that nothing was split."""
    print(f"split taken 512^3 V({ns},{ns})", flush=True)
    hists = []
    for split in (1, 0):
        ctx = mg.Context(0)
        ctx.set_tuning(f"split fp64 {split}\n")
        hists.append(mg.solve(rho, 1.0 / N, "fixed", fixed_cycles=40, npre=ns, npost=ns, ctx=ctx)[1])
        ctx.close()
    assert len(hists[0]) == len(hists[1]) == 41
    assert hists[0] != hists[1]


def test_split_passes_are_timed_512(mg, rho):
    """Every record counts one (split) pass per cycle, and the passes fit into the cycles' own times."""
    print("split timing 512^3", flush=True)
    ctx = mg.Context(0)
    ctx.set_kernel_timing(True)
    for _ in range(2):
        phi, hist, st = mg.solve(rho, 1.0 / N, "fixed", fixed_cycles=3, ctx=ctx)
    cyc, recs = ctx.last_timing()[2], ctx.kernel_timing()
    print([(r["name"], r["launches"], round(r["total_ms"], 4)) for r in recs], flush=True)
    assert st == mg.MG_OK and len(recs) == 2 and len(cyc) == 3
    assert all(r["launches"] == 3 and r["total_ms"] > 0 for r in recs)
    assert sum(r["total_ms"] / 3 for r in recs) < 1.02 * statistics.median(cyc)
    ctx.set_kernel_timing(False)
    again, hist2, _ = mg.solve(rho, 1.0 / N, "fixed", fixed_cycles=3, ctx=ctx)
    assert torch.equal(again, phi) and hist2 == hist
