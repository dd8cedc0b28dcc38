"""Refined meshes over a 16^3 root grid, whose middle of a V-cycle is one workgroup in global memory
(its arrays do not fit in LDS, as those of smaller root grids do): V-cycles, and the full-multigrid start,
whose Octet levels run their own cycles there.  Histories and potentials as the oracle's, to the bounds of
every refined-mesh check."""
import math

import numpy as np
import pytest

from oracle import amr
from parity import rel

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BOXES = [((5, 5, 6), (9, 9, 9)), ((11, 11, 13), (16, 17, 17))]
KINDS = {"periodic": [amr.PERIODIC] * 6, "fixed": [amr.FIXED] * 6,
         "mixed": [amr.ZERO_GRADIENT, amr.FIXED, amr.PERIODIC, amr.PERIODIC, amr.FIXED, amr.ZERO_GRADIENT]}


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("mode", ["mgi", "fmg"])
@pytest.mark.parametrize("kname", list(KINDS))
@pytest.mark.parametrize("levels", [1, 2])
def test_amr_root_16_matches_oracle(levels, kname, mode):
    import paper_2302_13903_amd as mg
    print(f"amr root 16^3 levels={levels} {kname} {mode}", flush=True)
    NB, nb, boxes, kinds = 16, 2, BOXES[:levels], KINDS[kname]
    m = amr.AmrMesh(NB, nb, boxes)
    rho = []
    for l in range(m.Lam + 1):
        x, y, z = m.centres(l)
        Z, Y, X = np.meshgrid(z, y, x, indexing="ij")
        r2 = (X - 0.45) ** 2 + (Y - 0.47) ** 2 + (Z - 0.5) ** 2
        rho.append(np.exp(-r2 / (2 * 0.06 ** 2)) + 0.3 * np.sin(2 * math.pi * X))
    rng = np.random.default_rng(levels)
    faces = [rng.uniform(-0.5, 0.5, (NB * nb,) * 2) if k == amr.FIXED else None for k in kinds]
    bf = amr.FaceArrays([f if f is not None else np.zeros((NB * nb,) * 2) for f in faces]) \
        if any(f is not None for f in faces) else None
    ref, rh = amr.solve(m, rho, kinds, bf, cycles=3, mode=mode)
    phi, hist, st = mg.amr_solve(mg.amr_mesh(NB, nb, boxes), [dev(r) for r in rho], kinds,
                                 fixed_b=[None if f is None else dev(f) for f in faces], fixed_cycles=3, mode=mode)
    torch.cuda.synchronize()
    assert st == mg.MG_OK and len(hist) == len(rh) == 4
    for a, b in zip(hist, rh):
        assert abs(a - b) <= 1e-6 * b + 1e-12, (hist, rh)
    assert rel([p.cpu().numpy() for p in phi], ref) < 1e-10
