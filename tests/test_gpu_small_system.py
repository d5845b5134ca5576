"""Small systems take their dipole product in few launches (tiles and spread together, the column
transforms together, and below 2,048 slots the rest of a PCG iteration in one workgroup): parity of
the product and of the solve with the FP64 oracle on both sides of the limits of that route, at the
bars of the path's other comparisons with the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2011_01207_amd import amoeba, synth
from parity_util import assert_fields

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

DEV = "cuda:0"
# atoms and grid on both sides of the limits: 64-atom blocks, 2,048 slots, 2,304 column points
SYSTEMS = [(21, 18.63, (24, 24, 24)), (216, 18.63, (20, 28, 21)), (682, 27.34, (30, 30, 30)),
           (683, 27.34, (36, 64, 30)), (700, 27.4, (48, 48, 28)), (700, 27.4, (48, 49, 28))]


def system(waters, box, grid):
    s = synth.water_box(waters, box, grid[0], 3, "water")
    s.grid = grid
    return s


@pytest.mark.parametrize("waters,box,grid", SYSTEMS, ids=lambda v: str(v))
def test_small_product_and_solve_match_the_oracle(waters, box, grid):
    s = system(waters, box, grid)
    mu = 0.05 * np.random.default_rng(5).standard_normal((s.n, 3))
    ref = O.matvec(s, mu, "spme")
    e_ref = O.perm_field(s, "spme")
    mu_ref, _, _ = O.pcg(s, e_ref, "spme", tol_debye=1e-10)
    for prec in ("fp64", "mixed"):
        print(f"[gpu] small system N={s.n} grid={grid} {prec}", flush=True)
        ctx, t = amoeba.context_for(s, precision=prec, device=DEV)
        try:
            out = ctx.dipole_matvec(t["pos"], torch.tensor(mu, device=DEV))
            m, _, _, st = ctx.polarize(t["pos"], torch.tensor(e_ref, device=DEV), tol_debye=1e-7, max_iter=200)
        finally:
            ctx.close()
        assert st == amoeba.AMOEBA_OK
        assert_fields(out.cpu().numpy(), ref, 1e-12 if prec == "fp64" else 2e-6)
        err = O.rms_debye(m.cpu().numpy() - mu_ref)
        assert err < (2e-7 if prec == "fp64" else 1e-5), (prec, err)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_small_solve_without_a_product_and_at_its_limits(prec):
    """A start that is already converged, an iteration limit, and the error of a bad input."""
    s = system(216, 18.63, (24, 24, 24))
    ctx, t = amoeba.context_for(s, precision=prec, device=DEV)
    try:
        z = torch.zeros_like(t["pos"])
        mu, _, it, st = ctx.polarize(t["pos"], z)
        assert (it, st) == (0, amoeba.AMOEBA_OK) and float(mu.abs().max()) == 0.0
        e = ctx.perm_field(t["pos"], t["q"], t["dip"], t["quad"])
        mu, _, it, st = ctx.polarize(t["pos"], e, tol_debye=1e-9, max_iter=3)
        assert (it, st) == (3, amoeba.AMOEBA_NOT_CONVERGED)
        bad = e.clone()
        bad[7, 1] = float("nan")
        with pytest.raises(amoeba.AmoebaError) as ei:
            ctx.polarize(t["pos"], bad)
        assert ei.value.status == amoeba.AMOEBA_E_NUMERIC
        mu, _, _, st = ctx.polarize(t["pos"], e, tol_debye=1e-6)
        assert st == amoeba.AMOEBA_OK
    finally:
        ctx.close()
    ref, _, _ = O.pcg(s, e.cpu().numpy(), "spme", tol_debye=1e-9)
    assert O.rms_debye(mu.cpu().numpy() - ref) < 1e-6 * (1 if prec == "fp64" else 3)
