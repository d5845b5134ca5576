"""GPU parity of the plane path's transforms over the lengths its stages split differently: two
stages of the largest radices, three and four stages, odd lengths, and z lengths whose lines hold
more butterflies than a row workgroup has threads."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2011_01207_amd import amoeba, synth
from parity_util import assert_fields  # noqa: E402

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

DEV = "cuda:0"
GRIDS = [(36, 16, 18), (16, 10, 200), (125, 14, 27), (10, 250, 63), (200, 10, 36), (10, 12, 875), (24, 216, 16)]


@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: "x".join(map(str, g)))
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_reciprocal_field_of_transform_lengths(grid, prec):
    print(f"[gpu] transform lengths grid={grid} {prec}", flush=True)
    s = synth.water_box(216, 18.63, 24, 3, "water_648")
    s.grid = grid
    mu = np.random.default_rng(4).standard_normal((s.n, 3)) * 0.05
    ctx, t = amoeba.context_for(s, precision=prec, device=DEV)
    try:
        ctx.set_pme_path("planes")
        _, ek = ctx.dipole_field_parts(t["pos"], torch.tensor(mu, device=DEV))
    finally:
        ctx.close()
    # the tolerances of the path's other comparisons with the oracle: a transform's rounding grows
    # with the logarithm of its length only
    tol = 1e-11 if prec == "fp64" else 2e-5
    assert_fields(ek.cpu().numpy(), O.spme_field(s, dip=mu), tol)
