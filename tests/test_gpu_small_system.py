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


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_calls_out_of_workspace_leave_the_context_whole(prec):
    """Caps that end between any two of a call's buffers: each call either gives the uncapped context's
    result or refuses, a second time too, with no part of a set of buffers left to be taken for a whole one."""
    s = synth.water648()
    print(f"[gpu] workspace caps {prec}", flush=True)
    mu = torch.tensor(0.05 * np.random.default_rng(3).standard_normal((s.n, 3)), device=DEV)

    def calls(ctx):
        t = {k: torch.tensor(getattr(s, k), device=DEV) for k in ("pos", "q", "dip", "quad", "alpha", "thole", "sc_s")}
        csr = [torch.tensor(a, dtype=torch.int32, device=DEV) for a in (s.sc_ptr, s.sc_j)]
        return [lambda: ctx.set_atoms(t["alpha"], t["thole"], *csr, t["sc_s"]),
                lambda: ctx.build_blocklist(t["pos"]),
                lambda: ctx.perm_field(t["pos"], t["q"], t["dip"], t["quad"]),
                lambda: ctx.polarization_gradient(t["pos"], t["q"], t["dip"], t["quad"], mu),
                lambda: ctx.guess_set_model(synth.guess_init_model()),
                lambda: ctx.guess_predict(t["pos"], mu)]

    def make(cap=0):
        return amoeba.Context(s.n, s.box, cutoff=s.cutoff, ewald_alpha=s.ewald_alpha, grid=s.grid, precision=prec,
                              max_workspace_bytes=cap)

    ctx = make()
    held, want = [ctx.info()["workspace_bytes"]], []
    for f in calls(ctx):
        r = f()
        want.append(r.cpu().numpy() if isinstance(r, torch.Tensor) else None)
        held.append(ctx.info()["workspace_bytes"])
    ctx.close()
    refused = 0
    caps = np.concatenate([np.linspace(a, b, 12, endpoint=False) for a, b in zip(held[:-1], held[1:]) if b > a])
    for cap in caps.astype(np.int64):
        ctx = make(int(cap))
        try:
            for f, ref in zip(calls(ctx), want):
                left = None   # what a refused call leaves allocated, the same after a second one
                for _ in range(2):
                    try:
                        r = f()
                    except amoeba.AmoebaError as e:
                        assert e.status in (amoeba.AMOEBA_E_NOMEM, amoeba.AMOEBA_E_LIST, amoeba.AMOEBA_E_STATE), e
                        now = ctx.info()["workspace_bytes"]
                        assert now <= cap and left in (None, now)
                        left = now
                        refused += e.status == amoeba.AMOEBA_E_NOMEM
                    else:
                        if ref is not None:
                            assert_fields(r.cpu().numpy(), ref, 1e-11 if prec == "fp64" else 2e-5)
        finally:
            ctx.close()
    assert refused > len(caps)


def test_refused_atoms_leave_the_old_ones():
    """A longer pair list that is refused changes nothing of the one in use."""
    s = synth.water648()
    ctx, t = amoeba.context_for(s, precision="mixed", device=DEV)
    try:
        e = ctx.perm_field(t["pos"], t["q"], t["dip"], t["quad"])
        ptr = t["sc_ptr"].clone()
        ptr[-1] += 2
        sj = torch.cat([t["sc_j"], torch.full((2,), s.n, dtype=torch.int32, device=DEV)])
        with pytest.raises(amoeba.AmoebaError) as ei:
            ctx.set_atoms(t["alpha"], t["thole"], ptr, sj, torch.cat([t["sc_s"], t["sc_s"][:2]]))
        assert ei.value.status == amoeba.AMOEBA_E_INVALID
        assert torch.equal(ctx.perm_field(t["pos"], t["q"], t["dip"], t["quad"]), e)
        moved = t["pos"] + 0.01
        ctx.build_blocklist(moved)
        ctx.build_blocklist(t["pos"])
        assert torch.equal(ctx.perm_field(t["pos"], t["q"], t["dip"], t["quad"]), e)
    finally:
        ctx.close()


@pytest.mark.parametrize("waters", [832, 853])
def test_fp64_tiles_on_both_sides_of_few_blocks(waters):
    """FP64 permanent field and gradient of 39 and 40 blocks (four and eight waves to a block)."""
    s = system(waters, 18.63 * (waters / 216) ** (1 / 3), (32, 32, 32))
    print(f"[gpu] FP64 tiles N={s.n}", flush=True)
    mu = 0.05 * np.random.default_rng(3).standard_normal((s.n, 3))
    ctx, t = amoeba.context_for(s, precision="fp64", device=DEV)
    try:
        e = ctx.perm_field(t["pos"], t["q"], t["dip"], t["quad"])
        g = ctx.polarization_gradient(t["pos"], t["q"], t["dip"], t["quad"], torch.tensor(mu, device=DEV))
    finally:
        ctx.close()
    assert_fields(e.cpu().numpy(), O.perm_field(s, "spme"), 1e-11)
    assert_fields(g.cpu().numpy(), O.polar_gradient(s, mu, "spme"), 1e-10)
