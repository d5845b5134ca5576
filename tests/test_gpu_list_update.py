"""The buffered list kept across configurations (amoeba_update_blocklist): no rebuild while
every atom stays within buffer/2 of its position at the last build, a rebuild as soon as one
leaves it, and fields and solves against the oracle at every configuration in between."""
import dataclasses

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


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_update_keeps_the_list_until_an_atom_leaves_half_the_buffer(prec):
    s0 = dataclasses.replace(synth.water648(), buffer=1.0)
    rng = np.random.default_rng(5)
    print(f"[gpu] list update {prec}", flush=True)
    ctx, t = amoeba.context_for(s0, precision=prec, device=DEV)   # builds at s0
    assert not ctx.update_blocklist(t["pos"])                      # same positions
    tol = {"fp64": 1e-11, "mixed": 2e-5}[prec]
    walk = np.zeros_like(s0.pos)
    for k in range(4):
        walk += rng.normal(0.0, 0.02, s0.pos.shape)
        s = dataclasses.replace(s0, pos=np.mod(s0.pos + walk, s0.box))
        pos = torch.tensor(s.pos, device=DEV)
        assert not ctx.update_blocklist(pos), k                   # max move << 0.5 A
        assert ctx.info()["n_pairs"] == O.count_pairs(s)
        e_ref = O.perm_field(s, "spme")
        e = ctx.perm_field(pos, t["q"], t["dip"], t["quad"])
        assert_fields(e.cpu().numpy(), e_ref, tol, what=f"E_perm frame {k}")
    mu_ref, _, _ = O.pcg(s, e_ref, "spme", tol_debye=1e-10)
    mu, _, _, st = ctx.polarize(pos, e, tol_debye=1e-6)
    assert st == amoeba.AMOEBA_OK and O.rms_debye(mu.cpu().numpy() - mu_ref) < 2e-6
    # one atom 0.6 A from where it was at the build: the list is rebuilt
    far = s.pos.copy()
    far[17] = np.mod(s0.pos[17] + np.array([0.6, 0.0, 0.0]), s0.box)
    s2 = dataclasses.replace(s0, pos=far)
    pos2 = torch.tensor(far, device=DEV)
    with pytest.raises(amoeba.AmoebaError) as ei:                   # the plain calls refuse it
        ctx.perm_field(pos2, t["q"], t["dip"], t["quad"])
    assert ei.value.status == amoeba.AMOEBA_E_LIST
    assert ctx.update_blocklist(pos2)
    assert not ctx.update_blocklist(pos2)
    assert ctx.info()["n_pairs"] == O.count_pairs(s2)
    e2 = ctx.perm_field(pos2, t["q"], t["dip"], t["quad"])
    assert_fields(e2.cpu().numpy(), O.perm_field(s2, "spme"), tol, what="E_perm after the rebuild")
    ctx.close()


def test_update_builds_a_missing_list_and_rejects_bad_positions():
    s = synth.water648()
    ctx = amoeba.Context(s.n, s.box, cutoff=s.cutoff, ewald_alpha=s.ewald_alpha, grid=s.grid, precision="mixed")
    t = torch.tensor(s.pos, device=DEV)
    ctx.set_atoms(*(torch.tensor(a, device=DEV) for a in (s.alpha, s.thole)),
                  torch.tensor(s.sc_ptr, dtype=torch.int32, device=DEV),
                  torch.tensor(s.sc_j, dtype=torch.int32, device=DEV), torch.tensor(s.sc_s, device=DEV))
    assert ctx.update_blocklist(t)
    assert ctx.info()["n_pairs"] == O.count_pairs(s)
    bad = t.clone()
    bad[3, 2] = float("nan")
    with pytest.raises(amoeba.AmoebaError) as ei:
        ctx.update_blocklist(bad)
    assert ei.value.status == amoeba.AMOEBA_E_NUMERIC
    assert not ctx.update_blocklist(t)      # the list of the last build is still valid
    e = ctx.perm_field(t, *(torch.tensor(a, device=DEV) for a in (s.q, s.dip, s.quad)))
    assert_fields(e.cpu().numpy(), O.perm_field(s, "spme"), 2e-5)
    ctx.close()


@pytest.mark.parametrize("waters,cube,box,grid", [
    (1, 18.63, (18.63, 18.63, 18.63), (24, 24, 24)),
    (216, 18.63, (120.0, 120.0, 120.0), (48, 48, 48)),     # a droplet: most columns and cells empty
    (216, 18.63, (18.7, 18.7, 400.0), (20, 20, 320)),      # a slab: one column of the box holds many atoms
    (343, 21.8, (900.0, 21.9, 21.9), (720, 24, 24)),       # all atoms in few slices of x
    (8640, 63.7, (66.0, 64.0, 90.0), (64, 64, 96))],       # the grid of blocks, some of its cells empty
    ids=lambda v: str(v))
def test_order_of_uneven_systems(waters, cube, box, grid):
    """Buckets and cells that hold many atoms or none: every pair once, the product at the bars of
    its other comparison with the oracle, and the same bits from a second build, also after one that
    was refused for its positions (all of them, one of them not finite)."""
    s = synth.water_box(waters, cube, grid[0], 7, "water")
    s = dataclasses.replace(s, box=np.array(box), grid=grid, buffer=0.5)
    mu = 0.05 * np.random.default_rng(3).standard_normal((s.n, 3))
    ref = O.matvec(s, mu, "spme")
    for prec in ("fp64", "mixed"):
        print(f"[gpu] uneven system N={s.n} box={box} {prec}", flush=True)
        ctx, t = amoeba.context_for(s, precision=prec, device=DEV)
        try:
            out = ctx.dipole_matvec(t["pos"], torch.tensor(mu, device=DEV)).cpu().numpy()
            assert ctx.info()["n_pairs"] == O.count_pairs(s)
            for bad in (slice(None), slice(0, 1)):
                p = t["pos"].clone()
                p[bad] = float("nan")
                with pytest.raises(amoeba.AmoebaError) as ei:
                    ctx.build_blocklist(p)
                assert ei.value.status == amoeba.AMOEBA_E_NUMERIC
            ctx.build_blocklist(t["pos"])
            again = ctx.dipole_matvec(t["pos"], torch.tensor(mu, device=DEV)).cpu().numpy()
        finally:
            ctx.close()
        assert_fields(out, ref, 1e-12 if prec == "fp64" else 2e-6)
        if prec == "mixed":
            assert np.array_equal(out, again)   # fixed-point sums; FP64 sums follow the list's order
        else:
            assert_fields(again, ref, 1e-12)


def test_order_of_one_full_slice():
    """65,856 atoms in one slice of one column (a box 2e6 A long): their index orders them, and the list,
    here of blocks along the rows of a lattice, holds every pair and is the same from every build."""
    from scipy.spatial import cKDTree
    s = synth.water_box(28 ** 3, 28 * 3.1, 32, 5, "water")
    s = dataclasses.replace(s, box=np.array([2.0e6, 100.0, 100.0]), grid=(64, 32, 32), cutoff=4.0)
    mu = 0.05 * torch.tensor(np.random.default_rng(3).standard_normal((s.n, 3)), device=DEV)
    pairs = (cKDTree(s.pos).count_neighbors(cKDTree(s.pos), s.cutoff) - s.n) // 2
    out = []
    for _ in range(3):
        ctx, t = amoeba.context_for(s, precision="mixed", device=DEV)
        try:
            assert ctx.info()["n_pairs"] == pairs
            out.append(ctx.dipole_field_parts(t["pos"], mu)[0].cpu().numpy())
        finally:
            ctx.close()
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_masks_refreshed_ahead_of_the_flags(prec):
    """Calls on the same, on changed and on refused positions in every order, and after new atom
    parameters on the same positions: each gives what a context that saw only those positions gives."""
    s = dataclasses.replace(synth.water648(), buffer=1.0)
    rng = np.random.default_rng(12)
    at = [torch.tensor(np.mod(s.pos + d, s.box), device=DEV)
          for d in (0.0, 0.03 * rng.standard_normal(s.pos.shape))]
    stale, nan = at[0].clone(), at[0].clone()
    stale[5, 0] = (stale[5, 0] + 3.0) % float(s.box[0])
    nan[7, 2] = float("nan")
    mu = torch.tensor(0.05 * rng.standard_normal(s.pos.shape), device=DEV)
    want = []
    for scale in (1.0, 1.1):
        for p in at:
            ctx, t = amoeba.context_for(s, precision=prec, device=DEV)
            ctx.set_atoms(t["alpha"] * scale, t["thole"], t["sc_ptr"], t["sc_j"], t["sc_s"])
            want.append(ctx.dipole_matvec(p, mu).cpu().numpy())
            ctx.close()
    ctx, t = amoeba.context_for(s, precision=prec, device=DEV)
    try:
        for k, scale in ((0, 1.0), (0, 1.0), (1, 1.0), (stale, 4), (1, 1.0), (nan, 8), (stale, 4), (0, 1.0), (0, 1.1),
                         (1, 1.1), (1, 1.0), (nan, 8), (1, 1.1), (0, 1.0)):
            if not isinstance(k, int):
                with pytest.raises(amoeba.AmoebaError) as ei:
                    ctx.dipole_matvec(k, mu)
                assert ei.value.status == (amoeba.AMOEBA_E_LIST if scale == 4 else amoeba.AMOEBA_E_NUMERIC)
                continue
            ctx.set_atoms(t["alpha"] * scale, t["thole"], t["sc_ptr"], t["sc_j"], t["sc_s"])
            out = ctx.dipole_matvec(at[k], mu).cpu().numpy()
            ref = want[k + (2 if scale == 1.1 else 0)]
            if prec == "mixed":
                assert np.array_equal(out, ref)
            else:
                assert_fields(out, ref, 1e-12)
    finally:
        ctx.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_coordinates_of_any_magnitude(prec):
    """Coordinates far beyond what the wrapping resolves (a diverged trajectory) build a list and give
    a finite field, and the next ordinary positions the right one."""
    s = synth.water648()
    mu = 0.05 * np.random.default_rng(3).standard_normal((s.n, 3))
    ref = O.matvec(s, mu, "spme")
    m = torch.tensor(mu, device=DEV)
    ctx, t = amoeba.context_for(s, precision=prec, device=DEV)
    try:
        for size in (1e14, 1e16, 1e17, 1e18, 1e21, 1e40, 1e300):
            print(f"[gpu] coordinates of {size:g} {prec}", flush=True)
            rng = np.random.default_rng(int(np.log10(size)))
            far = s.pos.copy()
            for a in (5, 200, 647):
                far[a] = size * rng.uniform(-1.0, 1.0, 3)
            far[70, 1] = size
            pos = torch.tensor(far, device=DEV)
            ctx.update_blocklist(pos)
            assert torch.isfinite(ctx.dipole_matvec(pos, m)).all()
            ctx.build_blocklist(t["pos"])
            assert_fields(ctx.dipole_matvec(t["pos"], m).cpu().numpy(), ref, 1e-12 if prec == "fp64" else 2e-6)
    finally:
        ctx.close()


def test_first_flags_of_a_context_are_its_own():
    """A context of one checked call leaves its sequence number and flag word in host memory that the
    next context may be given: the first check there is made all the same."""
    s = synth.water648()
    t = [torch.tensor(a, device=DEV) for a in (s.alpha, s.thole)]
    csr = (torch.tensor(s.sc_ptr, dtype=torch.int32, device=DEV), torch.tensor(s.sc_j, dtype=torch.int32, device=DEV),
           torch.tensor(s.sc_s, device=DEV))
    for _ in range(4):
        ctx = amoeba.Context(s.n, s.box, grid=s.grid, precision="mixed")
        ctx.set_atoms(*t, *csr)
        ctx.close()
        ctx = amoeba.Context(s.n, s.box, grid=s.grid, precision="mixed")
        try:
            with pytest.raises(amoeba.AmoebaError) as ei:
                ctx.set_atoms(-t[0], t[1], *csr)
            assert ei.value.status == amoeba.AMOEBA_E_INVALID
        finally:
            ctx.close()


@pytest.mark.parametrize("spread,edge", [(60.0, 700.0), (300.0, 3000.0), (900.0, 2000.0), (900.0, 4000.0), (900.0, 9000.0)])
@pytest.mark.parametrize("along", [(1.0, 0.0, 0.0), (0.75, 0.45, 0.48)], ids=["axis", "oblique"])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_pairs_of_dilute_blocks(spread, edge, prec, along):
    """64 lone pairs near the cutoff, spread over hundreds of Angstrom, so that the offsets within a
    block dwarf the cutoff: the list and the masks hold exactly the pairs within it (no buffer)."""
    rng = np.random.default_rng(8)
    print(f"[gpu] dilute pairs spread={spread} edge={edge} {along} {prec}", flush=True)
    y, z = (a.ravel() for a in np.meshgrid(*2 * (np.linspace(-spread, spread, 8),), indexing="ij"))
    a = np.stack([rng.uniform(-0.3, 0.3, 64), y, z], 1) + rng.uniform(0.0, 0.3, 3)
    u = np.array(along) * np.where(rng.random((64, 3)) < 0.5, 1.0, [1.0, -1.0, -1.0])
    u /= np.linalg.norm(u, axis=1)[:, None]
    d = 7.0 + np.where(np.arange(64) % 2, -1.0, 1.0) * 10.0 ** rng.uniform(-9, -4, 64)
    pos = np.concatenate([a, a + d[:, None] * u]) + 0.37 * edge
    n = len(pos)
    ctx = amoeba.Context(n, (edge,) * 3, cutoff=7.0, grid=(32, 32, 32), precision=prec)
    try:
        one = torch.ones(n, dtype=torch.float64, device=DEV)
        ctx.set_atoms(one, 0.39 * one, torch.zeros(n + 1, dtype=torch.int32, device=DEV),
                      torch.zeros(0, dtype=torch.int32, device=DEV), torch.zeros(0, dtype=torch.float64, device=DEV))
        ctx.build_blocklist(torch.tensor(pos, device=DEV))
        assert ctx.info()["n_pairs"] == 32
    finally:
        ctx.close()


def test_checks_behind_a_long_queue():
    """Calls behind half a second of other work on their stream, far beyond the time the host watches for the
    flags: the same checks and results."""
    s = synth.water648()
    ctx, t = amoeba.context_for(s, precision="mixed", device=DEV)
    try:
        e = ctx.perm_field(t["pos"], t["q"], t["dip"], t["quad"])
        start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        for cycles in (10 ** 6, 10 ** 7):   # the first also loads the kernel
            start.record()
            torch.cuda._sleep(cycles)
            end.record()
            torch.cuda.synchronize()
        cycles = int(10 ** 7 * 500.0 / start.elapsed_time(end))
        torch.cuda._sleep(cycles)
        with pytest.raises(amoeba.AmoebaError) as ei:
            ctx.set_atoms(-t["alpha"], t["thole"], t["sc_ptr"], t["sc_j"], t["sc_s"])
        assert ei.value.status == amoeba.AMOEBA_E_INVALID
        torch.cuda._sleep(cycles)
        assert torch.equal(ctx.perm_field(t["pos"], t["q"], t["dip"], t["quad"]), e)
    finally:
        ctx.close()
