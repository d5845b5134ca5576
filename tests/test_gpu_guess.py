"""GPU parity of the learned initial guess against the FP64 oracle (features and bases, network
forward, loss gradient, Adam, feature statistics), its error paths, and what the trained network
gains: fewer PCG iterations than the zero guess on held-out configurations, with every starting
point converging to the same dipoles."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle as O
from oracle import guess as G
from paper_2011_01207_amd import amoeba, synth

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

DEV = "cuda:0"


def rel(a, b):
    a, b = np.asarray(a, dtype=np.float64), np.asarray(b, dtype=np.float64)
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def random_model(seed, scale=0.3):
    rng = np.random.default_rng(seed)
    m = synth.guess_init_model(seed=seed).astype(np.float64)
    m[G.NPARAM - 3 * 64 - 3:G.NPARAM] = rng.standard_normal(3 * 64 + 3) * scale   # non-zero last layer
    m[:G.NPARAM] += rng.standard_normal(G.NPARAM) * 0.05
    m[G.NPARAM:G.NPARAM + G.NFEAT] = rng.standard_normal(G.NFEAT) * 0.2
    m[G.NPARAM + G.NFEAT:] = rng.uniform(0.5, 2.0, G.NFEAT)
    return m.astype(np.float32)


def f32(x):
    return torch.tensor(np.ascontiguousarray(x, dtype=np.float32), device=DEV)


@pytest.fixture(scope="module")
def c1():
    s = synth.water648()
    e = O.perm_field(s, "spme")
    x, b = G.features(s, e)
    return s, e, x, b


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_features_and_bases_match_oracle(c1, prec):
    s, e, x_ref, b_ref = c1
    print(f"[gpu] guess features water_648 {prec}", flush=True)
    ctx, t = amoeba.context_for(s, precision=prec, device=DEV)
    feat, basis = ctx.guess_features(t["pos"], torch.tensor(e, device=DEV))
    x = feat.cpu().numpy().astype(np.float64)
    b = basis.cpu().numpy().astype(np.float64)
    tol = 3e-7 if prec == "fp64" else 3e-6
    for k in range(3):
        assert rel(b[:, k], b_ref[:, k]) < tol, (k, rel(b[:, k], b_ref[:, k]))
    ftol = 1e-6 if prec == "fp64" else 2e-5
    for f in range(G.NFEAT):
        scale = max(1.0, float(np.max(np.abs(x_ref[:, f]))))
        assert np.max(np.abs(x[:, f] - x_ref[:, f])) < ftol * scale, (f, np.max(np.abs(x[:, f] - x_ref[:, f])))
    ctx.close()


def test_forward_matches_oracle(c1):
    s, e, x_ref, b_ref = c1
    model = random_model(31)
    ctx, t = amoeba.context_for(s, precision="mixed", device=DEV)
    ctx.guess_set_model(model)
    x32, b32 = x_ref.astype(np.float32), b_ref.astype(np.float32)
    mu = ctx.guess_forward(f32(x32), f32(b32)).cpu().numpy()
    ref = G.forward(model.astype(np.float64), x32.astype(np.float64), b32.astype(np.float64))
    assert rel(mu, ref) < 2e-6
    assert np.array_equal(ctx.guess_get_model(), model)
    ctx.close()


@pytest.mark.parametrize("n,use_idx", [(1000, False), (333, True), (64, False), (1, False)])
def test_gradient_matches_oracle(n, use_idx):
    """Loss and gradient of a batch against FP64 backpropagation on the same FP32 inputs (the
    analytic gradient is pinned to central differences on the CPU); several chunks, a ragged
    last chunk, an index batch with repeats and a single sample."""
    rng = np.random.default_rng(40 + n)
    rows = 1200
    x = rng.standard_normal((rows, G.NFEAT)).astype(np.float32)
    b = (rng.standard_normal((rows, 3, 3)) * 0.1).astype(np.float32)
    y = (rng.standard_normal((rows, 3)) * 0.1).astype(np.float32)
    model = random_model(41)
    s = synth.water648()
    ctx, t = amoeba.context_for(s, precision="mixed", device=DEV)
    ctx.guess_set_model(model)
    if use_idx:
        idx = rng.integers(0, rows, n).astype(np.int32)
        loss, g = ctx.guess_gradient(f32(x), f32(b), f32(y), idx=torch.tensor(idx, device=DEV))
        sel = idx
    else:
        loss, g = ctx.guess_gradient(f32(x), f32(b), f32(y), n_batch=n)
        sel = np.arange(n)
    l_ref, g_ref = G.loss_grad(model.astype(np.float64), x[sel].astype(np.float64), b[sel].astype(np.float64),
                               y[sel].astype(np.float64))
    assert abs(loss - l_ref) < 1e-5 * l_ref
    g = g.cpu().numpy()
    assert rel(g, g_ref) < 1e-4, rel(g, g_ref)
    # reproducible bit for bit
    loss2, g2 = (ctx.guess_gradient(f32(x), f32(b), f32(y), idx=torch.tensor(idx, device=DEV)) if use_idx
                 else ctx.guess_gradient(f32(x), f32(b), f32(y), n_batch=n))
    assert loss2 == loss and np.array_equal(g2.cpu().numpy(), g)
    ctx.close()


def test_adam_steps_match_oracle():
    rng = np.random.default_rng(50)
    rows = 700
    x = rng.standard_normal((rows, G.NFEAT)).astype(np.float32)
    b = (rng.standard_normal((rows, 3, 3)) * 0.1).astype(np.float32)
    y = (rng.standard_normal((rows, 3)) * 0.1).astype(np.float32)
    model = random_model(51)
    s = synth.water648()
    ctx, t = amoeba.context_for(s, precision="mixed", device=DEV)
    ctx.guess_set_model(model)
    cur = model.astype(np.float64)
    m = np.zeros(G.NPARAM)
    v = np.zeros(G.NPARAM)
    for step in range(1, 4):
        _, g = ctx.guess_gradient(f32(x), f32(b), f32(y))
        ctx.guess_train_step(f32(x), f32(b), f32(y), lr=1e-3)
        cur, m, v = G.adam_step(cur, m, v, step, g.cpu().numpy().astype(np.float64), 1e-3)
        got = ctx.guess_get_model().astype(np.float64)
        assert np.max(np.abs(got - cur)) < 2e-6, (step, np.max(np.abs(got - cur)))
        cur = got
    ctx.close()


def test_fit_norm_matches_oracle(c1):
    s, e, x_ref, _ = c1
    ctx, t = amoeba.context_for(s, precision="mixed", device=DEV)
    ctx.guess_set_model(synth.guess_init_model())
    x32 = x_ref.astype(np.float32)
    ctx.guess_fit_norm(f32(x32))
    mean, inv = G.fit_norm(x32.astype(np.float64))
    got = ctx.guess_get_model()
    assert np.allclose(got[G.NPARAM:G.NPARAM + G.NFEAT], mean, rtol=1e-6, atol=1e-7)
    assert np.allclose(got[G.NPARAM + G.NFEAT:], inv, rtol=1e-5, atol=0)
    assert got[G.NPARAM + G.NFEAT + 1] == 0.0          # Thole a is constant in water
    ctx.close()


def test_guess_error_paths(c1):
    s, e, x_ref, b_ref = c1
    ctx, t = amoeba.context_for(s, precision="mixed", device=DEV)
    et = torch.tensor(e, device=DEV)
    with pytest.raises(amoeba.AmoebaError) as ei:
        ctx.polarize(t["pos"], et, guess_mode="learned")
    assert ei.value.status == amoeba.AMOEBA_E_STATE
    with pytest.raises(amoeba.AmoebaError) as ei:
        ctx.guess_set_model(np.zeros(10, np.float32))
    assert ei.value.status == amoeba.AMOEBA_E_INVALID
    bad = synth.guess_init_model()
    bad[5] = np.nan
    with pytest.raises(amoeba.AmoebaError) as ei:
        ctx.guess_set_model(bad)
    assert ei.value.status == amoeba.AMOEBA_E_NUMERIC
    model = random_model(60)
    ctx.guess_set_model(model)
    x, b = f32(x_ref), f32(b_ref)
    y = torch.zeros((s.n, 3), dtype=torch.float32, device=DEV)
    with pytest.raises(amoeba.AmoebaError) as ei:
        ctx.guess_train_step(x, b, y, 1e-3, idx=torch.tensor([0, 5, s.n], dtype=torch.int32, device=DEV))
    assert ei.value.status == amoeba.AMOEBA_E_INVALID
    assert np.array_equal(ctx.guess_get_model(), model)         # rejected step changed nothing
    with pytest.raises(amoeba.AmoebaError):
        ctx.guess_train_step(x, b, y, -1.0)
    ctx.close()


def make_trajectory_data(ctx, t, base, frames, tol=1e-8):
    out = []
    for p in frames:
        pos = torch.tensor(p, device=DEV)
        ctx.build_blocklist(pos)
        e = ctx.perm_field(pos, t["q"], t["dip"], t["quad"])
        mu, _, _, st = ctx.polarize(pos, e, tol_debye=tol)
        assert st == amoeba.AMOEBA_OK
        feat, basis = ctx.guess_features(pos, e)
        out.append({"pos": pos, "e": e, "mu": mu.clone(), "feat": feat, "basis": basis})
    return out


def train(ctx, data, steps=1500, batch=4096, lr=2e-3, seed=3):
    feat = torch.cat([d["feat"] for d in data])
    basis = torch.cat([d["basis"] for d in data])
    target = torch.cat([d["mu"] for d in data]).float()
    ctx.guess_set_model(synth.guess_init_model(seed=7))
    ctx.guess_fit_norm(feat)
    rng = np.random.default_rng(seed)
    losses = []
    for k in range(steps):
        idx = torch.tensor(rng.integers(0, feat.shape[0], batch).astype(np.int32), device=DEV)
        losses.append(ctx.guess_train_step(feat, basis, target, lr, idx=idx))
    return losses


def test_trained_guess_gains_over_zero_and_converges_to_same_dipoles():
    """Train on 18 configurations of a 0.02 A-step trajectory of the 648-atom box (targets: the
    solver's own converged dipoles), evaluate on the next 6: the learned guess needs fewer PCG
    iterations than the zero guess, its error is well below the untrained network's, and zero,
    previous-step, learned and judged starts all converge to the same dipoles."""
    base = synth.water648()
    frames = list(synth.trajectory(base, 24, 0.02, seed=104))
    print("[gpu] guess training water_648 trajectory", flush=True)
    # FP64 context: the targets are converged to 1e-8 D, below what FP32 pair math resolves
    ctx, t = amoeba.context_for(base, precision="fp64", device=DEV)
    data = make_trajectory_data(ctx, t, base, frames)
    tr, te = data[:18], data[18:]
    ctx.guess_set_model(synth.guess_init_model(seed=7))
    ctx.guess_fit_norm(torch.cat([d["feat"] for d in tr]))
    err0 = np.mean([O.rms_debye((ctx.guess_forward(d["feat"], d["basis"]).double() - d["mu"]).cpu().numpy())
                    for d in te])
    losses = train(ctx, tr)
    assert np.mean(losses[-50:]) < 0.5 * np.mean(losses[:50])
    err1 = np.mean([O.rms_debye((ctx.guess_forward(d["feat"], d["basis"]).double() - d["mu"]).cpu().numpy())
                    for d in te])
    assert err1 < 0.7 * err0, (err0, err1)
    its = {"zero": [], "given": [], "learned": [], "best": []}
    for k, d in enumerate(te):
        prev = data[18 + k - 1]["mu"]
        ref = d["mu"].cpu().numpy()
        ctx.build_blocklist(d["pos"])
        for mode in its:
            mu, _, it, st = ctx.polarize(d["pos"], d["e"], mu_guess=prev if mode in ("given", "best") else None,
                                         guess_mode=mode, tol_debye=1e-5)
            assert st == amoeba.AMOEBA_OK
            its[mode].append(it)
            # every start converges to the same dipoles: the stopping test holds for the true
            # residual, and the error, (alpha A)^-1 times it, stays within a few tolerances
            z = (t["alpha"][:, None] * (d["e"] - ctx.dipole_matvec(d["pos"], mu))).cpu().numpy()
            assert O.rms_debye(z) < 1e-5
            assert O.rms_debye(mu.cpu().numpy() - ref) < 3e-5
            if mode == "best":
                info = ctx.info()
                rf, rl = info["last_guess_rms_debye"]
                assert rf > 0 and rl > 0
                assert info["last_guess"] == (amoeba.AMOEBA_GUESS_LEARNED if rl < rf else amoeba.AMOEBA_GUESS_GIVEN)
    mean = {k: float(np.mean(v)) for k, v in its.items()}
    print("[gpu] mean iterations", mean, flush=True)
    assert mean["learned"] < mean["zero"]
    assert mean["best"] <= min(mean["learned"], mean["given"]) + 0.5
    ctx.close()


def test_predict_matches_features_and_forward(c1):
    s, e, x_ref, b_ref = c1
    model = random_model(70)
    ctx, t = amoeba.context_for(s, precision="fp64", device=DEV)
    ctx.guess_set_model(model)
    et = torch.tensor(e, device=DEV)
    mu0 = ctx.guess_predict(t["pos"], et).cpu().numpy()
    ref = G.forward(model.astype(np.float64), x_ref, b_ref)
    assert rel(mu0, ref) < 2e-5
    ctx.close()


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 8191, 16385])
def test_gradient_at_the_edges_of_its_tiles(n):
    """Batches around the 16-sample tiles, the 64 samples of a workgroup and the launch's workgroup
    limit (256 of them), drawn with repetition from more rows than the batch, against FP64
    backpropagation at the bars of the gradient's other comparison."""
    s = synth.water648()
    rng = np.random.default_rng(n)
    x = rng.standard_normal((5000, G.NFEAT)).astype(np.float32)
    b = (0.05 * rng.standard_normal((5000, G.NBASIS, 3))).astype(np.float32)
    y = (0.05 * rng.standard_normal((5000, 3))).astype(np.float32)
    idx = rng.integers(0, 5000, n).astype(np.int32)
    model = random_model(61)
    ctx, _ = amoeba.context_for(s, precision="mixed", device=DEV)
    try:
        ctx.guess_set_model(model)
        loss, g = ctx.guess_gradient(f32(x), f32(b), f32(y), idx=torch.tensor(idx, device=DEV))
        idx_bad = torch.tensor(idx, device=DEV)
        idx_bad[-1] = 5000
        with pytest.raises(amoeba.AmoebaError) as ei:
            ctx.guess_gradient(f32(x), f32(b), f32(y), idx=idx_bad)
        assert ei.value.status == amoeba.AMOEBA_E_INVALID
    finally:
        ctx.close()
    l_ref, g_ref = G.loss_grad(model.astype(np.float64), x[idx].astype(np.float64), b[idx].astype(np.float64),
                               y[idx].astype(np.float64))
    assert abs(loss - l_ref) < 1e-5 * l_ref
    assert rel(g.cpu().numpy(), g_ref) < 1e-4


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("waters,box", [(1, 18.63), (21, 18.63), (22, 18.63), (216, 18.63), (8640, 63.7)])
def test_radial_sums_on_both_sides_of_the_wave_limit(waters, box, prec):
    """The neighbour sums of one to four blocks (eight waves a block, with and without neighbours in
    other blocks) and of 405 blocks (four waves), against the FP64 sums of sampled atoms, at the bars
    of the features' other comparison."""
    s = synth.water_box(waters, box, 48, 3, "water")
    print(f"[gpu] radial sums N={s.n} {prec}", flush=True)
    ctx, t = amoeba.context_for(s, precision=prec, device=DEV)
    try:
        feat, _ = ctx.guess_features(t["pos"], torch.zeros_like(t["pos"]))
    finally:
        ctx.close()
    idx = np.unique(np.linspace(0, s.n - 1, 200).astype(np.int64))
    ref = G.radial_sums(s, idx)
    x = feat.cpu().numpy().astype(np.float64)[idx][:, 8:11]
    assert np.max(np.abs(x - ref)) < (1e-6 if prec == "fp64" else 2e-5) * max(1.0, float(np.max(ref)))


@pytest.mark.parametrize("path", ["planes", "bricks"])
def test_prediction_then_products_on_the_same_positions(path):
    """A prediction takes no reciprocal field; the calls after it on the same positions do, with the
    atoms where they are then: the bits of a context that never predicted."""
    s = synth.water648()
    pos2 = torch.tensor(np.mod(s.pos + 0.02 * np.random.default_rng(8).standard_normal(s.pos.shape), s.box), device=DEV)
    out = []
    for predict in (False, True):
        ctx, t = amoeba.context_for(dataclasses.replace(s, buffer=1.0), precision="mixed", device=DEV)
        try:
            ctx.set_pme_path(path)
            ctx.guess_set_model(random_model(71))
            ctx.perm_field(t["pos"], t["q"], t["dip"], t["quad"])
            if predict:
                ctx.guess_predict(pos2, torch.zeros_like(pos2))
            e = ctx.perm_field(pos2, t["q"], t["dip"], t["quad"])
            if predict:
                ctx.guess_predict(t["pos"], e)
            out.append((e.cpu().numpy(), ctx.dipole_matvec(t["pos"], 0.1 * e).cpu().numpy()))
        finally:
            ctx.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("waters,box", [(216, 18.63), (8640, 63.7)])
def test_radial_sums_repeat_bitwise(waters, box):
    """FP64 contexts: the same features from every call, and from a list of its own (eight and four waves
    to a block)."""
    s = synth.water_box(waters, box, 48, 3, "water")
    first = None
    for _ in range(2):
        ctx, t = amoeba.context_for(s, precision="fp64", device=DEV)
        try:
            for _ in range(10):
                feat, _ = ctx.guess_features(t["pos"], torch.zeros_like(t["pos"]))
                x = feat.cpu().numpy()[:, 8:11]
                first = x if first is None else first
                assert np.array_equal(x, first)
        finally:
            ctx.close()
