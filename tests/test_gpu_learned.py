"""Learned spectral preconditioner on the GPU against the FP64 oracle.

Float32 network kernels are held to float bounds: outputs to 1e-5, the
gradient to 1e-4 of its largest component, one Adam step to 1e-6. Recorded
spectra (double) to 1e-10 relative. A network with a zero output layer must
reproduce plain Fourier acceleration exactly, and corrupted weights must be
caught by the fallback.
"""
import numpy as np
import pytest

from oracle import landau, mlp
from paper_1208_1186_amd import gf, learn, synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ALPHA = 0.08


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gf.load()


def dev(a, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(a))
    if dtype is not None:
        t = t.to(dtype)
    return t.to("cuda:0")


def _rand_samples(dims, nsamp, seed):
    rng = np.random.default_rng(seed)
    tuples = mlp.folded_tuples(dims)
    psq = mlp.tuple_psq(dims, tuples)
    out = []
    for _ in range(nsamp):
        x = mlp.features(psq, 10.0 ** rng.uniform(-12, 0), float(rng.integers(0, 60)))
        a = rng.uniform(0.1, 2.0, len(tuples))
        b = a * rng.uniform(0.5, 1.5, len(tuples))
        c = b * b / a * rng.uniform(1.0, 2.0, len(tuples))
        out.append((x, a, b, c))
    return out


def _stack(samples):
    x = np.concatenate([s[0] for s in samples]).astype(np.float32)
    tgt = np.concatenate([np.stack([s[1], s[2], s[3]], 1) for s in samples]).astype(np.float32)
    off = np.cumsum([0] + [len(s[0]) for s in samples]).astype(np.int32)
    return x, tgt, off


def _params(seed, scale=0.05):
    rng = np.random.default_rng(seed)
    return (mlp.init_params(seed) + scale * rng.standard_normal(mlp.n_params())).astype(np.float32)


def test_forward_matches_oracle():
    dims = (6, 4, 4, 8)
    (x, _, _, _), = _rand_samples(dims, 1, 1)
    th = _params(2)
    n = len(x)
    out = torch.empty((n, 2), dtype=torch.float32, device="cuda:0")
    nb = gf.gf_mlp_workspace_bytes(n, 1)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda:0")
    th_d, x_d = dev(th), dev(x.astype(np.float32))  # held: a freed temporary's block is reused at once
    gf.gf_mlp_forward(th_d.data_ptr(), x_d.data_ptr(), n, out.data_ptr(), ws.data_ptr(), nb)
    _, _, want = mlp.forward(th.astype(np.float64), x.astype(np.float32).astype(np.float64))
    assert np.max(np.abs(out.cpu().numpy() - want)) < 1e-5


def test_loss_and_gradient_match_oracle():
    dims = (4, 6, 4, 4)
    samples = _rand_samples(dims, 5, 3)
    th = _params(4)
    x, tgt, off = _stack(samples)
    n = len(x)
    nb = gf.gf_mlp_workspace_bytes(n, len(samples))
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda:0")
    g = torch.empty(gf.gf_mlp_param_count(), dtype=torch.float32, device="cuda:0")
    th_d, x_d, t_d, o_d = dev(th), dev(x), dev(tgt), dev(off)
    loss = gf.gf_mlp_loss_grad(th_d.data_ptr(), x_d.data_ptr(), t_d.data_ptr(), o_d.data_ptr(), len(samples), n,
                               g.data_ptr(), ws.data_ptr(), nb)
    # the oracle sees exactly the float inputs the GPU saw
    samples64 = [(x[i:j].astype(np.float64), tgt[i:j, 0].astype(np.float64), tgt[i:j, 1].astype(np.float64),
                  tgt[i:j, 2].astype(np.float64)) for i, j in zip(off[:-1], off[1:])]
    th64 = th.astype(np.float64)
    assert loss == pytest.approx(mlp.loss(th64, samples64), rel=1e-5)
    want = mlp.loss_grad(th64, samples64)
    got = g.cpu().numpy().astype(np.float64)
    assert np.max(np.abs(got - want)) <= 1e-4 * np.max(np.abs(want))


@pytest.mark.parametrize("rows", [(1,), (15,), (17, 47), (64, 1), (20011, 20011)])
def test_row_groups_and_train_step(rows):
    """Where the passes' groups of 16 rows and their dealing to the blocks have edges (one row, part groups, more
    groups than the waves of the largest grid); the bounds of the tests above. The training step gives
    bitwise the gradient and the optimiser's step of the separate calls."""
    rng = np.random.default_rng(sum(rows))
    n, ns = sum(rows), len(rows)
    x = np.concatenate([rng.uniform(-0.5, 0.5, (n, 4)), rng.uniform(-1, 1, (n, 2))], 1).astype(np.float32)
    a = rng.uniform(0.1, 2.0, n)
    b = a * rng.uniform(0.5, 1.5, n)
    tgt = np.stack([a, b, b * b / a * rng.uniform(1.0, 2.0, n)], 1).astype(np.float32)
    off = np.cumsum((0,) + rows).astype(np.int32)
    th = _params(6)
    nb = gf.gf_mlp_workspace_bytes(n, ns)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda:0")
    g = torch.empty(gf.gf_mlp_param_count(), dtype=torch.float32, device="cuda:0")
    th_d, x_d, t_d, o_d = dev(th), dev(x), dev(tgt), dev(off)
    loss = gf.gf_mlp_loss_grad(th_d.data_ptr(), x_d.data_ptr(), t_d.data_ptr(), o_d.data_ptr(), ns, n, g.data_ptr(),
                               ws.data_ptr(), nb)
    samples64 = [(x[i:j].astype(np.float64),) + tuple(tgt[i:j, k].astype(np.float64) for k in range(3))
                 for i, j in zip(off[:-1], off[1:])]
    th64 = th.astype(np.float64)
    assert loss == pytest.approx(mlp.loss(th64, samples64), rel=1e-5)
    want = mlp.loss_grad(th64, samples64)
    assert np.max(np.abs(g.cpu().numpy() - want)) <= 1e-4 * np.max(np.abs(want))
    m0 = (0.1 * rng.standard_normal(th.size)).astype(np.float32)
    v0 = np.abs(0.1 * rng.standard_normal(th.size)).astype(np.float32)
    pa, ma, va, pb, mb, vb = dev(th), dev(m0), dev(v0), dev(th), dev(m0), dev(v0)
    gf.gf_mlp_adam(pa.data_ptr(), ma.data_ptr(), va.data_ptr(), g.data_ptr(), 3, 1e-3)
    g2 = torch.empty_like(g)
    gf.gf_mlp_train_step(pb.data_ptr(), mb.data_ptr(), vb.data_ptr(), 3, 1e-3, x_d.data_ptr(), t_d.data_ptr(),
                         o_d.data_ptr(), ns, n, g2.data_ptr(), ws.data_ptr(), nb)
    torch.cuda.synchronize()
    assert torch.equal(g, g2) and torch.equal(pa, pb) and torch.equal(ma, mb) and torch.equal(va, vb)


def test_every_row_of_a_long_batch_matches_oracle():
    """More groups of 16 rows than the waves of the forward pass's largest grid (4096), so that waves take a second
    group (the one whose features were fetched meanwhile), with a part group at the end: every output by itself,
    bound above. The backward pass's waves (2048) take up to three."""
    rows = (33001, 40007)
    n = sum(rows)
    rng = np.random.default_rng(21)
    x = np.concatenate([rng.uniform(-0.5, 0.5, (n, 4)), rng.uniform(-1, 1, (n, 2))], 1).astype(np.float32)
    a = rng.uniform(0.1, 2.0, n)
    b = a * rng.uniform(0.5, 1.5, n)
    tgt = np.stack([a, b, b * b / a * rng.uniform(1.0, 2.0, n)], 1).astype(np.float32)
    off = np.cumsum((0,) + rows).astype(np.int32)
    th = _params(13)
    nb = gf.gf_mlp_workspace_bytes(n, 2)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda:0")
    out = torch.full((n, 2), float("nan"), dtype=torch.float32, device="cuda:0")
    g = torch.empty(gf.gf_mlp_param_count(), dtype=torch.float32, device="cuda:0")
    th_d, x_d, t_d, o_d = dev(th), dev(x), dev(tgt), dev(off)
    gf.gf_mlp_forward(th_d.data_ptr(), x_d.data_ptr(), n, out.data_ptr(), ws.data_ptr(), nb)
    th64, x64 = th.astype(np.float64), x.astype(np.float64)
    assert np.max(np.abs(out.cpu().numpy() - mlp.forward(th64, x64)[2])) < 1e-5
    gf.gf_mlp_loss_grad(th_d.data_ptr(), x_d.data_ptr(), t_d.data_ptr(), o_d.data_ptr(), 2, n, g.data_ptr(),
                        ws.data_ptr(), nb)
    want = mlp.loss_grad(th64, [(x64[i:j],) + tuple(tgt[i:j, k].astype(np.float64) for k in range(3))
                                for i, j in zip(off[:-1], off[1:])])
    assert np.max(np.abs(g.cpu().numpy() - want)) <= 1e-4 * np.max(np.abs(want))


def test_partial_gradients_stay_short():
    """A float partial gradient is a sum of at most 512 rows in an accumulator and 4 of those, however large the batch;
    the rest is double. With 2^24 equal rows every term of a parameter's gradient has the same size and sign, so
    against 2^9 such rows (16 in an accumulator) the gradient may differ by (516 + 16 + 1) 2^-24 relative, the 1 for
    the row's output gradient, which scales by a power of two."""
    ns, th = 64, _params(12)
    th[64 * 6 + 64 + 64 * 64 + 64 + 64:][:64] = 0.0  # W3[1]: the first rows' second output gradient stays out of the sums
    x0 = np.array([0.3, -0.2, 0.4, 0.1, 0.6, 0.25], np.float32)
    t0 = np.array([0.7, 0.9, 1.6], np.float32)
    out = []
    for n in (1 << 9, 1 << 24):
        x_d = torch.from_numpy(x0).cuda().repeat(n, 1)
        t_d = torch.from_numpy(t0).cuda().repeat(n, 1)
        o_d = torch.arange(ns + 1, dtype=torch.int32, device="cuda:0") * (n // ns)
        nb = gf.gf_mlp_workspace_bytes(n, ns)
        ws = torch.empty(nb, dtype=torch.uint8, device="cuda:0")
        g = torch.empty(gf.gf_mlp_param_count(), dtype=torch.float32, device="cuda:0")
        th_d = dev(th)
        gf.gf_mlp_loss_grad(th_d.data_ptr(), x_d.data_ptr(), t_d.data_ptr(), o_d.data_ptr(), ns, n, g.data_ptr(),
                            ws.data_ptr(), nb)
        out.append(g.cpu().numpy().astype(np.float64))
    assert np.all(np.isfinite(out[0])) and np.max(np.abs(out[0])) > 0.0
    err = np.abs(out[1] - out[0])
    print("largest relative difference", np.max(err / np.maximum(np.abs(out[0]), 1e-30)))
    assert np.all(err <= 533 * 2.0 ** -24 * np.abs(out[0]))


@pytest.mark.parametrize("rows", [1, 16, 17, 79])
def test_saturated_units_keep_the_gradient_finite(rows):
    """Infinite weights of layer 1 saturate their units (tanh = +-1, slope 0): outputs and gradient stay finite, also
    where the last group of 16 rows is part empty; the bounds of the tests above."""
    rng = np.random.default_rng(rows)
    x = np.concatenate([rng.uniform(0.1, 0.5, (rows, 4)), rng.uniform(-1, 1, (rows, 2))], 1).astype(np.float32)
    a = rng.uniform(0.1, 2.0, rows)
    b = a * rng.uniform(0.5, 1.5, rows)
    tgt = np.stack([a, b, b * b / a * 1.5], 1).astype(np.float32)
    th = _params(11)
    th[3 * 6 + 2], th[40 * 6] = np.inf, -np.inf  # W1[3, 2], W1[40, 0]
    th[64 * 6 + 21] = np.inf                     # b1[21]
    nb = gf.gf_mlp_workspace_bytes(rows, 1)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda:0")
    g = torch.empty(gf.gf_mlp_param_count(), dtype=torch.float32, device="cuda:0")
    o = torch.empty((rows, 2), dtype=torch.float32, device="cuda:0")
    th_d, x_d, t_d, o_d = dev(th), dev(x), dev(tgt), dev(np.array([0, rows], np.int32))
    gf.gf_mlp_forward(th_d.data_ptr(), x_d.data_ptr(), rows, o.data_ptr(), ws.data_ptr(), nb)
    gf.gf_mlp_loss_grad(th_d.data_ptr(), x_d.data_ptr(), t_d.data_ptr(), o_d.data_ptr(), 1, rows, g.data_ptr(),
                        ws.data_ptr(), nb)
    th64 = th.astype(np.float64)
    x64 = x.astype(np.float64)
    want = mlp.loss_grad(th64, [(x64,) + tuple(tgt[:, k].astype(np.float64) for k in range(3))])
    assert np.all(np.isfinite(want))
    assert np.max(np.abs(o.cpu().numpy() - mlp.forward(th64, x64)[2])) < 1e-5
    assert np.max(np.abs(g.cpu().numpy() - want)) <= 1e-4 * np.max(np.abs(want))


def test_adam_step_matches_oracle():
    rng = np.random.default_rng(5)
    n = gf.gf_mlp_param_count()
    th = rng.standard_normal(n).astype(np.float32)
    gr = rng.standard_normal(n).astype(np.float32)
    m = (0.1 * rng.standard_normal(n)).astype(np.float32)
    v = np.abs(0.1 * rng.standard_normal(n)).astype(np.float32)
    p_d, m_d, v_d, g_d = dev(th), dev(m), dev(v), dev(gr)
    gf.gf_mlp_adam(p_d.data_ptr(), m_d.data_ptr(), v_d.data_ptr(), g_d.data_ptr(), 7, 1e-3)
    torch.cuda.synchronize()
    want, wm, wv = mlp.adam_step(th.astype(np.float64), gr.astype(np.float64), m.astype(np.float64),
                                 v.astype(np.float64), 7, 1e-3)
    assert np.max(np.abs(p_d.cpu().numpy() - want)) < 1e-6
    assert np.max(np.abs(m_d.cpu().numpy() - wm)) < 1e-6


@pytest.mark.parametrize("dims", [(8, 4, 6, 4), (8, 8, 8, 8)])
def test_recorded_spectra_match_oracle(dims):
    sig = 0.7
    u = synth.make_config(dims, 11)
    links = dev(u)
    fx = gf.GaugeFixer(links, "fp64_18", flags=gf.FLAG_RECORD_SPECTRA)
    rec, theta = fx.record(3, sig)
    rec = rec.cpu().numpy()
    tuples = mlp.folded_tuples(dims)
    kern = landau.fa_kernel(dims) * sig
    cur = u
    specs, probes = [], []
    for k in range(4):
        specs.append(mlp.packed_spectrum(landau.divergence(cur)))
        if k < 3:
            assert theta[k] == pytest.approx(landau.theta(cur), rel=1e-12)
            up, *_ = landau.fa_step(cur, ALPHA, kernel=kern)
            probes.append(mlp.packed_spectrum(landau.divergence(up)))
            cur, *_ = landau.fa_step(cur, ALPHA)
    for k in range(3):
        p, c = mlp.record(specs[k], specs[k + 1], dims, tuples)
        e, _ = mlp.record(probes[k], probes[k], dims, tuples)
        scale = np.max(np.abs(p))
        assert np.max(np.abs(rec[k, :, 0] - p)) <= 1e-10 * scale
        assert np.max(np.abs(rec[k, :, 1] - c)) <= 1e-10 * scale
        assert np.max(np.abs(rec[k, :, 2] - e)) <= 1e-10 * scale
    # the probe steps were undone: the links were advanced by exactly the plain updates
    assert np.max(np.abs(links.cpu().numpy() - cur)) < 1e-12
    # training rows assembled on the GPU match the oracle's features and loss coefficients
    n, every = 2, 1
    X = torch.empty((n * len(tuples), 6), dtype=torch.float32, device="cuda:0")
    TG = torch.empty((n * len(tuples), 3), dtype=torch.float32, device="cuda:0")
    rec_d, th_d = dev(rec), dev(theta)
    gf.gf_mlp_make_samples(rec_d.data_ptr(), 3, th_d.data_ptr(), 0, every, n, 0, sig, dims, X.data_ptr(),
                           TG.data_ptr())
    X, TG = X.cpu().numpy(), TG.cpu().numpy()
    psq = mlp.tuple_psq(dims, tuples)
    for k in range(n):
        rows = slice(k * len(tuples), (k + 1) * len(tuples))
        assert np.max(np.abs(X[rows] - mlp.features(psq, theta[k], k))) < 1e-6
        want = mlp.targets(rec[k, :, 0], rec[k + 1, :, 0], rec[k, :, 2], sig)
        for j in range(3):
            assert np.max(np.abs(TG[rows, j] - want[j])) <= 1e-6 * np.max(np.abs(want[0])), (k, j)
    # a sample needs the record after it
    xb = torch.empty((2 * len(tuples), 6), dtype=torch.float32, device="cuda:0")
    tb = torch.empty((2 * len(tuples), 3), dtype=torch.float32, device="cuda:0")
    with pytest.raises(gf.GfError):
        gf.gf_mlp_make_samples(rec_d.data_ptr(), 3, th_d.data_ptr(), 1, 1, 2, 0, sig, dims, xb.data_ptr(),
                               tb.data_ptr())


@pytest.mark.parametrize("dims", [(8, 8, 8, 8), (12, 8, 6, 4), (32, 32, 32, 32)])
def test_multiplier_table_matches_oracle(dims):
    """The inference table (matrix-core layer 2) against the oracle's multipliers at the current theta, k."""
    u = synth.make_config(dims, 14)
    links = dev(u)
    fx = gf.GaugeFixer(links, "fp64_18", flags=gf.FLAG_LEARNED)
    p = _params(15, scale=0.2)
    p_d = dev(p)
    fx.set_weights(p_d, enable=False)
    fx.iterate(2)
    theta, _ = fx.quality()
    tuples = mlp.folded_tuples(dims)
    out = torch.empty(len(tuples), dtype=torch.float64, device="cuda:0")
    gf.gf_mlp_multipliers(fx.ctx, out.data_ptr())
    got = out.cpu().numpy() * np.prod(dims)  # the table includes the inverse FFT's 1/V
    psq = mlp.tuple_psq(dims, tuples)
    p2 = psq.sum(1)
    m0 = np.where(p2 > 0, 0.5 * ALPHA * 16.0 / np.where(p2 > 0, p2, 1.0), 0.0)
    x = mlp.features(psq, theta, 2).astype(np.float32).astype(np.float64)
    want = mlp.multipliers(p.astype(np.float64), x, m0)
    assert got[0] == 0.0
    rel = np.abs(got[1:] - want[1:]) / want[1:]
    assert rel.max() < 2e-5, rel.max()


def test_zero_output_network_is_plain_fa():
    u = synth.make_config((8, 8, 8, 8), 12)
    p = learn.init_params(3)  # zero output layer
    r0, _, l0 = learn.solve(u)
    r1, _, l1 = learn.solve(u, params=torch.from_numpy(p).cuda())
    assert r1.iters == r0.iters and r1.fallbacks == 0
    assert torch.equal(l0, l1)


def test_fallback_rescues_corrupted_weights():
    u = synth.make_config((8, 8, 8, 8), 13)
    p = learn.init_params(4)
    p[-130:-2] = 5.0  # W3: every output pushed far from zero
    p[-2:] = 3.0
    res, _, links = learn.solve(u, params=torch.from_numpy(p).cuda())
    assert res.status == gf.GF_OK and res.theta < 1e-15
    assert res.fallbacks >= 1
    assert landau.theta(links.cpu().numpy()) < 1e-15


@pytest.fixture(scope="module")
def trained():
    """The learned workload's recipe: 500 plain-FA trajectories of 16^4 lattices (seeds 1..500) recorded and
    trained on with the library's kernels."""
    print("training on 500 16^4 trajectories", flush=True)
    params, info = learn.train_default((16, 16, 16, 16), log=lambda m: print(m, flush=True))
    print(info, flush=True)
    return params, info


def test_trained_network_gains_over_plain_fa(trained):
    """Held-out 16^4 configurations solved with and without the trained network: fewer iterations in
    total, theta < 1e-15 by the oracle."""
    params, info = trained
    assert info["trajectories"] == 500 and info["loss_first_last"][1] < info["loss_first_last"][0]
    dims = (16, 16, 16, 16)
    plain, learned = 0, 0
    for seed in (800, 801, 802):
        u = synth.make_config(dims, seed)
        r0, _, _ = learn.solve(u)
        r1, _, links = learn.solve(u, params=params)
        assert r0.status == gf.GF_OK and r1.status == gf.GF_OK
        assert landau.theta(links.cpu().numpy()) < 1e-15
        plain += r0.iters
        learned += r1.iters
    print(f"plain {plain} learned {learned} iterations", flush=True)
    assert learned < plain


@pytest.mark.parametrize("dims,seed,eps", [((32, 32, 32, 32), 10000, synth.EPS_P059),
                                           ((48, 48, 48, 8), 20000, synth.EPS_P060)])
def test_trained_network_converges_on_evaluation_lattices(trained, dims, seed, eps):
    """The evaluation lattices of the learned workload (larger than the 16^4 training lattices): the learned
    solve (with its plain-FA fallback) reaches theta < 1e-15 by the oracle and keeps the plaquette."""
    from oracle import observables
    params, _ = trained
    u = synth.make_config(dims, seed, eps)
    r0, _, _ = learn.solve(u)
    r1, _, links = learn.solve(u, params=params)
    out = links.cpu().numpy()
    print(f"{dims}: plain {r0.iters}, learned {r1.iters} iterations, {r1.fallbacks} fallbacks", flush=True)
    assert r1.status == gf.GF_OK and r1.theta < 1e-15
    assert landau.theta(out) < 1e-15
    assert abs(observables.plaquette(out) - observables.plaquette(u)) < 1e-12
