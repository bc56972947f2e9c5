"""Surrogate network kernels and scorer vs the FP64 oracle, and what the
trained surrogate gains over random proposals."""
import numpy as np
import pytest

import oracle
from oracle import surrogate as S
from synth import sbm, workload
from tests.conftest import to_dev

pytestmark = pytest.mark.gpu

IN, H = 21, 256


def _data(B, seed):
    import torch
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((B, IN)).astype(np.float32)
    t = (np.sin(X[:, 0]) + 0.3 * X[:, 1] * X[:, 2]).astype(np.float32)
    return X, t, torch.from_numpy(X).cuda(), torch.from_numpy(t).cuda()


def test_mlp_init_is_glorot(lne, ctx):
    p = lne.mlp_init(ctx, IN, H, seed=3).cpu().numpy()
    lay, n = S.layout(IN, H)
    assert len(p) == n == lne.mlp_param_count(IN, H)
    o, k = lay["W1"]
    a = np.sqrt(6 / (IN + H))
    assert np.abs(p[o:o + k]).max() <= a and abs(np.std(p[o:o + k]) - a / np.sqrt(3)) < 0.05 * a
    o, k = lay["b2"]
    assert np.all(p[o:o + k] == 0)


@pytest.mark.parametrize("B", [1, 37, 1024])
def test_mlp_forward_and_gradient_match_oracle(lne, ctx, B):
    p = lne.mlp_init(ctx, IN, H, seed=B)
    X, t, Xd, td = _data(B, B)
    pn = p.cpu().numpy().astype(np.float64)
    y = lne.mlp_forward(ctx, IN, H, p, Xd).cpu().numpy()
    y0, _ = S.forward(pn, X.astype(np.float64), IN, H)
    np.testing.assert_allclose(y, y0, rtol=1e-4, atol=1e-5)
    g, loss = lne.mlp_grad(ctx, IN, H, p, Xd, td)
    l0, g0 = S.loss_and_grad(pn, X.astype(np.float64), t.astype(np.float64), IN, H)
    assert abs(loss.item() - l0) <= 1e-4 * max(l0, 1e-3)
    g = g.cpu().numpy()
    assert np.linalg.norm(g - g0) <= 1e-4 * np.linalg.norm(g0)


@pytest.mark.parametrize("n_in,h,B", [(1, 1, 1), (3, 17, 16), (21, 64, 33), (40, 130, 100),
                                      (21, 300, 17), (5, 320, 48), (21, 321, 20)])
def test_network_at_the_edges_of_its_tiles(lne, ctx, n_in, h, B):
    """Odd widths and batches around the 16-row, 16-column and 32-column tiles,
    the widest fused network (320) and the first that is not (321).  Each sum
    has at most 1 + max(n_in, h, B) terms of relative rounding u = 2^-24; the
    three chained layers and the sums over rows stay within 1e-4 in norm."""
    import torch
    rng = np.random.default_rng(h)
    p = lne.mlp_init(ctx, n_in, h, seed=h)
    p += 0.05 * torch.from_numpy(rng.standard_normal(p.numel()).astype(np.float32)).cuda()
    X = rng.standard_normal((B, n_in)).astype(np.float32)
    t = rng.standard_normal(B).astype(np.float32)
    pn = p.cpu().numpy().astype(np.float64)
    Xd, td = torch.from_numpy(X).cuda(), torch.from_numpy(t).cuda()
    y0, _ = S.forward(pn, X.astype(np.float64), n_in, h)
    y = lne.mlp_forward(ctx, n_in, h, p, Xd).cpu().numpy()
    np.testing.assert_allclose(y, y0, rtol=1e-4, atol=1e-5)
    g, loss = lne.mlp_grad(ctx, n_in, h, p, Xd, td)
    l0, g0 = S.loss_and_grad(pn, X.astype(np.float64), t.astype(np.float64), n_in, h)
    assert abs(loss.item() - l0) <= 1e-4 * max(l0, 1e-3)
    assert np.linalg.norm(g.cpu().numpy() - g0) <= 1e-4 * np.linalg.norm(g0)


@pytest.mark.parametrize("n_in,h,B,fused", [
    (21, 8, 8192, "fg"), (21, 8, 8193, "g"), (32, 48, 8193, "fg"), (33, 16, 4097, "g"),
    (64, 31, 4096, "fg"), (65, 31, 4096, "g"), (65, 32, 4096, "fg"), (600, 63, 65, "g"),
    (600, 16, 17, ""), (600, 17, 17, "g"), (600, 128, 512, "g"), (600, 64, 513, "fg"), (600, 129, 16, "fg")])
def test_network_on_both_sides_of_the_fused_kernel(lne, n_in, h, B, fused):
    """Forward pass (f) and gradient (g) by the fused kernel and by launches per
    layer, each where its rule has it; bars as in the test above."""
    import torch
    c = lne.Context()
    c.prof_enable()
    rng = np.random.default_rng(h)
    p = lne.mlp_init(c, n_in, h, seed=h)
    X = rng.standard_normal((B, n_in)).astype(np.float32)
    t = rng.standard_normal(B).astype(np.float32)
    pn = p.cpu().numpy().astype(np.float64)
    Xd, td = torch.from_numpy(X).cuda(), torch.from_numpy(t).cuda()
    y0, _ = S.forward(pn, X.astype(np.float64), n_in, h)
    y = lne.mlp_forward(c, n_in, h, p, Xd).cpu().numpy()
    assert c.prof_get("mlp_rows")[1] == int("f" in fused)
    np.testing.assert_allclose(y, y0, rtol=1e-4, atol=1e-5)
    c.prof_reset()
    g, loss = lne.mlp_grad(c, n_in, h, p, Xd, td)
    assert c.prof_get("mlp_wgrad")[1] == int("g" in fused)
    l0, g0 = S.loss_and_grad(pn, X.astype(np.float64), t.astype(np.float64), n_in, h)
    assert abs(loss.item() - l0) <= 1e-4 * max(l0, 1e-3)
    assert np.linalg.norm(g.cpu().numpy() - g0) <= 1e-4 * np.linalg.norm(g0)
    c.close()


@pytest.mark.parametrize("B", [(1 << 26) - 16, (1 << 26) - 15, (1 << 26) + 1])
def test_forward_of_batches_around_a_launch_of_threads(lne, ctx, B):
    """64 threads a row fill a launch (2^32 threads) at 2^26 rows; more go
    through the launches per layer.  The network is a sum of two GELUs, summed
    by torch in double precision; u = 2^-24, a dozen operations."""
    import torch
    p = torch.tensor([1.0, -0.5, 0.1, 0.2, 0.7, 0.3, -0.4, 0.9, 0.0, 0.1, 1.5, -0.8, 0.25],
                     device="cuda")
    assert p.numel() == lne.mlp_param_count(1, 2)
    X = torch.linspace(-3, 3, B, device="cuda").unsqueeze(1)
    y = lne.mlp_forward(ctx, 1, 2, p, X)
    gelu = torch.nn.functional.gelu
    q = p.double()
    for rows in (slice(0, 1 << 16), slice(B // 2, B // 2 + 4096), slice(B - 4096, B)):
        h = gelu(X[rows].double() @ q[0:2].view(1, 2) + q[2:4])
        h = gelu(h @ q[4:8].view(2, 2) + q[8:10])
        ref = h @ q[10:12] + q[12]
        assert (y[rows].double() - ref).abs().max() <= 64 * 2.0 ** -24
    del X, y
    torch.cuda.empty_cache()


def test_adam_step_matches_oracle(lne, ctx):
    import torch
    p = lne.mlp_init(ctx, IN, H, seed=9)
    X, t, Xd, td = _data(64, 9)
    m = torch.zeros_like(p)
    v = torch.zeros_like(p)
    pn = p.cpu().numpy().astype(np.float64)
    mn = np.zeros_like(pn)
    vn = np.zeros_like(pn)
    for step in range(1, 4):
        g, _ = lne.mlp_grad(ctx, IN, H, p, Xd, td)
        lne.mlp_adam(ctx, p, g, m, v, step, 1e-3)
        pn, mn, vn = S.adam_step(pn, g.cpu().numpy().astype(np.float64), mn, vn, step, 1e-3)
    np.testing.assert_allclose(p.cpu().numpy(), pn, rtol=1e-5, atol=1e-6)


def test_training_fits_a_smooth_target(lne, ctx):
    import torch
    p = lne.mlp_init(ctx, IN, H, seed=1)
    X, t, Xd, td = _data(512, 1)
    m = torch.zeros_like(p)
    v = torch.zeros_like(p)
    first = None
    for step in range(1, 301):
        g, loss = lne.mlp_grad(ctx, IN, H, p, Xd, td)
        first = first if first is not None else loss.item()
        lne.mlp_adam(ctx, p, g, m, v, step, 1e-3)
    assert loss.item() < 0.05 * first


@pytest.mark.parametrize("noise", [1.6, 2.5])
def test_scorer_matches_liblinear(lne, ctx, noise):
    """Multi-label data (1-3 labels per row, features = sum of label centres
    + noise) that is not separable: the GPU scorer and LIBLINEAR agree."""
    import torch
    rng = np.random.default_rng(int(noise * 10))
    n, L, d = 3000, 12, 24
    Y = np.zeros((n, L), dtype=np.uint8)
    for i in range(n):
        Y[i, rng.choice(L, rng.integers(1, 4), replace=False)] = 1
    centers = rng.standard_normal((L, d))
    X = (Y @ centers + noise * rng.standard_normal((n, d))).astype(np.float32)
    perm = rng.permutation(n)
    tr, te = np.sort(perm[:600]), np.sort(perm[600:])
    f_ref = S.score_micro_f1(X, Y, tr, te)
    f = lne.score_micro_f1(ctx, torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda(),
                           torch.from_numpy(tr).cuda(), torch.from_numpy(te).cuda())
    assert 0.2 < f_ref < 0.99
    assert abs(f - f_ref) <= 0.02, (f, f_ref)


def test_batched_scorer_equals_single_calls(lne, ctx):
    """Several embeddings scored in one call give each embedding's own score
    (the weight-gradient row chunks differ between the calls, so logits agree
    to rounding and micro-F1 to a few test rows); more than 64 labels take
    the in-memory logits path."""
    import torch
    rng = np.random.default_rng(5)
    for L in (12, 80):
        n, d = 2000, 16
        Y = np.zeros((n, L), dtype=np.uint8)
        for i in range(n):
            Y[i, rng.choice(L, rng.integers(1, 3), replace=False)] = 1
        centers = rng.standard_normal((L, d))
        Xs = np.stack([(Y @ centers + s * rng.standard_normal((n, d))).astype(np.float32)
                       for s in (0.8, 1.5, 3.0)])
        perm = rng.permutation(n)
        tr = torch.from_numpy(np.sort(perm[:400])).cuda()
        te = torch.from_numpy(np.sort(perm[400:])).cuda()
        Yd = torch.from_numpy(Y).cuda()
        fb = lne.score_micro_f1(ctx, torch.from_numpy(Xs).cuda(), Yd, tr, te)
        fs = [lne.score_micro_f1(ctx, torch.from_numpy(x).cuda(), Yd, tr, te) for x in Xs]
        assert len(fb) == 3
        assert fb[0] > fb[1] > fb[2]
        np.testing.assert_allclose(fb, fs, atol=3.0 / (1600 * 1.5))


def test_search_arms_run_end_to_end(lne, ctx):
    """Pretraining pairs from batched runs, the plain sequential arm and the
    batched surrogate arm on a small graph: shapes, monotone clocks, scores in
    [0, 1] and the batched arm reusing one captured graph per round shape."""
    from paper_2302_07084_amd import search
    rng = np.random.default_rng(3)
    fam = [_task(lne, ctx, intra, seed=40 + i) for i, intra in enumerate((0.45, 0.55))]
    F, y = search.pretrain_pairs(ctx, fam, 8, rng, max_batch=4)
    assert F.shape == (16, search.IN_DIM) and y.shape == (16,)
    sur = search.Surrogate(ctx, seed=1)
    sur.set_scaler(F)
    sur.add(F, y)
    sur.fit(epochs=50)
    task = _task(lne, ctx, 0.5, seed=50)
    sa, ta, ea = search.plain_sequential_search(ctx, task, search.sample_trials(rng, 3))
    assert sa.shape == (3, len(task.splits)) and np.all(np.diff(ta) > 0) and ea > 0
    tb, sb, stb, eb, setup = search.batched_surrogate_search(ctx, task, sur, 8, rng, per_round=4)
    assert len(tb) == 8 and sb.shape == (8, len(task.splits))
    assert np.all(np.diff(stb) >= 0) and eb > 0 and setup > 0
    assert np.all((sa >= 0) & (sa <= 1)) and np.all((sb >= 0) & (sb <= 1))
    assert len(sur.y) == 16                        # refits leave the pretraining set as it was


def test_scorer_rejects_bad_indices(lne, ctx):
    import torch
    X = torch.zeros((10, 4), device="cuda")
    Y = torch.zeros((10, 3), dtype=torch.uint8, device="cuda")
    Y[:, 0] = 1
    with pytest.raises(lne.LneError):
        lne.score_micro_f1(ctx, X, Y, torch.tensor([0, 1, 99], device="cuda"),
                           torch.tensor([2, 3], device="cuda"))


def _task(lne, ctx, intra, seed):
    from paper_2302_07084_amd import search
    n_b, bs, deg = 10, 200, 10
    n = n_b * bs
    g = sbm([bs] * n_b, intra * deg / (bs - 1), (1 - intra) * deg / (n - bs), seed=seed)
    base = dict(T=10, M=20 * 10 * g.m, b=1, C=float(np.log(g.n)), d=32, oversample=10, q=1,
                seed=seed, precision="f32")
    return search.Task.make(ctx, g, base, train_ratio=0.5, seed=seed)


def test_surrogate_beats_random_proposals(lne, ctx):
    """Pretrained on plain-method trials of other graphs (scores standardised
    within each graph, i.e. the relative quality of a trial on its graph),
    the surrogate's top proposals on held-out graphs score higher than random
    proposals with the same budget: over five held-out graphs (other block
    mixes and seeds) the paired per-graph gain has a 95% t-interval above 0,
    and its predictions rank random trials (positive mean Spearman
    correlation)."""
    import scipy.stats
    from paper_2302_07084_amd import search
    rng = np.random.default_rng(0)
    sur = search.Surrogate(ctx, seed=0)
    F, y = [], []
    for i, intra in enumerate((0.42, 0.46, 0.5, 0.54, 0.58, 0.62)):
        task = _task(lne, ctx, intra, seed=10 + i)
        trials, scores = search.random_search(ctx, task, 64, rng)
        F.append(search.features(task, trials))
        y.extend(search.standardize(scores))
    F = np.concatenate(F)
    sur.set_scaler(F)
    sur.add(F, y)
    sur.fit(epochs=800)
    gains, rhos = [], []
    for i, intra in enumerate((0.44, 0.48, 0.52, 0.56, 0.6)):
        task = _task(lne, ctx, intra, seed=30 + i)
        rtrials, rscores = search.random_search(ctx, task, 32, rng)
        cand = search.sample_trials(rng, 4096)
        pred = sur.predict(search.features(task, cand))
        picks = [cand[j] for j in np.argsort(-pred)[:16]]
        sscores = [search.evaluate(ctx, task, t) for t in picks]
        gains.append(np.mean(sscores) - np.mean(rscores))
        rhos.append(scipy.stats.spearmanr(sur.predict(search.features(task, rtrials)), rscores)[0])
        print(f"intra {intra}: random mean {np.mean(rscores):.4f} best {max(rscores):.4f} | "
              f"surrogate mean {np.mean(sscores):.4f} best {max(sscores):.4f} | rho {rhos[-1]:.2f}",
              flush=True)
    g = np.asarray(gains)
    half = scipy.stats.t.ppf(0.975, len(g) - 1) * g.std(ddof=1) / np.sqrt(len(g))
    print(f"gain {g.mean():.4f} +- {half:.4f} (95%), per graph {np.round(g, 4)}", flush=True)
    assert g.mean() - half > 0, (g.mean(), half, gains)
    assert np.mean(rhos) > 0.1, rhos
