"""lne_graph_stats (the search's graph descriptors) against the oracle's
graph_stats on the same graphs: degree moments, median and Hill exponent to
rounding, the closed-wedge count exactly (the same Philox draws on both
sides), and the spectral gap of the same subspace iteration to 1e-9."""
import math

import numpy as np
import pytest

from oracle import graphstats as gst
from synth import graphs as sg
from tests import graphs_small as gs
from tests.conftest import to_dev

pytestmark = pytest.mark.gpu

GRAPHS = {
    "complete12": lambda: gs.complete(12),
    "cycle12": lambda: gs.cycle(12),
    "path30": lambda: gs.path(30),
    "star50": lambda: gs.star(50),
    "sbm2000": lambda: sg.sbm([100] * 20, 0.2, 0.01, seed=3),
    "chunglu4000": lambda: sg.chung_lu(4000, 40000, 2.1, seed=2),   # isolated vertices too
}


@pytest.mark.parametrize("name", list(GRAPHS))
def test_graph_stats_match_oracle(lne, ctx, name):
    g = GRAPHS[name]()
    W, iters, seed = 3000, 200, 7
    rp, col = to_dev(g)
    got = lne.graph_stats(ctx, rp, col, seed=seed, wedges=W, iters=iters)
    ref = gst.graph_stats(g, seed=seed, wedges=W, iters=iters)
    print(name, "gpu", got, "oracle", ref, flush=True)
    np.testing.assert_allclose(got[:6], ref[:6], rtol=1e-12, atol=1e-14)
    assert round(got[6] * W) == gst.wedge_closed(g, seed, W)
    assert abs(got[7] - ref[7]) <= 1e-9


def test_graph_stats_rejects_bad_input(lne, ctx):
    import torch
    g = gs.cycle(8)
    rp, col = to_dev(g)
    with pytest.raises(lne.LneError):
        lne.graph_stats(ctx, rp, col, wedges=0)
    with pytest.raises(lne.LneError):
        lne.graph_stats(ctx, rp, col, iters=0)
    empty_rp = torch.zeros(5, dtype=torch.int64, device="cuda")
    empty_col = torch.zeros(0, dtype=torch.int32, device="cuda")
    with pytest.raises(lne.LneError):
        lne.graph_stats(ctx, empty_rp, empty_col)


@pytest.mark.parametrize("n", [5000, (1 << 20) + 7])
@pytest.mark.parametrize("hub", [65, 64])
def test_spectral_step_with_and_without_a_hub(lne, ctx, n, hub):
    """A star of `hub` leaves beside a path: rows taken by one, two or four groups
    of lanes, as the largest degree and the number of rows have it."""
    e = np.stack([np.arange(hub + 1, n - 1), np.arange(hub + 2, n)], 1)
    star = np.stack([np.zeros(hub, int), np.arange(1, hub + 1)], 1)
    g = gs.from_edges(n, np.concatenate([star, e]).tolist())
    rp, col = to_dev(g)
    got = lne.graph_stats(ctx, rp, col, seed=7, wedges=100, iters=3)
    assert abs(got[7] - (1.0 - gst.spectral_lambda2(g, 7, 3))) <= 1e-9


@pytest.mark.parametrize("n", [(1 << 24) + 1, (1 << 26) + 5])
def test_spectral_step_of_a_graph_of_many_vertices(lne, ctx, n):
    """One step on a cycle whose rows outnumber the waves of a launch (and, the
    larger, a launch's threads at a wave a row): S_2 of (X + A X / 2) / 2 from
    the Gaussian start, the Gram matrix summed by torch; its n products of
    terms of one size are off by less than 1e-9 of it however they are
    summed."""
    import torch
    i = torch.arange(n, device="cuda", dtype=torch.int32)
    col = torch.stack([torch.where(i == 0, 1, i - 1), torch.where(i == n - 1, n - 2, i + 1)], 1)
    col[0] = torch.tensor([1, n - 1])
    col[n - 1] = torch.tensor([0, n - 2])
    rp = 2 * torch.arange(n + 1, device="cuda", dtype=torch.int64)
    got = lne.graph_stats(ctx, rp, col.reshape(-1).contiguous(), seed=3, wedges=100, iters=1)
    del i, col, rp
    X = lne.gaussian(ctx, n, 16, 3, torch.float64)
    Y = X.roll(1, 0)
    Y += X.roll(-1, 0)
    Y.mul_(0.5).add_(X).mul_(0.5)
    S2 = torch.linalg.eigvalsh(Y.T @ Y)[-2].sqrt().item()
    assert abs((2.0 - got[7]) / 2.0 - S2) <= 1e-9 * S2
    assert got[6] == 0.0
    del X, Y
    torch.cuda.empty_cache()


@pytest.mark.parametrize("name", ["edges12", "k88", "cycle12"])
def test_a_block_that_loses_rank_is_seen_after_two_steps(lne, name):
    """The operator has fewer than 16 directions that do not vanish: the steps
    by CholeskyQR are left after the second, whatever their number."""
    g = {"edges12": gs.from_edges(24, [(2 * i, 2 * i + 1) for i in range(12)]),
         "k88": gs.from_edges(16, [(i, 8 + j) for i in range(8) for j in range(8)]),
         "cycle12": gs.cycle(12)}[name]
    rp, col = to_dev(g)
    c = lne.Context()
    c.prof_enable()
    for iters in (2, 3, 40):
        c.prof_reset()
        got = lne.graph_stats(c, rp, col, seed=7, wedges=10, iters=iters)
        # (a second pass where the next product is the last)
        assert c.prof_get("chol_inv")[1] == (2 if iters != 3 else 3)
        assert abs(got[7] - (1.0 - gst.spectral_lambda2(g, 7, iters))) <= 1e-9
    c.close()


@pytest.mark.parametrize("seed", [37904, 43290, 21102])
def test_spectral_gap_from_an_ill_conditioned_start(lne, ctx, seed):
    """A 16 x 16 Gaussian start whose condition number is 3 10^5 to 9 10^5,
    found by search over seeds: one Cholesky pass (and one eigSVD) leaves it
    orthonormal to 10^-5 only.  On the complete graph every direction but one
    has the eigenvalue -1/15, so two steps give the gap 1 + 1/15 itself; bar:
    1,000 roundings."""
    rp, col = to_dev(gs.complete(16))
    got = lne.graph_stats(ctx, rp, col, seed=seed, wedges=10, iters=2)
    assert abs(got[7] - (1.0 + 1.0 / 15.0)) <= 1000 * 2.0 ** -53
