"""The work that stands for this library's use, for timing it and comparing its results.

Each case is one call (or the pair of calls of a training step) of the public
Python entry points on inputs that are already on the GPU.  The sizes are
those of the repository's own configurations: the 1,000-vertex graph of the
smoke test, the BlogCatalog-like graph, the benchmark's 10-million-vertex
graph, the precision configuration's dense blocks, the batched-trials graph
and the surrogate of the hyperparameter search.  A case names its entry point
(`call`) and its sizes; `draw` gives further cases between the smallest and
the largest, odd sizes among them.

Inputs are made on the GPU from the seed alone: Chung-Lu power-law graphs and
planted-partition graphs (simple, undirected, rows ascending), dense blocks
with decaying singular values as a power iteration meets them, embeddings with
planted labels, and a half-trained surrogate network.
"""
import ctypes
import math

import numpy as np
import torch

import paper_2302_07084_amd as lne

IN_DIM = 21      # surrogate inputs: 10 length weights, k, theta, mu, 8 graph descriptors
SHORT = (0.3, 0.7)   # length weights of the benchmark (walks of one or two edges)
LABELS = 50

TYPES = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}


def listed():
    return [
        # A whole embedding of a small graph in double precision: the call of a
        # program that embeds many small graphs, where latency and launches count.
        dict(name="embed_small_f64", call="embed", graph="blocks", n=1000, m=9500, blocks=10,
             intra=0.75, T=10, lengths="uniform", mult=100, d=32, oversample=10, q=1, cheb_k=10,
             precision="f64", weights=0),
        # A whole embedding of an ordinary graph (BlogCatalog's size) with long walks.
        dict(name="embed_mid_f32", call="embed", graph="power", n=10_000, m=330_000, gamma=2.2,
             T=10, lengths="uniform", mult=20, d=128, oversample=10, q=1, cheb_k=10,
             precision="f32", weights=0),
        # The benchmark's workload, the largest graph: one embedding step.
        dict(name="embed_large_f32", call="embed", graph="power", n=10_000_000, m=200_000_000,
             gamma=2.1, T=5, lengths="short", mult=4, d=128, oversample=10, q=1, cheb_k=10,
             precision="f32", weights=0),
        # The sparsifier stage alone on a weighted graph (sampling, aggregation, Eq. (1)).
        dict(name="sparsify_weighted", call="sparsify", graph="power", n=1_000_000, m=20_000_000,
             gamma=2.1, T=5, lengths="short", mult=4, precision="f32", weights=16),
        # The orthonormaliser of a power step on the precision configuration's block in BF16.
        dict(name="orthonormalize_bf16", call="orthonormalize", n=1_000_000, k=266,
             precision="bf16"),
        # The same in single precision, at the width that the default dimension gives.
        dict(name="orthonormalize_f32", call="orthonormalize", n=2_000_003, k=138,
             precision="f32"),
        # The Gram-based SVD that ends every embedding, on a tall block of the default dimension.
        dict(name="eigsvd_f32", call="eigsvd", n=100_000, k=128, precision="f32"),
        # Spectral propagation of an embedding made elsewhere, on a graph of ordinary size.
        dict(name="propagate_f32", call="propagate", graph="power", n=1_000_000, m=20_000_000,
             gamma=2.1, d=128, cheb_k=10, precision="f32", weights=0),
        # A round of the hyperparameter search: several trials of one graph in one batch.
        dict(name="batch_trials", call="batch", graph="blocks", n=100_000, m=1_500_000, blocks=50,
             intra=0.3, T=10, mult=10, d=128, oversample=10, q=1, trials=8),
        # One training step of the search's surrogate on the pairs of eight graphs.
        dict(name="surrogate_step", call="surrogate", batch=512, hidden=256),
        # Link-prediction ranks of held-out edges among corrupted ones.
        dict(name="link_rank_f32", call="link", n=10_000_000, d=32, held_out=10_000,
             corrupted=1000, precision="f32"),
        # The descriptors of a graph that the surrogate reads (one call for each new graph).
        dict(name="graph_descriptors", call="stats", graph="blocks", n=30_000, m=450_000,
             blocks=30, intra=0.34, wedges=2000, iters=200),
    ]


def _spread(rng, lo, hi):
    """A whole number between lo and hi, spread over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["embed", "embed", "embed", "sparsify", "orthonormalize", "eigsvd",
                       "propagate", "propagate", "batch", "surrogate", "link", "stats"])
    c = dict(call=call)
    if call in ("embed", "sparsify", "propagate"):
        n = _spread(rng, 1000, 2_000_000)
        c.update(graph=rng.choice(["power", "blocks"]), n=n, m=int(n * rng.uniform(8, 25)))
        if c["graph"] == "power":
            c.update(gamma=round(rng.uniform(2.1, 2.5), 2))
        else:
            c.update(blocks=rng.randint(5, 50), intra=round(rng.uniform(0.3, 0.8), 2))
        c.update(weights=rng.choice([0, 0, 16]))
    if call in ("embed", "sparsify"):
        c.update(T=rng.choice([2, 5, 10]), lengths=rng.choice(["uniform", "short"]))
        # samples in all: between the benchmark's 4 T m and 100 T m on small graphs
        c.update(mult=max(1, min(100, int(2e8 / (c["T"] * c["m"])))) if c["m"] > 500_000
                 else rng.randint(4, 20))
    if call == "embed":
        c.update(d=rng.choice([16, 32, 33, 64, 96, 100, 128]), oversample=10,
                 q=rng.choice([1, 1, 2]), cheb_k=rng.choice([0, 5, 10, 10]),
                 precision=rng.choice(["f32", "f32", "f64"]))
    elif call == "sparsify":
        c.update(precision=rng.choice(["f32", "f32", "f64"]))
    elif call == "propagate":
        c.update(d=rng.choice([16, 32, 33, 64, 100, 128, 200]), cheb_k=rng.randint(3, 12),
                 precision=rng.choice(["f32", "f32", "f64"]))
    elif call in ("orthonormalize", "eigsvd"):
        c.update(n=_spread(rng, 3000, 3_000_000), k=rng.choice([16, 32, 42, 74, 128, 138, 200, 266]),
                 precision=rng.choice(["f32", "f32", "f64", "bf16"] if call == "orthonormalize"
                                      else ["f32", "f32", "f64"]))
    elif call == "batch":
        n = _spread(rng, 2000, 100_000)
        c.update(graph="blocks", n=n, m=int(n * rng.uniform(10, 18)), blocks=rng.randint(10, 50),
                 intra=round(rng.uniform(0.28, 0.5), 2), T=10, mult=rng.randint(5, 20),
                 d=rng.choice([32, 64, 128]), oversample=10, q=1, trials=rng.randint(2, 8))
    elif call == "surrogate":
        c.update(batch=_spread(rng, 16, 4096), hidden=rng.choice([64, 128, 256]))
    elif call == "link":
        c.update(n=_spread(rng, 10_000, 10_000_000), d=rng.choice([16, 32, 50, 64, 100, 128]),
                 held_out=_spread(rng, 200, 10_000), corrupted=_spread(rng, 50, 1000),
                 precision=rng.choice(["f32", "f32", "f64"]))
    else:
        n = _spread(rng, 2000, 100_000)
        c.update(graph="blocks", n=n, m=int(n * rng.uniform(10, 18)), blocks=rng.randint(10, 50),
                 intra=round(rng.uniform(0.28, 0.5), 2), wedges=2000,
                 iters=rng.choice([100, 150, 200]))
    return c


# ---- inputs -------------------------------------------------------------------
def _power_draw(n, m, gamma):
    """Sampler of vertex ids with weight (x + i0)^(-1 / (gamma - 1)), i0 such that
    the largest expected degree is sqrt(2m)."""
    alpha = 1.0 / (gamma - 1.0)
    beta = 1.0 - alpha
    lo, hi = 1e-9, float(n)
    for _ in range(100):
        i0 = math.sqrt(lo * hi)
        z = ((n + i0) ** beta - i0 ** beta) / beta
        w0 = ((1 + i0) ** beta - i0 ** beta) / beta
        lo, hi = (i0, hi) if 2.0 * m * w0 / z > math.sqrt(2.0 * m) else (lo, i0)
    low = hi ** beta
    span = (n + hi) ** beta - low

    def ids(count, gen):
        u = torch.rand(count, generator=gen, device="cuda", dtype=torch.float64)
        return (u.mul_(span).add_(low).pow_(1.0 / beta).sub_(hi)).long().clamp_(0, n - 1)
    return ids


def make_graph(case, gen):
    """(row offsets int64, columns int32, block of each vertex or None) of a simple
    undirected graph with case["m"] edges, rows ascending."""
    n, m = case["n"], case["m"]
    label = None
    if case["graph"] == "blocks":
        B = case["blocks"]
        label = torch.arange(n, device="cuda") * B // n
        first = (torch.arange(B + 1, device="cuda") * n + B - 1) // B

        def pairs(count):
            a = torch.randint(n, (count,), generator=gen, device="cuda")
            b = torch.randint(n, (count,), generator=gen, device="cuda")
            same = torch.rand(count, generator=gen, device="cuda") < case["intra"]
            s = first[label[a]]
            inside = s + b % (first[label[a] + 1] - s)
            return a, torch.where(same, inside, b)
    else:
        ids = _power_draw(n, m, case["gamma"])

        def pairs(count):
            return ids(count, gen), ids(count, gen)
    keys = torch.empty(0, dtype=torch.int64, device="cuda")
    want = int(1.05 * m) + 64
    while keys.numel() < m:
        a, b = pairs(want)
        k = torch.minimum(a, b) * n + torch.maximum(a, b)
        k = k[a != b]
        del a, b
        keys = torch.unique(torch.cat([keys, k]))
        del k
        want = max(int(1.5 * (m - keys.numel())), m // 20) + 64
    keep = torch.rand(keys.numel(), generator=gen, device="cuda")
    # exactly m of the distinct pairs, chosen uniformly
    cut = torch.kthvalue(keep, m).values if keys.numel() < 1 << 24 else torch.sort(keep).values[m - 1]
    keys = keys[keep <= cut][:m]
    del keep
    a, b = keys // n, keys % n
    both = torch.sort(torch.cat([keys, b * n + a])).values
    del keys, a, b
    row = both // n
    col = (both - row * n).to(torch.int32)
    del both
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rowptr[1:] = torch.cumsum(torch.bincount(row, minlength=n), 0)
    del row
    if m > 5_000_000:
        torch.cuda.empty_cache()
    return rowptr, col, label


def _arc_weights(case, rowptr, col):
    """Symmetric integer weights 1..case["weights"] from a hash of each pair."""
    n = case["n"]
    row = torch.repeat_interleave(torch.arange(n, device="cuda"), rowptr.diff())
    c = col.long()
    h = torch.minimum(row, c) * 0x1F123BB5 + torch.maximum(row, c) * 0x2545F491
    h = (h ^ (h >> 15)) * 0x2C1B3C6D
    h = (h ^ (h >> 12)) & 0x7FFFFFFF
    return (1 + h % case["weights"]).to(torch.int32)


def _params(case, seed):
    T = case.get("T", 1)
    s = np.full(T, 1.0 / T)
    if case.get("lengths") == "short":
        s = np.zeros(T)
        s[:2] = SHORT
    return dict(T=T, s=s, M=case.get("mult", 1) * T * case["m"], b=1, C=math.log(case["n"]),
                d=case.get("d", 1), oversample=case.get("oversample", 0), q=case.get("q", 1),
                cheb_k=case.get("cheb_k", 0), theta=0.5, mu=0.2, seed=seed,
                precision=case.get("precision", "f32"))


def _tall(case, gen):
    """n x k block whose singular values fall as a power iteration's product has them
    (power law over two decades), rows padded to whole cache lines."""
    n, k = case["n"], case["k"]
    dt = TYPES[case["precision"]]
    per = 128 // torch.empty(0, dtype=dt).element_size()
    ld = -(-k // per) * per
    Y = torch.zeros(n, ld, dtype=dt, device="cuda")
    s = 1000.0 * (1.0 + torch.arange(k, device="cuda", dtype=torch.float64)) ** -0.9
    V = torch.linalg.qr(torch.randn(k, k, generator=gen, device="cuda", dtype=torch.float64))[0]
    W = (s[:, None] * V).float()
    for i in range(0, n, 1 << 19):
        G = torch.randn(min(1 << 19, n - i), k, generator=gen, device="cuda") / math.sqrt(n)
        Y[i:i + G.shape[0], :k] = (G @ W).to(dt)
    return Y[:, :k]


def _trials(case, seed):
    r = np.random.default_rng(seed)
    return [dict(s=r.dirichlet(np.ones(case["T"])), k=int(r.integers(1, 21)),
                 theta=float(r.random()), mu=float(0.5 * r.random()))
            for _ in range(case["trials"])]


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _surrogate_inputs(case, gen):
    H, B = case["hidden"], case["batch"]
    count = lne.mlp_param_count(IN_DIM, H)
    rnd = lambda *shape: torch.randn(*shape, generator=gen, device="cuda")  # noqa: E731
    p = torch.cat([rnd(IN_DIM * H) / math.sqrt(IN_DIM), 0.1 * rnd(H), rnd(H * H) / math.sqrt(H),
                   0.1 * rnd(H), rnd(H) / math.sqrt(H), 0.1 * rnd(1)]).contiguous()
    assert p.numel() == count
    g = 0.05 * rnd(count)
    return dict(p=p, X=rnd(B, IN_DIM), t=rnd(B), m=0.3 * g, v=(0.5 + torch.rand(
        count, generator=gen, device="cuda")) * g * g + 1e-6)


def prepare(case, seed):
    gen = _generator(seed)
    call = case["call"]
    s = dict(case=case, ctx=lne.Context())
    if call == "surrogate":
        s.update(_surrogate_inputs(case, gen))
        return s
    if call == "link":
        n, d = case["n"], case["d"]
        X = torch.randn(n, d, generator=gen, device="cuda", dtype=TYPES[case["precision"]])
        X *= (1.0 + torch.arange(d, device="cuda")) ** -0.5
        ids = _power_draw(n, 20 * n, 2.1)
        s.update(X=X, pos=torch.stack([ids(case["held_out"], gen), ids(case["held_out"], gen)],
                                      1).to(torch.int32),
                 neg=torch.randint(n, (case["held_out"], case["corrupted"]), generator=gen,
                                   device="cuda").to(torch.int32))
        return s
    if call in ("orthonormalize", "eigsvd"):
        s.update(Y=_tall(case, gen))
        return s
    rowptr, col, _ = make_graph(case, gen)
    s.update(rowptr=rowptr, col=col, weight=None)
    if case.get("weights"):
        s["weight"] = _arc_weights(case, rowptr, col)
    if call == "batch":
        # the search keeps one batch per graph: its sampling pass is made once
        p = _params(case, seed)
        s.update(trials=_trials(case, seed),
                 batch=lne.Batch(s["ctx"], rowptr, col, p, case["trials"]))
    elif call == "propagate":
        p = _params(case, seed)
        p["flags"] = lne.FLAG_NO_FINAL_EIGSVD
        X0 = torch.randn(case["n"], case["d"], generator=gen, device="cuda",
                         dtype=TYPES[case["precision"]])
        X0 *= (1.0 + torch.arange(case["d"], device="cuda")) ** -0.5
        s.update(params=p, X0=X0)
    else:
        s.update(params=_params(case, seed))
    if call == "sparsify":
        # at most two entries per sample
        cap = min(2 * s["params"]["M"], case["n"] ** 2)
        s.update(out=(torch.zeros(case["n"] + 1, dtype=torch.int64, device="cuda"),
                      torch.zeros(cap, dtype=torch.int32, device="cuda"),
                      torch.zeros(cap, dtype=TYPES[case["precision"]], device="cuda")))
    return s


# ---- one pass -------------------------------------------------------------------
def run(state):
    case, ctx = state["case"], state["ctx"]
    call = case["call"]
    if call == "embed":
        return lne.embed(ctx, state["rowptr"], state["col"], state["params"],
                         weight=state["weight"])
    if call == "sparsify":
        # the matrix into the program's own buffers, which hold the largest it can be
        M, stats = lne.sparsify_log(ctx, state["rowptr"], state["col"], state["params"],
                                    weight=state["weight"])
        rp, c, v = state["out"]
        ctx.check(ctx.L.lne_csr_copy(ctx.h, ctypes.byref(M.s), rp.data_ptr(), c.data_ptr(),
                                     v.data_ptr()), "csr_copy")
        M.free()
        return rp, c, v, stats
    if call == "orthonormalize":
        return lne.orthonormalize(ctx, state["Y"])
    if call == "eigsvd":
        return lne.eigsvd(ctx, state["Y"])
    if call == "propagate":
        return lne.propagate(ctx, state["rowptr"], state["col"], state["params"], state["X0"],
                             weight=state["weight"])
    if call == "batch":
        return state["batch"].run(state["trials"], graph=True)[0]
    if call == "surrogate":
        H = case["hidden"]
        g, loss = lne.mlp_grad(ctx, IN_DIM, H, state["p"], state["X"], state["t"])
        lne.mlp_adam(ctx, state["p"], g, state["m"], state["v"], 100, 1e-3)
        return g, loss, state["p"], state["m"], state["v"]
    if call == "link":
        return lne.link_rank(ctx, state["X"], state["pos"], state["neg"])
    return lne.graph_stats(ctx, state["rowptr"], state["col"], seed=7, wedges=case["wedges"],
                           iters=case["iters"])


# ---- what one pass cannot do without ----------------------------------------------
def work(case):
    """Inputs read once and outputs written once; multiply-adds of the products that
    the method is made of.  The products with the sampled matrix are left out of
    "flops": its size is known only once it has been sampled."""
    call = case["call"]
    es = {"f64": 8, "f32": 4, "bf16": 2}[case.get("precision", "f32")]
    if call == "surrogate":
        B, H = case["batch"], case["hidden"]
        count = IN_DIM * H + H + H * H + H + H + 1
        return dict(bytes=4.0 * (B * (IN_DIM + 1) + 7 * count),
                    flops=6.0 * B * (IN_DIM * H + H * H + H))
    if call == "link":
        pairs = case["held_out"] * (case["corrupted"] + 1)
        return dict(bytes=float(pairs * (es * case["d"] + 4) + 8 * case["held_out"]),
                    flops=2.0 * pairs * case["d"])
    if call in ("orthonormalize", "eigsvd"):
        n, k = case["n"], case["k"]
        if call == "orthonormalize":   # two passes of Gram and projection
            return dict(bytes=2.0 * n * k * es, flops=2 * (n * k * (k + 1.0) + n * k * (k + 1.0)))
        return dict(bytes=2.0 * n * k * es + 8.0 * k * (k + 1), flops=n * k * (k + 1.0)
                    + 2.0 * n * k * k + 9.0 * k ** 3)
    n, arcs = case["n"], 2 * case["m"]
    graph = 8.0 * (n + 1) + 4.0 * arcs * (2 if case.get("weights") else 1)
    if call == "stats":
        return dict(bytes=graph + 64.0, flops=case["iters"] * 16 * (2.0 * arcs + 4.0 * 16 * n))
    if call == "sparsify":
        return dict(bytes=graph + 8.0 * (n + 1) + (4 + es) * 2.0 * arcs, flops=0.0)
    d = case["d"]
    steps = 2 * case["cheb_k"] + 1 if case.get("cheb_k") else 0
    if call == "propagate":
        return dict(bytes=graph + 2.0 * n * d * es, flops=2.0 * arcs * d * steps)
    kp = d + case["oversample"]
    # per embedding: an orthonormalisation, the eigen-solve's Gram, and U S^1/2
    dense = 4.0 * n * kp * kp + 1.0 * n * kp * kp + 2.0 * n * kp * d + (3.0 * n * d * d if steps else 0)
    if call == "batch":
        t = case["trials"]
        return dict(bytes=graph + 4.0 * t * n * d, flops=t * (dense + 2.0 * arcs * d * 21))
    return dict(bytes=graph + float(n * d * es), flops=dense + 2.0 * arcs * d * steps)


# ---- the same outputs in 64 bits ---------------------------------------------------
def _exact_orthonormalize(Y):
    Y = Y.double()
    for _ in range(2):
        Y = Y @ torch.linalg.inv(torch.linalg.cholesky(Y.T @ Y, upper=True))
    return Y


def _exact_propagate(case, s):
    """D^-1 A (X0 - sum_n c_n T_n(x) X0), x = ((I - D^-1 A) - mu)^2 / 2 - 1, with
    c_n = (2 - [n = 0]) (-1)^n e^(-theta/2) I_n(theta)."""
    p, X0 = s["params"], s["X0"].double()
    w = torch.ones(s["col"].numel(), dtype=torch.float64, device="cuda") if s["weight"] is None \
        else s["weight"].double()
    A = torch.sparse_csr_tensor(s["rowptr"], s["col"].long(), w, (case["n"], case["n"]))
    deg = (A @ torch.ones(case["n"], 1, dtype=torch.float64, device="cuda"))[:, 0]
    inv = torch.where(deg > 0, 1.0 / deg, 0.0)[:, None]
    walk = lambda Z: inv * (A @ Z)  # noqa: E731
    shifted = lambda Z: (1.0 - p["mu"]) * Z - walk(Z)  # noqa: E731
    x = lambda Z: 0.5 * shifted(shifted(Z)) - Z  # noqa: E731

    def bessel(n, t):
        return sum((t / 2) ** (2 * j + n) / (math.factorial(j) * math.factorial(j + n))
                   for j in range(40))
    c = [(1 if i == 0 else 2) * (-1) ** i * math.exp(-p["theta"] / 2) * bessel(i, p["theta"])
         for i in range(p["cheb_k"] + 1)]
    a, b = X0, x(X0)
    out = X0 - c[0] * a - c[1] * b
    for i in range(2, p["cheb_k"] + 1):
        a, b = b, 2.0 * x(b) - a
        out -= c[i] * b
    return walk(out)


def _exact_surrogate(case, s):
    H = case["hidden"]
    p = s["p"].double().requires_grad_(True)
    W1, b1, W2, b2, W3, b3 = torch.split(p, [IN_DIM * H, H, H * H, H, H, 1])
    gelu = torch.nn.functional.gelu
    h = gelu(s["X"].double() @ W1.view(IN_DIM, H) + b1)
    h = gelu(h @ W2.view(H, H) + b2)
    loss = ((h @ W3 + b3 - s["t"].double()) ** 2).mean()
    g, = torch.autograd.grad(loss, p)
    b1m, b2m, step, lr, eps = 0.9, 0.999, 100, 1e-3, 1e-8
    m = b1m * s["m"].double() + (1 - b1m) * g
    v = b2m * s["v"].double() + (1 - b2m) * g * g
    q = p.detach() - lr * (m / (1 - b1m ** step)) / ((v / (1 - b2m ** step)).sqrt() + eps)
    return g, loss.detach().reshape(1), q, m, v


def exact(case, seed):
    """Whole embeddings and trials, sampled matrices and sampled descriptors have no value
    here: singular vectors carry a sign, and samples are the library's own draws."""
    call = case["call"]
    if call not in ("orthonormalize", "eigsvd", "propagate", "surrogate"):
        return None
    if call == "propagate" and case["m"] * case["d"] * case["cheb_k"] > 4e10:
        return None
    s = prepare(case, seed)
    if call == "surrogate":
        return _exact_surrogate(case, s)
    if call == "propagate":
        return _exact_propagate(case, s)
    if call == "orthonormalize":
        return _exact_orthonormalize(s["Y"])
    lam = torch.linalg.eigvalsh(s["Y"].double().T @ s["Y"].double())
    return None, lam.flip(0).clamp_min(0).sqrt(), None
