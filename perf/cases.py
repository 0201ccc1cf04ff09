"""The workloads by which this framework's speed is judged, through its public entry points.

Kinds of case:
  price   exact price of every move of given solutions, every price returned (a caller with its own solutions)
  sweep   exact best move of every chain of a running search (the benchmark's step)
  search  GVNS iterations, plain or best-of-G (Algorithm 2), then the chains' costs and the best solution
  learned the learned move scorer fitted on a minibatch epoch, its scores, then GVNS iterations with it

A case's T is a comma-separated list of horizons; every instance of a batch draws its K from K..K_hi and its T
from the list.  The data are drawn as the repository's synthetic instances are.
"""
import numpy as np

from paper_1704_05132_amd import vns
from paper_1704_05132_amd.instances import draw_instance, random_pattern

INF = np.iinfo(np.int64).max


def _case(kind, K, T, n_inst=1, chains=1, K_hi=0, **more):
    return dict(kind=kind, n_inst=n_inst, K=K, K_hi=K_hi or K, T=str(T), chains=chains, **more)


def listed():
    return [
        # the smallest call: one small instance's moves priced once, where launches and copies are all there is
        dict(_case("price", 10, 12, decode=0), name="price_10x12"),
        # the paper's instance size: every move of one solution, every price wanted
        dict(_case("price", 300, 52, decode=0), name="price_300x52"),
        # the disposal reading of the decode with unit costs, on a population of solutions
        dict(_case("price", 100, 52, chains=16, decode=2, unit_costs=True), name="price_disposal_100x52_c16"),
        # the best move of every product of a 64-chain search
        dict(_case("sweep", 100, 52, chains=64, spread=8, products=True), name="sweep_100x52_c64"),
        # many uneven instances with short horizons
        dict(_case("sweep", 10, "12,24,52", n_inst=1024, chains=8, K_hi=200, spread=4, products=False),
             name="sweep_short_1024x8"),
        # the benchmark's shape: large uneven instances, horizons of one and two years of weeks
        dict(_case("sweep", 100, "52,104", n_inst=256, chains=16, K_hi=1000, group=16, products=False),
             name="sweep_long_256x16"),
        # a single small search, its iterations' records wanted
        dict(_case("search", 10, 12, iters=500, nb="1,2", trace=True), name="search_10x12"),
        # the 64-chain search of one instance, iterations computed side by side
        dict(_case("search", 100, 52, chains=64, iters=200, waves=4, spec_iters=12), name="search_100x52_c64"),
        # batched search, short horizons
        dict(_case("search", 10, "12,24,52", n_inst=512, chains=8, K_hi=200, iters=50, waves=2, lds=0, state=0),
             name="search_short_512x8"),
        # batched search, large instances
        dict(_case("search", 100, "52,104", n_inst=64, chains=16, K_hi=1000, iters=50, waves=2, lds=0, state=0),
             name="search_long_64x16"),
        # the paper's multi-GPU scheme on its instance size: best of 4 shakes an iteration
        dict(_case("search", 300, 52, n_inst=27, chains=2, iters=50, waves=2, best_of=4), name="best_of_4_300x52"),
        # the learned search: fit the scorer, score, search
        dict(_case("learned", 100, 52, chains=64, iters=50, waves=4, spec_iters=8, rows=65536, batch=4096),
             name="learned_100x52_c64"),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["price", "price", "sweep", "sweep", "sweep", "search", "search", "search", "learned"])
    T = ",".join(str(t) for t in sorted({_log(rng, 4, 128) for _ in range(rng.choice([1, 1, 2, 3]))}))
    if kind == "price":
        return _case(kind, _log(rng, 3, 400), T.split(",")[0], chains=_log(rng, 1, 16),
                     decode=rng.choice([0, 0, 0, 1, 2, 3]), unit_costs=rng.random() < 0.3)
    if kind == "learned":
        return _case(kind, _log(rng, 20, 200), T.split(",")[-1], chains=_log(rng, 4, 64), iters=_log(rng, 10, 60),
                     waves=4, spec_iters=rng.choice([1, 4, 8]), rows=_log(rng, 5000, 100000), batch=4096)
    n = _log(rng, 1, 200 if kind == "sweep" else 48)
    K = _log(rng, 8, 300)
    many = dict(n_inst=n, K_hi=_log(rng, K, 2 * K))
    if kind == "sweep":
        launch = rng.choice([dict(spread=4), dict(spread=8), dict(group=4), dict(group=16), dict(incremental=True)])
        return _case(kind, K, T, chains=_log(rng, 1, 16), products=rng.random() < 0.5, **launch, **many)
    chains = _log(rng, 1, 16)
    form = rng.choice(["plain", "plain", "spec", "best"])
    more = dict(waves=2, lds=0, state=0) if n * chains > 64 else dict(waves=rng.choice([4, 8]))
    if form == "spec":
        more["spec_iters"] = rng.choice([4, 12])
    if form == "best":
        many["n_inst"], chains, more["best_of"] = min(n, 16), min(chains, 4), rng.choice([2, 4])
    return _case(kind, K, T, chains=chains, iters=_log(rng, 10, 60), **more, **many)


def _instances(case, rng):
    Ts = [int(t) for t in case["T"].split(",")]
    sizes = np.random.default_rng([case["n_inst"], case["K"], case["K_hi"], *Ts])   # the case's, whatever the seed
    many = case["n_inst"] > 1
    out = []
    for _ in range(case["n_inst"]):
        K = int(sizes.integers(case["K"], case["K_hi"] + 1))
        inst = draw_instance(rng, K, int(sizes.choice(Ts)), *((0.1, 0.9) if many else (0.2, 0.8)))
        if case.get("unit_costs"):
            inst.pM, inst.pR = rng.integers(0, 20, K).astype(np.int32), rng.integers(0, 20, K).astype(np.int32)
        inst.strict, inst.dispose = bool(case.get("decode", 0) & 1), bool(case.get("decode", 0) & 2)
        out.append(inst)
    return out


def _patterns(case, inst, rng):
    """One solution per chain.  Under the strict reading an interval short of returns is infeasible, so those
    solutions only manufacture."""
    got = [random_pattern(inst, rng) for _ in range(case["chains"])]
    return [(a, np.zeros_like(b)) if inst.strict else (a, b) for a, b in got]


def _options(case):
    keys = dict(spread=vns.OPT_EVAL_SPREAD, group=vns.OPT_EVAL_GROUP, incremental=vns.OPT_EVAL_INCREMENTAL,
                waves=vns.OPT_RUN_WAVES, lds=vns.OPT_RUN_LDS, state=vns.OPT_STATE_LDS,
                spec_iters=vns.OPT_SPEC_ITERS, best_of=vns.OPT_BEST_OF)
    return {opt: int(case[k]) for k, opt in keys.items() if k in case}


def _training_rows(case, seed):
    """Rows with the scorer's features (move type, setups, demand and returns, costs, distances to the nearest
    setups) and a cost change that depends on them."""
    rng = np.random.default_rng([seed, 77])
    n = case["rows"]
    X = np.zeros((n, 16), np.float32)
    X[np.arange(n), rng.integers(0, 4, n)] = 1
    X[:, 4:6] = rng.random((n, 2)) < (0.4, 0.3)
    X[:, 6:10] = rng.integers(0, 201, (n, 4)) / 200
    X[:, 10:12] = rng.integers(200, 2001, (n, 2)) / 2000
    X[:, 12:14] = rng.integers(1, 7, (n, 2)) / 8
    X[:, 14:16] = rng.integers(0, 8, (n, 2)) / 52
    y = X @ rng.normal(0, 1, 16) + rng.normal(0, 0.5, n)
    return X, np.ascontiguousarray(y, np.float32)


def prepare(case, seed):
    rng = np.random.default_rng([seed, 1704])
    insts = _instances(case, rng)
    ctx = vns.Context(insts, seed=seed, chains=case["chains"], trace=bool(case.get("trace", False)),
                      nb_list=[int(b) for b in case.get("nb", "1,2,4").split(",")], options=_options(case))
    state = dict(case=case, ctx=ctx)
    if case["kind"] == "price":
        for g, (zM, zR) in enumerate(_patterns(case, insts[0], rng)):
            ctx.set_solution(g, zM, zR)
    elif case["kind"] == "sweep":
        ctx.run(5)   # solutions as a search holds them: local optima
    elif case["kind"] == "learned":
        ctx.set_option(vns.OPT_LEARNED, 100)
        ctx.mlp_init(seed)
        state["X"], state["y"] = _training_rows(case, seed)
    return state


def run(state):
    case, ctx = state["case"], state["ctx"]
    kind = case["kind"]
    if kind == "price":
        return ctx.eval_neighbourhood(7)
    if kind == "sweep":
        got = ctx.eval_neighbourhood(7, slot_prices=False, prod_best=case["products"])
        return {k: v for k, v in got.items() if v is not None}
    out = {}
    if kind == "learned":
        out["loss"] = ctx.mlp_train(state["X"], state["y"], epochs=1, batch=case["batch"], lr=2e-3, seed=11)
        out["weights"] = ctx.mlp_get()
        out["scores"] = ctx.mlp_score(state["X"])
    ctx.run(case["iters"])
    out["F"], out["F_best"] = ctx.costs()
    best = int(np.argmin(out["F_best"][:case["chains"]]))   # the first instance's best chain
    out["zM"], out["zR"] = ctx.solution(best, vns.SOLUTION_BEST)
    if case.get("trace"):
        rec = ctx.trajectory(best)
        out["records"] = {k: rec[k].copy() for k in rec.dtype.names}
    return out


def work(case):
    """Bytes: instances, solutions and outputs once.  Operations: a move's exact price takes at least the few
    dozen that its own setup interval and the next one need (30 here); three moves per period and product, and
    in a search about two passes over the moves of the three products an iteration shakes."""
    Ts = [int(t) for t in case["T"].split(",")]
    T = sum(Ts) / len(Ts)
    products = case["n_inst"] * (case["K"] + case["K_hi"]) / 2
    pairs, chains = products * case["chains"], case["n_inst"] * case["chains"]
    data = products * (8 * T + 32) + pairs * 40
    if case["kind"] == "price":
        return dict(bytes=data + pairs * (32 * T + 12) + chains * 12, flops=pairs * 3 * T * 30)
    if case["kind"] == "sweep":
        return dict(bytes=data + (pairs * 12 if case["products"] else 0) + chains * 12, flops=pairs * 3 * T * 30)
    flops = chains * case["iters"] * case.get("best_of", 1) * 3 * 2 * 3 * T * 30
    moved = data + pairs * 40
    if case["kind"] == "learned":   # forward and backward of 5184 multiply-adds a row, then forward again
        flops += case["rows"] * 10368 * 4
        moved += case["rows"] * 72 + 5313 * 4
    return dict(bytes=moved, flops=flops)


def _decode(T, D, R, c, zM, zR, strict, dispose):
    """Costs of patterns zM, zR [P, T] bool of products with D, R [P, T] and parameters c [P] each."""
    P = len(zM)
    PR = np.cumsum(R, 1)
    lim, XR, lsR, lastM, A1, A2 = (np.zeros(P, np.int64) for _ in range(6))
    open_ = np.ones(P, bool)      # no manufacturing lot may make this interval's demand
    bad = np.zeros(P, bool)
    xr_end, lot_at = np.zeros((P, T), np.int64), np.zeros((P, T), np.int64)
    for t in range(T):
        m, r = zM[:, t], zR[:, t]
        lim = np.where(m, XR, lim)
        lastM = np.where(m, t, lastM)
        open_ = ~m & (open_ | (r if strict else False))
        lim = np.where(r, PR[:, t], lim)
        lsR = np.where(r, t, lsR)
        xn = np.minimum(XR + D[:, t], lim)
        u = xn - XR
        XR = xn
        A1 += u * lsR
        A2 += (D[:, t] - u) * lastM
        bad |= open_ & (D[:, t] > u)
        xr_end[:, t], lot_at[:, t] = u, lsR
    n = np.arange(T)
    cost = (c["kM"] * zM.sum(1) + c["kR"] * zR.sum(1) + c["hM"] * ((D * n).sum(1) - A1 - A2) +
            c["hR"] * (PR.sum(1) - T * XR + A1) + c["pM"] * (D.sum(1) - XR) + c["pR"] * XR)
    if dispose:   # stock that no later lot needs: the least stock from a period on
        made = np.zeros((P, T), np.int64)
        np.add.at(made, (np.arange(P)[:, None], lot_at), xr_end)
        stock = PR - np.cumsum(made, 1)
        cost -= c["hR"] * np.minimum.accumulate(stock[:, ::-1], 1).sum(1)
    return np.where(bad, INF, cost)


def exact(case, seed):
    if case["kind"] == "learned":
        return _exact_learned(case, seed)
    if case["kind"] != "price":
        return None   # whole numbers that follow from a search
    rng = np.random.default_rng([seed, 1704])
    inst = _instances(case, rng)[0]
    K, T = inst.K, inst.T
    if K * T * T * case["chains"] * 4 > 3e8:
        return None
    pM, pR = inst.unit_costs()
    par = dict(kM=inst.kM, kR=inst.kR, hM=inst.hM, hR=inst.hR, pM=pM, pR=pR)

    def rep(a, n):
        return np.repeat(np.asarray(a, np.int64), n, 0)

    out = dict(slot_price=[], prod_best=[], prod_best_slot=[], best=[], best_slot=[])
    for zM, zR in _patterns(case, inst, rng):
        zM, zR = zM.astype(bool), zR.astype(bool)
        base = _decode(T, rep(inst.D, 1), rep(inst.R, 1), {k: rep(v, 1) for k, v in par.items()}, zM, zR, inst.strict,
                       inst.dispose)
        mm, mr = np.repeat(zM[:, None], 4 * T, 1), np.repeat(zR[:, None], 4 * T, 1)
        valid = np.ones((K, 4 * T), bool)
        t = np.arange(T)
        mm[:, t, t] ^= True
        mr[:, T + t, t] ^= True
        for z, block in ((mm, 2), (mr, 3)):
            for s in range(T - 1):
                l = block * T + s
                valid[:, l] = z[:, l, s] != z[:, l, s + 1]
                z[:, l, [s, s + 1]] = z[:, l, [s + 1, s]]
            valid[:, block * T + T - 1] = False
        c = _decode(T, rep(inst.D, 4 * T), rep(inst.R, 4 * T), {k: rep(v, 4 * T) for k, v in par.items()},
                    mm.reshape(-1, T), mr.reshape(-1, T), inst.strict, inst.dispose).reshape(K, 4 * T)
        price = np.where(valid & (c != INF), base.sum() - base[:, None] + np.where(c == INF, 0, c), INF)
        slot = price.argmin(1)
        low = price[np.arange(K), slot]
        out["slot_price"].append(price.reshape(-1))
        out["prod_best"].append(low)
        out["prod_best_slot"].append(np.where(low == INF, -1, slot).astype(np.int32))
        out["best"].append(np.array([price.min()]))
        out["best_slot"].append(np.array([price.reshape(-1).argmin() if price.min() != INF else -1], np.int32))
    return {k: np.concatenate(v) for k, v in out.items()}


def _exact_learned(case, seed):
    """The scorer's epoch (Adam over minibatches in the documented row order) and scores in float64."""
    u64 = (1 << 64) - 1

    def uniform(i):
        z = (seed + (i + 1) * 0x9E3779B97F4A7C15) & u64
        z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & u64
        z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & u64
        return ((z ^ (z >> 31)) >> 11) * 2.0 ** -53

    p = np.zeros(vns.MLP_PARAMS)
    cut = dict(W1=(0, 16, 64), W2=(1088, 64, 64), W3=(5248, 64, 1))
    for off, fan, wide in cut.values():
        for j in range(fan * wide):
            p[off + j] = np.sqrt(6.0 / fan) * (2 * uniform(off + j) - 1)
    X, y = _training_rows(case, seed)
    X, y = X.astype(np.float64), y.astype(np.float64)

    def layers(x):
        W1, W2, W3 = (p[o:o + a * b].reshape(a, b) for o, a, b in cut.values())
        z1 = x @ W1 + p[1024:1088]
        h1 = np.maximum(z1, 0)
        z2 = h1 @ W2 + p[5184:5248]
        h2 = np.maximum(z2, 0)
        return W2, W3, z1, h1, z2, h2, (h2 @ W3)[:, 0] + p[5312]

    n, batch = len(X), min(case["batch"], len(X))
    mul = 1000003
    while np.gcd(mul, n) != 1:
        mul += 2
    s = (11 * 0x9E3779B97F4A7C15 + 1) & u64
    s ^= s >> 33
    s = (s * 0xFF51AFD7ED558CCD) & u64
    s ^= s >> 33
    order = (mul * np.arange(n, dtype=object) + s % n) % n
    order = order.astype(np.int64)
    m, v, loss = np.zeros_like(p), np.zeros_like(p), 0.0
    for step, at in enumerate(range(0, n, batch), 1):
        rows = order[at:at + batch]
        W2, W3, z1, h1, z2, h2, score = layers(X[rows])
        e = score - y[rows]
        loss = float((e * e).mean())
        ds = 2 * e / len(rows)
        d2 = (z2 > 0) * ds[:, None] * W3[:, 0]
        d1 = (z1 > 0) * (d2 @ W2.T)
        g = np.concatenate([(X[rows].T @ d1).ravel(), d1.sum(0), (h1.T @ d2).ravel(), d2.sum(0), h2.T @ ds, [ds.sum()]])
        m = 0.9 * m + 0.1 * g
        v = 0.999 * v + 0.001 * g * g
        p = p - 2e-3 * (m / (1 - 0.9 ** step)) / (np.sqrt(v / (1 - 0.999 ** step)) + 1e-8)
    return dict(loss=loss, weights=p.copy(), scores=layers(X)[-1], F=None, F_best=None, zM=None, zR=None)
