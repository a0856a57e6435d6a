"""The work that a user of this library has it do, as timed cases.

A memetic run (Algorithm 1) is a sequence of generations; these cases are its
parts, each through the public entry points a program calls: the population
searches (k-COL and weighted), the uneven batch, the steps that make and keep
a generation, the diversity steps, and the two offspring scorers with their
products.  ``draw`` gives more cases of the same ranges.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2109_05948_amd as dlm

MLP = (256, 128, 64)  # widths of the per-class scorer
KINDS = ("diversity", "learn", "multi", "net_learn", "net_score", "product", "reproduce", "score", "tabu", "wvcp")


def listed():
    return [
        # the smallest search: a few dozen individuals of a small graph at a number of colours it does not
        # reach; latency per move decides, most of the card idles
        {"name": "tabu_100", "kind": "tabu", "n": 100, "p": 0.5, "k": 15, "pop": 64, "iters": 5000},
        # the benchmark's population on the shape of DSJC500.5, with a shorter budget
        {"name": "tabu_500", "kind": "tabu", "n": 500, "p": 0.5, "k": 49, "pop": 8192, "iters": 16000},
        # the local search of the memetic loop on the shape of DSJC1000.5 (99 % of a generation's time)
        {"name": "tabu_1000", "kind": "tabu", "n": 1000, "p": 0.5, "k": 85, "pop": 2048, "iters": 8000},
        # an uneven batch: graphs of many sizes and densities, one persistent launch
        {"name": "uneven_12", "kind": "multi", "graphs": 12, "nmin": 100, "nmax": 1000, "pop": 64, "rate": 16},
        # the weighted search on the shape of the weighted G(300, 0.3), ten rounds
        {"name": "wvcp_300", "kind": "wvcp", "n": 300, "p": 0.3, "pop": 4096, "iters": 300, "rounds": 10},
        # a generation around the search: pairs, crossover, selection, gather, population update
        {"name": "reproduce_1000", "kind": "reproduce", "n": 1000, "k": 85, "pop": 8192, "per_pair": 4},
        # the offspring of one generation scored by the per-class network
        {"name": "score_1000", "kind": "score", "n": 1000, "k": 85, "count": 32768},
        # one training batch of the per-class network
        {"name": "learn_1000", "kind": "learn", "n": 1000, "k": 85, "count": 1024},
        # one generation's diversity steps: new distances, spacing update, gathers, nearest neighbours
        {"name": "diversity_500", "kind": "diversity", "n": 500, "k": 49, "pop": 4096, "near": 16},
        # the paper's network scoring offspring, k-COL depth for 500 vertices
        {"name": "net_score_500", "kind": "net_score", "n": 500, "k": 49, "count": 2048, "depth": "col"},
        # the same network, one training batch of the paper's size
        {"name": "net_learn_500", "kind": "net_learn", "n": 500, "k": 49, "count": 100, "depth": "col"},
        # one of its products alone: the weight gradient X^T dZ of a 2500 -> 1000 layer over 100 colourings
        {"name": "product_wgrad", "kind": "product", "m": 2500, "n": 1000, "k": 4900, "akc": False, "bkc": False},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _colours(n, p):
    """About the number of colours a good search reaches on G(n, p)."""
    b = -math.log1p(-p)
    ln = math.log(n) / b
    return max(2, int(round(n / max(1.0, 2 * ln - 2 * math.log(max(ln, 1.001)) / b - 1))))


def draw(rng):
    kind = rng.choice(["tabu", "tabu", "tabu", "multi", "wvcp", "wvcp", "reproduce", "score", "learn", "diversity",
                       "net_score", "net_learn", "product"])
    if kind == "tabu":
        n, p = _log(rng, 60, 1000), round(rng.uniform(0.1, 0.9), 2)
        k = max(2, _colours(n, p) + rng.randint(0, 3))
        # a longer row or a larger graph costs more a move; tables past 2^17 entries leave the wave's tier
        top = 60e6 if n <= 500 else 12e6
        if n * ((k + 3) & ~3) > (1 << 17):
            top = 3e6
        iters = _log(rng, 500, 16000)
        return {"kind": kind, "n": n, "p": p, "k": k, "pop": _log(rng, 1, max(1, min(8192, int(top / iters)))),
                "iters": iters}
    if kind == "multi":
        nmin = _log(rng, 60, 400)
        return {"kind": kind, "graphs": rng.randint(2, 12), "nmin": nmin, "nmax": rng.randint(nmin, 1000),
                "pop": _log(rng, 4, 64), "rate": rng.randint(4, 16)}
    if kind == "wvcp":
        n, p = _log(rng, 60, 500), round(rng.uniform(0.1, 0.7), 2)
        if 1.6 * _colours(n, p) * n * 2 > 100000:
            p = 0.3
        iters, rounds = rng.randint(50, 300), rng.randint(2, 10)
        return {"kind": kind, "n": n, "p": p, "pop": _log(rng, 8, max(8, min(4096, int(6e6 * (300 / n) ** 2 / (iters * rounds))))),
                "iters": iters, "rounds": rounds}
    if kind in ("reproduce", "score"):
        n = _log(rng, 60, 1000)
        k = max(2, _colours(n, rng.uniform(0.1, 0.6)))
        if kind == "score":
            return {"kind": kind, "n": n, "k": k, "count": _log(rng, 16, 32768)}
        return {"kind": kind, "n": n, "k": k, "pop": _log(rng, 16, 8192), "per_pair": rng.choice([2, 4])}
    if kind == "learn":
        n = _log(rng, 60, 1000)
        return {"kind": kind, "n": n, "k": max(2, _colours(n, rng.uniform(0.1, 0.6))), "count": _log(rng, 32, 1024)}
    if kind == "diversity":
        n = _log(rng, 60, 1000)
        k = max(2, min(120, _colours(n, rng.uniform(0.1, 0.6))))
        return {"kind": kind, "n": n, "k": k, "pop": _log(rng, 64, 4096 if n <= 500 else 2048), "near": rng.choice([8, 16, 32])}
    if kind in ("net_score", "net_learn"):
        n = rng.randint(60, 500)
        k = max(2, min(49, _colours(n, rng.uniform(0.2, 0.5))))
        count = _log(rng, 16, 2048) if kind == "net_score" else rng.randint(16, 100)
        return {"kind": kind, "n": n, "k": k, "count": count, "depth": rng.choice(["col", "wvcp"])}
    # a layer's forward product (both operands along K), its weight gradient (neither) or its input gradient
    akc, bkc = rng.choice([(True, True), (False, False), (True, True)])
    return {"kind": kind, "m": _log(rng, 100, 5000), "n": _log(rng, 100, 2500), "k": _log(rng, 250, 5000), "akc": akc, "bkc": bkc}


# ---------------------------------------------------------------- inputs, from the seed alone
def _rng(case, seed):
    return np.random.default_rng([seed, KINDS.index(case["kind"])])


def _gnp(rng, n, p, parts=None):
    """Symmetric CSR of G(n, p); with ``parts`` only pairs of different parts are joined."""
    a = np.triu(rng.random((n, n), dtype=np.float32) < p, 1)
    if parts is not None:
        a &= parts[:, None] != parts[None, :]
    a |= a.T
    ptr = np.zeros(n + 1, np.int32)
    np.cumsum(a.sum(1), out=ptr[1:])
    return ptr, np.nonzero(a)[1].astype(np.int32)


def _start(rng, pop, n, k):
    return torch.from_numpy(rng.integers(0, k, (pop, n)).astype(np.int16)).cuda()


def _relatives(rng, pop, n, k):
    """Colourings as a searched population has them: families of near relatives."""
    roots = rng.integers(0, k, (max(1, pop // 32), n))
    out = roots[rng.integers(0, roots.shape[0], pop)]
    other = rng.random((pop, n)) < rng.uniform(0.02, 0.5, (pop, 1))
    out[other] = rng.integers(0, k, int(other.sum()))
    return out.astype(np.int16)


def _mlp_weights(rng, n):
    out = {}
    for i, (a, b) in enumerate(((n, MLP[0]), (MLP[0], MLP[1]), (MLP[1], MLP[2]), (MLP[2], 1)), 1):
        s = 1.0 / math.sqrt(a)
        out[("W%d" if i < 4 else "w%d") % i] = rng.uniform(-s, s, (a, b) if i < 4 else (a,)).astype(np.float32)
        out["b%d" % i] = rng.uniform(-s, s, (b,)).astype(np.float32)
    return out


def _net_widths(case):
    n = case["n"]
    return [10 * n, 5 * n] + [2 * n] * 5 + [n, n // 2, 1] if case["depth"] == "col" else [5 * n, 2 * n, n, n // 2, 1]


def _net_weights(rng, n, k, widths):
    """Fresh weights, with the running estimates that a normalised network has on random colourings."""
    out, a = {}, n
    mean, var = 1.0 / k, (1.0 / k) / 3
    for j, b in enumerate(widths):
        s = np.float32(1.0 / math.sqrt(a))
        for nm, shape in (("L", (a, b)), ("G", (a, b)), ("b", (b,))):
            out[f"{nm}{j}"] = (rng.random(shape, dtype=np.float32) * 2 - 1) * s
        if j < len(widths) - 1:
            out[f"g{j}"] = rng.uniform(0.8, 1.2, b).astype(np.float32)
            out[f"m{j}"] = rng.uniform(-0.2, 0.2, b).astype(np.float32)
            drift = out[f"L{j}"].sum(0, dtype=np.float64) + out[f"G{j}"].sum(0, dtype=np.float64)
            out[f"rm{j}"] = (mean * drift + out[f"b{j}"]).astype(np.float32)
            out[f"rv{j}"] = np.full(b, var, np.float32)
            mean, var = 0.32, 0.14  # of a leaky rectifier on unit normal values, through weights of variance 1/3
        a = b
    return out


def _bf16(rng, rows, cols):
    return torch.from_numpy(rng.standard_normal((rows, cols), dtype=np.float32)).cuda().bfloat16()


def _product_inputs(case, seed):
    rng = _rng(case, seed)
    m, n, k = case["m"], case["n"], case["k"]
    return (_bf16(rng, *((m, k) if case["akc"] else (k, m))), _bf16(rng, *((n, k) if case["bkc"] else (k, n))))


def _learn_inputs(case, seed):
    """Weights, colourings and standardised targets of a scorer."""
    rng = _rng(case, seed)
    n, k, count = case["n"], case["k"], case["count"]
    if case["kind"].startswith("net"):
        w = _net_weights(rng, n, k, _net_widths(case))
    else:
        w = _mlp_weights(rng, n)
    cols = torch.from_numpy(_relatives(rng, count, n, k)).cuda()
    return w, cols, torch.from_numpy(rng.standard_normal(count, dtype=np.float32)).cuda()


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("score", "learn"):
        w, cols, tgt = _learn_inputs(case, seed)
        s = dlm.Scorer(case["n"], case["k"], w, max_batch=case["count"] if kind == "learn" else 1024, widths=MLP)
        return {"case": case, "scorer": s, "cols": cols, "targets": tgt}
    if kind in ("net_score", "net_learn"):
        w, cols, tgt = _learn_inputs(case, seed)
        s = dlm.InvNet(case["n"], case["k"], _net_widths(case), w, max_batch=min(case["count"], 1024))
        return {"case": case, "scorer": s, "cols": cols, "targets": tgt}
    if kind == "product":
        a, b = _product_inputs(case, seed)
        return {"case": case, "a": a, "b": b,
                "ws": torch.empty(8 * case["m"] * case["n"], dtype=torch.float32, device="cuda")}
    rng = _rng(case, seed)
    st = {"case": case, "seed": int(rng.integers(1 << 40))}
    if kind == "tabu":
        st["graph"] = dlm.Graph(case["n"], *_gnp(rng, case["n"], case["p"]))
        st["start"] = _start(rng, case["pop"], case["n"], case["k"])
    elif kind == "wvcp":
        n, pop = case["n"], case["pop"]
        ptr, col = _gnp(rng, n, case["p"])
        st["graph"] = dlm.Graph(n, ptr, col, rng.integers(1, 101, n).astype(np.int32))
        st["start"], used = dlm.init_population(st["graph"], 0, pop, seed=st["seed"], mode="greedy")
        st["k"] = int(used.max().item())
    elif kind == "multi":
        jobs = []
        sizes = np.random.default_rng(case["graphs"])  # the shapes are the case's, the edges the seed's
        for i in range(case["graphs"]):
            n = int(sizes.integers(case["nmin"], case["nmax"] + 1))
            p, hidden = float(sizes.uniform(0.1, 0.9)), int(sizes.integers(5, 61))
            if i % 2:  # a hidden colouring
                k, csr = hidden, _gnp(rng, n, 0.5, rng.integers(0, hidden, n))
            else:
                k, csr = _colours(n, p), _gnp(rng, n, p)
            jobs.append({"graph": dlm.Graph(n, *csr), "k": k, "iters": case["rate"] * n, "seed": st["seed"] + i,
                         "colors": torch.empty((case["pop"], n), dtype=torch.int16, device="cuda")})
            jobs[-1]["start"] = _start(rng, case["pop"], n, k)
        st["plan"] = dlm.MultiBatch(jobs)
    elif kind == "reproduce":
        n, k, pop = case["n"], case["k"], case["pop"]
        st["graph"] = dlm.Graph(n, *_gnp(rng, n, 0.5))
        st["cols"] = torch.from_numpy(_relatives(rng, pop, n, k)).cuda()
        st["scores"] = torch.from_numpy(rng.standard_normal(pop * case["per_pair"], dtype=np.float32)).cuda()
        st["f"], st["f_off"] = (torch.from_numpy(rng.integers(0, 80, pop).astype(np.int32)).cuda() for _ in range(2))
    else:  # diversity
        n, k, pop = case["n"], case["k"], case["pop"]
        both = torch.from_numpy(_relatives(rng, 2 * pop, n, k)).cuda()
        st["cols"], st["off"] = both[:pop].clone(), both[pop:].clone()
        st["f"], st["f_off"] = (torch.from_numpy(rng.integers(0, 80, pop).astype(np.int32)).cuda() for _ in range(2))
        st["pool"], st["next"] = (torch.zeros((2 * pop, 2 * pop), dtype=torch.int32, device="cuda") for _ in range(2))
        dlm.partition_distance(st["cols"], k, out=st["pool"][:pop, :pop])
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "tabu":
        o = dlm.tabu_batch(st["graph"], st["start"].clone(), case["k"], case["iters"], st["seed"])
        return {x: o[x] for x in ("colors", "f_best", "iters", "stats", "hash")}
    if kind == "wvcp":
        o = dlm.wvcp_batch(st["graph"], st["start"].clone(), st["k"], case["iters"], case["rounds"], st["seed"])
        return {x: o[x] for x in ("colors", "best_legal", "stats", "hash")}
    if kind == "multi":
        plan = st["plan"]
        for j in plan.jobs:
            j["colors"].copy_(j["start"])
        plan.launch()
        return [[j[x] for x in ("colors", "f_best", "iters_out", "stats", "hash")] for j in plan.jobs]
    if kind == "reproduce":
        pop, per = case["pop"], case["per_pair"]
        pairs = dlm.random_pairs(pop, st["seed"], 1)
        children = dlm.gpx_batch(st["graph"], case["k"], st["cols"], pairs, per, st["seed"], child_base=pop * per)
        idx = dlm.select(st["scores"], pop * per, pop, "top")
        off = dlm.gather_rows(children, idx)
        cols, f = dlm.pop_update(st["cols"], st["f"], off, st["f_off"])
        return {"children": children, "idx": idx, "off": off, "cols": cols, "f": f}
    if kind in ("score", "net_score"):
        return st["scorer"].score(st["cols"])
    if kind in ("learn", "net_learn"):
        return st["scorer"].grad(st["cols"], st["targets"])
    if kind == "product":
        return dlm.gemm_bf16(st["a"], st["b"], case["m"], case["n"], case["k"], case["akc"], case["bkc"], workspace=st["ws"])
    pop, k, pool, nxt = case["pop"], case["k"], st["pool"], st["next"]
    dlm.partition_distance(st["cols"], k, st["off"], out=pool[:pop, pop:])
    dlm.partition_distance(st["off"], k, out=pool[pop:, pop:], upper_only=True)
    pick, spaced = dlm.spacing_update(st["f"], st["f_off"], pool, pop, case["n"] // 10)
    dlm.gather_distances(pool, pick, out=nxt[:pop, :pop])
    cols, f = dlm.gather_pool(st["cols"], st["f"], st["off"], st["f_off"], pick)
    near = dlm.nearest(nxt, case["near"], p=pop)
    return {"dist": nxt[:pop, :pop], "pick": pick, "spaced": spaced, "cols": cols, "f": f, "near": near}


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    kind = case["kind"]
    if kind == "tabu":
        n, k, pop, iters = case["n"], case["k"], case["pop"], case["iters"]
        deg = case["p"] * (n - 1)
        # candidates of about a twelfth of the vertices, two table updates per neighbour of the moved vertex
        return {"bytes": 4 * pop * n + 4 * n * deg + 80 * pop, "flops": pop * iters * (5.0 * n / 12 * k + 4 * deg)}
    if kind == "wvcp":
        n, pop, it = case["n"], case["pop"], case["iters"] * case["rounds"]
        deg, k = case["p"] * (n - 1), _colours(n, case["p"])
        # what a move changes: its neighbours' two table entries, and two candidates of every vertex
        return {"bytes": 4 * pop * n + 4 * n * deg + 80 * pop, "flops": pop * it * (4 * deg + 8.0 * n + 5.0 * deg / k * k)}
    if kind == "multi":
        n = 0.5 * (case["nmin"] + case["nmax"])
        moves = case["graphs"] * case["pop"] * case["rate"] * n
        return {"bytes": case["graphs"] * (4 * case["pop"] * n + 2 * n * n), "flops": moves * (5.0 * n / 12 * 0.1 * n + 2 * n)}
    if kind == "reproduce":
        n, k, pop, per = case["n"], case["k"], case["pop"], case["per_pair"]
        return {"bytes": 2 * n * (pop * 2 + pop * per * 2 + pop * 2), "flops": float(pop) * per * (3 * n + k * k)}
    if kind in ("score", "learn"):
        n, k, c = case["n"], case["k"], case["count"]
        rows = 2.0 * k * MLP[0] * MLP[1] + 2 * MLP[1] * MLP[2] + n * MLP[0]
        weights = 4 * (n * MLP[0] + MLP[0] * MLP[1] + MLP[1] * MLP[2])
        t = kind == "learn"
        return {"bytes": 2 * n * c + weights * (2 if t else 1), "flops": c * rows * (3 if t else 1)}
    if kind == "diversity":
        n, k, pop = case["n"], case["k"], case["pop"]
        pairs = 1.5 * pop * pop
        return {"bytes": 4 * pairs + 8 * pop * pop + 8 * pop * n, "flops": pairs * (n + 2.0 * k * k)}
    if kind in ("net_score", "net_learn"):
        a, prod, par = case["n"], 0, 0
        for j, b in enumerate(_net_widths(case)):
            prod += 2.0 * case["count"] * (case["k"] + 1) * a * b * (1 if kind == "net_score" else 3 if j else 2)
            par += 2 * a * b
            a = b
        return {"bytes": 2 * case["n"] * case["count"] + par * (2 if kind == "net_score" else 6), "flops": prod}
    m, n, k = case["m"], case["n"], case["k"]
    return {"bytes": 2 * (m * k + n * k) + 4 * m * n, "flops": 2.0 * m * n * k}


# ---------------------------------------------------------------- the same in 64 bits
def _lrelu(x):
    return torch.where(x > 0, x, 0.2 * x)


def _one_hot(cols, k):
    """[count][k][n] class indicators in 64 bits."""
    return (cols[:, None, :] == torch.arange(k, device=cols.device, dtype=cols.dtype)[None, :, None]).double()


def _mlp(w, x):
    z = _lrelu(_lrelu(x @ w["W1"] + w["b1"]) @ w["W2"] + w["b2"]).sum(1)
    return _lrelu(z @ w["W3"] + w["b3"]) @ w["w4"] + w["b4"]


def _net(w, x, last, batch_stats):
    for j in range(last + 1):
        z = x @ w[f"L{j}"] + (x.mean(1) @ w[f"G{j}"])[:, None, :] + w[f"b{j}"]
        if j == last:
            return z[..., 0].mean(1)
        if batch_stats:
            mu, var = z.mean((0, 1)), z.var((0, 1), unbiased=False)
        else:
            mu, var = w[f"rm{j}"], w[f"rv{j}"]
        x = _lrelu((z - mu) / torch.sqrt(var + 1e-5) * w[f"g{j}"] + w[f"m{j}"])


def exact(case, seed):
    kind = case["kind"]
    if kind == "product":
        a, b = (t.double() for t in _product_inputs(case, seed))
        return (a if case["akc"] else a.T) @ (b.T if case["bkc"] else b)
    if kind not in ("score", "learn", "net_score", "net_learn"):
        return None  # whole numbers
    w, cols, tgt = _learn_inputs(case, seed)
    w = {x: torch.from_numpy(v).cuda().double() for x, v in w.items()}
    net, last = kind.startswith("net"), len(_net_widths(case)) - 1 if kind.startswith("net") else 0
    if kind.endswith("score"):
        f = (lambda x: _net(w, x, last, False)) if net else (lambda x: _mlp(w, x))
        return torch.cat([f(_one_hot(c, case["k"])) for c in cols.split(256)])
    if net:
        names = [f"{x}{j}" for j in range(last + 1) for x in ("LGbgm" if j < last else "LGb")]
    else:
        names = ["W1", "b1", "W2", "b2", "W3", "b3", "w4", "b4"]
    for x in names:
        w[x].requires_grad_(True)
    if net:
        loss = ((_net(w, _one_hot(cols, case["k"]), last, True) - tgt.double()) ** 2).mean()
        loss.backward()
        total = loss.detach().reshape(1)
    else:
        total = torch.zeros(1, dtype=torch.float64, device="cuda")
        for c, t in zip(cols.split(128), tgt.double().split(128)):
            loss = ((_mlp(w, _one_hot(c, case["k"])) - t) ** 2).sum() / case["count"]
            loss.backward()
            total += loss.detach()
    return torch.cat([w[x].grad.reshape(-1) for x in names]), total
