"""Performance cases of the Ant System library: what a user has it do.

Four kinds of case, each through the public entry points:

* ``solve``      one instance from its distance matrix to its best tour: a
                 ``Colony`` is built, runs ``iters`` iterations of one of the
                 three construction rules with one of the update variants, and
                 the best tour, its length and the final pheromone are read
                 (what a program that keeps or checkpoints its result does);
* ``construct``  one construction of a colony in mid-search, with every
                 ant's tour read back (a program with a local search of its
                 own between construction and update);
* ``resume``     a checkpoint restored into a colony that then runs on;
* ``batch``      many uneven instances advanced together by one ``Batch``;
* ``served``     requests through the continuous-batching ``Server``.

Sizes are those of the repository's workloads (n = m = 100, 1000, 2400; 50 to
1000 cities in a batch with 25 iterations; 100 to 3000 cities served with 50
iterations), with ragged ones beside them.
"""
from __future__ import annotations

import numpy as np
import torch

import tsp_inputs
from paper_1101_2678_amd.aco import Batch, Colony
from paper_1101_2678_amd.serve import Request, Server

SIDE = 1_000_000


# --------------------------------------------------------------------- cases
def _solve(n, iters, m=None, rule="r64", update="gather", layout="uniform", alpha=1, beta=2,
           rho=0.5, nn=30, side=SIDE):
    return {"kind": "solve", "n": n, "m": n if m is None else m, "iters": iters, "rule": rule,
            "update": update, "layout": layout, "alpha": alpha, "beta": beta, "rho": rho,
            "nn": nn, "side": side}


def _construct(n, m=None, rule="r64", layout="uniform", at=5, nn=30):
    return {"kind": "construct", "n": n, "m": n if m is None else m, "rule": rule,
            "layout": layout, "at": at, "nn": nn, "alpha": 1, "beta": 2, "rho": 0.5,
            "side": SIDE}


def _resume(n, iters, m=None, at=10, layout="uniform", update="gather"):
    return {"kind": "resume", "n": n, "m": n if m is None else m, "iters": iters, "at": at,
            "layout": layout, "update": update, "alpha": 1, "beta": 2, "rho": 0.5, "side": SIDE}


def _many(kind, count, lo, hi, iters, sizes_seed):
    return {"kind": kind, "count": count, "n_lo": lo, "n_hi": hi, "iters": iters,
            "sizes_seed": sizes_seed}


def listed():
    cases = [
        # the smallest instance of the paper's range and its iteration count:
        # launches and latency
        ("solve n100", _solve(100, 10, side=10_000)),
        # a ragged size with more ants than cities, other exponents and the
        # direct atomic update
        ("solve n333 ragged", _solve(333, 15, m=500, update="atomic_direct", alpha=2, beta=3,
                                     rho=0.3)),
        # the middle of the range, both layouts, gather and shared-memory
        # atomic updates
        ("solve n1000", _solve(1000, 20)),
        ("solve n1000 cluster", _solve(1000, 20, update="atomic", layout="cluster")),
        # the paper's largest instance
        ("solve n2400", _solve(2400, 20)),
        # its two other construction rules at the same size
        ("nn n2400", _solve(2400, 20, rule="nn")),
        ("product n2400", _solve(2400, 20, rule="product")),
        # the largest size that is served, with a served request's iterations
        ("solve n3000 cluster", _solve(3000, 50, layout="cluster")),
        # one construction in mid-search with its tours read, odd size
        ("construct n1511", _construct(1511)),
        # a checkpoint restored and continued
        ("resume n500", _resume(500, 10)),
        # many uneven instances in one batch
        ("batch 64", _many("batch", 64, 50, 1000, 25, 7)),
        # requests through the server
        ("served 10", _many("served", 10, 100, 3000, 50, 5)),
    ]
    return [dict(c, name=name) for name, c in cases]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["solve"] * 5 + ["construct", "resume", "batch", "served"])
    layout = rng.choice(["uniform", "cluster"])
    if kind == "solve":
        rule = rng.choice(["r64", "r64", "r64", "nn", "product"])
        n = _log_int(rng, 50, 2400 if rule == "product" else 3000)
        m = n if rng.random() < 0.5 else rng.randint(max(2, n // 2), n)
        return _solve(n, rng.randint(5, 50 if rule != "product" else 40), m=m, rule=rule,
                      update=rng.choice(["gather", "gather", "atomic", "atomic_direct"]),
                      layout=layout, alpha=rng.choice([1, 1, 1, 2]),
                      beta=rng.choice([2, 2, 3, 4]), rho=rng.choice([0.1, 0.3, 0.5, 0.5, 0.7]),
                      nn=rng.choice([15, 20, 30, 40]))
    if kind == "construct":
        return _construct(_log_int(rng, 50, 3000), rule=rng.choice(["r64", "r64", "nn", "product"]),
                          layout=layout, at=rng.randint(0, 20), nn=rng.choice([15, 30, 40]))
    if kind == "resume":
        return _resume(_log_int(rng, 50, 2000), rng.randint(5, 20), at=rng.randint(1, 15),
                       layout=layout, update=rng.choice(["gather", "atomic"]))
    if kind == "batch":
        return _many("batch", rng.randint(8, 64), 50, _log_int(rng, 200, 1000),
                     rng.randint(5, 25), rng.randint(0, 999))
    return _many("served", rng.randint(4, 8), 100, _log_int(rng, 400, 2400), rng.randint(10, 50),
                 rng.randint(0, 999))


def _sizes(case):
    return [int(x) for x in tsp_inputs.log_uniform_sizes(case["count"], case["n_lo"],
                                                          case["n_hi"], case["sizes_seed"])]


# ------------------------------------------------------------------- prepare
def _dist(n, layout, side, seed):
    return tsp_inputs.instance(n, layout, side=side, seed=seed)[1]


def _colony(case, dist, seed):
    return Colony(dist, case["m"], case["alpha"], case["beta"], case["rho"], seed=seed,
                  atomic=case.get("update", "gather") != "gather")


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("batch", "served"):
        dists = [_dist(n, "uniform" if q % 2 else "cluster", SIDE, 1000 * seed + q)
                 for q, n in enumerate(_sizes(case))]
        state = {"case": case, "seed": seed, "dists": dists}
        if kind == "served":
            state["server"] = Server(pool_bytes=2 << 30)
        return state
    dist = _dist(case["n"], case["layout"], case["side"], seed)
    state = {"case": case, "seed": seed, "dist": dist}
    if kind == "construct":  # a colony after `at` iterations
        col = _colony(case, dist, seed)
        if case["rule"] == "nn":
            col.attach_nn(case["nn"])
        col.solve(case["at"], "gather", "nn" if case["rule"] == "nn" else "r64")
        state["colony"] = col
    elif kind == "resume":  # a checkpoint after `at` iterations, and a colony to take it
        col = _colony(case, dist, seed)
        tour, length = col.solve(case["at"], case["update"])
        state["checkpoint"] = (col.tau(), col.iteration, length, tour)
        state["colony"] = col
    return state


# ----------------------------------------------------------------------- run
def _read(col, tour, length):
    return {"tour": tour, "length": length, "tau": col.tau()}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "solve":
        col = _colony(case, state["dist"], state["seed"])
        if case["rule"] == "nn":
            col.attach_nn(case["nn"])
        return _read(col, *col.solve(case["iters"], case["update"], case["rule"]))
    if kind == "construct":
        col = state["colony"]
        {"r64": col.construct, "nn": col.construct_nn,
         "product": col.construct_product}[case["rule"]](case["at"])
        tours, lens = col.tours()
        return {"tours": tours, "lens": lens}
    if kind == "resume":
        col = state["colony"]
        col.restore(*state["checkpoint"])
        return _read(col, *col.solve(case["iters"], case["update"]))
    if kind == "batch":
        batch = Batch(state["dists"], [dict(m=d.shape[0], seed=state["seed"] + q)
                                       for q, d in enumerate(state["dists"])])
        batch.run(case["iters"])
        best = [batch.best(q) for q in range(batch.count)]
    else:
        best = _serve(state["server"], [
            Request(rid=q, arrival=0.0, dist=d, m=d.shape[0], iters=case["iters"],
                    seed=state["seed"] + q) for q, d in enumerate(state["dists"])])
    return {"tours": np.concatenate([t for t, _ in best]), "lens": np.array([x for _, x in best])}


def _serve(server, requests):
    """Every request submitted as soon as the server takes it, its result read
    and its slot released when it is done."""
    waiting, by_slot, best = list(requests), {}, {}
    while len(best) < len(requests):
        while waiting:
            slot = server.submit(waiting[0])
            if slot is None:
                break
            by_slot[slot] = waiting.pop(0)
        server.step()
        for slot, rid in server.collect():
            best[rid] = server.result(slot, by_slot.pop(slot).n)
            server.release(slot)
    return [best[q] for q in range(len(requests))]


# ---------------------------------------------------------------------- work
def work(case):
    """Bytes: each input matrix read once, each output written once.  Flops:
    one addition (product rule: one multiplication and one comparison) per
    unvisited city of every selection, n / 2 of them on average; the candidate
    rule needs at most its list."""
    kind = case["kind"]
    if kind in ("batch", "served"):
        ns = _sizes(case)
        return {"bytes": sum(4 * n * n + 2 * (n + 1) for n in ns),
                "flops": case["iters"] * sum(n * n * n / 2 for n in ns)}
    n, m = case["n"], case["m"]
    steps = m * (n - 1) * case.get("iters", 1)
    per = {"nn": min(case.get("nn", 0), n / 2), "product": n}.get(case.get("rule"), n / 2)
    if kind == "construct":
        return {"bytes": 4 * n * n + 2 * m * (n + 1) + 8 * m, "flops": steps * per}
    return {"bytes": 8 * n * n + 2 * (n + 1), "flops": steps * per}


# --------------------------------------------------------------------- exact
# The pheromone after a solve in 64 bits.  Which edges receive deposits
# depends on the selections, whose definition fixes every binary32 operation;
# the tours are therefore drawn by that definition (in plain torch, all ants
# of a step at once), and the pheromone they give is accumulated in binary64.
_MASK = 0xFFFFFFFF


def _philox(seed, c0, c1, c2, c3):
    """The four words of Philox4x32-10 (int64 tensors holding 32-bit words)."""
    k0, k1 = seed & _MASK, seed >> 32
    for _ in range(10):
        a, b = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = (((b >> 32) & _MASK) ^ c1 ^ k0, b & _MASK,
                          ((a >> 32) & _MASK) ^ c3 ^ k1, a & _MASK)
        k0, k1 = (k0 + 0x9E3779B9) & _MASK, (k1 + 0xBB67AE85) & _MASK
    return c0, c1, c2, c3


def _s64(x):
    """The 64-wide binary32 prefix tree of the roulette, on the last axis."""
    x = x.unflatten(-1, (4, 16))
    for s in (1, 2, 4, 8):
        x = x + torch.nn.functional.pad(x[..., :-s], (s, 0))
    r0, r1, r2 = x[..., 0, 15:], x[..., 1, 15:], x[..., 2, 15:]
    y = r1 + r0
    return torch.cat([x[..., 0, :], x[..., 1, :] + r0, x[..., 2, :] + y, (x[..., 3, :] + r2) + y],
                     dim=-1)


def _roulette(w, live, u):
    """One selection per row of w (rows x 64 blocks; weights of the rest +0)."""
    s = _s64(w.unflatten(-1, (-1, 64)))
    blocks = s.shape[-2]
    t = torch.nn.functional.pad(s[..., 63], (0, 64 - blocks))
    i = _s64(t)[:, :blocks]
    prefix = (torch.nn.functional.pad(i[:, :-1], (1, 0))[..., None] + s).flatten(-2)
    hit = (prefix > (u * i[:, -1])[:, None]) & live
    last = live.shape[1] - 1 - live.flip(1).to(torch.uint8).argmax(1)
    return torch.where(hit.any(1), hit.to(torch.uint8).argmax(1), last)


def _tours(case, choice, lists, seed, it):
    """All tours of iteration `it`; choice: n x (n rounded up to 64), binary32."""
    n, m, dev = case["n"], case["m"], choice.device
    ant = torch.arange(m, device=dev)
    zero = torch.zeros_like(ant)
    cur = (_philox(seed, zero, ant, zero + it, zero)[0] * n) >> 32
    step = torch.arange(n, device=dev)[:, None] + zero
    u = (_philox(seed, step, ant + 0 * step, it + 0 * step, 0 * step)[0] >> 8).float() * 2.0**-24
    live = torch.zeros(m, choice.shape[1], dtype=torch.bool, device=dev)
    live[:, :n] = True
    tours = [cur]
    for s in range(1, n):
        live[ant, cur] = False
        row = choice[cur] * live
        if case["rule"] == "r64":
            cur = _roulette(row, live, u[s])
        elif case["rule"] == "nn":
            cities = lists[cur]
            near = torch.nn.functional.pad(live.gather(1, cities), (0, 64 - cities.shape[1]))
            w = torch.nn.functional.pad(row.gather(1, cities), (0, 64 - cities.shape[1]))
            r = _roulette(w, near, u[s]).clamp(max=cities.shape[1] - 1)
            # every list entry visited: the live city of largest choice, lowest index
            best = torch.where(live, row, torch.full_like(row, -1.0)).argmax(1)
            cur = torch.where(near.any(1), cities.gather(1, r[:, None])[:, 0], best)
        else:
            block = torch.arange(choice.shape[1] // 4, device=dev) + 0 * ant[:, None]
            x = torch.stack(_philox(seed, 0 * block + s, ant[:, None] + 0 * block, 0 * block + it,
                                    1 + block), dim=-1).flatten(1)
            product = row * ((x >> 8).float() * 2.0**-24)
            cur = torch.where(live, product, torch.full_like(product, -1.0)).argmax(1)
        tours.append(cur)
    return torch.stack(tours, dim=1)


def exact(case, seed):
    cost = case.get("n", 0) * (case.get("iters", 0) + case.get("at", 0))
    cost *= {"nn": 2, "product": 4}.get(case.get("rule"), 1)
    if case["kind"] not in ("solve", "resume") or cost > 25_000:
        return None
    case = dict({"rule": "r64", "at": 0, "nn": 0}, **case)
    n, m, dev = case["n"], case["m"], "cuda" if torch.cuda.is_available() else "cpu"
    dist = _dist(n, case["layout"], case["side"], seed)
    left, at, cnn = np.ones(n, bool), 0, 0
    for _ in range(n - 1):  # nearest-neighbour tour from city 0
        left[at] = False
        to = int(np.where(left, dist[at], 2**31 - 1).argmin())
        cnn, at = cnn + int(dist[at, to]), to
    cnn += int(dist[at, 0])
    lists = torch.from_numpy(np.argsort(dist + 0, axis=1, kind="stable")).to(dev)
    lists = lists[lists != torch.arange(n, device=dev)[:, None]].view(n, n - 1)[:, :case["nn"]]
    d = torch.from_numpy(dist).to(dev).double()
    d.fill_diagonal_(1.0)
    off = 1.0 - torch.eye(n, device=dev)
    power = torch.ones_like(d)
    for _ in range(case["beta"]):
        power = power * d
    heur = (1.0 / power).float() * off
    rho = float(np.float32(case["rho"]))
    keep = torch.tensor(np.float32(1.0 - rho), device=dev)
    tau = torch.full((n, n), m / cnn, dtype=torch.float64, device=dev)  # 64 bits throughout
    held = tau.float()                                                  # as the colony holds it
    width = -(-n // 64) * 64
    for it in range(case["at"] + case["iters"]):
        power = held * held if case["alpha"] == 2 else held if case["alpha"] else held * 0 + 1
        choice = torch.nn.functional.pad(power * heur, (0, width - n))
        a = _tours(case, choice, lists, seed, it)
        b = a.roll(-1, 1)
        length = (d[a, b]).sum(1)
        sums = []
        for dep in (1.0 / length, (1.0 / length).float().double()):
            s = torch.zeros(n * n, dtype=torch.float64, device=dev)
            s.index_add_(0, (a * n + b).flatten(), dep.repeat_interleave(n))
            sums.append(s.view(n, n) + s.view(n, n).T)
        tau = tau * (1.0 - rho) + sums[0]
        held = ((held * keep).double() + sums[1]).float()
    return {"tour": None, "length": None, "tau": tau.cpu().numpy()}
