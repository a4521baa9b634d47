"""Selections through the short lists of the choice rows (shortlist.hpp),
against the oracle, at the sizes and rows where a list can go wrong: the block
and workgroup bounds of its construction, rows of equal weights (no edge
between them, so the list stays empty or partial), rows of a few positive
weights, weights that span the binary32 range, and rows whose sums could
overflow, which must not be selected from by list."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import tsp_inputs
from gpu_helpers import ORACLE_THREADS, assert_same_f32

pytestmark = pytest.mark.gpu

CONSTRUCT = {"product": (lambda c, it: c.construct_product(it), oracle.construct_product),
             "r64": (lambda c, it: c.construct(it), oracle.construct)}


def pheromone(kind, n, rng):
    """A symmetric pheromone matrix; None keeps the colony's own."""
    if kind == "own":
        return None
    if kind == "zero":
        t = np.zeros((n, n))
    elif kind == "sparse":  # a few positive entries a row, the rest 0
        t = np.where(rng.random((n, n)) < 3.0 / n, 1.0, 0.0)
    elif kind == "wide":
        t = 10.0 ** rng.uniform(-44, 17, (n, n))
    elif kind == "steep":  # converged: each city two strong edges
        t = 1e-6 * rng.random((n, n))
        ring = rng.permutation(n)
        t[ring, np.roll(ring, 1)] = 1.0
    else:  # "huge": squares and sums near the top of binary32
        t = np.full((n, n), 1e18)
    t = np.maximum(t, t.T)
    return t.astype(np.float32)


def check(rule, dist, m, alpha, beta, kind, iters=2, seed=3):
    from paper_1101_2678_amd.aco import Colony

    n = dist.shape[0]
    construct, reference = CONSTRUCT[rule]
    tau = pheromone(kind, n, np.random.default_rng(n))
    ref = oracle.init(dist, m, alpha, beta, 0.5, seed)
    col = Colony(dist, m, alpha, beta, 0.5, seed, atomic=False)
    if tau is not None:
        col.restore(tau, 0)
        ref.tau, ref.choice = tau, oracle.choice(tau, dist, alpha, beta)
    for it in range(iters):
        tours, lens = reference(ref.choice, dist, m, seed, it, threads=ORACLE_THREADS)
        construct(col, it)
        got, got_lens = col.tours()
        assert np.array_equal(got, tours) and np.array_equal(got_lens, lens), (rule, n, kind, it)
        if kind == "huge":
            break  # the oracle's update refuses nothing here, but tau stops meaning anything
        ref.tau, ref.choice = oracle.update(ref.tau, tours, lens, dist, 0.5, alpha, beta)
        col.update("gather")
        assert_same_f32(col.tau(), ref.tau, f"tau {rule} n={n} {kind} it={it}")
    col.close()


@pytest.mark.parametrize("rule", sorted(CONSTRUCT))
@pytest.mark.parametrize("n", [3, 62, 63, 64, 65, 257, 1023, 1024, 1025, 2560, 2561, 4096])
def test_sizes(rule, n):
    m = 40 if n < 1024 else 12
    _, d = tsp_inputs.instance(n, "cluster" if n % 2 else "uniform", seed=n)
    check(rule, d, m, 1, 2, "own", iters=2 if n < 4096 else 1)


@pytest.mark.parametrize("rule", sorted(CONSTRUCT))
@pytest.mark.parametrize("kind", ["zero", "sparse", "wide", "steep", "huge"])
@pytest.mark.parametrize("n,alpha,beta", [(70, 1, 2), (300, 2, 4), (600, 1, 0), (1100, 1, 3)])
def test_weights(rule, kind, n, alpha, beta):
    _, d = tsp_inputs.instance(n, "uniform", side=20_000, seed=5)
    check(rule, d, 24, alpha, beta, kind)


@pytest.mark.parametrize("n", [257, 511, 512, 513, 1025, 1537, 1999, 2000, 2049, 3073])
def test_general_steps_between_list_steps(n):
    """Rows that start every roulette step from the lists, at the pass bounds:
    steps the list does not settle rebuild the visited bits."""
    _, d = tsp_inputs.instance(n, "uniform", seed=n)
    check("r64", d, 24 if n < 1024 else 8, 1, 2, "steep")


@pytest.mark.parametrize("rule", sorted(CONSTRUCT))
@pytest.mark.parametrize("kind", ["own", "zero", "sparse", "wide", "steep", "huge"])
@pytest.mark.parametrize("n", [2560, 2561, 3001, 3585])
def test_wide_lists(rule, kind, n):
    _, d = tsp_inputs.instance(n, "cluster", seed=n)
    check(rule, d, 8, 1, 2, kind, iters=1)


@pytest.mark.parametrize("rule", sorted(CONSTRUCT))
@pytest.mark.parametrize("side,beta", [(8, 2), (20, 2), (33, 0)])
def test_equal_weights(rule, side, beta):
    xy = np.array([(x, y) for x in range(side) for y in range(side)], np.int64) * 10
    check(rule, tsp_inputs.euc2d(xy), 30, 1, beta, "own")


@pytest.mark.parametrize("kind", ["own", "steep"])
@pytest.mark.parametrize("n,m", [(320, 8), (321, 9), (512, 8), (512, 9), (513, 8)])
def test_few_ants(kind, n, m):
    """Ant counts on each side of the line below which short rows have no lists,
    after a product construction has built lists that are then out of date."""
    from paper_1101_2678_amd.aco import Colony

    _, d = tsp_inputs.instance(n, "uniform", seed=n)
    tau = pheromone(kind, n, np.random.default_rng(n))
    ref = oracle.init(d, m, 1, 2, 0.5, 3)
    col = Colony(d, m, 1, 2, 0.5, 3, atomic=False)
    steep = pheromone("steep", n, np.random.default_rng(n + 1))
    col.restore(steep, 0)
    col.construct_product(0)
    col.restore(ref.tau if tau is None else tau, 0)
    if tau is not None:
        ref.choice = oracle.choice(tau, d, 1, 2)
    tours, lens = oracle.construct(ref.choice, d, m, 3, 0, threads=ORACLE_THREADS)
    col.construct(0)
    got, got_lens = col.tours()
    assert np.array_equal(got, tours) and np.array_equal(got_lens, lens)
    col.close()


@pytest.mark.parametrize("alpha,beta", [(0, 0), (1, 0), (2, 0)])
@pytest.mark.parametrize("n,m", [(63, 63), (65, 65), (333, 333), (1000, 60), (2561, 8)])
def test_product_rows_of_equal_weights(n, m, alpha, beta):
    """Product constructions that start on whole rows, because all weights are
    equal, and where tau counts may go over to the lists as it gathers."""
    _, d = tsp_inputs.instance(n, "uniform", seed=n)
    check("product", d, m, alpha, beta, "own", iters=8 if n < 400 else 2)
