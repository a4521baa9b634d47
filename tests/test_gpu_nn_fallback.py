"""Candidate-list construction where most steps leave the list: the largest
unvisited city from the row's short list (rows of more than 1280 cities) or
from the whole row, against the oracle, with equal choice values, zero rows and
rows that must not be selected from by list."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import tsp_inputs
from gpu_helpers import ORACLE_THREADS
from test_gpu_shortlist import pheromone

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,alpha,beta", [(1280, 1, 2), (1281, 1, 2), (1300, 2, 4), (2600, 1, 0)])
@pytest.mark.parametrize("kind", ["own", "zero", "sparse", "wide", "steep", "huge"])
def test_fallback(n, alpha, beta, kind):
    from paper_1101_2678_amd.aco import Colony

    _, d = tsp_inputs.instance(n, "cluster", side=20_000, seed=n)
    ref = oracle.init(d, 12, alpha, beta, 0.5, 4)
    col = Colony(d, 12, alpha, beta, 0.5, 4, atomic=False)
    tau = pheromone(kind, n, np.random.default_rng(n))
    if tau is not None:
        col.restore(tau, 0)
        ref.choice = oracle.choice(tau, d, alpha, beta)
    for nn in (1, 5):
        col.attach_nn(nn)
        col.construct_nn(3)
        tours, lens = oracle.construct_nn(ref.choice, d, oracle.nn_lists(d, nn), 12, 4, 3,
                                          threads=ORACLE_THREADS)
        got, got_lens = col.tours()
        assert np.array_equal(got, tours) and np.array_equal(got_lens, lens), (n, kind, nn)


@pytest.mark.parametrize("n,alpha,beta", [(1281, 1, 2), (1300, 2, 4), (2600, 1, 1)])
@pytest.mark.parametrize("kind", ["own", "zero", "sparse", "wide", "steep", "huge"])
def test_fallback_by_list(n, alpha, beta, kind):
    """As above with as many ants as have the lists built."""
    from paper_1101_2678_amd.aco import Colony

    _, d = tsp_inputs.instance(n, "cluster", side=20_000, seed=n)
    ref = oracle.init(d, 64, alpha, beta, 0.5, 4)
    col = Colony(d, 64, alpha, beta, 0.5, 4, atomic=False)
    tau = pheromone(kind, n, np.random.default_rng(n))
    if tau is not None:
        col.restore(tau, 0)
        ref.choice = oracle.choice(tau, d, alpha, beta)
    for nn in (1, 5):
        col.attach_nn(nn)
        col.construct_nn(3)
        tours, lens = oracle.construct_nn(ref.choice, d, oracle.nn_lists(d, nn), 64, 4, 3,
                                          threads=ORACLE_THREADS)
        got, got_lens = col.tours()
        assert np.array_equal(got, tours) and np.array_equal(got_lens, lens), (n, kind, nn)
    col.close()


@pytest.mark.parametrize("m,beta", [(63, 2), (64, 2), (64, 0), (63, 0)])
def test_rule_of_the_lists(m, beta):
    """Ant counts and weights on each side of the rule, after a product
    construction on other weights has built lists that are then out of date."""
    from paper_1101_2678_amd.aco import Colony

    n, nn = 1300, 8
    _, d = tsp_inputs.instance(n, "cluster", seed=7)
    ref = oracle.init(d, m, 1, beta, 0.5, 5)
    lists = oracle.nn_lists(d, nn)
    col = Colony(d, m, 1, beta, 0.5, 5, atomic=False)
    col.attach_nn(nn)
    other = np.random.default_rng(1).random((n, n)).astype(np.float32)
    col.restore(np.maximum(other, other.T), 0)
    col.construct_product(0)
    col.restore(ref.tau, 0)
    tours, lens = oracle.construct_nn(ref.choice, d, lists, m, 5, 0, ORACLE_THREADS)
    col.construct_nn(0)
    got, got_lens = col.tours()
    assert np.array_equal(got, tours) and np.array_equal(got_lens, lens)
    col.close()
