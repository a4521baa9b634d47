"""Batches that run long enough for their roulette steps to start from the short
lists, at the pass bounds and in an order where colonies with lists stand
behind colonies without, against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import tsp_inputs
from gpu_helpers import ORACLE_THREADS, assert_same_f32

pytestmark = pytest.mark.gpu


def check_batch(spec, iters, configure=None, runs=2):
    """spec: (n, m) per instance; `iters` iterations in `runs` calls."""
    from paper_1101_2678_amd.aco import Batch

    dists = [tsp_inputs.instance(n, "cluster" if n % 2 else "uniform", seed=n + m)[1]
             for n, m in spec]
    params = [dict(m=m, alpha=1, beta=2, rho=0.5, seed=n) for n, m in spec]
    b = Batch(dists, params)
    for r in range(runs):
        if configure:
            configure(b, r)
        b.run(iters // runs, graph=r % 2 == 0)
        b.sync()
    for q, ((n, m), d) in enumerate(zip(spec, dists)):
        st = oracle.solve(d, m, 1, 2, 0.5, n, iters, threads=ORACLE_THREADS)
        assert_same_f32(b.tau(q), st.tau, f"n={n} m={m} tau")
        assert b.best(q)[1] == st.best_len and np.array_equal(b.best(q)[0], st.best_tour), n
        assert b.iteration(q) == iters
    b.close()


@pytest.mark.parametrize("sizes", [(256, 257, 320, 321), (512, 513), (1024, 1025), (1536, 1537)])
def test_long_batches_at_the_pass_bounds(sizes):
    check_batch([(n, 24) for n in sizes], 24)


@pytest.mark.parametrize("sizes", [(2048, 2049, 600), (2561, 330), (3584, 3585)])
def test_long_batches_of_long_rows(sizes):
    """Rows of four to eight passes, whose flags lie behind the staged block (up to
    seven passes) or behind the tour."""
    check_batch([(n, 10) for n in sizes], 18)


@pytest.mark.parametrize("ants", [3072, 3073])
def test_long_batches_on_each_side_of_the_staging(ants):
    """Batches of as many ants as keep whole rows in LDS, and of one more."""
    check_batch([(600, 20), (400, 20), (1100, 20), (1024, 20), (100, ants - 80)], 20)


def test_lists_behind_colonies_without():
    """The colonies of 600 and 330 cities at tile 4 and those of up to 256 have
    no lists, nor has the one of 400 with 8 ants; those of 700, 500 and 300 do."""
    from paper_1101_2678_amd import aco

    aco.set_tile(550, 650, 4)
    aco.set_tile(330, 340, 4)
    try:
        check_batch([(200, 20), (330, 20), (600, 20), (500, 20), (400, 8), (700, 20), (300, 20)],
                    24)
    finally:
        aco.reset_tiles()


def test_lists_follow_the_tile_policy():
    """A configuration that takes the lists from a colony and gives them back."""
    def configure(b, r):
        b.set_config(0, (0, 1024, -1)[r])

    check_batch([(600, 20), (300, 16)], 30, configure, runs=3)


def test_batch_without_lists():
    check_batch([(60, 30), (256, 24), (17, 5)], 6)
