"""Initialisation at its bounds: the row lists' threads (256 keys), the list
entries staged for the nearest-neighbour tour (32 to n = 2350, then 16) and a
batch whose colonies lie on both sides of them, against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import tsp_inputs
from gpu_helpers import bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 33, 34, 256, 257, 512, 2340, 2350, 2351, 2352, 2360, 4096])
def test_tau0_and_choice(n):
    from paper_1101_2678_amd.aco import Colony

    # clusters: the tour leaves its lists often
    _, d = tsp_inputs.instance(n, "cluster", side=5_000, seed=n)
    ref = oracle.init(d, 7, 1, 2, 0.5, 1)
    col = Colony(d, 7, 1, 2, 0.5, 1, atomic=False)
    assert np.array_equal(bits(col.tau()), bits(ref.tau))
    assert np.array_equal(bits(col.choice()), bits(ref.choice))


def test_equal_distances():
    """A lattice: many equal keys but for the city index."""
    from paper_1101_2678_amd.aco import Colony

    xy = np.array([(x, y) for x in range(24) for y in range(24)], np.int64) * 10
    d = tsp_inputs.euc2d(xy)
    ref = oracle.init(d, 5, 1, 2, 0.5, 1)
    col = Colony(d, 5, 1, 2, 0.5, 1, atomic=False)
    assert np.array_equal(bits(col.tau()), bits(ref.tau))
    for nn in (1, 31, 64):
        col.attach_nn(nn)
        assert np.array_equal(col.nn_lists(), oracle.nn_lists(d, nn))


def test_batch():
    from paper_1101_2678_amd.aco import Batch

    sizes = [3, 2350, 64, 2400, 257, 900]
    dists = [tsp_inputs.instance(n, "cluster", seed=n)[1] for n in sizes]
    batch = Batch(dists, [dict(m=4 + q, rho=0.25, beta=3) for q in range(len(sizes))])
    for q, d in enumerate(dists):
        ref = oracle.init(d, 4 + q, 1, 3, 0.25, 1)
        assert np.array_equal(bits(batch.tau(q)), bits(ref.tau))


@pytest.mark.parametrize("layout", ["uniform", "cluster"])
def test_served(layout):
    """The server's initialisation walks the lists where they lie: nothing
    staged in LDS beside the ticks of other requests."""
    from paper_1101_2678_amd.serve import Request, Server, run_open_loop

    reqs = [Request(rid=q, arrival=0.0, m=5 + q, iters=1, seed=q + 1,
                    dist=tsp_inputs.instance(n, layout, side=5_000, seed=n)[1])
            for q, n in enumerate([3, 33, 34, 300, 1025, 2350, 2400, 3100])]
    server = Server(pool_bytes=1 << 30, max_slots=8)
    run_open_loop(server, reqs, keep_tau=True)
    server.close()
    for r in reqs:
        st = oracle.solve(r.dist, r.m, 1, 2, 0.5, r.seed, 1)
        assert np.array_equal(bits(r.extra["tau"]), bits(st.tau)), r.n
        assert r.best_len == st.best_len


@pytest.mark.parametrize("n", [6, 64, 257, 700, 4096])
def test_lists_of_few_entries(n):
    """On each side of the length up to which every entry is a minimum of the
    workgroup."""
    from paper_1101_2678_amd.aco import Colony

    _, d = tsp_inputs.instance(n, "cluster", side=60 * n, seed=n)
    col = Colony(d, 3, 1, 2, 0.5, 1, atomic=False)
    for nn in (1, 2, 4, 5):
        col.attach_nn(nn)
        assert np.array_equal(col.nn_lists(), oracle.nn_lists(d, nn)), nn
    col.close()
