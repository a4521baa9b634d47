"""Matrices read back through the neighbour tables (large, no construction
pending and none captured), in pieces, and by rows: the read changes nothing that
a later call sees, replays of captured calls among them."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import tsp_inputs
from gpu_helpers import ORACLE_THREADS, assert_same_f32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m", [(511, 511), (513, 513), (700, 3), (700, 700), (1000, 1024),
                                 (1100, 1101)])
def test_reads_between_calls(n, m):
    from paper_1101_2678_amd.aco import Colony

    _, d = tsp_inputs.instance(n, "uniform", seed=n)
    ref = oracle.init(d, m, 1, 2, 0.5, 1)
    col = Colony(d, m, 1, 2, 0.5, 1)
    for it in range(2):
        assert_same_f32(col.tau(), ref.tau, "tau before")
        assert_same_f32(col.choice(), ref.choice, "choice before")
        col.construct(it)
        assert_same_f32(col.tau(), ref.tau, "tau, construction pending")
        tours, lens = oracle.construct(ref.choice, d, m, 1, it, threads=ORACLE_THREADS)
        ref.tau, ref.choice = oracle.update(ref.tau, tours, lens, d, 0.5, 1, 2)
        col.update("gather" if it else "atomic")
        assert_same_f32(col.tau(), ref.tau, "tau after")
        assert_same_f32(col.choice(), ref.choice, "choice after")
        got, got_lens = col.tours()
        assert np.array_equal(got, tours) and np.array_equal(got_lens, lens)


def test_batch_reads_between_runs():
    from paper_1101_2678_amd.aco import Batch

    dists = [tsp_inputs.instance(n, "uniform", seed=n)[1] for n in (700, 64)]
    params = [dict(m=700), dict(m=20)]
    read, alone = Batch(dists, params), Batch(dists, params)
    for _ in range(2):
        read.run(1)
        read.tau(0), read.tau(1)
        alone.run(1)
    for q in (0, 1):
        assert_same_f32(read.tau(q), alone.tau(q), f"instance {q}")
        assert np.array_equal(read.best(q)[0], alone.best(q)[0])


def test_tours_after_autotune():
    """The batch tuner repeats constructions of one state; what it leaves are
    the tours of the last iteration that it advances by."""
    from paper_1101_2678_amd import aco

    sizes = (70, 333, 600)
    dists = [tsp_inputs.instance(n, "uniform", seed=n)[1] for n in sizes]
    params = [dict(m=n, alpha=1, beta=2, rho=0.5, seed=n) for n in sizes]
    tuned, plain = aco.Batch(dists, params), aco.Batch(dists, params)
    tuned.autotune([(0, -1), (8, 0), (16, 1024)], iters=2)
    plain.run(9, graph=False)
    plain.sync()
    for q in range(len(sizes)):
        assert tuned.iteration(q) == plain.iteration(q) == 9
        for a, b in zip(tuned.tours(q), plain.tours(q)):
            assert np.array_equal(a, b)
        assert_same_f32(tuned.tau(q), plain.tau(q), f"instance {q}")
    tuned.close()
    plain.close()


@pytest.mark.parametrize("kind,n,m", [("gather", 513, 600), ("atomic", 1500, 1500),
                                      ("noalloc", 1000, 1024), ("gather", 2600, 2600)])
def test_read_between_capture_and_replay(kind, n, m):
    """A captured update uses the neighbour tables of the construction before
    it whenever it is replayed: matrices read after the capture, and between
    replays of a captured construction and a captured update, leave them."""
    import torch
    from paper_1101_2678_amd.aco import Colony

    _, d = tsp_inputs.instance(n, "uniform", seed=n)
    stream = torch.cuda.Stream()
    ref = oracle.init(d, m, 1, 2, 0.5, 1)
    col = Colony(d, m, 1, 2, 0.5, 1, atomic=kind == "atomic", stream=stream)
    update = col.update_atomic_noalloc if kind == "noalloc" else lambda: col.update(kind)

    def capture(call):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream, capture_error_mode="thread_local"):
            call()
        return graph

    def replay(graph):
        with torch.cuda.stream(stream):
            graph.replay()
        stream.synchronize()

    def check(what):
        assert_same_f32(col.tau(), ref.tau, f"tau {what}")
        assert_same_f32(col.choice(), ref.choice, f"choice {what}")

    check("before any capture")
    col.construct(0)
    captured_update = capture(update)
    captured_construct = capture(lambda: col.construct(1))
    for it in range(2 if n < 2000 else 1):
        check(f"before replay {it}")
        if it:
            replay(captured_construct)
            check("between replays")
        tours, lens = oracle.construct(ref.choice, d, m, 1, it, threads=ORACLE_THREADS)
        got, got_lens = col.tours()
        assert np.array_equal(got, tours) and np.array_equal(got_lens, lens)
        ref.tau, ref.choice = oracle.update(ref.tau, tours, lens, d, 0.5, 1, 2)
        replay(captured_update)
        check(f"after replay {it}")
    col.close()
