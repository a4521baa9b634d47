"""The roulette steps of short rows (one city of every 64-city block per lane,
construct_flat.hpp) and of rows of one to three passes (visited set as factors,
construct_masked.hpp) at the edges of their blocks and passes, against the
oracle."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import tsp_inputs
from gpu_helpers import compare_run

pytestmark = pytest.mark.gpu

EDGES = [2, 63, 64, 65, 127, 128, 129, 191, 192, 193, 256, 257, 319, 320, 321]
PASSES = [385, 511, 512, 513, 1023, 1024, 1025, 1535, 1536, 1537]


@pytest.mark.parametrize("n", EDGES + PASSES)
def test_select(n):
    import torch
    from paper_1101_2678_amd import aco
    from test_gpu_parity import _adversarial_rows

    rows, feas, u = _adversarial_rows(n, 1500, np.random.default_rng(9000 + n))
    feas[::97] = 0  # no feasible city
    args = [torch.from_numpy(a).cuda() for a in (rows, feas, u)]
    got = aco.test_select(*args).cpu().numpy()
    assert (got == oracle.r64_select_batch(rows, feas, u)).all()


BATCHED = [255, 257, 320, 321, 385, 511, 512, 513, 1000, 1023, 1024, 1025, 1500, 1535, 1536, 1537,
           2400, 4096]


@pytest.mark.parametrize("n,tile", [(n, 8) for n in BATCHED] + [(n, 4) for n in BATCHED if n <= 1024])
def test_select_batched(n, tile):
    """The same rows through the batched launch's code, which keeps the bits, with
    as many rows as a launch stores whole in LDS, and with more."""
    import torch
    from paper_1101_2678_amd import aco
    from test_gpu_parity import _adversarial_rows

    rows, feas, u = _adversarial_rows(n, 3073, np.random.default_rng(9000 + n))
    feas[::97] = 0  # no feasible city
    args = [torch.from_numpy(a).cuda() for a in (rows, feas, u)]
    want = oracle.r64_select_batch(rows, feas, u)
    got = aco.test_select(*args, tile=tile, batched=True).cpu().numpy()
    assert (got == want).all()
    got = aco.test_select(*[a[:3072] for a in args], tile=tile, batched=True).cpu().numpy()
    assert (got == want[:3072]).all()


def test_select_batched_non_monotone_prefix():
    """Rows with a block whose tree prefix exceeds a later one."""
    import torch
    from paper_1101_2678_amd import aco

    rng = np.random.default_rng(78)
    rows = []
    while len(rows) < 200:
        w = rng.random(64).astype(np.float32)
        w[63] = 0
        s = oracle.s64(w)
        if (s[:63] > s[63]).any():
            rows.append(np.concatenate([rng.random(64 * (5 + len(rows) % 19)).astype(np.float32),
                                        w]))
    for k in range(19):
        part = np.array([r for r in rows if len(r) == 64 * (6 + k)])
        feas = np.ones(part.shape, np.uint8)
        u = np.full(len(part), 1.0 - 2.0**-24, np.float32)
        args = [torch.from_numpy(a).cuda() for a in (part, feas, u)]
        want = oracle.r64_select_batch(part, feas, u)
        assert (aco.test_select(*args, batched=True).cpu().numpy() == want).all()
        assert (aco.test_select(*args).cpu().numpy() == want).all()


@pytest.mark.parametrize("n", [100, 320, 321, 513, 1025, 1537])
def test_select_ignores_infeasible_weights(n):
    """A city that may not be chosen counts for nothing, whatever its weight."""
    import torch
    from paper_1101_2678_amd import aco
    from test_gpu_parity import _adversarial_rows

    rng = np.random.default_rng(n)
    rows, feas, u = _adversarial_rows(n, 300, rng)
    dirty = np.where(feas != 0, rows, rng.choice(np.float32([np.inf, np.nan, 3e38]), rows.shape))
    args = [torch.from_numpy(a).cuda() for a in (dirty.astype(np.float32), feas, u)]
    got = aco.test_select(*args).cpu().numpy()
    assert (got == oracle.r64_select_batch(np.where(feas != 0, rows, np.float32(0)), feas, u)).all()


@pytest.mark.parametrize("n", [n for n in EDGES if n > 2])
def test_parity(n):
    _, d = tsp_inputs.instance(n, "cluster" if n % 2 else "uniform", side=10_000, seed=n + 1)
    compare_run(d, 70, 1, 2, 0.5, seed=n, iters=2, kinds=("gather",))


@pytest.mark.parametrize("n", PASSES)
def test_parity_passes(n):
    _, d = tsp_inputs.instance(n, "uniform", seed=n + 2)
    compare_run(d, 20, 1, 2, 0.5, seed=n, iters=2, kinds=("gather",))


@pytest.mark.parametrize("kind", ["own", "steep"])
@pytest.mark.parametrize("n,m", [(520, 3072), (520, 3073), (1030, 2048), (1030, 2049)])
def test_many_ants(kind, n, m):
    """The ant counts on each side of the line between factors and bits, on
    whole rows and from the lists."""
    from test_gpu_shortlist import check

    _, d = tsp_inputs.instance(n, "uniform", seed=n + m)
    check("r64", d, m, 1, 2, kind, iters=1)


@pytest.mark.parametrize("n", [600, 1000, 1100, 1500])
def test_many_ants_stay_resident(n):
    """A launch of more ants than fit one round with the factors keeps as many
    on a compute unit as the bits allow."""
    from paper_1101_2678_amd.aco import Colony

    def ants_per_cu(m):
        c = Colony(tsp_inputs.instance(n, "uniform", seed=n)[1], m, 1, 2, 0.5, 1, atomic=False)
        text = c.describe()
        c.close()
        return int(text.split("ants_per_cu=")[1].split()[0])

    assert ants_per_cu(n) * 256 >= n
    assert ants_per_cu(16384) >= 20


@pytest.mark.parametrize("n,m", [(2100, 2380), (2100, 2381), (2600, 1924), (3100, 1613),
                                 (4096, 1220), (4096, 1221)])
def test_whole_rows_on_each_side_of_the_memory_bound(n, m):
    """Rows of five to eight passes that no list settles, loaded in one burst
    and with few loads in flight (from m n = 5e6 on)."""
    from paper_1101_2678_amd.aco import Colony

    _, d = tsp_inputs.instance(n, "uniform", seed=n)
    ref = oracle.init(d, m, 0, 1, 0.5, 7)
    col = Colony(d, m, 0, 1, 0.5, 7, atomic=False)
    col.construct(2)
    tours, lens = col.tours()
    for k in np.linspace(0, m - 1, 9).astype(int):
        tour, length = oracle.construct_ant(ref.choice, d, 7, 2, int(k))
        assert np.array_equal(tours[k], tour) and lens[k] == length, k
    col.close()


@pytest.mark.parametrize("n,m,tile,layout", [
    (100, 10, 4, "flat"), (256, 10, 8, "flat"), (257, 10, 8, "factors"), (320, 10, 4, "flat"),
    (321, 10, 4, "bits"), (512, 65535, 8, "factors"), (1000, 3072, 8, "factors"),
    (1000, 3073, 8, "bits"), (1536, 2048, 8, "factors"), (1536, 2049, 8, "bits"),
    (1537, 10, 8, "bits")])
def test_described_layout(n, m, tile, layout):
    from paper_1101_2678_amd import aco

    aco.set_tile(n, n, tile)
    try:
        col = aco.Colony(tsp_inputs.instance(n, "uniform", seed=n)[1], m, 1, 2, 0.5, 1,
                         atomic=False)
        assert f"layout={layout}" in col.describe().split()
        col.close()
    finally:
        aco.reset_tiles()
