"""Per-run statistics of a population restarted from given rows (de_load_population
and de_evolve with no generations): best value with its lowest index, accepted
count and first hits, whatever the number and size of the runs.
"""
import numpy as np
import pytest

from tests.gpu_helpers import host, make_de

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU (run with -m 'not gpu' on CPU)")
    yield


# one large run, few runs that do not divide the waves, runs of every group
# width, more runs than groups, and populations beyond one workgroup's
@pytest.mark.parametrize("runs,NP", [
    (1, 4), (1, 64), (1, 16384), (2, 8192), (3, 5000), (5, 65), (15, 257),
    (16, 33), (17, 63), (31, 32), (64, 16), (100, 7), (255, 4), (256, 64),
    (257, 5), (4096, 4), (3276, 5), (2, 8193),
])
def test_restarted_statistics(runs, NP):
    D = 5
    de, _, _ = make_de(runs=runs, NP=NP, D=D, seed=2)
    de.generation(1)
    pop = host(de.population()).copy()
    rng = np.random.default_rng(runs * NP)
    # the lowest value twice in some runs, and rows that are not numbers
    pop[::3, NP // 2] = pop[::3, NP - 1]
    pop[1::5, rng.integers(0, NP)] = np.nan
    de.load_population(pop, 4)
    fit = host(de.fitness())
    f = np.where(np.isnan(fit), np.inf, fit)
    idx = f.argmin(axis=1)
    acc, best = de.stats()
    assert list(acc) == [0] * runs
    assert list(best) == [float(f[r, idx[r]]) for r in range(runs)]
    assert de.best_f64()[1] == list(idx)
    target = float(np.median(f.min(axis=1)))
    done, hits = de.evolve(0, target=target, check_every=1)
    assert done == 0
    want = np.where(f.min(axis=1) <= target, 4, -1)
    np.testing.assert_array_equal(np.asarray(hits), want)
    de.close()


# evolve in chunks against single steps: runs that fit one workgroup each and
# more, posts by the launch itself and behind it, hits posted and copied
@pytest.mark.parametrize("runs,NP,D", [
    (256, 6, 3), (257, 6, 3), (4096, 4, 2), (5000, 4, 2), (65536, 4, 1),
    (65537, 4, 1),
])
def test_first_hits_of_many_runs(runs, NP, D):
    a, _, _ = make_de(runs=runs, NP=NP, D=D, seed=8)
    b, _, _ = make_de(runs=runs, NP=NP, D=D, seed=8)
    best = [host(b.fitness()).min(axis=1)]
    for _ in range(12):
        b.generation(1)
        best.append(host(b.fitness()).min(axis=1))
    best = np.array(best)
    target = float(np.float32(np.quantile(best[6], 0.5)))
    done, hits = a.evolve(12, target=target, check_every=5)
    assert done == 12
    hit = best <= target
    want = np.where(hit.any(axis=0), hit.argmax(axis=0), -1)
    np.testing.assert_array_equal(np.asarray(hits), want)
    np.testing.assert_array_equal(host(a.population()), host(b.population()))
    assert a.stats() == b.stats()
    a.close()
    b.close()
