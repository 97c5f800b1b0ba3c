"""The FP32 rotation product (DE_GEMM_FP32) through the C ABI: operands of all
24 bits, whatever the sizes of R's entries, and values that depend on the row
and R alone.

Bars.  u = 2^-24 bounds the relative error of one FP32 rounding.
  - A row with a single coordinate in play has z_i = R_ij y_j: one rounding
    (none where the entry is a power of two).  A relative error e of z and the
    rounding of 3z move f = z^2 + sin^2(3z) by at most 2 e + 3 (e + u) / |z|
    relative, the rounding of the sum by u.  |z| >= 64: 1.05 u for an exact z,
    3.1 u for a rounded one.  |z| in [1, 2]: at most 9 u, and 3 u for the
    sine's series.
  - A dense row's z_i carries the errors of a chain of D fused additions
    (root mean square sqrt(D / 6) u of the row's size, independent between the
    D columns of the sum: 2 sqrt(D / 6) u / sqrt(D) in f), and its f those of
    5 additions over a block's columns, up to 3 blocks and 16 slots, each of
    at most f in size: sqrt(24 / 3) u.
"""
import numpy as np
import pytest

import oracle
from tests import test_gpu_kernel_edges as edges
from tests.gpu_helpers import FP32_RTOL, HI, LO, host, host_threads

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU (run with -m 'not gpu' on CPU)")
    yield


def _handle(D, R, o=None, NP=8, lo=LO, hi=HI):
    from paper_2405_16551_amd.de import DifferentialEvolution
    o = np.zeros(D, np.float32) if o is None else o
    return DifferentialEvolution(runs=1, NP=NP, D=D, F=0.5, CR=0.9, lo=lo,
                                 hi=hi, seed=1, kind="rot_osc", o=o, R=R,
                                 gemm_prec="fp32")


def _single(rng, n, D, lo, hi):
    """n rows with one coordinate in play, of random mantissa and sign."""
    X = np.zeros((n, D), np.float32)
    j = rng.integers(0, D, n)
    X[np.arange(n), j] = (rng.uniform(lo, hi, n)
                          * rng.choice((-1.0, 1.0), n)).astype(np.float32)
    return X, j


def _rel(f, X, R):
    o = np.zeros(R.shape[0], np.float32)
    fo = oracle.objective_batch(oracle.OBJ_ROT_OSC, X.astype(np.float64), o, R,
                                nthreads=host_threads())
    return np.abs(f.astype(np.float64) - fo) / fo


# the widths of every form of the tile; 400 rows, and more 32-row tiles than
# compute units
SIZES = [(32, 400), (100, 400), (129, 8300), (256, 400), (333, 400),
         (512, 8300), (513, 8300), (700, 400), (1000, 400), (1000, 8300),
         (1152, 400)]


@pytest.mark.parametrize("D,n", SIZES)
def test_operands_keep_all_their_bits(D, n):
    rng = np.random.default_rng(D + n)
    X, j = _single(rng, n, D, 64.0, 128.0)
    perm = rng.permutation(D)
    # a permutation: z is the coordinate itself
    R = np.zeros((D, D), np.float32)
    R[perm, np.arange(D)] = 1.0
    de = _handle(D, R)
    assert _rel(host(de.eval(X)), X, R).max() <= 1.06 * U
    de.close()
    # any entries: one rounding of z
    R[perm, np.arange(D)] = rng.uniform(1.0, 2.0, D).astype(np.float32)
    de = _handle(D, R)
    assert _rel(host(de.eval(X)), X, R).max() <= 3.11 * U
    de.close()


@pytest.mark.parametrize("D,n", SIZES)
@pytest.mark.parametrize("decades", [6, 9, 20])
def test_small_rows_of_R_keep_their_bits(D, n, decades):
    rng = np.random.default_rng(D + n + decades)
    scale = np.logspace(0, -decades, D)[rng.permutation(D)].astype(np.float32)
    R = np.diag(scale)
    X, j = _single(rng, n, D, 1.0, 2.0)
    X[np.arange(n), j] /= scale[j]
    # beside a weak coordinate in play the strong ones are zero, and the same
    # rows with every other weak coordinate in play too
    de = _handle(D, R)
    assert _rel(host(de.eval(X)), X, R).max() <= 12 * U
    Y = (rng.uniform(1.0, 2.0, (n, D)) / scale).astype(np.float32)
    r = _rel(host(de.eval(Y)), Y, R)
    assert r.max() <= (12 + 24) * U
    de.close()


# next to the largest float: the high part must not round beyond it.  |z| ~ 3e7,
# where the sine's argument carries no bits: f by z^2, at the bar of a step
@pytest.mark.parametrize("D,n", SIZES)
def test_largest_operands(D, n):
    rng = np.random.default_rng(D + n)
    top = np.finfo(np.float32).max
    X, j = _single(rng, n, D, 3.2e38, 3.4e38)
    X[0, j[0]] = top
    R = np.diag(rng.uniform(1e-31, 2e-31, D).astype(np.float32))
    de = _handle(D, R)
    assert _rel(host(de.eval(X)), X, R).max() <= FP32_RTOL
    de.close()
    de = _handle(D, np.zeros_like(R))
    assert (host(de.eval(X)) == 0.0).all()
    de.close()
    R = np.diag(np.full(D, top))
    X[np.arange(n), j] = 1e-31
    de = _handle(D, R)
    assert _rel(host(de.eval(X)), X, R).max() <= FP32_RTOL
    de.close()


@pytest.mark.parametrize("D,n", SIZES)
def test_error_of_a_dense_rotation(D, n):
    rng = np.random.default_rng(D + n)
    q, _ = np.linalg.qr(rng.standard_normal((D, D)))
    R = np.ascontiguousarray(q.astype(np.float32))
    X = rng.uniform(-5.0, 5.0, (n, D)).astype(np.float32)
    de = _handle(D, R)
    r = _rel(host(de.eval(X)), X, R)
    bar = U * np.sqrt(4.0 / 6.0 + 24.0 / 3.0)
    rms = float(np.sqrt(np.mean(r ** 2)))
    print(f"D {D} rows {n}: rms {rms:.2e} bar {bar:.2e}", flush=True)
    assert rms <= bar
    de.close()


# run 0 of a handle of one run equals run 0 of a handle of many, and the value
# of a row does not depend on how many rows are evaluated with it, at the
# widths of 513 to 1024 coordinates too
@pytest.mark.parametrize("NP,D,many,jde", [
    (33, 513, 130, None), (65, 640, 90, True), (64, 700, 129, None),
    (97, 769, 70, None), (33, 1000, 130, None), (40, 1024, 129, True),
])
def test_values_do_not_depend_on_the_number_of_runs(NP, D, many, jde):
    edges.test_few_tiles_equal_many("fp32", NP, D, many, jde)
