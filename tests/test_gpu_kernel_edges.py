"""Edges of tiles, chunks and dispatch rules of the GPU kernels, through the
C ABI, against the FP64 oracle or against the form that a smaller call takes.

Bars are those of the paths' own parity tests: 1e-5 relative for f of the
FP32 paths, 8 * 2^-8 / sqrt(D) for the BF16 rotation product, 2e-5 for the
composition objective, 4 * 2^-8 of the absolute-value network for the BF16
models; forms that perform the same operations in the same order are equal
bit for bit.
"""
import numpy as np
import pytest

import oracle
from tests import test_gpu_surrogate as sur
from tests import test_gpu_batch as batch
from tests.gpu_helpers import (FP32_RTOL, FP32_TIE_SHARE, HI, LO,
                               compare_generation, host, host_threads,
                               make_de)
from tests.test_gpu_parity import bf16_rtol

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU (run with -m 'not gpu' on CPU)")
    yield


# ---- rotated objective: tiles and the selection of a wave's rows -------------

@pytest.mark.parametrize("prec,runs,NP,D,CR", [
    # FP32 product: FP32 MFMA up to 31 coordinates, split halves from 32 on;
    # paired build up to 128; one column block per wave up to 256, then two
    ("fp32", 2, 33, 31, 0.9), ("fp32", 2, 65, 32, 0.9),
    ("fp32", 2, 40, 33, 0.5), ("fp32", 1, 97, 127, 0.9),
    ("fp32", 1, 70, 129, 0.9), ("fp32", 2, 45, 256, 0.3),
    ("fp32", 2, 39, 257, 0.9), ("fp32", 1, 64, 512, 0.9),
    ("fp32", 1, 33, 513, 1.0), ("fp32", 1, 37, 1025, 0.9),
    # rewriting several rows at a time: one, two and three 256-coordinate
    # chunks a row, many rows accepted or stale
    ("bf16", 2, 130, 200, 0.5), ("bf16", 2, 129, 400, 0.9),
    ("bf16", 2, 65, 600, 0.2), ("bf16", 1, 100, 900, 0.9),
])
def test_rotated_tile_edges(prec, runs, NP, D, CR):
    de, o, R = make_de(runs=runs, NP=NP, D=D, CR=CR, seed=11, kind="rot_osc",
                       gemm_prec=prec)
    de.generation(2)
    g = de.gen
    pop32 = host(de.population()).copy()
    fit_prev = host(de.fitness()).copy()
    de.generation(1)
    res = compare_generation(
        host(de.population()), host(de.fitness()), pop32, fit_prev, F=0.5,
        CR=CR, seed=11, gen=g, kind=oracle.OBJ_ROT_OSC, o=o, R=R,
        f_rtol=FP32_RTOL if prec == "fp32" else bf16_rtol(D))
    res.check(f"{prec} {runs}x{NP}x{D}",
              share=FP32_TIE_SHARE if prec == "fp32" else None)
    de.close()


# FP32 product, padded widths 640..1024 with more 32-row tiles than compute
# units: 64-row tiles.  3 x 2753 rows: 261 tiles of 32, last tiles of one row;
# D = 512 and 1025 lie outside (32-row tiles), 513 and 1024 are the ends,
# 768 / 769 the change from three column blocks per wave to four
@pytest.mark.parametrize("D", [512, 513, 768, 769, 1024, 1025])
def test_tall_tile_edges(D):
    runs, NP = 3, 2753
    de, o, R = make_de(runs=runs, NP=NP, D=D, seed=4, kind="rot_osc",
                       gemm_prec="fp32")
    de.generation(1)
    g = de.gen
    pop32 = host(de.population()).copy()
    fit_prev = host(de.fitness()).copy()
    de.generation(1)
    pop, fit = host(de.population()).copy(), host(de.fitness()).copy()
    # whole last tiles and the row beside them, and every 37th row
    rows = [(r, i) for r in range(runs)
            for i in sorted(set(range(0, NP, 37)) | set(range(2680, NP)))]
    pick = np.array(rows)
    f_own = oracle.objective_batch(
        oracle.OBJ_ROT_OSC, pop[pick[:, 0], pick[:, 1]].astype(np.float64),
        o, R, nthreads=host_threads())
    np.testing.assert_allclose(fit[pick[:, 0], pick[:, 1]], f_own,
                               rtol=FP32_RTOL, atol=0)
    np.testing.assert_allclose(
        host(de.eval(pop.reshape(-1, D))).reshape(runs, NP)[
            pick[:, 0], pick[:, 1]], f_own, rtol=FP32_RTOL, atol=0)
    # the step: kept rows exact, replaced rows the oracle's trial
    res = compare_generation(pop, fit, pop32, fit_prev, F=0.5, CR=0.9, seed=4,
                             gen=g, kind=oracle.OBJ_ROT_OSC, o=o, R=R,
                             f_rtol=FP32_RTOL, rows=rows)
    res.check(f"tall D={D}", share=FP32_TIE_SHARE)
    # control parameters per individual that never change: the same step
    jd, _, _ = make_de(runs=runs, NP=NP, D=D, seed=4, kind="rot_osc",
                       gemm_prec="fp32",
                       jde=dict(F_lo=0.1, F_span=0.9, tau_F=0.0, tau_CR=0.0))
    jd.generation(2)
    np.testing.assert_array_equal(host(jd.population()), pop)
    np.testing.assert_array_equal(host(jd.fitness()), fit)
    de.close()
    jd.close()


# the split product's scales: rows next to the optimum beside rows of the
# whole box in one tile, coordinates of very different sizes in one row, rows
# of zeros, and R scaled up and down
@pytest.mark.parametrize("D,n,rscale", [
    (32, 70, 1.0), (100, 33, 2.0 ** -20), (333, 65, 1000.0), (700, 70, 1.0),
    (700, 8193, 1.0),
])
def test_split_product_scales(D, n, rscale):
    from paper_2405_16551_amd import instances
    from paper_2405_16551_amd.de import DifferentialEvolution
    o, R = instances.make_instance("rot_osc", D, 1)
    R = (R * np.float32(rscale)).astype(np.float32)
    de = DifferentialEvolution(runs=1, NP=8, D=D, F=0.5, CR=0.9, lo=LO, hi=HI,
                               seed=1, kind="rot_osc", o=o, R=R,
                               gemm_prec="fp32")
    rng = np.random.default_rng(D + n)
    X = rng.uniform(LO, HI, (n, D)).astype(np.float32)
    scale = np.logspace(-5, 0, n)[rng.permutation(n)][:, None]
    X = (o + (X - o) * scale).astype(np.float32)
    X[1::3] = (o + (X[1::3] - o) * 10.0 ** rng.uniform(-6, 0, X[1::3].shape)
               ).astype(np.float32)
    X[::32] = o
    f = host(de.eval(X)).astype(np.float64)
    pick = np.unique(np.r_[0:min(n, 70), max(0, n - 70):n])
    fo = oracle.objective_batch(oracle.OBJ_ROT_OSC, X[pick].astype(np.float64),
                                o, R, nthreads=host_threads())
    assert (f[::32] == 0.0).all()
    np.testing.assert_allclose(f[pick], fo, rtol=FP32_RTOL, atol=0)
    de.close()


# ---- separable objective: the resident form, and evolve's chunks -------------

# quads of a row that fill their lanes or leave one for the donor draw, rows
# of several passes over a block's threads; the last case does not fit LDS and
# has more than 16384 rows
@pytest.mark.parametrize("runs,NP,D", [
    (2, 20, 1), (3, 33, 12), (3, 33, 13), (2, 257, 16), (2, 50, 17),
    (2, 70, 29), (2, 40, 61), (2, 25, 124), (2, 20, 128), (2, 20, 250),
    (5, 4001, 3),
])
def test_resident_and_evolve_equal_single_steps(runs, NP, D):
    a, _, _ = make_de(runs=runs, NP=NP, D=D, seed=6)
    b, _, _ = make_de(runs=runs, NP=NP, D=D, seed=6)
    done, hits = a.evolve(65, target=-1.0, check_every=30)
    assert done == 65 and all(h < 0 for h in hits)
    for _ in range(65):
        b.generation(1)
    np.testing.assert_array_equal(host(a.population()), host(b.population()))
    np.testing.assert_array_equal(host(a.fitness()), host(b.fitness()))
    assert list(a.stats()[1]) == list(b.stats()[1])
    a.close()
    b.close()


# ---- mixed batch: tile lists dealt by runs -----------------------------------

# one run; fewer runs than XCDs; one run with most of the tiles; more runs
# than a multiple of eight
@pytest.mark.parametrize("sizes", [
    [(64, 30)], [(40, 10), (33, 100), (70, 50)],
    [(1024, 100)] + [(32, 10)] * 4, [(32, 30)] * 17,
])
def test_batch_runs_do_not_depend_on_their_place(sizes):
    specs = [(NP, D, 0.5, 0.9) for NP, D in sizes]
    b, inst = batch.make_batch(specs, plan=batch.all_variants(specs, 1))
    b.generation(3)
    g = b.gen
    before = [(host(b.population(r)).copy(), host(b.fitness(r)).copy())
              for r in range(len(specs))]
    b.generation(1)
    for r, (NP, D, F, CR) in enumerate(specs):
        o, R = inst[D]
        res = compare_generation(
            host(b.population(r))[None], host(b.fitness(r))[None],
            before[r][0][None], before[r][1][None], F=F, CR=CR, seed=1, gen=g,
            kind=oracle.OBJ_ROT_OSC, o=o, R=R, f_rtol=bf16_rtol(D), run0=r)
        assert res.n == NP
    b.close()


# ---- surrogate ---------------------------------------------------------------

# 16-row blocks, 64-coordinate parts and component pairs that are not full
@pytest.mark.parametrize("D,n,rows", [
    (1, 1, 1), (2, 3, 17), (15, 2, 16), (17, 9, 33), (63, 4, 15), (64, 8, 48),
    (65, 1, 31), (100, 9, 1), (128, 5, 70), (129, 2, 17), (200, 3, 33),
])
def test_composition_edges(D, n, rows):
    s, comp = sur.make_sur(runs=1, NP=8, D=D, n=n)
    rng = np.random.default_rng(D + n)
    X = rng.uniform(LO, HI, (rows, D)).astype(np.float32)
    X[rows // 2] = comp[0][n - 1] + np.float32(1e-3)
    f = host(s.eval(X)).astype(np.float64)
    np.testing.assert_allclose(f, sur.comp_f(X, comp), rtol=sur.F_RTOL,
                               atol=1e-30)
    s.close()


# tiles of 128 rows; rows that cannot be read four coordinates at a time;
# widths with and without a compiled form
@pytest.mark.parametrize("D,H,n", [
    (33, 32, 1), (20, 64, 127), (97, 128, 129), (128, 256, 257),
    (100, 256, 385), (130, 96, 70),
])
def test_inference_edges(D, H, n):
    import torch
    from paper_2405_16551_amd import de as lib
    s, _ = sur.make_sur(runs=2, NP=64, D=D, hidden=H, steps=3, warmup_gens=1)
    s.generation(3)
    theta, _, _, _ = s.get_model()
    rng = np.random.default_rng(n)
    X = rng.uniform(LO, HI, (n, D)).astype(np.float32)
    ld = D + 1 + D % 2  # odd row length, first row off by one float
    buf = torch.zeros(1 + n * ld, dtype=torch.float32, device=s.device)
    buf[1:].view(n, ld)[:, :D] = torch.from_numpy(X).to(s.device)
    for run in range(2):
        y = host(s.predict(run, X))
        yo = oracle.mlp_forward(theta[run].astype(np.float64), X, D=D, H=H,
                                lo=LO, hi=HI)
        bound = 4 * 2.0 ** -8 * sur.abs_scale(theta[run], X, D, H)
        assert (np.abs(y - yo) <= bound).all()
        y2 = torch.empty(n, dtype=torch.float32, device=s.device)
        lib._check(lib._lib.de_sur_predict(
            s.handle, run, buf.data_ptr() + 4, n, ld, y2.data_ptr(), s._s()),
            "de_sur_predict")
        np.testing.assert_array_equal(host(y2), y)
        # a row's value does not depend on the rows beside it
        np.testing.assert_array_equal(host(s.predict(run, X[n // 2:])),
                                      y[n // 2:])
    s.close()


# minibatches below, between and above the compiled gradient forms, widths
# that leave column blocks partly empty
@pytest.mark.parametrize("D,H,B", [(33, 32, 32), (100, 256, 64),
                                   (97, 128, 96), (128, 256, 160)])
def test_training_edges(D, H, B):
    sur.test_adam_step_matches_oracle(D, H, B)


# candidates: two rows or one row per wave instruction (up to 32 4-groups, or
# more), rows of one to three passes, last waves with rows left over
@pytest.mark.parametrize("NP,D,k", [(5, 1, 1), (9, 127, 3), (11, 128, 4),
                                    (7, 129, 1), (13, 257, 2), (6, 600, 3)])
def test_candidate_edges(NP, D, k):
    s, comp = sur.make_sur(runs=2, NP=NP, D=D, n=1, hidden=32, k=k, F=0.6,
                           CR=0.8, seed=3, warmup_gens=100, steps=0, batch=32,
                           archive=64)
    s.generation(1)
    g = s.gen
    pop32, fit32 = host(s.population()).copy(), host(s.fitness()).copy()
    theta, _, _, _ = s.get_model()
    s.generation(1)
    cand, pred, choice = s.last()
    O, R, bias, sigma = comp
    out = oracle.sur_generation(pop32, fit32, theta, k=k, F=0.6, CR=0.8, lo=LO,
                                hi=HI, seed=3, gen=g, use_model=False, H=32,
                                O=O, R=R, bias=bias, sigma=sigma, nthreads=8)
    assert (pred == 0).all() and (choice == 0).all()
    # one rounding of the difference and one of the fused result, every
    # operand within the box
    tol = 2.0 ** -22 * HI * (1 + 2 * 0.6)
    assert (np.abs(cand - out["cand"]) <= tol).all()
    s.close()


# run groups: calls of 32 generations and more on BF16 rows of more than 896
# coordinates, the second call with a measured offset; 17 runs: groups of 8
# and 9; a shorter call between them goes unsplit
@pytest.mark.parametrize("jde", [None, True])
def test_long_calls_equal_single_steps(jde):
    kw = dict(runs=17, NP=1000, D=900, seed=3, kind="rot_osc",
              gemm_prec="bf16", jde=jde)
    a, _, _ = make_de(**kw)
    b, _, _ = make_de(**kw)
    for n in (32, 3, 33):
        a.generation(n)
        host(a.fitness())
    for _ in range(68):
        b.generation(1)
    np.testing.assert_array_equal(host(a.population()), host(b.population()))
    np.testing.assert_array_equal(host(a.fitness()), host(b.fitness()))
    assert a.stats() == b.stats()
    a.close()
    b.close()


# BF16 tiles of 32 rows while they find a compute unit each, else of 64; split
# FP32 tiles of 16 waves likewise, else of 8: run 0
# of a handle of one run equals run 0 of a handle of many, at the rule's edge
# (256 tiles of 32 rows on 256 compute units), in paired and chunked builds
@pytest.mark.parametrize("prec,NP,D,many,jde", [
    ("bf16", 8192, 10, 2, None), ("bf16", 250, 100, 33, None),
    ("bf16", 33, 128, 130, True), ("bf16", 65, 129, 90, None),
    ("bf16", 64, 333, 129, True), ("bf16", 33, 1000, 130, None),
    ("bf16", 32, 1152, 257, None),
    ("fp32", 8192, 32, 2, None), ("fp32", 250, 100, 33, True),
    ("fp32", 33, 128, 130, None), ("fp32", 65, 200, 90, True),
    ("fp32", 64, 333, 129, None), ("fp32", 50, 512, 129, True),
    ("fp32", 33, 1100, 130, None),
])
def test_few_tiles_equal_many(prec, NP, D, many, jde):
    kw = dict(NP=NP, D=D, seed=13, kind="rot_osc", gemm_prec=prec, jde=jde)
    a, _, _ = make_de(runs=1, **kw)
    b, _, _ = make_de(runs=many, **kw)
    a.generation(6)
    b.generation(6)
    np.testing.assert_array_equal(host(a.population())[0],
                                  host(b.population())[0])
    np.testing.assert_array_equal(host(a.fitness())[0], host(b.fitness())[0])
    # values of given rows: 33 rows, and more rows than 32 per compute unit
    x = host(b.population())[0]
    few = host(a.eval(x[:33]))
    np.testing.assert_array_equal(few, host(b.fitness())[0][:33])
    reps = -(-8200 // len(x))
    many_f = host(a.eval(np.tile(x, (reps, 1))))
    np.testing.assert_array_equal(many_f[:len(few)], few)
    a.close()
    b.close()
