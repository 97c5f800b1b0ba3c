"""Calls that run as two run groups (de.h, de_generation) equal, bit for bit,
those of a process in which none does (DE_STAGGER=0): tiles that leave a
quarter or more of the compute units idle in their last round, from 16
generations on (32 for a single round of rows of up to 128 coordinates), and full rounds of wide
BF16 rows, from 32 generations on.
"""
import json
import os
import subprocess
import sys

import pytest

from tests.gpu_helpers import make_de
from tests.test_gpu_stagger import ROOT

pytestmark = pytest.mark.gpu

# 256 compute units: 272 tiles of 64 rows unless stated; the last ones of a
# run are not full
CASES = [
    dict(runs=17, NP=1000, D=900, gemm_prec="bf16", gens=(16, 20)),
    dict(runs=2, NP=9000, D=641, gemm_prec="bf16", gens=(16, 17)),   # 282
    dict(runs=24, NP=1024, D=333, gemm_prec="bf16", jde=True, gens=(16, 16)),
    dict(runs=33, NP=1000, D=100, gemm_prec="bf16", gens=(16, 17)),  # 528
    dict(runs=17, NP=1000, D=100, gemm_prec="bf16", gens=(32, 33)),
    dict(runs=16, NP=1024, D=1000, gemm_prec="bf16", gens=(32, 40)),  # 256
    dict(runs=16, NP=1024, D=700, gemm_prec="bf16", jde=True, gens=(32, 33)),
    dict(runs=17, NP=1000, D=20, gemm_prec="fp32", gens=(16, 17)),
    dict(runs=17, NP=1000, D=100, gemm_prec="fp32", gens=(16, 17)),
    dict(runs=17, NP=1000, D=333, gemm_prec="fp32", jde=True, gens=(16, 17)),
    dict(runs=17, NP=1000, D=700, gemm_prec="fp32", gens=(16, 17)),
    dict(runs=17, NP=1000, D=1000, gemm_prec="fp32", gens=(16, 17)),
]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU (run with -m 'not gpu' on CPU)")
    yield


def digest(kw):
    """Populations, values and statistics after two calls, the second of
    which knows the first one's time per generation."""
    import hashlib

    import torch
    kw = dict(kw)
    gens = kw.pop("gens")
    de, _, _ = make_de(F=0.5, CR=0.9, seed=3, kind="rot_osc", **kw)
    for g in gens:
        de.generation(g)
        torch.cuda.synchronize()
    h = hashlib.sha256()
    h.update(de.population().cpu().numpy().tobytes())
    h.update(de.fitness().cpu().numpy().tobytes())
    acc, best = de.stats()
    de.close()
    assert sum(acc) > 0
    return [h.hexdigest(), list(acc), list(best)]


SCRIPT = r"""
import json, sys
sys.path.insert(0, sys.argv[1])
from tests.test_gpu_run_groups import CASES, digest
for kw in CASES:
    print(json.dumps(digest(kw)), flush=True)
"""


def test_run_groups_equal_single_launches():
    out = subprocess.run([sys.executable, "-c", SCRIPT, ROOT],
                         env=dict(os.environ, DE_STAGGER="0"), cwd=ROOT,
                         capture_output=True, text=True, timeout=240)
    assert out.returncode == 0, out.stderr[-2000:]
    want = [json.loads(ln) for ln in out.stdout.splitlines()
            if ln.startswith("[")]
    assert len(want) == len(CASES)
    for kw, ref in zip(CASES, want):
        print(kw, flush=True)
        mine = json.loads(json.dumps(digest(kw)))
        assert mine == ref, kw
