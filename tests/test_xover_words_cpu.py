"""Crossover draws with shared rounds, compiled for the host: equal to the
whole block and to the oracle's Philox, bit for bit.  Runs on CPU."""
import os
import subprocess

import numpy as np
import pytest

import oracle

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_shared_rounds_give_the_block(tmp_path):
    exe = tmp_path / "xover_words"
    try:
        subprocess.run(["hipcc", "-O2", "-I",
                        os.path.join(ROOT, "paper_2405_16551_amd", "csrc"),
                        "-o", str(exe),
                        os.path.join(HERE, "pins", "xover_words.cpp")],
                       check=True, capture_output=True, timeout=600)
    except (OSError, subprocess.CalledProcessError) as e:  # pragma: no cover
        pytest.skip(f"hipcc unavailable: {e}")
    rng = np.random.default_rng(4)
    q = rng.integers(0, 2**32, (4000, 6), dtype=np.uint64)
    q[:, 0] >>= 8  # run numbers share their word with the tag
    q[0] = 0
    q[1] = [(1 << 24) - 1] + [2**32 - 1] * 5
    q[2] = [0, 0, 0, 2**32 - 1, 0, 2**32 - 1]
    out = subprocess.run([str(exe)], text=True, check=True,
                         capture_output=True, timeout=600,
                         input="\n".join(" ".join(map(str, r))
                                         for r in q.tolist()) + "\n")
    got = np.array([ln.split() for ln in out.stdout.splitlines()],
                   dtype=np.uint64).astype(np.uint32)
    assert got.shape == (4000, 8)
    np.testing.assert_array_equal(got[:, :4], got[:, 4:])
    # the crossover block's counter: (q, indiv, gen, 3 << 24 | run)
    ctr = np.stack([q[:, 3], q[:, 2], q[:, 1], q[:, 0] | (3 << 24)], 1)
    np.testing.assert_array_equal(
        got[:, :4], oracle.philox(ctr.astype(np.uint32),
                                  q[:, 4:6].astype(np.uint32)))
