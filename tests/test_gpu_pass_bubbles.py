"""The test pass of a small box with many small bubbles beside one with two (ratio within a process):
a wave that meets dozens of bubbles must not sum them up one after the other."""
import time

import numpy as np
import pytest

from paper_1708_01608_amd import sc

pytestmark = pytest.mark.gpu


def _pass_us(n):
    rng = np.random.default_rng(1)
    g = sc.Sim(q=9, nx=64, ny=64, tau=0.9, amp=1e-3, seed=3, K=10)
    c = np.stack([rng.integers(0, 64, n), rng.integers(0, 64, n), np.zeros(n)], 1).astype(float)
    g.seed_nuclei(c, np.full(n, 2.6), np.zeros(n), 0.0)
    best = 1e9
    for _ in range(10):
        t0 = time.perf_counter()
        for _ in range(10):
            g.test_pass()
        best = min(best, time.perf_counter() - t0)
    bubbles = len(g.bubbles())
    g.close()
    return best / 10 * 1e6, bubbles


def test_many_bubbles_are_not_summed_one_by_one():
    (two, b2), (many, bn) = _pass_us(2), _pass_us(64)
    print(f"[gpu] pass of 64^2: {b2} bubbles {two:.1f} us, {bn} bubbles {many:.1f} us", flush=True)
    assert b2 == 2 and bn > 16
    assert many < 2.6 * two
