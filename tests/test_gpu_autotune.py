"""The tuner keeps what is fastest, the shape a box has by default included: the fitted tile of a small
D3Q19 box (which no candidate comes near), and the several steps a launch of a D2Q9 box; for the
handle and for the ones that follow it; and its table's smallest time is the kept shape's."""
import time

import numpy as np
import pytest

from paper_1708_01608_amd import sc, workloads

pytestmark = pytest.mark.gpu


def _step_us(g, n=400):
    g.step(n)
    best = 1e9
    for _ in range(5):
        t0 = time.perf_counter()
        g.step(n)
        best = min(best, time.perf_counter() - t0)
    return best / n * 1e6


@pytest.mark.parametrize("kw,count", [
    (dict(), 108), (dict(storage="f16"), 108), (dict(gravity=(0.0, 0.0, -1e-5)), 72),
    (dict(two_component=workloads.MIXTURE, G=0.0, rho_l=1.0, rho_g=0.05), 60)])
def test_the_fitted_tile_is_kept_when_it_is_the_fastest(kw, count):
    box = dict(q=19, nx=41, ny=39, nz=35, tau=0.9, K=0)
    g = sc.Sim(**box, **kw)
    cfg = g.step_config()
    before = g.get_populations()
    print(f"[gpu] autotune {box} {sorted(kw)}: fitted tile {cfg}", flush=True)
    table = g.autotune(trials=20)
    assert np.array_equal(g.get_populations(), before)
    best = min(table, key=lambda e: e["us"])
    print(f"kept {g.step_config()} {best['us']:.2f} us of {len(table)}", flush=True)
    assert g.step_config() == cfg == (*best["tile"], best["variant"])
    assert len(table) == count
    h = sc.Sim(**box, **kw)  # and for the next handle of the box
    assert h.step_config() == cfg
    # a handle that was given a slow tile gets the fitted one back
    variant = 4 if "two_component" in kw else 1
    s = sc.Sim(**box, **kw, tile=(64, 4, 16), variant=variant)
    s.autotune(trials=20)
    assert s.step_config() == cfg
    for x in (g, h, s):
        x.close()


@pytest.mark.parametrize("compute", ["f64", "f32"])
def test_several_steps_a_launch_stand_against_single_ones(compute):
    box = dict(q=9, nx=130, ny=126, tau=0.9, K=0, compute=compute)
    g = sc.Sim(**box)
    fast = _step_us(g)
    g.autotune(trials=20)
    h = sc.Sim(**box)
    s = sc.Sim(**box, tile=(64, 1, 4), variant=1)
    slow = _step_us(s)
    s.autotune(trials=20)
    times = [_step_us(x) for x in (g, h, s)]
    print(f"[gpu] 130 x 126 {compute}: {fast:.2f} us a step by default, {slow:.2f} with a tile given; "
          f"tuned {[round(t, 2) for t in times]}", flush=True)
    assert slow > 1.5 * fast and max(times) < 1.25 * fast
    ref = sc.Sim(**box, tile=(64, 1, 4), variant=1)
    ref.step(s.t)
    assert np.array_equal(ref.get_populations(), s.get_populations())
    for x in (g, h, s, ref):
        x.close()
