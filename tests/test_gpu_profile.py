"""Counts of the kernel classes: every time step and every fed step once, whether the source runs by
itself or is added by the step that follows, and whether steps share launches."""
import numpy as np
import pytest

from paper_1708_01608_amd import sc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q,shape,radius,storage", [
    (19, (48, 48, 48), 14.0, "f32"),   # many fed nodes: the source is added by the step after
    (19, (48, 48, 48), 14.0, "f16"),
    (19, (96, 64, 64), 8.0, "f32"),    # few: by itself (a bubble that the 60 steps do not dissolve)
    (9, (96, 80, 1), 12.0, "f32")])
def test_every_fed_step_is_counted(q, shape, radius, storage):
    nx, ny, nz = shape
    print(f"[gpu] profile counts {q} {shape} {storage}", flush=True)
    g = sc.Sim(q=q, nx=nx, ny=ny, nz=nz, tau=0.9, amp=1e-3, seed=2, K=25, storage=storage,
               rho_l=1.80)
    g.seed_nuclei(np.array([[nx / 2, ny / 2, nz // 2]]), np.array([radius]), np.array([1e6]), 1e-4)
    g.profile(True)
    g.step(60)  # two passes, and a call that ends between them
    counts = [g.profile_read(c) for c in (sc.SC_KERNEL_STEP, sc.SC_KERNEL_SOURCE,
                                          sc.SC_KERNEL_TEST)]
    assert [n for _, n in counts] == [60, 60, 2]
    assert all(ms > 0 for ms, _ in counts)
    g.close()
