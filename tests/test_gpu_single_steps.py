"""The tile of a D2Q9 box's single steps (those that a source or a test pass follows): no wider than
its rows need, as few rows a block as its lanes allow, and the bits of a fixed tile."""
import numpy as np
import pytest

from paper_1708_01608_amd import sc

pytestmark = pytest.mark.gpu


# rows of part of a wave, of just over one and two; few, many and very many lanes
@pytest.mark.parametrize("box,rows", [((4, 2100), 1), ((16, 20000), 4), ((33, 10000), 2),
                                      ((65, 3000), 2), ((130, 4096), 4), ((900, 900), 4),
                                      ((128, 128), 1)])
def test_single_steps_take_a_tile_of_the_rows_width(box, rows):
    nx, ny = box
    print(f"[gpu] single steps {box}", flush=True)
    out = []
    for kw in (dict(tuned=False), dict(tile=(64, 1, 8), variant=1)):
        g = sc.Sim(q=9, nx=nx, ny=ny, nz=1, tau=0.9, amp=1e-3, seed=5, K=0, **kw)
        g.seed_nuclei(np.array([[nx - 1, 1, 0], [nx // 2, ny // 2, 0]], dtype=float),
                      np.full(2, min(6.0, nx / 4.0)), np.full(2, 1.0), 1e-3)
        cfg = g.step_config()
        for _ in range(5):
            g.step(1)
        out.append(g.get_populations())
        g.close()
        if "tile" not in kw:
            assert cfg[0] == (64 if nx <= 64 else 128 if nx <= 128 else 256) and cfg[2] == rows
    assert np.array_equal(out[0], out[1])
