"""What the choice of a D3Q19 box's tile adds to the creation of a simulation (beside one that is
given its tile): some ten thousand shapes are estimated, in a few tens of microseconds."""
import time

import pytest

from paper_1708_01608_amd import sc

pytestmark = pytest.mark.gpu


def _create_us(**kw):
    best = 1e9
    for _ in range(30):  # (the binding's streams take turns, and memory is kept by stream)
        t0 = time.perf_counter()
        g = sc.Sim(q=19, nx=300, ny=9, nz=300, **kw)
        dt = time.perf_counter() - t0
        g.close()
        best = min(best, dt)
    return best * 1e6


def test_the_choice_of_a_tile_is_quick():
    for _ in range(2):  # a first round fills the allocator's caches
        fitted, given = _create_us(tuned=False), _create_us(tile=(32, 8, 16), variant=1)
    print(f"[gpu] sc_create 300 x 9 x 300: fitted {fitted:.0f} us, tile given {given:.0f} us",
          flush=True)
    assert fitted - given < 45.0
