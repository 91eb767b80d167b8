"""Several D2Q9 steps in one launch give the bits of one step at a time: boxes smaller than a tile's
rim, tiles that overhang the box, step counts that split unevenly between launches and test passes,
a source that stops mid-chunk, gravity, every storage and arithmetic type; and under a barrier,
whose fix-up needs single steps once bubbles meet."""
import numpy as np
import pytest

from paper_1708_01608_amd import sc

pytestmark = pytest.mark.gpu

BOXES = [(4, 4), (5, 31), (17, 6), (66, 41), (128, 128), (131, 257), (300, 700)]
KINDS = {"f32": {}, "f32_f32": dict(compute="f32"), "f16": dict(storage="f16"),
         "bf16": dict(storage="bf16"), "gravity": dict(gravity=(1e-4, -2e-4, 0.0))}


def _run(shape, schedule, K, budget=0.0, **kw):
    nx, ny = shape
    g = sc.Sim(q=9, nx=nx, ny=ny, nz=1, tau=0.9, amp=1e-3, seed=9, K=K, **kw)
    c = np.array([[nx - 1, 1, 0], [nx // 2, ny // 2, 0]], dtype=float)
    g.seed_nuclei(c, np.full(2, min(6.0, min(shape) / 4.0)), np.full(2, budget), 1e-3)
    for n in schedule:
        g.step(n)
    out = [g.get_populations(), g.last_labels(), np.array(g.nuclei(2)[1])]
    t = g.t
    g.close()
    return out, t


@pytest.mark.parametrize("shape", BOXES)
@pytest.mark.parametrize("kind", list(KINDS))
def test_several_steps_a_launch_give_the_same_bits(shape, kind):
    kw = KINDS[kind]
    print(f"[gpu] multi-step {shape} {kind}", flush=True)
    for K, schedule in ((0, (1, 2, 7, 13)), (10, (3, 7, 25)), (7, (30,))):
        got, t = _run(shape, schedule, K, **kw)
        ref, tr = _run(shape, schedule, K, tile=(64, 1, 4), variant=1, **kw)
        assert t == tr == sum(schedule)
        for a, b in zip(got, ref):
            assert np.array_equal(a, b), (K, schedule)


@pytest.mark.parametrize("budget", [4.5e-3, 1.0])
def test_steps_around_the_source(budget):
    """The agent feeds for 4.5 steps, then the rest of the chunk is free of it; or at every step."""
    print(f"[gpu] multi-step source budget {budget}", flush=True)
    got, _ = _run((96, 70), (23, 18), 10, budget=budget)
    ref, _ = _run((96, 70), (23, 18), 10, budget=budget, tile=(64, 1, 4), variant=1)
    for a, b in zip(got, ref):
        assert np.array_equal(a, b)


def test_steps_under_a_barrier():
    kw = dict(barrier=True, corona=3)

    def run(**k):
        g = sc.Sim(q=9, nx=120, ny=60, nz=1, amp=1e-3, seed=2, K=5, **kw, **k)
        g.seed_nuclei([[40, 30, 0], [72, 30, 0]], [13.0, 13.0], [0.0, 0.0], 0.0)
        g.step(47)
        return g.get_populations(), g.owner()

    print("[gpu] multi-step barrier", flush=True)
    got, ref = run(), run(tile=(64, 1, 4), variant=1)
    assert len(np.unique(got[1])) == 3  # two owned bubbles: the frontier is in use
    for a, b in zip(got, ref):
        assert np.array_equal(a, b)
