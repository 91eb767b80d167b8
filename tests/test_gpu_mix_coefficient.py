"""The mixture's force coefficient -tau G_cross under FP32 arithmetic: where a tile of the kernel with
one component a wave is given, the FP64 product rounded once (two strengths whose products round to
the same FP32 value step to the same bits); by default and with both components a thread, the
product of the rounded factors, whatever tile the box is fitted with."""
import numpy as np
import pytest

from paper_1708_01608_amd import sc

pytestmark = pytest.mark.gpu

TAU, PAIR = 0.9, (1.5, 1.50000006)


def _run(G, storage, shape=(70, 40, 30), **kw):
    nx, ny, nz = shape
    g = sc.Sim(q=19, nx=nx, ny=ny, nz=nz, tau=TAU, G=0.0, rho_l=1.0, rho_g=0.05, amp=1e-3,
               seed=11, K=0, two_component=(G, TAU, 1.0, 0.05), storage=storage, **kw)
    g.seed_nuclei(np.array([[nx / 2, ny / 2, nz // 2], [2.0, 3.0, 0.0]]), np.full(2, 9.0),
                  np.zeros(2), 0.0)
    g.step(30)
    out = np.stack([g.get_populations(), g.get_gas_populations()])
    g.close()
    return out


def test_the_strengths_tell_the_roundings_apart():
    f = np.float32
    once = [f(-(TAU * g)) for g in PAIR]
    factors = [f(-f(TAU)) * f(g) for g in PAIR]
    assert once[0] == once[1] and factors[0] != factors[1]


@pytest.mark.parametrize("storage", ["f16", "bf16"])
def test_the_coefficient_of_each_call(storage):
    print(f"[gpu] mixture coefficient {storage}", flush=True)
    once = [_run(G, storage, tile=(64, 4, 16), variant=v) for v in (4, 5) for G in PAIR]
    assert all(np.array_equal(once[0], o) for o in once[1:])
    factors = [[_run(G, storage, **kw) for kw in (dict(tuned=False),
                                                  dict(tile=(32, 8, 16), variant=1),
                                                  dict(tile=(32, 8, 16), variant=3))]
               for G in PAIR]
    for runs in factors:
        assert all(np.array_equal(runs[0], r) for r in runs[1:])
    assert not np.array_equal(factors[0][0], factors[1][0])


def test_a_fitted_tile_that_is_also_a_given_one():
    # 128 nodes a row: the fitted tile is one of the fixed ones, and by default still the default's
    g = sc.Sim(q=19, nx=128, ny=32, nz=32, two_component=(1.5, TAU, 1.0, 0.05), storage="f16",
               tuned=False)
    cfg = g.step_config()
    g.close()
    shape = (128, 32, 32)
    by_default = _run(1.5, "f16", shape, tuned=False)
    assert np.array_equal(by_default, _run(1.5, "f16", shape, tile=(32, 8, 16), variant=1))
    if cfg[3] >= 4 and cfg[:2] in ((32, 4), (32, 8), (64, 4), (64, 8), (128, 4)):
        given = _run(1.5, "f16", shape, tile=cfg[:3], variant=cfg[3])
        assert np.array_equal(given, _run(PAIR[1], "f16", shape, tile=cfg[:3], variant=cfg[3]))
