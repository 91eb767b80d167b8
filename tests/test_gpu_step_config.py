"""The tile that sc_step_config reports can be given back: to a handle of the same box, of another
storage type, and without the variant; and tiles that are not the box's stay refused."""
import numpy as np
import pytest

from paper_1708_01608_amd import sc, workloads

pytestmark = pytest.mark.gpu

SPLIT_TILES = [(32, 4), (32, 8), (64, 4), (64, 8), (128, 4)]
MIX = dict(two_component=workloads.MIXTURE, G=0.0, rho_l=1.0, rho_g=0.05)


def _state(g):
    g.step(12)
    out = [g.get_populations()]
    if g.params.components == 2:
        out.append(g.get_gas_populations())
    return out


@pytest.mark.parametrize("shape", [(41, 39, 35), (203, 18, 9), (5, 37, 6), (64, 64, 64)])
@pytest.mark.parametrize("kw", [{}, dict(storage="bf16"), dict(gravity=(0.0, 0.0, -1e-5)), MIX,
                                dict(MIX, storage="f16")])
def test_the_reported_tile_is_accepted(shape, kw):
    nx, ny, nz = shape
    box = dict(q=19, nx=nx, ny=ny, nz=nz, tau=0.9, seed=4, K=5, tuned=False)
    g = sc.Sim(**box, **kw)
    cfg = g.step_config()
    print(f"[gpu] step config {shape} {sorted(kw)}: {cfg}", flush=True)
    ref = _state(g)
    g.close()
    for given in (dict(tile=cfg[:3], variant=cfg[3]), dict(tile=cfg[:3]),
                  dict(tile=(*cfg[:2], max(1, cfg[2] - 1)), variant=cfg[3])):
        h = sc.Sim(**box, **kw, **given)
        assert h.step_config()[:3] == tuple(given["tile"])
        # (16-bit mixtures on a fixed tile of the kernel with one component a wave: given, it has the
        # force coefficient rounded once, by default the default's)
        if not (kw.get("storage") == "f16" and cfg[:2] in SPLIT_TILES and "variant" in given):
            assert all(np.array_equal(a, b) for a, b in zip(_state(h), ref))
        h.close()
    other = dict(kw, storage="f16" if kw.get("storage", "f32") == "f32" else "f32")
    h = sc.Sim(**box, **other, tile=cfg[:3], variant=cfg[3])
    assert h.step_config() == cfg
    h.close()


@pytest.mark.parametrize("tile,variant", [((48, 8, 16), 1), ((40, 3, 1), 1), ((41, 24, 1), 3),
                                          ((41, 4, 1), 2), ((1025, 1, 1), 1), ((4, 4, 4), 1)])
def test_other_tiles_stay_refused(tile, variant):
    with pytest.raises(sc.ScError) as ei:
        sc.Sim(q=19, nx=41, ny=39, nz=35, tile=tile, variant=variant)
    assert ei.value.code == sc.SC_E_INVAL
