"""Tiles fitted to the box: the shape an untuned D3Q19 box gets (any width, height and number of
planes, last tiles ragged in every direction) gives the bits of a power-of-two tile.

The boxes: a row narrower than a wave, one a little wider, one that needs two tiles, odd sides
throughout, planes fewer than a chunk, and a box whose cells are fewer than a tile's threads.
"""
import numpy as np
import pytest

from paper_1708_01608_amd import sc, workloads

pytestmark = pytest.mark.gpu

BOXES = [(5, 37, 6), (67, 40, 30), (203, 18, 9), (300, 23, 5), (61, 5, 47), (4, 4, 4), (33, 97, 31)]


def _run(shape, steps=12, **kw):
    nx, ny, nz = shape
    two = kw.get("two_component")
    if two is not None:
        kw.update(G=0.0, rho_l=1.0, rho_g=0.05)
    g = sc.Sim(q=19, nx=nx, ny=ny, nz=nz, tau=0.9, amp=1e-3, seed=7, K=4, **kw)
    c = np.array([[nx - 1, 1, nz // 2], [nx // 2, ny // 2, 0]], dtype=float)
    g.seed_nuclei(c, np.full(2, min(3.0, min(shape) / 3.0)), np.full(2, 1e-2), 1e-4)
    g.step(steps)
    out = [g.get_populations(), g.last_labels()]
    if two is not None:
        out.append(g.get_gas_populations())
    cfg = g.step_config()
    g.close()
    return out, cfg


@pytest.mark.parametrize("shape", BOXES)
@pytest.mark.parametrize("kind", ["f32", "f32_f32", "f16", "bf16", "gravity", "mix_f32", "mix_f16"])
def test_fitted_tile_gives_the_bits_of_a_fixed_one(shape, kind):
    kw = {"f32": {}, "f32_f32": dict(compute="f32"), "f16": dict(storage="f16"),
          "bf16": dict(storage="bf16"), "gravity": dict(gravity=(1e-5, 0.0, -2e-5)),
          "mix_f32": dict(two_component=workloads.MIXTURE),
          "mix_f16": dict(two_component=workloads.MIXTURE, storage="f16")}[kind]
    print(f"[gpu] fitted tile {shape} {kind}", flush=True)
    got, cfg = _run(shape, tuned=False, **kw)
    ref, _ = _run(shape, tile=(32, 8, 16), variant=1, **kw)
    if min(shape) > 4:  # the smallest box has too few cells for a fitted tile
        assert cfg[0] * cfg[1] <= 1024 and cfg[:2] != (32, 8)
    for a, b in zip(got, ref):
        assert np.array_equal(a, b), cfg
