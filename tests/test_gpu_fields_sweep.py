"""The one-sweep 3D field kernels at the sizes where they can go wrong (tiles narrower than a wave,
rows in two tiles, ragged last tiles and chunks, a box smaller than a tile's ring), against the same
formulas in numpy from the populations.

Tolerances: rho and u are FP64 results rounded to FP32 (2^-24 = 6e-8 relative; u is off by that of
its own size and by FP64 rounding, 1e-13, of order-one terms); p and lap are FP64 sums of up to 19
order-one terms (1e-13)."""
import numpy as np
import pytest

from paper_1708_01608_amd import sc, workloads

pytestmark = pytest.mark.gpu

BOXES = [(4, 4, 4), (5, 37, 6), (203, 18, 9), (300, 7, 5), (33, 97, 31), (64, 64, 13)]


def _near(v, e):
    """v at x + e on the box ([nz, ny, nx])."""
    return np.roll(v, (-e[2], -e[1], -e[0]), (0, 1, 2))


def _gradient(v, e, w):
    return [sum(w[i] * e[i][c] * _near(v, e[i]) for i in range(1, 19)) for c in range(3)]


@pytest.mark.parametrize("shape", BOXES)
@pytest.mark.parametrize("kind", ["f32", "f16", "gravity", "mix_f32", "mix_bf16"])
def test_fields_and_laplacian_of_the_populations(shape, kind):
    nx, ny, nz = shape
    kw = {"f32": {}, "f16": dict(storage="f16"), "gravity": dict(gravity=(1e-4, 0.0, -2e-4)),
          "mix_f32": dict(two_component=workloads.MIXTURE),
          "mix_bf16": dict(two_component=workloads.MIXTURE, storage="bf16")}[kind]
    mix = kind.startswith("mix")
    if mix:
        kw.update(G=0.0, rho_l=1.0, rho_g=0.05)
    print(f"[gpu] field sweep {shape} {kind}", flush=True)
    g = sc.Sim(q=19, nx=nx, ny=ny, nz=nz, tau=0.9, amp=1e-2, seed=3, K=0, **kw)
    g.seed_nuclei([[nx - 1, 0, nz // 2]], [min(3.0, min(shape) / 3.0)], [0.0], 0.0)
    g.step(3)
    rho, u, _ = g.fields()
    p, lap = g.laplacian_p()
    e, w = sc.lattice(19)
    box = (nz, ny, nx)
    f = g.get_populations().reshape(19, *box)
    r = f.sum(0)
    j = [np.tensordot(e[:, c].astype(float), f, 1) for c in range(3)]
    if mix:
        fv = g.get_gas_populations().reshape(19, *box)
        rv, Gx = fv.sum(0), workloads.MIXTURE[0]
        gl, gv = _gradient(r, e, w), _gradient(rv, e, w)
        j = [j[c] + np.tensordot(e[:, c].astype(float), fv, 1) for c in range(3)]
        ref_u = [(j[c] - 0.5 * Gx * (r * gv[c] + rv * gl[c])) / (r + rv) for c in range(3)]
        ref_p = (r + rv) / 3.0 + Gx / 3.0 * r * rv
        assert np.abs(g.gas_density().reshape(box) - rv).max() <= 1e-7 * np.abs(rv).max()
    else:
        psi, G = 1.0 - np.exp(-r), -5.0
        gr = kw.get("gravity", (0.0, 0.0, 0.0))
        F = [-G * psi * v + (r - g.rho0) * gr[c] for c, v in enumerate(_gradient(psi, e, w))]
        ref_u = [(j[c] + 0.5 * F[c]) / r for c in range(3)]
        ref_p = r / 3.0 + G / 6.0 * psi * psi
    ref_lap = 6.0 * sum(w[i] * (_near(ref_p, e[i]) - ref_p) for i in range(1, 19))
    assert np.abs(rho.reshape(box) / r - 1.0).max() <= 1e-7
    for c in range(3):
        assert np.all(np.abs(u[c].reshape(box) - ref_u[c]) <= 1e-7 * np.abs(ref_u[c]) + 1e-13)
    assert np.abs(p.reshape(box) - ref_p).max() <= 1e-13
    assert np.abs(lap.reshape(box) - ref_lap).max() <= 1e-13
