"""Tiles and chunks of the one-sweep 3D field kernels: boxes large enough for a full block a CU with
many planes, and smaller ones with thin chunks and several blocks a CU, ragged in y and z.  The
Laplacian against the stencil applied to the returned p, p and rho against the populations.

Tolerances: p is an FP64 function of a 19-term FP64 sum (order one: 1e-13), lap a 19-term FP64 sum of
differences of p, times 6 (1e-13), rho the FP64 sum rounded to FP32 (6e-8 relative)."""
import pytest
import torch

from paper_1708_01608_amd import sc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(256, 219, 37), (131, 67, 66), (40, 61, 71), (24, 200, 17)])
def test_tiles_of_the_field_sweep(shape):
    nx, ny, nz = shape
    print(f"[gpu] field tiles {shape}", flush=True)
    g = sc.Sim(q=19, nx=nx, ny=ny, nz=nz, tau=0.9, amp=1e-2, seed=3, K=0)
    g.seed_nuclei([[nx - 1, 0, nz // 2]], [min(shape) / 4.0], [0.0], 0.0)
    g.step(2)
    box = (nz, ny, nx)
    p = torch.full((g.N,), 9.0, dtype=torch.float64, device="cuda")
    lap, rho = torch.full_like(p, 9.0), torch.full((g.N,), 9.0, device="cuda")
    u = torch.full((3, g.N), 9.0, device="cuda")
    g.laplacian_p_device(p, lap)
    g.fields_device(rho, u)
    r = torch.from_numpy(g.get_populations().reshape(19, -1)).cuda().double().sum(0)
    psi = 1.0 - torch.exp(-r)
    ref_p = r / 3.0 - 5.0 / 6.0 * psi * psi
    assert float((p - ref_p).abs().max()) <= 1e-13
    assert float(((rho.double() - r) / r).abs().max()) <= 6e-8
    e, w = sc.lattice(19)
    pb = p.reshape(box)
    acc = torch.zeros_like(pb)
    for i in range(1, 19):
        near = torch.roll(pb, (-int(e[i][2]), -int(e[i][1]), -int(e[i][0])), (0, 1, 2))
        acc += float(w[i]) * (near - pb)
    assert float((lap.reshape(box) - 6.0 * acc).abs().max()) <= 1e-13
    # u moved: the momentum of the pulled populations plus half the force, per density
    psb = psi.reshape(box)
    f = torch.from_numpy(g.get_populations().reshape(19, -1)).cuda().double()
    for c in range(3):
        j = sum(float(e[i][c]) * f[i] for i in range(19) if e[i][c])
        grad = torch.zeros_like(psb)
        for i in range(1, 19):
            if e[i][c]:
                near = torch.roll(psb, (-int(e[i][2]), -int(e[i][1]), -int(e[i][0])), (0, 1, 2))
                grad += float(w[i]) * float(e[i][c]) * near
        ref = (j + 0.5 * 5.0 * psi * grad.reshape(-1)) / r
        assert float((u[c].double() - ref).abs().max()) <= 6e-8 * (1.0 + float(ref.abs().max()))
