"""The mixture's force coefficient -tau G_cross enters the step with one rounding to the arithmetic
type: two strengths whose products round to the same FP32 value step to the same bits (with each
factor rounded first they would not), in every mixture kernel."""
import numpy as np
import pytest

from paper_1708_01608_amd import sc

pytestmark = pytest.mark.gpu

TAU, PAIR = 0.9, (1.5, 1.50000006)


def test_the_strengths_tell_the_roundings_apart():
    f = np.float32
    once = [f(-(TAU * g)) for g in PAIR]
    thrice = [f(-f(TAU)) * f(g) for g in PAIR]
    assert once[0] == once[1] and thrice[0] != thrice[1]


@pytest.mark.parametrize("storage", ["f16", "bf16"])
@pytest.mark.parametrize("q,kw", [
    (19, dict(tuned=False)), (19, dict(tile=(32, 8, 16), variant=1)),
    (19, dict(tile=(32, 8, 16), variant=3)), (19, dict(tile=(64, 4, 16), variant=4)),
    (19, dict(tile=(64, 4, 16), variant=5)), (9, dict(tuned=False))])
def test_equal_products_step_to_equal_bits(q, kw, storage):
    print(f"[gpu] mixture coefficient q={q} {kw} {storage}", flush=True)
    nx, ny, nz = (70, 40, 30) if q == 19 else (160, 130, 1)
    out = []
    for G in PAIR:
        g = sc.Sim(q=q, nx=nx, ny=ny, nz=nz, tau=TAU, G=0.0, rho_l=1.0, rho_g=0.05, amp=1e-3,
                   seed=11, K=0, two_component=(G, TAU, 1.0, 0.05), storage=storage, **kw)
        g.seed_nuclei(np.array([[nx / 2, ny / 2, nz // 2], [2.0, 3.0, 0.0]]), np.full(2, 9.0),
                      np.zeros(2), 0.0)
        g.step(30)
        out.append((g.get_populations(), g.get_gas_populations()))
        g.close()
    assert all(np.array_equal(a, b) for a, b in zip(*out))
