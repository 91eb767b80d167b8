"""Few boxes run with wide workgroups, many with narrow ones: the same boxes alone and beside so many
small ones that the other width is taken must give the same bits (a node's arithmetic does not
depend on the width; the totals are summed in another order: N roundings of FP64)."""
import numpy as np
import pytest

from paper_1708_01608_amd import sc, workloads as W

pytestmark = pytest.mark.gpu

# nx, ny, radius (negative: noise only, no gas)
BOXES = [(4, 4, -1.0), (5, 200, -1.0), (85, 31, 6.0), (86, 33, 6.0), (129, 40, 9.0), (255, 21, 4.0),
         (256, 64, 12.0), (200, 5, -1.0), (64, 65, 7.0), (192, 80, 14.0)]
MANY = 8192  # boxes of 4 x 4 beside them


def _run(boxes, max_steps, K, compute):
    n = len(boxes)
    rg, rl = W.coexistence_densities(-5.0)
    spec = W.BatchSpec(nx=np.array([b[0] for b in boxes]), ny=np.array([b[1] for b in boxes]),
                       G=np.full(n, -5.0), radius=np.array([b[2] for b in boxes]),
                       gap=np.full(n, 4), rho_l=np.full(n, rl), rho_g=np.full(n, rg),
                       seed=np.arange(3, 3 + n, dtype=np.int64), tau=0.9, max_steps=max_steps, K=K)
    b = sc.Batch(spec, compute=compute)
    res, _ = b.run()
    rho = [b.density(k) for k in range(len(BOXES))]
    b.close()
    return res[:len(BOXES)], rho


@pytest.mark.parametrize("compute", ["auto", "f32"])
@pytest.mark.parametrize("max_steps,K", [(1, 100), (60, 5), (23, 3)])
def test_width_does_not_change_a_box(max_steps, K, compute):
    print(f"[gpu] batch widths: {max_steps} steps, a pass every {K}, {compute}", flush=True)
    few, rho_few = _run(BOXES, max_steps, K, compute)
    many, rho_many = _run(BOXES + [(4, 4, -1.0)] * MANY, max_steps, K, compute)
    for k, (nx, ny, _) in enumerate(BOXES):
        assert np.array_equal(rho_few[k], rho_many[k]), BOXES[k]
        mass = float(np.sum(np.abs(rho_few[k].astype(np.float64))))
        for name, a in few[k].items():
            b = many[k][name]
            if name == "totals":
                assert np.max(np.abs(np.asarray(a) - np.asarray(b))) <= 2.0 ** -52 * nx * ny * mass
            else:
                assert a == b or (a != a and b != b), (BOXES[k], name, a, b)
