"""The batch's two-step sweep (two time steps per pass over a box, the second pulled from LDS) at
the sizes where it can go wrong: boxes of one, two and many rows a block, fewer blocks than the
pipeline is deep, a last block that wraps around, a full-width row; odd and even step counts, odd
test cadences (single steps in between).  Every node against the oracle, FP32 storage with FP64
arithmetic (the parity tests' 1e-5)."""
import numpy as np
import pytest

from oracle import OracleSim
from paper_1708_01608_amd import sc, workloads as W

pytestmark = pytest.mark.gpu

# nx, ny, radius (negative: noise only, no gas)
BOXES = [(4, 4, -1.0), (5, 7, -1.0), (64, 4, -1.0), (9, 64, -1.0), (85, 31, 6.0), (86, 33, 6.0),
         (129, 40, 9.0), (256, 21, 4.0), (200, 5, -1.0), (64, 65, 7.0)]


def _spec(max_steps, K):
    n = len(BOXES)
    rg, rl = W.coexistence_densities(-5.0)
    return W.BatchSpec(nx=np.array([b[0] for b in BOXES]), ny=np.array([b[1] for b in BOXES]),
                       G=np.full(n, -5.0), radius=np.array([b[2] for b in BOXES]),
                       gap=np.full(n, 10), rho_l=np.full(n, rl), rho_g=np.full(n, rg),
                       seed=np.arange(3, 3 + n, dtype=np.int64), tau=0.9, max_steps=max_steps, K=K)


@pytest.mark.parametrize("max_steps,K", [(1, 100), (2, 100), (7, 100), (24, 100), (23, 3), (24, 1),
                                         (22, 8)])
def test_two_step_sweep_matches_oracle(max_steps, K):
    spec = _spec(max_steps, K)
    print(f"[gpu] batch sweep: {max_steps} steps, a pass every {K}", flush=True)
    b = sc.Batch(spec)
    res, _ = b.run()
    for k in range(spec.n):
        s = spec.instance(k)
        assert res[k]["steps_run"] == max_steps and res[k]["status"] == 0
        o = OracleSim(9, s.nx, s.ny, 1, s.tau, s.G, s.rho_l, s.rho_g, s.amp, s.seed, 0.0, 0, 8)
        o.seed_nuclei(s.centres, s.radii, s.budgets, 0.0)
        o.step(max_steps)
        ro, _, _ = o.fields()
        err = float(np.max(np.abs(b.density(k).astype(np.float64) - ro) / ro))
        assert err <= 1e-5, (BOXES[k], err)
    b.close()
