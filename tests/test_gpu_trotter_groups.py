"""Phase form of the product formulas over the counts of modes whose groups of
modes per pass differ: one short group, full groups and a short slowest one, one
mode per pass; against the CPU FP64 oracle, forward and LCAM gradient."""
import numpy as np
import pytest

import scp_inputs as si
from oracle import lcam, trotter
from oracle.system import OracleSystem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# 10 steps, every amplitude through some 10^3 rounded FP64 operations of relative size 1e-16
TOL = 1e-12


@pytest.mark.parametrize("order", ["q1", "q2"])
@pytest.mark.parametrize("d,n", [(2, 2), (2, 4), (2, 6), (2, 8), (3, 6), (4, 5), (5, 4)])
def test_groups_of_modes(d, n, order):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_18155_amd as scp
    s = si.transmon_ring(si.rng_for(7, d * 100 + n), n, d, 0.2, 10, ring=False)
    s = si._finish(s, [d] * n, target=si.cz_target(n))
    o = OracleSystem(s)
    rng = np.random.default_rng(d * 10 + n)
    x = rng.normal(size=(o.D, 2)) + 1j * rng.normal(size=(o.D, 2))
    x /= np.linalg.norm(x, axis=0)
    g = scp.System(s)
    psi = torch.tensor(np.ascontiguousarray(x.T), device="cuda")
    U = g.propagate_trotter(psi, order)
    ref = trotter.propagate(o, order, psi0=x)
    err = float(np.abs(U.cpu().numpy().T - ref).max())
    print(f"[groups] d={d} n={n} {order} err {err:.1e}", flush=True)
    assert err <= TOL
    if n <= 4:
        cot = rng.normal(size=(o.D, 2)) + 1j * rng.normal(size=(o.D, 2))
        grad = g.trotter_adjoint(psi, torch.tensor(np.ascontiguousarray(cot.T), device="cuda"), order)
        want = lcam.gradient(o, order, cot, x)
        assert np.abs(grad - want).max() <= 1e-9 * np.abs(want).max()
    g.close()
