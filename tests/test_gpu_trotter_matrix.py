"""Product formulas in the matrix form (d = 4, 5, couplings that do not
commute): against the CPU FP64 oracle over fibre counts below, at and above a
tile of 16, pairs in either orientation and between distant modes, several
couplings on a pair, and the smallest number of pairs."""
import numpy as np
import pytest

import scp_inputs as si
from oracle import trotter
from oracle.system import OracleSystem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-11   # at most 20 steps of 3 pieces: some 10^4 rounded FP64 operations (1e-16) per amplitude


@pytest.fixture(scope="module")
def scp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_18155_amd as m
    return m


CASES = [(4, 3, [(0, 1), (1, 2)], 12), (4, 3, [(1, 0), (0, 1), (2, 0)], 12),
         (4, 4, [(0, 1), (0, 1), (1, 2), (3, 2)], 8), (4, 5, [(0, 4), (4, 1), (2, 1), (3, 2)], 4),
         (5, 3, [(0, 1), (2, 1)], 12), (5, 3, [(0, 1), (1, 2), (0, 2)], 20),
         (5, 4, [(0, 1), (2, 1), (2, 3), (3, 0)], 4)]


@pytest.mark.parametrize("order", ["q1", "q2", "q4", "q4j"])
@pytest.mark.parametrize("d,n,edges,steps", CASES)
def test_matches_the_oracle(scp, d, n, edges, steps, order):
    desc = si.random_raw_system(60 + d * 10 + n, [d] * n, 0, 0.1 * steps, steps, env="gauss")
    rng = np.random.default_rng(d * 10 + n)
    # operators alternate along the list, so that terms on a shared mode do not commute
    desc["couplings"] = [{"i": i, "j": j, "op_i": ("n", "phi")[e % 2], "op_j": ("phi", "n")[e % 2],
                          "g": float(rng.uniform(.1, .4))} for e, (i, j) in enumerate(edges)]
    o = OracleSystem(desc)
    cols = sorted({0, o.D // 3, o.D - 1})
    g = scp.System(desc)
    psi = scp.basis_columns(g.D, cols, dtype=torch.complex128)
    U = g.propagate_trotter(psi, order)
    ref = trotter.propagate(o, order, psi0=np.eye(o.D)[:, cols].astype(complex))
    err = float(np.abs(U.cpu().numpy().T - ref).max())
    same = torch.equal(U, g.propagate_trotter(psi, order, psiT=psi))     # in place
    print(f"[trotter matrix] d={d} n={n} {order} err {err:.1e}", flush=True)
    assert err <= TOL and same
    g.close()
