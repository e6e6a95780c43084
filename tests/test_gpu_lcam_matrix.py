"""LCAM where the sweep runs in the matrix form (three modes and more of four and
five levels, several pairs): one pass and two, three pieces, a short last slot, one
column and many, against the CPU FP64 oracle; both entries bitwise equal; several
rounds against one walk of all columns (a gradient is the sum of its columns')."""
import numpy as np
import pytest

import scp_inputs as si
from oracle import lcam
from oracle.system import OracleSystem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# FP64 throughout: some 10^5 rounded operations of 1e-16 relative size per
# amplitude, and cancellation in the reduced matrices
TOL = 1e-9


@pytest.fixture(scope="module")
def scp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_18155_amd as m
    return m


def _case(n, d, S, N):
    s = si.fluxonium_chain(si.rng_for(8, N), n, d, 0.02 * N, N, n_basis_gauss=3, amp=0.03,
                           drive_modes=(0, n - 1))
    rng = np.random.default_rng(S + N)
    x, lam = ((rng.normal(size=(d ** n, S)) + 1j * rng.normal(size=(d ** n, S))) for _ in range(2))
    return si._finish(s, [d] * n, target=si.cz_target(n)), x / np.linalg.norm(x, axis=0), lam


def dev(a):
    return torch.tensor(np.ascontiguousarray(a.T), device="cuda")


@pytest.mark.parametrize("order,n,d,S,N", [("q1", 3, 4, 100, 7), ("q2", 3, 4, 100, 7), ("q4", 3, 4, 60, 7),
                                           ("q1", 3, 5, 100, 7), ("q2", 3, 5, 60, 7), ("q4", 3, 5, 3, 7),
                                           ("q1", 3, 4, 1, 1), ("q2", 4, 4, 2, 9)])
def test_gradient(scp, order, n, d, S, N):
    desc, x, lam = _case(n, d, S, N)
    o = OracleSystem(desc)
    ref = lcam.gradient(o, order, lam, x)
    g = scp.System(desc)
    got = g.trotter_adjoint(dev(x), dev(lam), order)
    fin = g.trotter_adjoint_final(g.propagate_trotter(dev(x), order), dev(lam), order)
    rel = np.abs(got - ref).max() / np.abs(ref).max()
    print(f"[lcam matrix] {order} n={n} d={d} S={S} N={N} rel {rel:.1e}", flush=True)
    assert rel <= TOL and np.array_equal(got, fin)
    g.close()


# rounds of 3 x 64 steps (100 columns) and 10 x 20 or 10 x 40 (28)
@pytest.mark.parametrize("order", ["q1", "q2", "q4"])
@pytest.mark.parametrize("d,N", [(4, 200), (4, 400), (5, 200)])
def test_rounds_add_up_to_one_walk(scp, order, d, N):
    desc, x, lam = _case(3, d, 128, N)
    g = scp.System(desc)
    parts = [g.trotter_adjoint(dev(x[:, a:b]), dev(lam[:, a:b]), order) for a, b in ((0, 100), (100, 128))]
    ref = g.trotter_adjoint(dev(x), dev(lam), order)
    rel = np.abs(sum(parts) - ref).max() / np.abs(ref).max()
    print(f"[lcam matrix] rounds {order} d={d} N={N} rel {rel:.1e}", flush=True)
    assert rel <= TOL
    g.close()
