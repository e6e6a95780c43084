"""The LCAM walk in slots side by side: the gradient against the CPU FP64
oracle where the split into rounds and slots can go wrong (fewer steps than
slots, a last slot or round that is short, one column, the most columns that
take slots), and both entries bitwise equal."""
import numpy as np
import pytest

import scp_inputs as si
from oracle import lcam, trotter
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


@pytest.mark.parametrize("order,n,d,S,N", [("q2", 2, 3, 1, 1), ("q2", 2, 3, 1, 2), ("q1", 3, 3, 1, 300),
                                           ("q4", 2, 4, 5, 33), ("q2", 2, 5, 100, 200),
                                           ("q2", 3, 2, 127, 130), ("q2", 2, 3, 128, 70)])
def test_gradient(scp, order, n, d, S, N):
    s = si.fluxonium_chain(si.rng_for(8, N), n, d, 0.02 * N, N, n_basis_gauss=3, amp=0.03,
                           drive_modes=(0,))
    desc = si._finish(s, [d] * n, target=si.cz_target(n))
    o = OracleSystem(desc)
    rng = np.random.default_rng(S + N)
    x = rng.normal(size=(o.D, S)) + 1j * rng.normal(size=(o.D, S))
    lam = rng.normal(size=(o.D, S)) + 1j * rng.normal(size=(o.D, S))
    x /= np.linalg.norm(x, axis=0)
    ref = lcam.gradient(o, order, lam, x)
    g = scp.System(desc)
    dev = lambda a: torch.tensor(np.ascontiguousarray(a.T), device="cuda")
    got = g.trotter_adjoint(dev(x), dev(lam), order)
    fin = g.trotter_adjoint_final(g.propagate_trotter(dev(x), order), dev(lam), order)
    rel = np.abs(got - ref).max() / np.abs(ref).max()
    print(f"[lcam slots] {order} n={n} d={d} S={S} N={N} rel {rel:.1e}", flush=True)
    assert rel <= TOL and np.array_equal(got, fin)
    g.close()
