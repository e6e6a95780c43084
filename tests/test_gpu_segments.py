"""The gather engine walks checkpoint segments side by side after a costate
sweep: the gradient against the CPU FP64 oracle where the split can go wrong
(one column, one segment, segments of one step, an interval beyond the run,
more columns than fill a round, a step count that no block size divides)."""
import numpy as np
import pytest

import scp_inputs as si
from oracle.adjoint import gradient
from oracle.system import OracleSystem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GRAD_TOL = 1e-4


@pytest.fixture(scope="module")
def scp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_18155_amd as m
    return m


@pytest.mark.parametrize("n_steps", [1, 3, 65])
@pytest.mark.parametrize("S,ce", [(1, 0), (1, 1), (5, 4), (64, 7), (64, 70), (300, 1), (300, 13)])
def test_gradient_of_a_random_costate(scp, S, ce, n_steps):
    s = si.fluxonium_chain(si.rng_for(8, 5), 3, 4, 0.02 * n_steps, n_steps, n_basis_gauss=3, amp=0.03,
                           drive_modes=(0, 2))
    desc = si._finish(s, [4] * 3, target=si.cz_target(3))
    rng = np.random.default_rng(S * 100 + ce)
    o = OracleSystem(desc)
    x = rng.normal(size=(o.D, S)) + 1j * rng.normal(size=(o.D, S))
    lam = rng.normal(size=(o.D, S)) + 1j * rng.normal(size=(o.D, S))
    x /= np.linalg.norm(x, axis=0)
    lam /= np.linalg.norm(lam, axis=0)
    ref, _ = gradient(o, lam, x)
    g = scp.System(desc)
    g.set_engine("gather")
    opts = g.opts(S, ckpt_every=ce, with_ckpt=1)
    ws = g.workspace(opts, with_grad=True)
    dev = lambda a: torch.tensor(np.ascontiguousarray(a.T), dtype=torch.complex64, device="cuda")
    g.propagate(dev(x), opts=opts, workspace=ws)
    a = g.adjoint(dev(lam), opts, ws)
    b = g.adjoint(dev(lam), opts, ws)          # the checkpoints serve again
    assert np.array_equal(a, b)
    rel = np.abs(a - ref).max() / np.abs(ref).max()
    print(f"[segments] S={S} ce={ce} N={n_steps} rel {rel:.1e}", flush=True)
    assert rel <= GRAD_TOL
    g.close()
