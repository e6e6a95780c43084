"""Forward of a small device (D < 64) split over time: against the CPU FP64
oracle at the edges of its split (the fewest steps, one step per run, runs of
unequal length, groups of one), every compiled d, one column and many, in place,
modes of different truncations."""
import numpy as np
import pytest

import scp_inputs as si
from oracle.rk4 import propagate
from oracle.system import OracleSystem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# |V| T stays below 10; at most 30 rounded FP32 terms per evaluation (6e-8 each)
U_TOL = 2e-5


@pytest.fixture(scope="module")
def scp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_18155_amd as m
    return m


def _check(scp, desc, S):
    o = OracleSystem(desc)
    rng = np.random.default_rng(S)
    x = rng.normal(size=(o.D, S)) + 1j * rng.normal(size=(o.D, S))
    x /= np.linalg.norm(x, axis=0)
    ref = propagate(o, x)
    g = scp.System(desc)
    psi = torch.tensor(np.ascontiguousarray(x.T), dtype=torch.complex64, device="cuda")
    U = g.propagate(psi)
    g.set_engine("register")
    V = g.propagate(psi)                      # the serial chain of steps
    g.set_engine("auto")
    same = torch.equal(U, g.propagate(psi, psiT=psi))
    err = float(np.abs(U.cpu().numpy().T - ref).max())
    print(f"[split] D={o.D} N={desc['n_steps']} S={S} err {err:.1e}", flush=True)
    assert err <= U_TOL and float((U - V).abs().max()) <= U_TOL and same
    g.close()


@pytest.mark.parametrize("n_steps,S", [(63, 3), (64, 1), (65, 16), (257, 5), (300, 40), (513, 2)])
def test_edges_of_the_split(scp, n_steps, S):
    s = si.transmon_ring(si.rng_for(7, 1), 2, 4, 0.02 * n_steps, n_steps)
    _check(scp, si._finish(s, [4, 4], target=si.cz_target(2)), S)


@pytest.mark.parametrize("dims", [(2,), (2, 2, 2, 2, 2), (3, 3, 3), (4, 4), (5, 5), (5,)])
@pytest.mark.parametrize("S", [1, 70])
def test_shapes(scp, dims, S):
    s = si.random_raw_system(len(dims) * 10 + dims[0], list(dims), len(dims) - 1, 4.0, 100, env="gauss")
    _check(scp, s, S)


def test_other_envelopes(scp):
    # piecewise-constant pulses change within and at the ends of the runs
    _check(scp, si.random_raw_system(3, [3, 3], 1, 3.0, 150, env="pwc", n_pieces=7), 9)
