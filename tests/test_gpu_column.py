"""Forward of closed systems of eight three-level modes (D = 6561) whose terms
are real and odd: one workgroup per column, the elements of the first two modes'
digits within a thread.  Chains and rings, one and two couplings on a pair,
undriven modes, one step and many, columns of any number and in place, against
the CPU FP64 oracle; the frame switch returns to the general stepper on the same
workspace."""
import numpy as np
import pytest

import scp_inputs as si
from oracle.rk4 import propagate
from oracle.system import OracleSystem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# |V| T stays below 10; at most 40 rounded FP32 terms per evaluation (6e-8 each)
U_TOL = 2e-5


def _desc(ring, per_pair, imag, driven, steps):
    s = si.random_raw_system(80 + steps, [3] * 8, 8, 0.02 * steps, steps, env="gauss")
    odd = (np.add.outer(np.arange(3), np.arange(3)) % 2).astype(float)
    for m in s["modes"]:
        n_op, p_op = m["ops"]["n"] * odd, m["ops"]["phi"] * odd
        m["ops"]["n"] = (1j * n_op.imag if imag else n_op.real).astype(np.complex128)
        m["ops"]["phi"] = p_op.real.astype(np.complex128)
    pairs = [(i, i + 1) for i in range(7)] + ([(7, 0)] if ring else [])
    s["couplings"] = [{"i": i, "j": j, "op_i": op, "op_j": op, "g": 0.1 + 0.02 * i + 0.05 * k}
                      for i, j in pairs for k, op in enumerate(("n", "phi")[:per_pair])]
    s["drives"] = [dict(s["drives"][m], op="phi") for m in driven]
    return s


@pytest.mark.parametrize("ring,per_pair,imag,driven,steps,S", [
    (True, 1, False, range(8), 20, 3), (False, 2, True, (0, 1, 5), 11, 2),
    (True, 2, True, (2, 7), 1, 1), (False, 1, False, (), 6, 2)])
def test_forward_matches_the_oracle(ring, per_pair, imag, driven, steps, S):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_18155_amd as scp
    desc = _desc(ring, per_pair, imag, driven, steps)
    o = OracleSystem(desc)
    rng = np.random.default_rng(S)
    x = rng.normal(size=(o.D, S)) + 1j * rng.normal(size=(o.D, S))
    x /= np.linalg.norm(x, axis=0)
    ref = propagate(o, x)
    g = scp.System(desc)
    assert g.real_frame
    psi = torch.tensor(np.ascontiguousarray(x.T), dtype=torch.complex64, device="cuda")
    opts = g.opts(S)
    ws = g.workspace(opts)
    for real in (True, False):
        g.set_real_frame(real)
        U = g.propagate(psi, opts=opts, workspace=ws)
        err = float(np.abs(U.cpu().numpy().T - ref).max())
        print(f"[column] ring={ring} steps={steps} real={real} {err:.1e}", flush=True)
        assert err <= U_TOL
    g.set_real_frame(True)
    U = g.propagate(psi)
    assert torch.equal(U, g.propagate(psi, psiT=psi))
    g.close()
