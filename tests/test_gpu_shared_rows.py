"""Gather engine, real form, six four-level modes (D = 4096): a thread's four
elements differ in the first mode's digit alone and share the other modes' rows.
Chains and rings (the wrap pair reads along the first mode too), one and two
couplings on a pair, the first mode driven or not, real and imaginary operators,
checkpoint intervals with a remainder, against the CPU FP64 oracle; the gradient
does not depend on the interval."""
import numpy as np
import pytest

import scp_inputs as si
from oracle.adjoint import loss_and_grad
from oracle.system import OracleSystem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# |V| T stays below 10; at most 40 rounded FP32 terms per evaluation (6e-8 each)
U_TOL = 2e-5
GRAD_TOL = 1e-4


def _desc(ring, per_pair, imag, driven, steps):
    s = si.random_raw_system(60 + steps, [4] * 6, 6, 0.02 * steps, steps, env="gauss")
    odd = (np.add.outer(np.arange(4), np.arange(4)) % 2).astype(float)
    for m in s["modes"]:
        n_op, p_op = m["ops"]["n"] * odd, m["ops"]["phi"] * odd
        m["ops"]["n"] = (1j * n_op.imag if imag else n_op.real).astype(np.complex128)
        m["ops"]["phi"] = p_op.real.astype(np.complex128)
    pairs = [(i, i + 1) for i in range(5)] + ([(5, 0)] if ring else [])
    s["couplings"] = [{"i": i, "j": j, "op_i": op, "op_j": op, "g": 0.1 + 0.02 * i + 0.05 * k}
                      for i, j in pairs for k, op in enumerate(("n", "phi")[:per_pair])]
    s["drives"] = [dict(s["drives"][m], op="phi") for m in driven]
    return s


@pytest.mark.parametrize("ring,per_pair,imag,driven,steps", [
    (True, 2, True, (0, 3), 11), (True, 1, False, range(6), 7), (False, 2, False, (2, 5), 5),
    (False, 1, True, (0,), 1)])
def test_forward_and_gradient_match_the_oracle(ring, per_pair, imag, driven, steps):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_18155_amd as scp
    desc = _desc(ring, per_pair, imag, driven, steps)
    L, F, tau, U_ref, g_ref = loss_and_grad(OracleSystem(desc))
    g = scp.System(desc)
    assert g.real_frame
    psi0 = scp.basis_columns(g.D, desc["columns"])
    grads = []
    for ce in (0, 1, 4):
        opts = g.opts(psi0.shape[0], with_ckpt=1, ckpt_every=ce)
        assert g.engine(opts, with_grad=True) == "gather"
        ws = g.workspace(opts, with_grad=True)
        U = g.propagate(psi0, opts=opts, workspace=ws)
        cot = torch.empty_like(U)
        scp.fidelity(U, scp.Target(desc["comp_rows"], desc["comp_cols"], desc["target"]),
                     cotangent=cot)
        grads.append(g.adjoint(cot, opts, ws))
        err = float(np.abs(U.cpu().numpy().T - U_ref).max())
        rel = float(np.abs(grads[-1] - g_ref).max() / np.abs(g_ref).max())
        print(f"[shared] ring={ring} ce={ce} U {err:.1e} grad {rel:.1e}", flush=True)
        assert err <= U_TOL and rel <= GRAD_TOL
        assert np.array_equal(grads[0], grads[-1])
    g.close()
