"""Gather engine over the closed shapes that no other test takes: two-level
devices of 6 to 10 modes (one-entry rows, a single wave at D = 64, ten digits) in
the general, parity and real forms, and the real form's larger shapes, several
elements per thread and a partly filled last one among them.  Chains and rings,
one and two couplings on a pair, checkpoint intervals with a remainder, forward
and gradient against the CPU FP64 oracle."""
import numpy as np
import pytest

import scp_inputs as si
from oracle.adjoint import gradient
from oracle.rk4 import propagate
from oracle.system import OracleSystem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# |V| T is about 1: at most 40 rounded FP32 operations (6e-8) per evaluation on the
# way of an amplitude of at most 1
U_TOL = 40 * 6e-8
# a sensitivity is a sum of products of two such vectors, over which it may cancel by ten
GRAD_TOL = 10 * 2 * U_TOL


def _desc(d, n, form, ring, per_pair, steps):
    s = si.random_raw_system(d * 100 + n, [d] * n, n, 0.02 * steps, steps, env="gauss")
    odd = (np.add.outer(np.arange(d), np.arange(d)) % 2).astype(float)
    for m in s["modes"]:
        for k in ("n", "phi"):
            a = m["ops"][k] if form == "general" else m["ops"][k] * odd
            if form == "real":
                a = 1j * a.imag if k == "n" and n % 2 else a.real
            m["ops"][k] = np.asarray(a, dtype=np.complex128)
    pairs = [(i, i + 1) for i in range(n - 1)] + ([(n - 1, 0)] if ring else [])
    s["couplings"] = [{"i": i, "j": j, "op_i": op, "op_j": op, "g": 0.1 + 0.02 * i + 0.05 * k}
                      for i, j in pairs for k, op in enumerate(("n", "phi")[:per_pair])]
    op = "n" if n == 10 else "phi"      # at most 16 operators in a gradient's tables
    s["drives"] = [dict(r, op=op) for r in s["drives"][:max(1, n - 2)]]
    return s


CASES = ([(2, 6, f, r, p) for f in ("general", "parity", "real") for r, p in ((True, 1), (False, 2))] +
         [(2, 7, "real", False, 2), (2, 8, "real", True, 1), (2, 8, "parity", False, 1),
          (2, 9, "real", True, 1), (2, 9, "general", False, 1), (2, 10, "real", True, 1),
          (2, 10, "real", False, 1), (2, 10, "parity", True, 1), (3, 6, "real", True, 2),
          (3, 7, "real", True, 1), (3, 7, "real", False, 2), (4, 4, "real", True, 2),
          (4, 5, "real", True, 1), (4, 5, "real", False, 2), (5, 3, "real", True, 2),
          (5, 4, "real", True, 2), (5, 5, "real", True, 1), (5, 5, "real", False, 2)])


@pytest.mark.parametrize("d,n,form,ring,per_pair", CASES)
def test_forward_and_gradient(d, n, form, ring, per_pair):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_18155_amd as scp
    desc = _desc(d, n, form, ring, per_pair, 7)
    o = OracleSystem(desc)
    rng = np.random.default_rng(d * 10 + n)
    S = 3
    x, lam = ((rng.normal(size=(o.D, S)) + 1j * rng.normal(size=(o.D, S))) for _ in range(2))
    x /= np.linalg.norm(x, axis=0)
    lam /= np.linalg.norm(lam, axis=0)
    x, lam = x.astype(np.complex64).astype(complex), lam.astype(np.complex64).astype(complex)
    U_ref = propagate(o, x)
    g_ref = np.asarray(gradient(o, lam, x, 3)[0])
    g = scp.System(desc)
    assert g.real_frame == (form == "real")
    g.set_engine("gather")
    dev = lambda a: torch.tensor(np.ascontiguousarray(a.T), dtype=torch.complex64, device="cuda")  # noqa: E731
    psi0, cot = dev(x), dev(lam)
    grads = []
    for ce in (0, 1, 5):
        opts = g.opts(S, with_ckpt=1, ckpt_every=ce)
        assert g.engine(opts, with_grad=True) == "gather"
        ws = g.workspace(opts, with_grad=True)
        U = g.propagate(psi0, opts=opts, workspace=ws)
        assert torch.equal(U, g.propagate(psi0))        # without checkpoints
        grads.append(g.adjoint(cot, opts, ws, psi0=psi0))
        err = float(np.abs(U.cpu().numpy().T - U_ref).max())
        rel = float(np.abs(grads[-1] - g_ref).max() / np.abs(g_ref).max())
        print(f"[shapes] d={d} n={n} {form} ce={ce} U {err:.1e} grad {rel:.1e}", flush=True)
        assert err <= U_TOL and rel <= GRAD_TOL
        assert np.array_equal(grads[0], grads[-1])
    g.close()
