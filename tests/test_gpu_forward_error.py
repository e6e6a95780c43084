"""Error of the forwards that run in another manner than the step-by-step ones
(split over time, real form, column kernel) at the size FP32 with a compensated
state allows, against the CPU FP64 oracle."""
import numpy as np
import pytest

import scp_inputs as si
from oracle.rk4 import propagate
from oracle.system import OracleSystem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# A coefficient's rounding repeats at every step and turns into an error of the
# angle of |V| T 6e-8 at most; the roundings of the evaluations are independent and
# together smaller.  |V| T <= 8 here (couplings of 0.3, drives of 0.4, operators of
# norm 2 and less, T = 1).
TOL = 2 * 8 * 6e-8


@pytest.mark.parametrize("d,n,n_steps,S", [(2, 1, 64, 1), (4, 2, 64, 16), (4, 2, 257, 5), (3, 3, 513, 3),
                                           (2, 5, 300, 40), (5, 2, 1000, 2), (3, 4, 50, 5), (4, 5, 30, 2),
                                           (5, 4, 30, 2), (3, 7, 20, 2), (4, 6, 20, 2), (3, 8, 20, 2)])
def test_error_of_the_final_states(d, n, n_steps, S):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_18155_amd as scp
    s = si.random_raw_system(d * 10 + n, [d] * n, n if n > 2 else n - 1, 1.0, n_steps, env="gauss")
    odd = (np.add.outer(np.arange(d), np.arange(d)) % 2).astype(float)
    for m in s["modes"]:
        for k in m["ops"]:
            m["ops"][k] = (m["ops"][k].real * odd).astype(np.complex128)
    for c in s["couplings"]:
        c["op_j"] = c["op_i"]
    o = OracleSystem(s)
    rng = np.random.default_rng(S)
    x = rng.normal(size=(o.D, S)) + 1j * rng.normal(size=(o.D, S))
    x = (x / np.linalg.norm(x, axis=0)).astype(np.complex64).astype(complex)
    g = scp.System(s)
    assert g.real_frame
    U = g.propagate(torch.tensor(np.ascontiguousarray(x.T), dtype=torch.complex64, device="cuda"))
    err = float(np.abs(U.cpu().numpy().T - propagate(o, x)).max())
    print(f"[error] d={d} n={n} N={n_steps} {err:.1e}", flush=True)
    assert err <= TOL
    g.close()
