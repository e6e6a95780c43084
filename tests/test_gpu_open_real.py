"""Open systems whose terms are real and odd take kernels on the density matrix
without its frame phases: every compiled shape, chains and rings, one and two
couplings on a pair, drives on some modes, either rate absent, one step and
checkpoint intervals with a remainder, and a non-Hermitian input, each against
the CPU FP64 oracle and in both frame settings."""
import numpy as np
import pytest

import scp_inputs as si
from oracle import lindblad as lb
from oracle.system import OracleSystem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# FP32 stages of about 50 rounded terms each with |V| T below 10, a compensated
# state: 50 * 6e-8 on entries below 1; the gradient is relative to its largest
# entry (the bars of the general open-system kernels)
ENTRY_TOL = 5e-6
GRAD_TOL = 1e-4

CASES = {
    # (d, N, ring, couplings per pair, imaginary n, driven modes, gamma1, gammaphi, steps)
    "d2x3": (2, 3, True, 1, False, (0, 1, 2), 0.04, 0.02, 60),
    "d2x4_phi": (2, 4, False, 2, True, (1, 3), 0.0, 0.03, 61),
    "d2x5": (2, 5, True, 2, False, (0, 4), 0.05, 0.0, 50),
    "d3x3_ring": (3, 3, True, 2, True, (0, 2), 0.03, 0.02, 70),
    "d3x3_one_step": (3, 3, False, 1, False, (1,), 0.03, 0.02, 1),
    "d3x4_chain": (3, 4, False, 2, True, (0, 2), 0.03, 0.02, 37),
    "d3x4_ring": (3, 4, True, 1, False, (0, 1, 2, 3), 0.04, 0.01, 26),
    "d3x4_no_rates": (3, 4, True, 2, False, (3,), 0.0, 0.0, 10),
    "d4x3": (4, 3, True, 2, True, (0, 1, 2), 0.03, 0.02, 40),
    "d4x3_undriven": (4, 3, False, 1, False, (), 0.03, 0.02, 17),
}


def _desc(d, n, ring, per_pair, imag, driven, g1, gp, steps):
    T = 0.02 * steps
    s = si.random_raw_system(d * 100 + n * 10 + steps, [d] * n, n, T, steps, env="gauss")
    odd = (np.add.outer(np.arange(d), np.arange(d)) % 2).astype(float)
    for k, m in enumerate(s["modes"]):
        n_op, p_op = m["ops"]["n"] * odd, m["ops"]["phi"] * odd
        m["ops"]["n"] = (1j * n_op.imag if imag else n_op.real).astype(np.complex128)
        m["ops"]["phi"] = p_op.real.astype(np.complex128)
        m["gamma1"], m["gammaphi"] = g1 * (1 + 0.3 * k), gp * (1 + 0.2 * k)
    pairs = [(i, i + 1) for i in range(n - 1)] + ([(n - 1, 0)] if ring else [])
    s["couplings"] = [{"i": i, "j": j, "op_i": op, "op_j": op, "g": 0.1 + 0.03 * i + 0.05 * k}
                      for i, j in pairs for k, op in enumerate(("n", "phi")[:per_pair])]
    s["drives"] = [dict(s["drives"][m], op="phi") for m in driven]
    return s


@pytest.mark.parametrize("name", sorted(CASES))
def test_states_and_gradient_match_oracle(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_18155_amd as scp
    desc = _desc(*CASES[name])
    sys_ = OracleSystem(desc)
    rng = np.random.Generator(np.random.PCG64(5))
    shape = (2, sys_.D, sys_.D)
    rho0 = rng.normal(size=shape) + 1j * rng.normal(size=shape)
    rho0 /= 4 * np.abs(rho0).max()
    lam = rng.normal(size=shape) + 1j * rng.normal(size=shape)
    ref, g_ref = lb.propagate(sys_, rho0), lb.gradient(sys_, lam, rho0)
    g = scp.System(desc)
    assert g.real_frame
    x = torch.tensor(rho0, dtype=torch.complex64, device="cuda").contiguous()
    c = torch.tensor(lam, dtype=torch.complex64, device="cuda").contiguous()
    for real in (True, False):
        g.set_real_frame(real)
        print(f"[open] {name} real={real}", flush=True)
        out = g.propagate_lindblad(x).cpu().numpy()
        grad = g.lindblad_adjoint(x, c)
        err = np.abs(out - ref).max()
        rel = np.abs(grad - g_ref).max() / np.abs(g_ref).max()
        print(f"[open] {name} real={real} rho {err:.1e} grad {rel:.1e}", flush=True)
        assert err <= ENTRY_TOL and rel <= GRAD_TOL
    g.close()
