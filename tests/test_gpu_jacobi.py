"""The one-workgroup eigensolver at the edges of its sizes: the smallest bases,
odd ones (one level rests per round), and the largest, through the dressed
energies of two coupled modes (vectors enter through the coupling), against
the CPU FP64 oracle."""
import numpy as np
import pytest

from oracle.spectrum import dressed_energies
from oracle.system import OracleSystem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# Jacobi's backward error is below K * sweeps * 1e-16 of the matrix norm:
# 96 * 10 * 1e-16 = 1e-13; the coupling adds as much again through the vectors
TOL = 1e-12


def _transmon(ncut, trunc):
    return {"kind": "transmon", "EC": 1.3, "EJ": 60.0, "ng": 0.1, "basis_dim": 2 * ncut + 1,
            "trunc": trunc}, 4 * 1.3 * (ncut + 0.1) ** 2 + 60.0


def _fluxonium(K, trunc):
    return {"kind": "fluxonium", "EC": 7.0, "EJ": 28.0, "EL": 4.0, "phiext": 2.9, "basis_dim": K,
            "trunc": trunc}, np.sqrt(8 * 7.0 * 4.0) * K + 28.0


@pytest.mark.parametrize("a,b", [(("t", 1, 2), ("t", 1, 2)), (("t", 2, 3), ("f", 4, 3)),
                                 (("f", 7, 5), ("t", 10, 5)), (("f", 33, 3), ("f", 80, 3)),
                                 (("f", 95, 5), ("f", 96, 5)), (("t", 47, 5), ("f", 65, 5))])
def test_dressed_energies_match_the_oracle(a, b):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_18155_amd as scp
    print(f"[jacobi] {a} {b}", flush=True)
    made = [(_transmon if k == "t" else _fluxonium)(n, t) for k, n, t in (a, b)]
    desc = {"modes": [m for m, _ in made], "drives": [], "T": 1.0, "n_steps": 1,
            "couplings": [{"i": 0, "j": 1, "op_i": "n", "op_j": "n", "g": 0.3}]}
    # n is imaginary in a fluxonium's basis and real in a transmon's: such a
    # mixed pair has a complex Hamiltonian, so it stays uncoupled here
    if a[0] != b[0]:
        desc["couplings"] = []
    g = scp.System(desc)
    E = g.energy_tensor()
    g.close()
    Eo = dressed_energies(OracleSystem(desc))[0]
    assert np.abs(E - Eo).max() <= TOL * max(s for _, s in made)
