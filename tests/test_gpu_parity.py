"""Devices whose operators connect levels of unlike parity only (transmons at
n_g = 0, fluxoniums at half flux, raw modes given so) take kernels that leave
the zero entries out; every other device takes the general ones.  Both against
the CPU FP64 oracle, on either side of the rule, on both engines."""
import copy
import math

import numpy as np
import pytest

import scp_inputs as si
from oracle.adjoint import loss_and_grad
from oracle.system import OracleSystem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# FP32 stages: at most 4 n_steps evaluations of about 30 rounded terms each,
# every one scaled by h |V|; with |V| T below 10 the worst case is 30 * 6e-8 * 10
U_TOL = 2e-5
GRAD_TOL = 1e-4


@pytest.fixture(scope="module")
def scp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_18155_amd as m
    return m


def _raw(d, n, real, even):
    """n raw modes of d levels, odd operators; ``even``: their (0, 0) entry
    relative to the largest entry."""
    s = si.random_raw_system(d * 10 + n, [d] * n, n - 1 if n < 3 else n, 4.0, 60, env="gauss")
    mask = (np.add.outer(np.arange(d), np.arange(d)) % 2).astype(float)
    for m in s["modes"]:
        for k in m["ops"]:
            a = m["ops"][k] * mask
            a = (a.real if real else a).astype(np.complex128)
            a[0, 0] = even * np.abs(a).max()
            m["ops"][k] = a
    return s


def _biased(kind):
    if kind == "transmon":
        s = si.transmon_ring(si.rng_for(7, 3), 4, 3, 4.0, 100)
        for m in s["modes"]:
            m["ng"] = 0.2
    else:
        s = si.fluxonium_chain(si.rng_for(8, 3), 3, 4, 4.0, 100, n_basis_gauss=3, amp=0.03)
        for m in s["modes"]:
            m["phiext"] = 0.93 * math.pi
    d = s["modes"][0]["trunc"]
    return si._finish(s, [d] * len(s["modes"]), target=si.cz_target(len(s["modes"])))


def _check(scp, desc, engine):
    L, F, tau, U_ref, g_ref = loss_and_grad(OracleSystem(desc))
    g = scp.System(desc)
    if engine == "gather" and (g.D < 64 or g.d == 2):
        g.close()
        pytest.skip("the gather engine takes D >= 64 and d >= 3")
    g.set_engine(engine)
    psi0 = scp.basis_columns(g.D, desc["columns"])
    opts = g.opts(psi0.shape[0], with_ckpt=1)
    ws = g.workspace(opts, with_grad=True)
    for real in ((True, False) if g.real_frame else (False,)):
        if g.real_frame != real:
            g.set_real_frame(real)
        U = g.propagate(psi0, opts=opts, workspace=ws)
        cot = torch.empty_like(U)
        scp.fidelity(U, scp.Target(desc["comp_rows"], desc["comp_cols"], desc["target"]),
                     cotangent=cot)
        grad = g.adjoint(cot, opts, ws)
        err = float(np.abs(U.cpu().numpy().T - U_ref).max())
        rel = float(np.abs(grad - g_ref).max() / np.abs(g_ref).max())
        print(f"[parity] {engine} real={real} U {err:.1e} grad {rel:.1e}", flush=True)
        assert err <= U_TOL and rel <= GRAD_TOL
    g.close()


@pytest.mark.parametrize("engine", ["register", "gather"])
@pytest.mark.parametrize("even", [0.0, 1e-9, 0.3])   # 0: odd operators; the others: not
@pytest.mark.parametrize("d,n,real", [(2, 2, True), (2, 6, False), (3, 3, True), (3, 4, False),
                                      (4, 2, True), (4, 3, False), (5, 2, False), (5, 3, True)])
def test_raw_modes_on_either_side_of_the_rule(scp, d, n, real, even, engine):
    _check(scp, _raw(d, n, real, even), engine)


@pytest.mark.parametrize("engine", ["register", "gather"])
@pytest.mark.parametrize("kind", ["transmon", "fluxonium"])
def test_biased_devices(scp, kind, engine):
    _check(scp, _biased(kind), engine)
