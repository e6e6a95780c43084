"""A raw mode's operators are taken as they are given: a NaN or an infinity in
any of their entries, also one between levels of like parity, makes the result
non-finite on every path (the kernels that leave such entries out run only
where they are zero)."""
import numpy as np
import pytest

import scp_inputs as si

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def scp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_18155_amd as m
    return m


# split over time, gather engine and its real form, column kernel
@pytest.mark.parametrize("d,n,n_steps", [(4, 2, 64), (3, 4, 10), (4, 4, 10), (3, 8, 3)])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("engine", ["auto", "register"])
def test_bad_even_entry_reaches_the_result(scp, d, n, n_steps, bad, engine):
    s = si.random_raw_system(d * 10 + n, [d] * n, n if n > 2 else 1, 0.05 * n_steps, n_steps, env="gauss")
    odd = (np.add.outer(np.arange(d), np.arange(d)) % 2).astype(float)
    for m in s["modes"]:
        for k in m["ops"]:
            m["ops"][k] = (m["ops"][k].real * odd).astype(np.complex128)
    for c in s["couplings"]:
        c["op_i"] = c["op_j"] = "n"
    s["modes"][0]["ops"]["n"][0, 0] = bad
    print(f"[nonfinite] d={d} n={n} {bad} {engine}", flush=True)
    g = scp.System(s)
    g.set_engine(engine)
    psi = scp.basis_columns(g.D, [0, 1])
    assert not torch.isfinite(torch.view_as_real(g.propagate(psi))).all()
    opts = g.opts(2, with_ckpt=1)
    with pytest.raises(scp.ScpError, match="ENONFINITE"):
        g.adjoint(psi, opts, g.workspace(opts, with_grad=True), psi0=psi)
    g.close()
