"""The automatic engine of a real device with odd operators: the gather engine up
to as many columns as it wins with, fewer for a gradient than for a forward where
a gradient's workgroups go in rounds; checkpoints are written by the engine that
the gradient runs on."""
import pytest

import scp_inputs as si

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n,fwd,grad", [(3, 4, 1024, 1024), (2, 9, 1024, 1024), (2, 10, 1024, 512),
                                          (3, 6, 1024, 768), (4, 5, 1024, 1024), (4, 6, 256, 256),
                                          (5, 5, 256, 128)])
def test_columns_of_the_gather_engine(d, n, fwd, grad):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2406_18155_amd as scp
    s = si.transmon_ring(si.rng_for(7, d * 100 + n), n, d, 0.1, 5)
    g = scp.System(si._finish(s, [d] * n, target=si.cz_target(n)))
    for most, opts, with_grad in ((fwd, {}, False), (grad, {"with_ckpt": 1}, False),
                                  (grad, {"with_ckpt": 1}, True), (grad, {}, True)):
        assert g.engine(g.opts(most, **opts), with_grad) == "gather"
        assert g.engine(g.opts(most + 1, **opts), with_grad) == "register"
    S = grad + 1
    x = torch.zeros(S, g.D, dtype=torch.complex64, device="cuda")
    x[:, 0] = 1
    opts = g.opts(S, with_ckpt=1)
    ws = g.workspace(opts, with_grad=True)
    U = g.propagate(x, opts=opts, workspace=ws)
    a, b = g.adjoint(U, opts, ws), g.adjoint(U, opts, ws, psi0=x)
    assert (a == b).all()
    g.close()
