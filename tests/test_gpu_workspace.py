"""Workspaces below the size of a call's own path: one made for the gradient does
for a forward, one for more columns does for fewer, and the register-layout
stepper's size always does, with that engine's results bit for bit; the gather
engine's adjoint runs with fewer segments side by side, with the same result."""
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


def _device(scp, d, n, n_steps, ng=0.0):
    s = si.transmon_ring(si.rng_for(7, d * 100 + n), n, d, 0.02 * n_steps, n_steps)
    for m in s["modes"]:
        m["ng"] = ng
    print(f"[workspace] d={d} n={n} N={n_steps} ng={ng}", flush=True)
    return scp.System(si._finish(s, [d] * n, target=si.cz_target(n)))


def _columns(g, S, seed=1):
    gen = torch.Generator().manual_seed(seed)
    x = torch.randn(S, g.D, 2, generator=gen)
    return torch.view_as_complex(x / x.norm(dim=(1, 2), keepdim=True)).contiguous().cuda()


def _bytes(n):
    return torch.empty(n, dtype=torch.uint8, device="cuda")


# time split, column kernel, gather engine
@pytest.mark.parametrize("d,n,S,n_steps", [(4, 2, 16, 1000), (3, 8, 1, 40), (4, 3, 8, 30)])
def test_gradient_workspace_does_for_the_forward(scp, d, n, S, n_steps):
    g = _device(scp, d, n, n_steps)
    opts = g.opts(S, with_ckpt=1)
    ws = g.workspace(opts, with_grad=True)
    for k in (S, max(1, S // 2)):
        x = _columns(g, k)
        U = g.propagate(x, opts=g.opts(k), workspace=ws)
        V = g.propagate(x, opts=g.opts(k, with_ckpt=1), workspace=ws)
        assert (U - V).abs().max().item() <= 2e-5   # paths differ by FP32 rounding
    g.close()


# columns on either side of the automatic choice
@pytest.mark.parametrize("d,n,most,fewer", [(4, 6, 257, 256), (3, 5, 1025, 1000), (3, 4, 300, 1)])
@pytest.mark.parametrize("grad", [False, True])
def test_workspace_for_more_columns_does_for_fewer(scp, d, n, most, fewer, grad):
    g = _device(scp, d, n, 64)
    ws = g.workspace(g.opts(most, with_ckpt=int(grad)), with_grad=grad)
    x = _columns(g, fewer)
    opts = g.opts(fewer, with_ckpt=int(grad))
    U = g.propagate(x, opts=opts, workspace=ws)
    if grad:
        g.adjoint(_columns(g, fewer, 2), opts, ws)
    assert torch.isfinite(torch.view_as_real(U)).all()
    g.close()


@pytest.mark.parametrize("d,n,S,n_steps,ng", [(4, 2, 16, 100, 0.0), (3, 4, 5, 40, 0.0), (3, 4, 5, 40, 0.2),
                                              (4, 4, 20, 30, 0.0), (3, 8, 2, 10, 0.0)])
def test_register_size_always_does(scp, d, n, S, n_steps, ng):
    g = _device(scp, d, n, n_steps, ng)
    x, cot = _columns(g, S), _columns(g, S, 2)

    def near(a, b, tol):   # either engine ran; they differ by FP32 rounding
        return (abs(a - b)).max() <= tol * abs(b).max()

    for ckpt, grad in ((0, False), (1, False), (1, True)):
        g.set_engine("register")
        opts = g.opts(S, with_ckpt=ckpt)
        ws = g.workspace(opts, with_grad=grad)
        U = g.propagate(x, opts=opts, workspace=ws)
        ref = g.adjoint(cot, opts, ws) if grad else None
        g.set_engine("auto")
        assert near(g.propagate(x, opts=opts, workspace=ws), U, 2e-5)
        if grad:
            assert near(g.adjoint(cot, opts, ws), ref, 1e-4)
            assert near(g.adjoint(cot, opts, ws, psi0=x), ref, 1e-4)
        tiny = ws[:ws.numel() // 2 if ckpt else 64]
        with pytest.raises(scp.ScpError, match="EINVAL.*workspace_bytes"):
            if grad:
                g.adjoint(cot, opts, tiny, psi0=x)
            else:
                g.propagate(x, opts=opts, workspace=tiny)
    # an adjoint takes the engine that wrote its checkpoints, whatever it has room for
    room = _bytes(max(g.workspace_bytes(opts, True), ws.numel()))
    g.propagate(x, opts=opts, workspace=room[:ws.numel()])
    assert near(g.adjoint(cot, opts, room), ref, 1e-4)
    g.close()


@pytest.mark.parametrize("d,n,S,ng", [(3, 4, 5, 0.0), (3, 4, 5, 0.2), (3, 7, 2, 0.0)])
def test_adjoint_with_fewer_segments(scp, d, n, S, ng):
    g = _device(scp, d, n, 40, ng)
    x, cot = _columns(g, S), _columns(g, S, 2)
    opts = g.opts(S, with_ckpt=1)
    assert g.engine(opts, with_grad=True) == "gather"
    full = g.workspace_bytes(opts, with_grad=True)
    ref = g.adjoint(cot, opts, _bytes(full), psi0=x)
    g.set_engine("gather")                             # no other engine to fall back on
    ws = _bytes(full)
    seg = S * 7 * 4 * g.D * 8                          # ceil(sqrt(40)) steps; six segments
    for k in range(1, 6):
        assert (ref == g.adjoint(cot, opts, ws[:full - k * seg + 255], psi0=x)).all()
    with pytest.raises(scp.ScpError, match="EINVAL.*workspace_bytes"):
        g.adjoint(cot, opts, ws[:full - 6 * seg], psi0=x)
    g.close()


def test_forward_workspace_of_the_column_kernel_is_bounded(scp):
    sizes = []
    for n_steps in (4000, 20000):
        g = _device(scp, 3, 8, n_steps)
        sizes.append(g.workspace_bytes(g.opts(3)))
        g.close()
    assert sizes[0] == sizes[1]


# the real form's forward goes in runs of steps, 4096 of them at D = 4096: one
# step in the last run, a run and a remainder, three runs
@pytest.mark.parametrize("n_steps", [4096, 4097, 5000, 8193])
def test_runs_of_steps_leave_no_trace(scp, n_steps):
    g = _device(scp, 4, 6, n_steps)
    S = 3
    x = _columns(g, S)
    opts = g.opts(S, with_ckpt=1)
    assert g.engine(opts) == "gather"
    U = g.propagate(x, opts=opts)                     # checkpoints: one run
    V = g.propagate(x, opts=g.opts(S))
    assert torch.equal(U, V) and torch.equal(V, g.propagate(x, psiT=x, opts=g.opts(S)))
    g.close()


def test_runs_of_steps_of_the_column_kernel(scp):
    g = _device(scp, 3, 8, 2700)                      # a run of 2557 steps and the rest
    x = _columns(g, 3)
    U = g.propagate(x)
    ref = g.propagate(x.to(torch.complex128)).to(torch.complex64)
    # amplitudes of about 0.01 (random columns of 6561), |V| T below 50, a few rounded
    # FP32 operations (6e-8) per evaluation: 0.01 * 50 * 10 * 6e-8
    assert (U - ref).abs().max().item() <= 3e-7
    g.close()


def _open_device(scp):
    s = si.transmon_ring(si.rng_for(7, 3), 3, 3, 1.0, 50)
    s = si.with_rates(s, si.open_rates(si.rng_for(9, 1), 3))
    return scp.System(si._finish(s, [3] * 3, target=si.cz_target(3)))


def test_open_system_in_the_size_of_the_tables(scp):
    g = _open_device(scp)
    x = scp.matrix_units(g.D, [0, 1])
    cot = torch.randn(x.shape, dtype=torch.complex64, generator=torch.Generator().manual_seed(3)).cuda()
    # |V| T below 10; at most 30 rounded FP32 terms per evaluation (6e-8 each)
    full = g.lindblad_workspace_bytes()
    R = g.propagate_lindblad(x)
    Q = g.propagate_lindblad(x, workspace=_bytes(full // 2))
    assert (R - Q).abs().max().item() <= 2e-5
    with pytest.raises(scp.ScpError, match="workspace"):
        g.propagate_lindblad(x, workspace=_bytes(full // 50))
    full = g.lindblad_adjoint_workspace_bytes(x.shape[0])
    ref = g.lindblad_adjoint(x, cot)
    grad = g.lindblad_adjoint(x, cot, workspace=_bytes(full - 256))
    assert abs(grad - ref).max() <= 1e-4 * abs(ref).max()
    with pytest.raises(scp.ScpError, match="workspace"):
        g.lindblad_adjoint(x, cot, workspace=_bytes(full // 3))
    g.close()


# either side of the columns that are walked in slots, one step and many rounds;
# fused operations in the split form and in the matrix form
@pytest.mark.parametrize("d,n,n_steps", [(3, 3, 1), (3, 3, 70), (4, 3, 400)])
def test_lcam_workspace_grows_with_the_columns(scp, d, n, n_steps):
    s = si.fluxonium_chain(si.rng_for(8, d), n, d, 0.01 * n_steps, n_steps, n_basis_gauss=3)
    g = scp.System(si._finish(s, [d] * n, target=si.cz_target(n)))
    for order in ("q1", "q2", "q4", "q4j"):
        sizes = [g.trotter_adjoint_workspace_bytes(order, k) for k in range(1, 300)]
        assert sizes == sorted(sizes)
    x, cot = (_columns(g, 86, k).to(torch.complex128) for k in (1, 2))
    ref = g.trotter_adjoint(x, cot, "q2")
    ws = _bytes(g.trotter_adjoint_workspace_bytes("q2", 130))
    assert (ref == g.trotter_adjoint(x, cot, "q2", workspace=ws)).all()
    g.close()
