"""What the server lends a gradient request beyond its reserved footprint (stage
inputs of further segments) never keeps another request waiting: as many run at
once as their footprints allow, and the results are bitwise those of the direct
path whether buffers were lent, taken back or neither."""
import numpy as np
import pytest

import scp_inputs as si
from test_gpu_serve import direct, scp  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _request(k):
    s = si.transmon_ring(si.rng_for(7, 40 + k), 7, 3, 2.0, 100)
    s = si._finish(s, [3] * 7, target=si.cz_target(7))
    s["columns"] = s["columns"][:64]                    # those of the first qubit at 0
    s["comp_rows"], s["comp_cols"] = s["comp_rows"][:64], list(range(64))
    s["target"] = np.asarray(s["target"])[:64, :64]
    return s


def _check(scp, res, reqs, ids, engine):
    for q, i in zip(reqs, ids):
        F, grad, _ = direct(scp, q, True, engine)
        assert res[i]["state"] == "done"
        assert res[i]["F"] == F and np.array_equal(res[i]["grad"], grad)


@pytest.mark.parametrize("engine", ["register", "auto"])
def test_as_many_run_as_the_footprints_allow(scp, engine):  # noqa: F811
    reqs = [_request(k) for k in range(4)]
    need = scp.serve.request_bytes(reqs[0], True)
    # the gather engine adds a costate per segment and the sums of the steps
    extra = 0 if engine == "register" else need // 2
    srv = scp.serve.Server(4 * (need + extra) + 4096, max_active=8, chunk_work=1e5, engine=engine)
    ids = [srv.submit(q, True) for q in reqs]
    assert srv.step() == (4, 0)
    _check(scp, scp.serve.drain(srv, ids), reqs, ids, engine)
    srv.close()


@pytest.mark.parametrize("engine", ["register", "auto"])
def test_lent_buffers_are_taken_back_for_a_queued_request(scp, engine):  # noqa: F811
    reqs = [_request(k) for k in range(3)]
    need = scp.serve.request_bytes(reqs[0], True)
    # room for further segments of the first in the free half, and for three requests without
    room = 3.6 if engine == "register" else 5.0
    srv = scp.serve.Server(int(room * need), max_active=8, chunk_work=2e5, engine=engine)
    ids = [srv.submit(reqs[0], True)]
    for _ in range(200):                                # into the reverse walk
        srv.step()
        if srv.result(ids[0])["F"] != 0.0:
            break
    srv.step()
    assert srv.result(ids[0])["state"] == "running"
    ids += [srv.submit(q, True) for q in reqs[1:]]
    assert srv.step() == (3, 0)
    _check(scp, scp.serve.drain(srv, ids), reqs, ids, engine)
    srv.close()


def test_a_refused_request_leaves_the_budget_alone(scp):  # noqa: F811
    # six levels: queued, refused when it is built
    good, bad = _request(0), _request(1)
    bad["modes"] = [dict(m, trunc=6) for m in bad["modes"][:2]]
    bad["couplings"], bad["drives"] = bad["couplings"][:1], bad["drives"][:2]
    bad["columns"], bad["comp_rows"], bad["comp_cols"] = [0, 1], [0, 1], [0, 1]
    bad["target"], bad["n_steps"] = np.eye(2), 300
    need = scp.serve.request_bytes(good, False)
    srv = scp.serve.Server(need + scp.serve.request_bytes(bad, False), max_active=8, chunk_work=1e4,
                           engine="register")
    ids = [srv.submit(q, False) for q in (good, bad, good)]
    assert srv.step() == (1, 1)              # the third waits for the first's memory
    assert srv.result(ids[0])["state"] == "running" and srv.result(ids[2])["state"] == "queued"
    with pytest.raises(scp.ScpError, match="d in"):
        srv.result(ids[1])
    srv.close()
