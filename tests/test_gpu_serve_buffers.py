"""A served gradient recomputes several segments side by side where the budget
has room for their stage inputs: with one buffer (the budget holds the request
alone), a few, and all it takes, in ticks of one segment and of many, the result
is bitwise that of the direct path."""
import numpy as np
import pytest

from test_gpu_serve import direct, scp, short_request  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chunk_work", [2e4, 3e6])
@pytest.mark.parametrize("room", [1.01, 3.0, None])
def test_any_number_of_buffers_gives_the_direct_result(scp, room, chunk_work):  # noqa: F811
    reqs = [short_request(0), short_request(5)]
    need = max(scp.serve.request_bytes(q, True) for q in reqs)
    budget = 64 << 30 if room is None else int(room * need)
    srv = scp.serve.Server(budget, max_active=2, chunk_work=chunk_work, engine="register")
    ids = [srv.submit(q, True) for q in reqs]
    res = scp.serve.drain(srv, ids)
    for q, i in zip(reqs, ids):
        F, grad, _ = direct(scp, q, True, "register")
        assert res[i]["state"] == "done"
        assert res[i]["F"] == F and np.array_equal(res[i]["grad"], grad)
    srv.close()
