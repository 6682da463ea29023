"""GPU tests of hybrid requests of the serving runtime: assembled together by
blocks with a gather, each bitwise as alone; and one whose row images do not
fit the server's memory, which assembles colour by colour."""
import numpy as np
import pytest

import meshgen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fe_ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2107_11541_amd as fe
    ctx = fe.Context(0)
    yield ctx
    torch.cuda.synchronize()


def submit(fe, srv, c, **kw):
    return srv.submit(fe.HYBRID if c.types is not None else c.nen, c.coords, c.conn, c.dirichlet, c.dt, c.u, c.rho, c.mu,
                      rtol=1e-9, max_iter=4000, want_mom_rhs=True,
                      **({"types": c.types} if c.types is not None else {}), **kw)


def test_hybrid_requests_together_equal_each_alone(fe_ctx):
    import paper_2107_11541_amd as fe
    cases = [meshgen.make_case(n, meshgen.HYBRID if i % 3 else meshgen.HEX08, 0.1, case_id=1200 + i, shuffle=True)
             for i, n in enumerate((4, 4, 5, 6, 7, 9, 4, 12, 8, 5, 6, 6))]
    srv = fe.Server(fe_ctx, hbm_budget=1 << 30, max_slots=16, host_threads=4)
    alone = [srv.wait(submit(fe, srv, c)) for c in cases]
    for _ in range(3):
        tickets = [submit(fe, srv, c) for c in cases]
        for c, t, want in zip(cases, tickets, alone):
            got = srv.wait(t)
            assert got["status"] == want["status"] == 0, got["message"]
            assert got["iterations"] == want["iterations"] and got["min_detJ"] == want["min_detJ"]
            assert np.array_equal(got["x"], want["x"]) and np.array_equal(got["mom_rhs"], want["mom_rhs"]), c.n_nodes
    srv.close()


def test_hybrid_request_that_fits_only_without_its_images(fe_ctx):
    """Budgets from one that is too small to one that holds all: the request is
    refused, then served colour by colour, then by blocks, with one result."""
    import paper_2107_11541_amd as fe
    c = meshgen.make_case(14, meshgen.HYBRID, 0.1, case_id=1220, shuffle=True)
    got = []
    for kb in range(1024, 24 << 10, 512):
        srv = fe.Server(fe_ctx, hbm_budget=kb << 10, max_slots=2, host_threads=2)
        try:
            r = srv.wait(submit(fe, srv, c))
        except fe.FeError as e:
            r = {"status": e.status}
        srv.close()
        if r["status"] == 0:
            got.append(r)
        else:
            assert not got   # a larger budget never refuses
    assert len(got) > 2
    for r in got:
        assert np.linalg.norm(r["x"] - got[-1]["x"]) <= 1e-6 * np.linalg.norm(got[-1]["x"])
        assert np.linalg.norm(r["mom_rhs"] - got[-1]["mom_rhs"]) <= 1e-12 * np.linalg.norm(got[-1]["mom_rhs"])
    # both forms were among them: their sums round differently
    assert not np.array_equal(got[0]["mom_rhs"], got[-1]["mom_rhs"])
