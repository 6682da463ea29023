"""GPU tests of the one-launch PCG (the matrix held in registers): the solves
of meshes that fit it against the general form (fe_cg_solve_noalloc), at the
sizes where its dispatch changes -- one group and several, each number of rows
per thread, the last size that fits and the first that does not -- for rows of
up to 16 and up to 27 entries, in FP64 and inside the mixed refinement.

The two forms run the same recurrence and differ in the order of their sums:
5 fixed iterations agree to 1e-12 relative (a row sums at most 27 products and
a dot at most 4e5 terms; the iterates of 5 steps amplify 2^-53 by far less than
the 1e4 left), converged solutions to the CG bound kappa rtol.
"""
import numpy as np
import pytest

import meshgen
from tests.gpu_helpers import dev, host, rel

pytestmark = pytest.mark.gpu

HEX, TET, HYB = meshgen.HEX08, meshgen.TET04, meshgen.HYBRID


@pytest.fixture(scope="module")
def fe_ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2107_11541_amd as fe
    ctx = fe.Context(0)
    yield ctx
    torch.cuda.synchronize()


def _system(fe, ctx, kind, n, renumber=True):
    c = meshgen.make_case(n, kind, 0.10, case_id=400 + n, shuffle=True)
    print(f"kind={kind} n={n} nodes={c.n_nodes} renumber={renumber}", flush=True)
    types = {"types": c.types} if c.types is not None else {}
    mesh = fe.Mesh(ctx, fe.HYBRID if c.types is not None else c.nen, c.coords, c.conn, c.dirichlet,
                   renumber=renumber, **types)
    u, rho = mesh.to_mesh(dev(c.u)), mesh.to_mesh(dev(c.rho))
    L, f, _ = fe.assemble(mesh, fe.POISSON, c.dt, u, rho)
    fe.apply_dirichlet(mesh, L, f)
    return mesh, L[0].contiguous(), f[0].contiguous()


def _check(fe, mesh, L, f):
    import torch
    xs, a = fe.cg_solve(mesh, L, f, rtol=0.0, max_iter=5)
    xg, b = fe.cg_solve_noalloc(mesh, L, f, rtol=0.0, max_iter=5)
    assert a["symmetric_spmv"] and a["iterations"] == b["iterations"] == 5
    assert rel(host(xs), host(xg)) <= 1e-12
    for key in ("rel_residual", "true_rel_residual"):
        assert abs(a[key] - b[key]) <= 1e-11 * b[key]
    # a first guess, and a solve to convergence
    g = torch.Generator().manual_seed(3)
    x0 = torch.rand(mesh.n_nodes, generator=g, dtype=torch.float64).cuda()
    xs, a = fe.cg_solve(mesh, L, f, x=x0.clone(), rtol=1e-9, max_iter=5000)
    xg, b = fe.cg_solve_noalloc(mesh, L, f, x=x0.clone(), rtol=1e-9, max_iter=5000)
    assert a["status"] == b["status"] == 0 and abs(a["iterations"] - b["iterations"]) <= 1
    assert a["true_rel_residual"] <= 2e-9 and rel(host(xs), host(xg)) <= 1e-5
    # no iteration at all: x unchanged, the residual of the guess
    xs, a = fe.cg_solve(mesh, L, f, x=x0.clone(), rtol=1e-9, max_iter=0, raise_on_noconv=False)
    assert a["iterations"] == 0 and a["status"] != 0 and torch.equal(xs, x0)
    xm, m = fe.cg_solve(mesh, L, f, rtol=1e-10, max_iter=20000, precision=fe.MIXED)
    xt, _ = fe.cg_solve_noalloc(mesh, L, f, rtol=1e-12, max_iter=20000)
    assert m["status"] == 0 and m["true_rel_residual"] <= 1e-10 and rel(host(xm), host(xt)) <= 1e-6


# rows per thread 1, 2, 4, 5, 6 (27 entries; 72^3 is the last cube that fits, 73^3 the
# first that does not) and up to 9 (16 entries; 79^3 and 84^3)
@pytest.mark.parametrize("kind,n", [(HEX, 4), (HEX, 5), (HEX, 9), (HEX, 23), (HEX, 31), (HEX, 63), (HEX, 66),
                                    (HEX, 72), (HEX, 73), (TET, 4), (TET, 24), (TET, 70), (TET, 79), (TET, 84),
                                    (HYB, 17)])
def test_one_launch_solve_equals_general(fe_ctx, kind, n):
    import paper_2107_11541_amd as fe
    mesh, L, f = _system(fe, fe_ctx, kind, n)
    _check(fe, mesh, L, f)
    mesh.close()


def test_halo_that_does_not_fit(fe_ctx):
    """Random numbering kept as it is: a group's rows touch more columns than
    its window holds, and the solve runs in several launches."""
    import paper_2107_11541_amd as fe
    mesh, L, f = _system(fe, fe_ctx, HEX, 26, renumber=False)
    _check(fe, mesh, L, f)
    mesh.close()


def test_breakdown_is_reported(fe_ctx):
    """A negative definite matrix: p . A p < 0 in the first iteration."""
    import paper_2107_11541_amd as fe
    mesh, L, f = _system(fe, fe_ctx, HEX, 8)
    with pytest.raises(fe.FeError) as e:
        fe.cg_solve(mesh, -L, f, rtol=1e-9, max_iter=100)
    assert "EBREAKDOWN" in str(e.value)
    x, info = fe.cg_solve(mesh, L, f, rtol=1e-9, max_iter=1000)   # and the mesh still solves
    assert info["status"] == 0 and np.isfinite(host(x)).all()
    mesh.close()
