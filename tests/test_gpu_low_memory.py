"""GPU tests of meshes without the gathers' work arrays, which are left out at
upload or freed later when a device allocation finds no room (made so here by
fe_test_fail_allocs): the element-vector passes, and the matrices of meshes
that else assemble by blocks, then run colour by colour.  Tolerances as in
tests/test_gpu_vector_passes.py and tests/test_gpu_matrix_blocks.py."""
import numpy as np
import pytest

import meshgen
import oracle
from tests.gpu_helpers import dev, host, make_mesh, mesh_fields, rel, rhs_user, row_scaled_err, user_order, values_user

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


def no_room(ctx, n):
    ctx.check(ctx.lib.fe_test_fail_allocs(ctx.h, n))


def check_operators(fe, mesh, c):
    f = mesh_fields(mesh, c)

    def user(t):
        return host(mesh.to_user(t.contiguous()))

    for form in range(4):
        want, mass = oracle.residual(c.coords, c.conn, c.u, c.rho, c.mu, c.types, form=form)
        got = user(fe.residual(mesh, f["u"], f["rho"], f["mu"], form=form))
        assert rel(got[:3], want) <= 1e-12 and rel(got[3], mass) <= 1e-12
    p = c.Y[0]
    assert rel(user(fe.gradient(mesh, mesh.to_mesh(dev(p)))), oracle.gradient(c.coords, c.conn, p, c.types)) <= 1e-12
    got = user(fe.scalar_residual(mesh, f["u"], f["rho"], f["Y"][0].contiguous(), float(c.D[0])))
    want, mass = oracle.scalar_residual(c.coords, c.conn, c.u, c.rho, p, float(c.D[0]), c.types)
    assert rel(got[0], want) <= 1e-12 and rel(got[1], mass) <= 1e-12
    _, _, _, F = oracle.assemble(c.coords, c.conn, oracle.OP_POISSON, c.dt, c.u, c.rho, None, types=c.types)
    assert rel(user(fe.divergence(mesh, c.dt, f["u"], f["rho"])), F[0]) <= 1e-12
    order, _, cols = user_order(mesh)
    for op in (fe.MOMENTUM, fe.SCALAR, fe.POISSON):
        kw = {"Y": c.Y, "D": c.D} if op == fe.SCALAR else {}
        rp, ci, V, B = oracle.assemble(c.coords, c.conn, op, c.dt, c.u, c.rho, c.mu, types=c.types, **kw)
        assert np.array_equal(cols, ci)
        kw = {"Y": f["Y"], "D": c.D} if op == fe.SCALAR else {}
        for precision, tol in ((fe.FP64, 1e-12), (fe.MIXED, 1e-5)):
            v, b, info = fe.assemble(mesh, op, c.dt, f["u"], f["rho"], f["mu"], precision=precision, **kw)
            assert info["first_bad_elem"] == -1 and info["min_detJ"] > 0
            vu, bu = values_user(mesh, host(v), order), rhs_user(mesh, host(b))
            for k in range(V.shape[0]):
                assert rel(vu[k], V[k]) <= tol and row_scaled_err(rp, vu[k], V[k]) <= tol
            for k in range(B.shape[0]):
                assert rel(bu[k], B[k]) <= tol


@pytest.mark.parametrize("renumber", [True, False])
@pytest.mark.parametrize("kind,n", [(8, 1), (8, 5), (4, 1), (4, 5), (6, 4), (5, 4), (0, 4), (0, 6)])
def test_upload_without_room_for_the_gathers(fe_ctx, kind, n, renumber):
    import paper_2107_11541_amd as fe
    c = meshgen.make_case(n, kind, 0.12, case_id=900 + n, shuffle=True, n_scalars=2)
    print(f"kind={kind} n={n} renumber={renumber}", flush=True)
    mesh = make_mesh(fe_ctx, c, renumber=renumber)
    whole = mesh.info()["device_bytes"]
    mesh.close()
    no_room(fe_ctx, 1)
    mesh = make_mesh(fe_ctx, c, renumber=renumber)
    assert mesh.info()["device_bytes"] < whole
    check_operators(fe, mesh, c)
    mesh.close()


@pytest.mark.parametrize("kind,n", [(8, 6), (4, 5), (0, 6)])
def test_later_allocation_takes_the_work_arrays(fe_ctx, kind, n):
    """A solve, a step and the block operator whose memory does not fit beside
    the work arrays: they go, the call succeeds, the mesh still assembles."""
    import paper_2107_11541_amd as fe
    c = meshgen.make_case(n, kind, 0.12, case_id=920 + n, shuffle=True, n_scalars=2)
    print(f"kind={kind} n={n}", flush=True)
    for call in ("solve", "step", "block"):
        other, mesh = make_mesh(fe_ctx, c), make_mesh(fe_ctx, c)
        f = mesh_fields(mesh, c)
        L, b, _ = fe.assemble(mesh, fe.POISSON, c.dt, f["u"], f["rho"])
        fe.apply_dirichlet(mesh, L, b)
        before = mesh.info()["device_bytes"], other.info()["device_bytes"]
        no_room(fe_ctx, 1)
        if call == "solve":
            x, info = fe.cg_solve(mesh, L[0], b[0], rtol=1e-10, max_iter=2000)
            assert info["status"] == 0 and info["true_rel_residual"] <= 2e-10
        elif call == "step":
            p = b[0].clone().zero_()
            fe.fractional_step(mesh, c.dt, f["rho"], f["mu"], L[0], f["u"].clone(), p, rtol=1e-8)
        else:
            v, r, info = fe.assemble_block(mesh, 0, c.dt, f["u"], f["rho"], f["mu"])
            m, s, _ = fe.assemble(mesh, fe.MOMENTUM, c.dt, f["u"], f["rho"], f["mu"])
            assert rel(host(v[:, 1, 1]), host(m[0])) <= 1e-12 and rel(host(r), host(s)) <= 1e-12
        assert other.info()["device_bytes"] < before[1]
        check_operators(fe, mesh, c)
        mesh.close()
        other.close()


def test_without_work_arrays_an_allocation_fails_as_such(fe_ctx):
    import paper_2107_11541_amd as fe
    c = meshgen.make_case(5, 8, 0.12, case_id=930, shuffle=True)
    no_room(fe_ctx, 1)
    mesh = make_mesh(fe_ctx, c)
    f = mesh_fields(mesh, c)
    L, b, _ = fe.assemble(mesh, fe.POISSON, c.dt, f["u"], f["rho"])
    fe.apply_dirichlet(mesh, L, b)
    no_room(fe_ctx, 1)
    with pytest.raises(fe.FeError) as e:
        fe.cg_solve(mesh, L[0], b[0])
    assert "ENOMEM" in str(e.value)
    x, info = fe.cg_solve(mesh, L[0], b[0], rtol=1e-9, max_iter=2000)
    assert info["status"] == 0
    mesh.close()
