"""GPU tests of the matrix assembly where its launch shape can go wrong: one
element, a block or group that is not full, several blocks whose rows are
gathered, rows longer than one pass of the gather and nodes of more than eight
blocks (shuffled elements in the caller's numbering), each element type and a
hybrid mesh.  Against the FP64 oracle: 1e-12 relative, in norm and per entry
scaled by its row's largest (<= 200 element contributions of ~1e3 roundings
each, 2e5 * 1.1e-16 = 2.2e-11 if all had the same sign, their square root,
~5e-14, if not); mixed precision: 1e-5 (FP32 products, ~80 ulp)."""
import numpy as np
import pytest

import meshgen
import oracle
from tests.gpu_helpers import host, make_mesh, mesh_fields, rel, rhs_user, row_scaled_err, user_order, values_user

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


@pytest.mark.parametrize("renumber", [True, False])
@pytest.mark.parametrize("kind,n", [(8, 1), (8, 2), (8, 4), (8, 5), (8, 9), (4, 1), (4, 3), (4, 6), (6, 1), (6, 4),
                                    (6, 7), (5, 1), (5, 3), (5, 6), (0, 4), (0, 5), (0, 7)])
def test_matrix_blocks_at_their_edges(fe_ctx, kind, n, renumber):
    import torch
    import paper_2107_11541_amd as fe
    c = meshgen.make_case(n, kind, 0.12, case_id=700 + n, shuffle=True, n_scalars=2, temperature=True)
    print(f"kind={kind} n={n} renumber={renumber}", flush=True)
    meshes = [make_mesh(fe_ctx, c, renumber=renumber)]
    if c.types is None:
        meshes.append(make_mesh(fe_ctx, c, renumber=renumber, coloured=True))
    for op in (fe.MOMENTUM, fe.SCALAR, fe.POISSON):
        kw = {"Y": c.Y, "D": c.D} if op == fe.SCALAR else {}
        rp, ci, V, B = oracle.assemble(c.coords, c.conn, op, c.dt, c.u, c.rho, c.mu, types=c.types, **kw)
        for mesh in meshes:
            f = mesh_fields(mesh, c)
            order, _, cols = user_order(mesh)
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
                again = fe.assemble(mesh, op, c.dt, f["u"], f["rho"], f["mu"], precision=precision, **kw)
                assert torch.equal(v, again[0]) and torch.equal(b, again[1])
    for mesh in meshes:
        mesh.close()


@pytest.mark.parametrize("count", [2, 3, 4, 5])
@pytest.mark.parametrize("n,renumber", [(1, True), (5, False), (9, True)])
def test_scalars_of_one_pass_equal_each_alone(fe_ctx, n, renumber, count):
    """Mixed HEX08 scalars share passes of up to three: bitwise what each gives alone."""
    import torch
    import paper_2107_11541_amd as fe
    c = meshgen.make_case(n, 8, 0.12, case_id=800 + n, shuffle=True, n_scalars=5)
    mesh = make_mesh(fe_ctx, c, renumber=renumber)
    f = mesh_fields(mesh, c)

    def run(a, b):
        v, r, info = fe.assemble(mesh, fe.SCALAR, c.dt, f["u"], f["rho"], Y=f["Y"][a:b].contiguous(), D=c.D[a:b],
                                 precision=fe.MIXED)
        return v, r, info["min_detJ"]

    V, B, det = run(0, count)
    for k in range(count):
        v, b, d = run(k, k + 1)
        assert torch.equal(V[k], v[0]) and torch.equal(B[k], b[0]) and d == det
    mesh.close()
