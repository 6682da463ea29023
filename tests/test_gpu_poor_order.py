"""GPU tests of single-type meshes whose elements and nodes come in an order of
poor locality and keep it: their matrices assemble by owner groups (plan.h,
max_images), those of the same mesh renumbered by blocks with a gather.
Against the FP64 oracle, tolerances as in tests/test_gpu_matrix_blocks.py."""
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


@pytest.mark.parametrize("kind,n", [(4, 5), (4, 9), (6, 8), (6, 13), (5, 5), (5, 9)])
def test_matrices_in_poor_order(fe_ctx, kind, n):
    import torch
    import paper_2107_11541_amd as fe
    c = meshgen.make_case(n, kind, 0.12, case_id=1000 + n, shuffle=True, n_scalars=2, temperature=True)
    print(f"kind={kind} n={n}", flush=True)
    x = fe.Plan(c.nen, c.coords, c.conn, renumber=False).export()
    images = int(np.diff(x["rowptr"]).astype(np.int64)[x["block_nodes"]].sum())
    assert images > 4.1 * x["rowptr"][-1]
    mesh = make_mesh(fe_ctx, c, renumber=False)
    # no images, which alone would take more than all the rest of the mesh
    assert mesh.info()["device_bytes"] < 8 * images + 4 * 8 * x["block_nodes"].size + 40 * mesh.nnz + 200 * mesh.n_elems
    f = mesh_fields(mesh, c)
    order, _, cols = user_order(mesh)
    for op in (fe.MOMENTUM, fe.SCALAR, fe.POISSON):
        kw = {"Y": c.Y, "D": c.D} if op == fe.SCALAR else {}
        rp, ci, V, B = oracle.assemble(c.coords, c.conn, op, c.dt, c.u, c.rho, c.mu, **kw)
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
    # an element turned inside out is found by its id
    bad = c.conn.copy()
    e = len(bad) // 2
    swap = {4: (0, 1, 3, 2), 6: (3, 4, 5, 0, 1, 2), 5: (3, 2, 1, 0, 4)}[kind]
    bad[e] = bad[e][list(swap)]
    other = fe.Mesh(fe_ctx, c.nen, c.coords, bad, c.dirichlet, renumber=False)
    with pytest.raises(fe.FeError) as err:
        fe.assemble(other, fe.MOMENTUM, c.dt, f["u"], f["rho"], f["mu"])
    assert "EBADELEM" in str(err.value) and str(e) in str(err.value)
    other.close()
    mesh.close()
