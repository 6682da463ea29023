"""GPU tests of the element-vector passes (residual with every operator
variant, gradient, divergence, scalar residual) where their launch shape can go
wrong: one element, a block that is not full, several blocks whose nodes are
gathered, each element type and a hybrid mesh, in the caller's numbering and in
the library's.  Against the FP64 oracle: relative 2-norm <= 1e-12 (the bound of
the other operators; ~30 contributions of ~1e3 roundings each per node)."""
import numpy as np
import pytest

import meshgen
import oracle
from tests.gpu_helpers import dev, host, make_mesh, mesh_fields, rel

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
@pytest.mark.parametrize("kind,n", [(8, 1), (8, 3), (8, 4), (8, 5), (8, 9), (4, 1), (4, 3), (6, 1), (6, 5), (5, 1),
                                    (5, 4), (0, 4), (0, 7)])
def test_vector_passes_at_block_edges(fe_ctx, kind, n, renumber):
    import torch
    import paper_2107_11541_amd as fe
    c = meshgen.make_case(n, kind, 0.12, case_id=500 + n, shuffle=True, n_scalars=1)
    print(f"kind={kind} n={n} renumber={renumber}", flush=True)
    mesh = make_mesh(fe_ctx, c, renumber=renumber)
    f = mesh_fields(mesh, c)

    def user(t):
        return host(mesh.to_user(t.contiguous()))

    for form in range(4):
        got = fe.residual(mesh, f["u"], f["rho"], f["mu"], form=form)
        want, mass = oracle.residual(c.coords, c.conn, c.u, c.rho, c.mu, c.types, form=form)
        assert rel(user(got)[:3], want) <= 1e-12 and rel(user(got)[3], mass) <= 1e-12
        assert torch.equal(got, fe.residual(mesh, f["u"], f["rho"], f["mu"], form=form))
    p = c.Y[0]
    assert rel(user(fe.gradient(mesh, mesh.to_mesh(dev(p)))), oracle.gradient(c.coords, c.conn, p, c.types)) <= 1e-12
    got = fe.scalar_residual(mesh, f["u"], f["rho"], f["Y"][0].contiguous(), float(c.D[0]))
    want, mass = oracle.scalar_residual(c.coords, c.conn, c.u, c.rho, p, float(c.D[0]), c.types)
    assert rel(user(got)[0], want) <= 1e-12 and rel(user(got)[1], mass) <= 1e-12
    _, _, _, F = oracle.assemble(c.coords, c.conn, oracle.OP_POISSON, c.dt, c.u, c.rho, None, types=c.types)
    assert rel(user(fe.divergence(mesh, c.dt, f["u"], f["rho"])), F[0]) <= 1e-12
    mesh.close()
