"""GPU tests of the 3x3-block operator's row groups: one element, a group that
is not full, several groups, and meshes on both sides of the size (2^16 element
nodes) from which groups have 256 lanes instead of 64, of each element type and
hybrid, in the caller's numbering (many elements to a group) and in the
library's.  Against the FP64 oracle: 1e-12 relative in norm (<= 200 element
contributions of ~1e3 roundings each at random, 5e-14)."""
import numpy as np
import pytest

import meshgen
import oracle
from tests.gpu_helpers import dev, host, make_mesh, rel, user_order

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


@pytest.mark.parametrize("kind,n,renumber", [(8, 1, True), (8, 3, False), (8, 20, True), (8, 21, True), (8, 21, False),
                                             (4, 1, True), (4, 13, True), (4, 15, True), (6, 1, True), (6, 18, True),
                                             (6, 19, True), (5, 1, True), (5, 12, True), (5, 14, False), (0, 4, False),
                                             (0, 14, True), (0, 16, True), (0, 16, False)])
def test_block_groups(fe_ctx, kind, n, renumber):
    import torch
    import paper_2107_11541_amd as fe
    c = meshgen.make_case(n, kind, 0.12, case_id=900 + n, shuffle=True, temperature=True)
    c.mu = np.random.default_rng(n).uniform(1e-2, 3e-2, c.n_nodes)
    print(f"kind={kind} n={n} renumber={renumber} E={c.n_elems}", flush=True)
    mesh = make_mesh(fe_ctx, c, renumber=renumber)
    u, rho, mu = (mesh.to_mesh(dev(np.ascontiguousarray(a))) for a in (c.u, c.rho, c.mu))
    order, _, cols = user_order(mesh)
    for form in range(4):
        V, B, info = fe.assemble_block(mesh, form, c.dt, u, rho, mu)
        rp, ci, Vo, Bo = oracle.assemble_block(c.coords, c.conn, form, c.dt, c.u, c.rho, c.mu, types=c.types)
        assert info["first_bad_elem"] == -1 and info["min_detJ"] > 0
        assert np.array_equal(cols, ci)
        assert rel(host(V).reshape(-1, 9)[order].reshape(-1), Vo.reshape(-1)) <= 1e-12
        assert rel(host(mesh.to_user(B)), Bo) <= 1e-12
        V2, B2, _ = fe.assemble_block(mesh, form, c.dt, u, rho, mu)
        assert torch.equal(V, V2) and torch.equal(B, B2)
    mesh.close()
