"""GPU tests of the 3x3-block operator where its form changes (plan.h, RowForm):
hybrid meshes from 2^18 element nodes on, whose plain operator (each task alone)
and full-stress operator (shared groups) are planned side by side, and meshes in
random order kept as it is.  Against the FP64 oracle at a sample of rows:
1e-12 of the sample's norm, as in tests/test_gpu_block_groups.py."""
import numpy as np
import pytest

import meshgen
import oracle
from tests.gpu_helpers import dev, host, make_mesh, rel, submesh_rows_typed

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


@pytest.mark.parametrize("kind,n,renumber", [(0, 25, True), (0, 25, False), (8, 22, False), (4, 8, False), (4, 16, False),
                                             (6, 10, False), (6, 19, False), (5, 8, False), (5, 14, False)])
def test_block_forms(fe_ctx, kind, n, renumber):
    import torch
    import paper_2107_11541_amd as fe
    c = meshgen.make_case(n, kind, 0.12, case_id=1100 + n, shuffle=True, temperature=True)
    r = np.random.default_rng(n)
    c.mu = r.uniform(1e-2, 3e-2, c.n_nodes)
    nodes = r.choice(c.n_nodes, 40, replace=False)
    coords, conn, types, loc, glob = submesh_rows_typed(c, nodes)
    sub = {"u": c.u[:, glob], "rho": c.rho[glob], "mu": c.mu[glob]}
    types = None if c.types is None else types
    mesh = make_mesh(fe_ctx, c, renumber=renumber)
    print(f"kind={kind} n={n} renumber={renumber} E={c.n_elems}", flush=True)
    u, rho, mu = (mesh.to_mesh(dev(np.ascontiguousarray(a))) for a in (c.u, c.rho, c.mu))
    rp, ci = mesh.pattern_host()
    where = np.empty(c.n_nodes, np.int64)
    where[mesh.node_perm] = np.arange(c.n_nodes)
    for form in (0, 3, 2, 1, 0):
        V, B, info = fe.assemble_block(mesh, form, c.dt, u, rho, mu)
        assert info["first_bad_elem"] == -1 and info["min_detJ"] > 0
        V2, B2, _ = fe.assemble_block(mesh, form, c.dt, u, rho, mu)
        assert torch.equal(V, V2) and torch.equal(B, B2)
        so, sc, Vo, Bo = oracle.assemble_block(coords, conn, form, c.dt, sub["u"], sub["rho"], sub["mu"], types=types)
        Vh, Bh = host(V).reshape(-1, 9), host(mesh.to_user(B))
        got, want = [], []
        for i in nodes:
            row, srow = where[i], loc[i]
            cols = mesh.node_perm[ci[rp[row]:rp[row + 1]]]
            order = np.argsort(cols)
            assert np.array_equal(np.sort(cols), np.sort(glob[sc[so[srow]:so[srow + 1]]]))
            sorder = np.argsort(glob[sc[so[srow]:so[srow + 1]]])
            got.append(Vh[rp[row]:rp[row + 1]][order].ravel())
            want.append(Vo.reshape(-1, 9)[so[srow]:so[srow + 1]][sorder].ravel())
        assert rel(np.concatenate(got), np.concatenate(want)) <= 1e-12
        assert rel(Bh[:, nodes], Bo[:, loc[nodes]]) <= 1e-12
    mesh.close()
