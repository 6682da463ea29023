"""GPU tests of the form that a PCG solve takes: in one launch where the matrix
fits the registers (csrc/resident.hip), three launches per iteration otherwise.
The context's profile tells them apart: slot 0 has one interval per solve in
one launch (FE_MIXED: per inner solve), one per iteration in the general form.
"""
import numpy as np
import pytest

import meshgen
from tests.gpu_helpers import dev, host, rel

pytestmark = pytest.mark.gpu

HEX, PEN, PYR, TET, HYB = meshgen.HEX08, meshgen.PEN06, meshgen.PYR05, meshgen.TET04, meshgen.HYBRID


@pytest.fixture(scope="module")
def fe_ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2107_11541_amd as fe
    ctx = fe.Context(0)
    yield ctx
    torch.cuda.synchronize()


def system(fe, ctx, kind, n, renumber=True, **kw):
    """A jittered cube's Poisson system with its boundary fixed: mesh, L, f."""
    c = meshgen.make_case(n, kind, 0.10, case_id=500 + n, shuffle=True)
    print(f"kind={kind} n={n} nodes={c.n_nodes} renumber={renumber} {kw}", flush=True)
    if c.types is not None:
        kw["types"] = c.types
    mesh = fe.Mesh(ctx, fe.HYBRID if c.types is not None else c.nen, c.coords, c.conn, c.dirichlet,
                   renumber=renumber, **kw)
    u, rho = mesh.to_mesh(dev(c.u)), mesh.to_mesh(dev(c.rho))
    L, f, _ = fe.assemble(mesh, fe.POISSON, c.dt, u, rho)
    fe.apply_dirichlet(mesh, L, f)
    return mesh, L[0].contiguous(), f[0].contiguous()


def solve(fe, mesh, L, f, **kw):
    """A solve's x, info and the intervals of profile slot 0."""
    mesh.ctx.profile(True)
    x, info = fe.cg_solve(mesh, L, f, **kw)
    launches = mesh.ctx.profile_read(0)[0]
    mesh.ctx.profile(False)
    return x, info, launches


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_general_upload_flag_holds_in_both_precisions(fe_ctx, precision):
    import paper_2107_11541_amd as fe
    prec = fe.MIXED if precision == "mixed" else fe.FP64
    mesh, L, f = system(fe, fe_ctx, HEX, 10, symmetric_spmv=False)
    x, info, launches = solve(fe, mesh, L, f, rtol=1e-10, max_iter=2000, precision=prec)
    assert info["status"] == 0 and launches >= info["iterations"] > info["outer_iterations"]
    mesh.close()
