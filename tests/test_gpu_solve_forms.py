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


def hooks(mesh, wait_us=50000.0, last_wait_us=50000.0, stopped=False):
    mesh.ctx.check(mesh.ctx.lib.fe_test_one_launch(mesh.h, wait_us, last_wait_us, int(stopped)))


def check_given_up(fe, mesh, L, f):
    """The solve starts from the first guess as passed in, whichever form runs in
    the end: 5 iterations agree with the general SpMV's to 1e-12 (see
    tests/test_gpu_resident.py).  Returns its intervals of slot 0."""
    import torch
    g = torch.Generator().manual_seed(5)
    x0 = torch.rand(mesh.n_nodes, generator=g, dtype=torch.float64).cuda()
    x, info, launches = solve(fe, mesh, L, f, x=x0.clone(), rtol=0.0, max_iter=5)
    xg, want = fe.cg_solve_noalloc(mesh, L, f, x=x0.clone(), rtol=0.0, max_iter=5)
    assert info["iterations"] == want["iterations"] == 5
    assert rel(host(x), host(xg)) <= 1e-12
    assert abs(info["true_rel_residual"] - want["true_rel_residual"]) <= 1e-11 * want["true_rel_residual"]
    return launches


# 23^3: several groups, each with rows for every thread; 4^3: one group (no meeting:
# only the stop word ends it early)
@pytest.mark.parametrize("n,kw", [(23, dict(stopped=True)), (4, dict(stopped=True)), (23, dict(wait_us=0.0)),
                                  (23, dict(last_wait_us=0.0))])
def test_solve_that_is_given_up(fe_ctx, n, kw):
    """Groups that start after the solve was given up leave at once; groups that
    wait too long give it up, at the first meeting or, some of them having
    stored x, at the last."""
    import paper_2107_11541_amd as fe
    mesh, L, f = system(fe, fe_ctx, HEX, n)
    hooks(mesh, **kw)
    # (at the last meeting a group gives up unless every other came before it)
    for _ in range(20):
        launches = check_given_up(fe, mesh, L, f)
        if launches != 1:
            break
    assert launches == 1 + 5   # the one given up, then one per iteration
    hooks(mesh)
    check_given_up(fe, mesh, L, f)
    mesh.close()


@pytest.mark.parametrize("kw", [dict(stopped=True), dict(wait_us=0.0)])
def test_mixed_solve_that_is_given_up(fe_ctx, kw):
    import paper_2107_11541_amd as fe
    mesh, L, f = system(fe, fe_ctx, HEX, 23)
    hooks(mesh, **kw)
    x, info, launches = solve(fe, mesh, L, f, rtol=1e-10, max_iter=5000, precision=fe.MIXED)
    assert info["status"] == 0 and info["true_rel_residual"] <= 1e-10 and launches > info["iterations"]
    xt, _ = fe.cg_solve_noalloc(mesh, L, f, rtol=1e-12, max_iter=5000)
    assert rel(host(x), host(xt)) <= 1e-6
    mesh.close()


def test_one_launch_form_comes_back_after_a_give_up(fe_ctx):
    """16 solves in the general form, then one launch again; a second give-up in
    a row doubles them."""
    import paper_2107_11541_amd as fe
    mesh, L, f = system(fe, fe_ctx, HEX, 9)

    def forms(k):
        return [solve(fe, mesh, L, f, rtol=0.0, max_iter=3)[2] for _ in range(k)]
    assert forms(1) == [1]
    hooks(mesh, stopped=True)
    assert forms(1 + 16 + 1 + 32) == [4] + 16 * [3] + [4] + 32 * [3]
    hooks(mesh)
    assert forms(2) == [1, 1]
    hooks(mesh, stopped=True)
    assert forms(1 + 16) == [4] + 16 * [3]
    mesh.close()


def test_refused_matrix_after_a_general_symmetric_solve(fe_ctx):
    """A matrix that fails the pair check, on a mesh whose last solves ran the
    symmetric SpMV in the general form: the general SpMV runs, on this matrix."""
    import torch
    import paper_2107_11541_amd as fe
    mesh, L, f = system(fe, fe_ctx, HEX, 9)
    hooks(mesh, stopped=True)
    for _ in range(17):
        assert solve(fe, mesh, L, f, rtol=0.0, max_iter=3)[1]["symmetric_spmv"]
    hooks(mesh)
    rp, ci = mesh.pattern_host()
    rows = np.repeat(np.arange(mesh.n_nodes), np.diff(rp))
    r = rows[int(np.argmax(np.where(ci != rows, np.abs(host(L)), 0.0)))]
    off = torch.tensor([p for p in range(rp[r], rp[r + 1]) if ci[p] != r], device=L.device)
    L2 = 3.0 * L
    L2[off] *= 1.0 + 1e-6
    x, info, _ = solve(fe, mesh, L2, f, rtol=0.0, max_iter=3)
    xg, _ = fe.cg_solve_noalloc(mesh, L2, f, rtol=0.0, max_iter=3)
    assert not info["symmetric_spmv"] and torch.equal(x, xg)
    mesh.close()


def _contexts(fe, k, kind=HEX, n=9):
    """k contexts on streams of their own, each with a mesh that has solved once."""
    import torch
    out = []
    for _ in range(k):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            ctx = fe.Context(0, st)
            mesh, L, f = system(fe, ctx, kind, n)
            x, info = fe.cg_solve(mesh, L, f, rtol=1e-9, max_iter=2000)
            st.synchronize()
        out.append((st, ctx, mesh, L, f, x, info))
    return out


def test_solves_of_several_contexts_at_once(fe_ctx):
    """Four threads solving at a time, each on its stream: every solve in one
    launch, with the bits of a solve alone."""
    import threading
    import torch
    import paper_2107_11541_amd as fe
    ws = _contexts(fe, 4, n=17)
    bad = []

    def go(st, ctx, mesh, L, f, x, info):
        with torch.cuda.stream(st):
            for _ in range(20):
                y, i, launches = solve(fe, mesh, L, f, rtol=1e-9, max_iter=2000)
                st.synchronize()
                if launches != 1 or i != info or not torch.equal(x, y):
                    bad.append((launches, i))
    threads = [threading.Thread(target=go, args=w) for w in ws]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
    for w in ws:
        w[2].close()
        w[1].close()


def test_work_queued_before_a_solve_holds_up_no_other_context(fe_ctx):
    """A solve queued behind other work of its stream (here a kernel that spins
    for about half a second) waits for it alone: another context solves
    meanwhile."""
    import threading
    import time
    import torch
    import paper_2107_11541_amd as fe
    ws = _contexts(fe, 5)
    a = ws[0]
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    with torch.cuda.stream(a[0]):
        torch.cuda._sleep(1000)   # (the kernel is loaded)
        a[0].synchronize()
        e0.record()
        torch.cuda._sleep(10_000_000)
        e1.record()
        a[0].synchronize()
    cycles = int(10_000_000 * 500.0 / e0.elapsed_time(e1))   # 500 ms
    print(f"500 ms are {cycles} cycles", flush=True)

    def beside(w):
        # whether w's stream runs beside a's (streams may share a hardware queue)
        with torch.cuda.stream(a[0]):
            torch.cuda._sleep(cycles // 5)
        t = time.perf_counter()
        with torch.cuda.stream(w[0]):
            w[5].add(1.0)
            w[0].synchronize()
        t = time.perf_counter() - t
        a[0].synchronize()
        return t < 0.05
    b = next((w for w in ws[1:] if beside(w)), None)
    if b is None:
        pytest.skip("no stream beside the first")
    done = threading.Event()

    def slow():
        with torch.cuda.stream(a[0]):
            x = torch.zeros_like(a[5])
            torch.cuda._sleep(cycles)
            fe.cg_solve(a[2], a[3], a[4], x=x, rtol=1e-9, max_iter=2000)
        done.set()
    t = threading.Thread(target=slow)
    with torch.cuda.stream(b[0]):
        x = torch.zeros_like(b[5])
        t.start()
        time.sleep(0.1)
        y, info = fe.cg_solve(b[2], b[3], b[4], x=x, rtol=1e-9, max_iter=2000)
        b[0].synchronize()
        assert not done.is_set() and info["status"] == 0
    t.join()
    for w in ws:
        w[2].close()
        w[1].close()


def test_solve_on_a_stream_with_few_cus(fe_ctx):
    """A stream masked to 64 CUs: a matrix that needs more groups than that runs
    in the general form, one that does not in one launch, and the mesh that was
    planned on the masked stream in one launch on another."""
    import ctypes
    import torch
    import paper_2107_11541_amd as fe
    hip = ctypes.CDLL("libamdhip64.so")
    h, mask = ctypes.c_void_p(), (ctypes.c_uint32 * 8)(*([0xff] * 8))
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(h), 8, mask) == 0
    st = torch.cuda.ExternalStream(h.value)
    with torch.cuda.stream(st):
        ctx = fe.Context(0, st)
        for n, one in ((9, True), (60, False)):   # 4 groups; 222 on the whole device
            mesh, L, f = system(fe, ctx, HEX, n)
            x, info, launches = solve(fe, mesh, L, f, rtol=0.0, max_iter=5)
            assert launches == (1 if one else 5)
            xg, _ = fe.cg_solve_noalloc(mesh, L, f, rtol=0.0, max_iter=5)
            assert rel(host(x), host(xg)) <= 1e-12
            st.synchronize()
            ctx.check(ctx.lib.fe_ctx_set_stream(ctx.h, ctypes.c_void_p(fe_ctx.stream.cuda_stream)))
            assert solve(fe, mesh, L, f, rtol=0.0, max_iter=5)[2] == 1
            torch.cuda.synchronize()
            ctx.check(ctx.lib.fe_ctx_set_stream(ctx.h, h))
            mesh.close()
        ctx.close()
    assert hip.hipStreamDestroy(h) == 0


# rows of 27 entries: 72^3 is the last cube that fits the registers in FP64, 85^3 in
# FP32; rows of 15: 82^3 in FP64
@pytest.mark.parametrize("kind,n,fp64,mixed", [(HEX, 4, True, True), (HEX, 23, True, True), (HEX, 72, True, True),
                                               (HEX, 73, False, True), (HEX, 86, False, False), (TET, 24, True, True),
                                               (TET, 82, True, True), (TET, 83, False, True), (PEN, 12, True, True),
                                               (PYR, 12, True, True), (HYB, 17, True, True)])
def test_form_by_size(fe_ctx, kind, n, fp64, mixed):
    import paper_2107_11541_amd as fe
    mesh, L, f = system(fe, fe_ctx, kind, n)
    _, info, launches = solve(fe, mesh, L, f, rtol=0.0, max_iter=5)
    assert info["symmetric_spmv"] and launches == (1 if fp64 else 5)
    _, info, launches = solve(fe, mesh, L, f, rtol=0.0, max_iter=5, precision=fe.MIXED)
    assert info["iterations"] == 5 and launches == (1 if mixed else 5)
    mesh.close()


def test_form_of_a_halo_that_does_not_fit(fe_ctx):
    import paper_2107_11541_amd as fe
    mesh, L, f = system(fe, fe_ctx, HEX, 26, renumber=False)
    for precision in (fe.FP64, fe.MIXED):
        assert solve(fe, mesh, L, f, rtol=0.0, max_iter=5, precision=precision)[2] == 5
    mesh.close()


# the general form's symmetric SpMV on every pattern: small meshes by giving the
# one launch up, and one too large for it
@pytest.mark.parametrize("kind,n", [(HEX, 14), (TET, 24), (PEN, 16), (PYR, 12), (HYB, 12), (PYR, 60)])
def test_symmetric_spmv_of_the_general_form(fe_ctx, kind, n):
    import paper_2107_11541_amd as fe
    mesh, L, f = system(fe, fe_ctx, kind, n)
    hooks(mesh, stopped=True)
    solve(fe, mesh, L, f, rtol=0.0, max_iter=1)
    xs, info, launches = solve(fe, mesh, L, f, rtol=0.0, max_iter=5)
    xg, want = fe.cg_solve_noalloc(mesh, L, f, rtol=0.0, max_iter=5)
    assert info["symmetric_spmv"] and not want["symmetric_spmv"] and launches == 5
    assert rel(host(xs), host(xg)) <= 1e-12
    assert abs(info["rel_residual"] - want["rel_residual"]) <= 1e-12 * want["rel_residual"]
    mesh.close()
