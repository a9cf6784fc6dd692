"""The order in which the stencils visit the lattice and how they deal right-
hand sides to waves: lattices of several slabs whose sites do not fill the
last wave, blocks of every width class (4, 2 and 1 chunks per block).  FP64
iterates against the oracle to 1e-12 (the bound of the other operator tests);
every source of a block bit for bit what it is alone."""

import numpy as np
import pytest

from lattice_inputs import make_gauge, random_spinor

pytestmark = pytest.mark.gpu

KAPPA, MU = 0.1632, 0.004
# several slabs of 3, 2 and 7 planes (whole lattice and half), ragged waves
LATTICES = [(10, 6, 12, 6), (14, 10, 4, 6), (6, 18, 14, 4)]


def _ctx(dims):
    import paper_1211_0126_amd as tq
    U = make_gauge(dims, 0.25, 17)
    ctx = tq.tm_create(dims, KAPPA, MU, -1)
    tq.tm_gauge_load(ctx, U)
    return ctx, U


@pytest.mark.parametrize("dims", LATTICES)
def test_operator_in_slab_order(orc, dims):
    import torch
    import paper_1211_0126_amd as tq
    ctx, U = _ctx(dims)
    x = random_spinor(dims, 5, 3)
    y = tq.tm_dslash(ctx, tq.OP_MDAGM, tq.PREC_F64, torch.from_numpy(x).cuda()).cpu().numpy()
    ctx.close()
    for r in range(3):
        ref = orc.apply_op(dims, -1, KAPPA, MU, tq.OP_MDAGM, U, x[r])
        assert np.linalg.norm(y[r] - ref) < 1e-12 * np.linalg.norm(ref)


@pytest.mark.parametrize("dims", LATTICES)
@pytest.mark.parametrize("n", [1, 2, 3, 4, 6, 8])
def test_evenodd_blocks(orc, dims, n):
    import torch
    import paper_1211_0126_amd as tq
    ctx, U = _ctx(dims)
    ids = [3 * i + 1 for i in range(n)]

    def solve(prec, which, block):
        p = tq.solve_params(prec=prec, tol=0.0, max_iter=3, rhs_block=block, solver=tq.SOLVER_CG_EO, true_resid=0)
        return tq.tsm_solve_batch(ctx, p, 29, which)[0]

    x = solve(tq.PREC_F64, ids, n)
    ref, _ = orc.cgnr_eo(dims, -1, KAPPA, MU, U, orc.noise_z4(dims, 29, ids[-1]), 0.0, 3)
    assert np.linalg.norm(x[-1].cpu().numpy() - ref) < 1e-12 * np.linalg.norm(ref)
    for prec in (tq.PREC_F64, tq.PREC_F32, tq.PREC_F16):
        for nr in (1, 2):
            if n % nr == 0:
                tq.tm_set_lane_rhs(ctx, prec, nr)
                x = solve(prec, ids, n)
                for i in range(n):
                    assert torch.equal(x[i], solve(prec, ids[i:i + 1], 1)[0]), (prec, nr, i)
    ctx.close()


@pytest.mark.parametrize("prec", [0, 1, 2, 3])
@pytest.mark.parametrize("n", [1, 2, 3])
def test_canonical_fields_at_any_alignment(prec, n):
    """Canonical fields in place (16-byte aligned) and through the staging
    buffers (views one complex number further): the same kernel arithmetic,
    bit for bit, and the native layout's result."""
    import torch
    import paper_1211_0126_amd as tq
    dims = LATTICES[0]
    ctx, _ = _ctx(dims)
    x = torch.from_numpy(random_spinor(dims, 3, n)).cuda()
    if prec == tq.PREC_F32:
        x = x.to(torch.complex64)
    elif prec != tq.PREC_F64:
        x = torch.view_as_real(x).to(torch.float16 if prec == tq.PREC_F16 else torch.bfloat16).contiguous()
    step = 1 if x.is_complex() else 2
    odd = torch.empty(x.numel() + step, dtype=x.dtype, device="cuda")[step:].view(x.shape)
    odd.copy_(x)
    for op in (tq.OP_M, tq.OP_MDAG, tq.OP_MDAGM, tq.OP_HOP):
        y = tq.tm_dslash(ctx, op, prec, x)
        z = torch.empty(x.numel() + step, dtype=x.dtype, device="cuda")[step:].view(x.shape)
        assert torch.equal(y, tq.tm_dslash(ctx, op, prec, odd, out=z))
        assert torch.equal(y, tq.tm_dslash(ctx, op, prec, odd))
        assert torch.equal(y, tq.tm_dslash(ctx, op, prec, x, out=z))
        nb = tq.tm_field_bytes(ctx, prec, n, tq.LAYOUT_NATIVE)
        a, b = (torch.empty(nb, dtype=torch.uint8, device="cuda") for _ in range(2))
        tq.tm_field_convert(ctx, prec, n, True, x, a)
        tq.tm_dslash(ctx, op, prec, a, out=b, layout=tq.LAYOUT_NATIVE, nrhs=n)
        tq.tm_field_convert(ctx, prec, n, False, b, z)
        assert torch.equal(y, z)
    ctx.close()


@pytest.mark.parametrize("solver", [0, 2])
@pytest.mark.parametrize("prec", [0, 1, 2, 3])
def test_small_and_large_launches_agree(orc, solver, prec):
    """One source alone (a direction per wave, reductions merged into the CG
    kernels) and in a block of 16 (one lane per site, reductions launched): the
    same iterate bit for bit, after a truncation and after a converged solve."""
    import torch
    import paper_1211_0126_amd as tq
    dims = (16, 16, 16, 12)
    ctx, U = _ctx(dims)
    ids = list(range(16))
    for kw in (dict(tol=0.0, max_iter=3), dict(tol=1e-2)):
        def solve(which):
            p = tq.solve_params(prec=prec, rhs_block=16, solver=solver, true_resid=0, **kw)
            return tq.tsm_solve_batch(ctx, p, 29, which)[:2]
        x, st = solve(ids)
        for i in (0, 7, 15):
            y, sy = solve(ids[i:i + 1])
            assert torch.equal(x[i], y[0]) and st[i]["iters"] == sy[0]["iters"], (kw, i)
        if prec == 0 and kw["tol"] == 0.0:
            f = orc.cgnr_eo if solver else orc.cgnr
            ref, _ = f(dims, -1, KAPPA, MU, U, orc.noise_z4(dims, 29, 7), 0.0, 3)
            assert np.linalg.norm(x[7].cpu().numpy() - ref) < 1e-12 * np.linalg.norm(ref)
    ctx.close()


@pytest.mark.parametrize("dims,nrhs", [((10, 14, 18, 20), 7), ((8, 10, 12, 10), 7), ((16, 16, 10, 6), 7)])
@pytest.mark.parametrize("adjoint", [False, True])
def test_network_right_hand_sides_per_block(orc, dims, nrhs, adjoint):
    """Transport layers with 4, 1 and 2 right-hand sides per block (ragged last
    tiles, pairs and a single one): each field as when it is given alone."""
    import torch
    import paper_1211_0126_amd as tq
    ctx, U = _ctx(dims)
    widths = [1, 2, 2, 1]
    rng = np.random.default_rng(3)
    n = orc.net_weight_count(widths)
    tq.tm_precond_set(ctx, widths, 0.3 * (rng.standard_normal(n) + 1j * rng.standard_normal(n)))
    x = torch.from_numpy(random_spinor(dims, 5, nrhs)).cuda()
    y = tq.tm_precond_apply(ctx, x, adjoint=adjoint)
    for r in range(nrhs):
        assert torch.equal(y[r], tq.tm_precond_apply(ctx, x[r:r + 1].contiguous(), adjoint=adjoint)[0]), r
    ctx.close()


@pytest.mark.parametrize("graphs", [False, True])
@pytest.mark.parametrize("maxit", [1, 2, 8, 9, 21])
def test_cg_steps_finished_in_the_next_launch(orc, maxit, graphs):
    """Lattices of few waves (the last one ragged): the direction and the stop
    test of a step are formed by the next one's first stencil, the last step of
    a chunk by a launch of its own.  Truncated inside and at the ends of chunks,
    repeated, eager and captured: FP64 iterates against the oracle (1e-12) and
    FP32 ones against FP64 (2e-5: FP32 rounding over 21 steps)."""
    import torch
    import paper_1211_0126_amd as tq
    dims = (3, 5, 4, 6)
    U = make_gauge(dims, 0.25, 17)
    stream = torch.cuda.Stream()  # (graphs need a stream of their own)
    with torch.cuda.stream(stream):
        ctx = tq.tm_create(dims, KAPPA, MU, -1, stream=stream)
        tq.tm_gauge_load(ctx, U)
        n0 = tq.tm_set_graphs(ctx, graphs)
        ref, _ = orc.cgnr(dims, -1, KAPPA, MU, U, orc.noise_z4(dims, 29, 7), 0.0, maxit)
        for prec, tol in ((tq.PREC_F64, 1e-12), (tq.PREC_F32, 2e-5)):
            p = tq.solve_params(prec=prec, tol=0.0, max_iter=maxit, rhs_block=4, true_resid=0)
            for _ in range(3):
                x, st, _ = tq.tsm_solve_batch(ctx, p, 29, [7, 8])
                assert st[0]["iters"] == maxit
                assert np.linalg.norm(x[0].cpu().numpy() - ref) < tol * np.linalg.norm(ref)
        assert (tq.tm_set_graphs(ctx) > n0) == graphs
        ctx.close()


@pytest.mark.parametrize("solver,kw,bound", [
    # M^dag M >= (2 kappa mu)^2 and |M| < 2.4: two solutions with true residuals
    # below 1e-10 differ by less than 2e-10 * 2.4 / (2 kappa mu) = 3.7e-7
    (2, dict(tol=1e-10, max_iter=-1, reliable=1, delta=0.1), 4e-7),
    # the same directions and step lengths, FP32 sums of five terms
    (0, dict(tol=0.0, max_iter=5), 1e-5)])
def test_kept_directions_only_where_the_workspace_has_room(solver, kw, bound):
    """16-bit solves that keep their directions in a ring where the workspace has
    room, and where it lacks a MiB for that update x in every iteration."""
    import paper_1211_0126_amd as tq
    dims = (8, 8, 8, 8)
    U = make_gauge(dims, 0.25, 17)
    p = tq.solve_params(prec=tq.PREC_F16, rhs_block=8, solver=solver, **kw)
    x, size = [], None
    for _ in range(2):
        ctx = tq.tm_create(dims, KAPPA, MU, -1, workspace_bytes=size)
        tq.tm_gauge_load(ctx, U)
        for _ in range(2):
            y, st, _ = tq.tsm_solve_batch(ctx, p, 29, list(range(8)))
            assert all(s["converged"] for s in st) or kw["tol"] == 0.0
            x.append(y.cpu())
        use = ctx.workspace_usage()
        size = use["persistent"] + use["peak_scratch"] - (1 << 20)
        ctx.close()
    assert (x[0] == x[1]).all() and (x[2] == x[3]).all()
    assert (x[0] - x[2]).norm() < bound * x[0].norm()
