"""CG launches too large for the direction-per-wave kernels, at every lane width
(1, 2, 4 sources) and every dealing of waves (4, 2 and 1 chunks of sources per
block), on a lattice that leaves its last wave ragged; the operator at two
fields per lane; and the steps that small launches fold into the next one.

Every source of a block is bit for bit what it is alone, where the
direction-per-wave kernels solve it; FP64 iterates against the oracle to 1e-12
(the bound of the other operator tests)."""

import numpy as np
import pytest

from lattice_inputs import make_gauge, random_spinor

pytestmark = pytest.mark.gpu

KAPPA, MU = 0.1632, 0.004
# 9240 half sites (145 groups of 64, the last of 24), 18480 sites (289, 48);
# launches of more than 1536 groups have a lane per site
DIMS = (6, 10, 14, 22)


def _ctx(dims):
    import paper_1211_0126_amd as tq
    U = make_gauge(dims, 0.25, 17)
    ctx = tq.tm_create(dims, KAPPA, MU, -1)
    tq.tm_gauge_load(ctx, U)
    return ctx, U


@pytest.mark.parametrize("prec", [0, 1, 2, 3])
@pytest.mark.parametrize("solver,blocks", [(2, (11, 12, 14, 16)), (0, (6, 7, 8))])
def test_blocks_of_every_width(orc, solver, blocks, prec):
    import torch
    import paper_1211_0126_amd as tq
    ctx, U = _ctx(DIMS)
    groups = 145 if solver else 289
    assert min(blocks) * groups > 1536

    def solve(ids, kw):
        p = tq.solve_params(prec=prec, rhs_block=16, solver=solver, true_resid=0, **kw)
        return tq.tsm_solve_batch(ctx, p, 29, ids)[:2]

    for kw in (dict(tol=0.0, max_iter=3), dict(tol=1e-2)):
        alone = {i: solve([i], kw) for i in (0, 1, 5, max(blocks) - 1)}
        if prec == 0 and kw["tol"] == 0.0:
            f = orc.cgnr_eo if solver else orc.cgnr
            ref, _ = f(DIMS, -1, KAPPA, MU, U, orc.noise_z4(DIMS, 29, 5), 0.0, 3)
            assert np.linalg.norm(alone[5][0][0].cpu().numpy() - ref) < 1e-12 * np.linalg.norm(ref)
        for n in blocks:
            for nr in (1, 2, 4):
                if n % nr or (prec == 0 and nr > 1):
                    continue
                tq.tm_set_lane_rhs(ctx, prec, nr)
                tq.tm_profile_enable(ctx, True)
                x, st = solve(list(range(n)), kw)
                widths = {e["lane_rhs"] for e in tq.tm_profile_entries(ctx) if e["kc"] in ("dslash", "dslash_upd")}
                tq.tm_profile_enable(ctx, False)
                assert widths == {nr}
                for i, (y, sy) in alone.items():
                    if i < n:
                        assert torch.equal(x[i], y[0]) and st[i]["iters"] == sy[0]["iters"], (kw, n, nr, i)
                tq.tm_set_lane_rhs(ctx, prec, 0)
    ctx.close()


@pytest.mark.parametrize("prec", [2, 3])
def test_operator_with_two_fields_per_lane(prec):
    """16 fields of a ragged volume: each operation on aligned, unaligned and
    native fields as on one field alone (one per lane), bit for bit."""
    import torch
    import paper_1211_0126_amd as tq
    dims, n = (15, 14, 13, 12), 16  # 32760 sites: 56 in the last wave
    ctx, _ = _ctx(dims)
    assert ctx.V * n >= 500000 and ctx.V % 64
    dt = torch.float16 if prec == tq.PREC_F16 else torch.bfloat16
    x = torch.view_as_real(torch.from_numpy(random_spinor(dims, 3, n)).cuda()).to(dt).contiguous()
    odd = torch.empty(x.numel() + 2, dtype=dt, device="cuda")[2:].view(x.shape)
    odd.copy_(x)
    z = torch.empty(x.numel() + 2, dtype=dt, device="cuda")[2:].view(x.shape)
    nb = tq.tm_field_bytes(ctx, prec, n, tq.LAYOUT_NATIVE)
    a, b = (torch.empty(nb, dtype=torch.uint8, device="cuda") for _ in range(2))
    tq.tm_field_convert(ctx, prec, n, True, x, a)
    for op in (tq.OP_M, tq.OP_MDAG, tq.OP_MDAGM, tq.OP_HOP):
        y = tq.tm_dslash(ctx, op, prec, x)
        for i in (0, 1, 14, 15):
            assert torch.equal(y[i], tq.tm_dslash(ctx, op, prec, x[i:i + 1].contiguous())[0]), (op, i)
        assert torch.equal(y, tq.tm_dslash(ctx, op, prec, odd, out=z)), op
        tq.tm_dslash(ctx, op, prec, a, out=b, layout=tq.LAYOUT_NATIVE, nrhs=n)
        tq.tm_field_convert(ctx, prec, n, False, b, z)
        assert torch.equal(y, z), op
    ctx.close()


@pytest.mark.parametrize("prec", [0, 1])
def test_folded_steps_are_those_of_larger_blocks(prec):
    """One source alone (210 groups: each step finished by the next one's first
    stencil), in a block of 4 (840: a direction per wave, three launches a step)
    and of 16 (3360: a lane per site), truncated and converged: the same bits."""
    import torch
    import paper_1211_0126_amd as tq
    ctx, _ = _ctx((10, 12, 8, 14))
    for kw in (dict(tol=0.0, max_iter=1), dict(tol=0.0, max_iter=7), dict(tol=1e-2), dict(tol=1e-5)):
        out = {}
        for n in (1, 4, 16):
            p = tq.solve_params(prec=prec, rhs_block=16, solver=tq.SOLVER_CG, true_resid=0, **kw)
            out[n] = tq.tsm_solve_batch(ctx, p, 29, list(range(n)))[:2]
        for n in (4, 16):
            assert torch.equal(out[n][0][0], out[1][0][0]), (kw, n)
            assert out[n][1][0]["iters"] == out[1][1][0]["iters"], (kw, n)
    ctx.close()


@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (16, 16, 16, 12), (16, 16, 16, 32), (16, 16, 16, 34)])
@pytest.mark.parametrize("solver", [0, 2])
def test_tracked_residuals_of_every_sum(dims, solver):
    """The true residual that a solve tracks (two arrays of 4 to 2176 partials:
    one pass of a wave, several, a block) is the one computed from the solution,
    to the rounding of five FP64 steps."""
    import paper_1211_0126_amd as tq
    ctx, _ = _ctx(dims)
    p = tq.solve_params(prec=tq.PREC_F64, tol=0.0, max_iter=5, rhs_block=2, solver=solver, stop=tq.STOP_TRUE,
                        true_resid=1)
    _, st, _ = tq.tsm_solve_batch(ctx, p, 29, [0, 1], want_solutions=False)
    ctx.close()
    for q in st:
        assert q["iters"] == 5 and abs(q["resid_iterated"] - q["resid_true"]) < 1e-12
