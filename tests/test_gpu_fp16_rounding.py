"""FP16 iterates of the CG kernels on the whole lattice (marching in time or
not) and of the even-odd tile kernels, bit for bit.

Which components of an FP16 field are rounded within the last multiply-add is
the compiler's choice and moves with the code around it; these solves amplify
such a change to 1e-4 of their norm.  The digests are of the FP32 solutions
after three steps on an 8^3 x 16 lattice."""

import hashlib

import pytest

from lattice_inputs import make_gauge

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("solver,nr,march,tiles,digest", [
    (0, 2, 8, 0, "df4e21e5c35ee9a46dc68992b8da8ac337baf87b0a59493cbcb5c435d6a50943"),
    (0, 2, 0, 0, "609706ff772ccb40aef6e5f4abb1f13937bbecbe81327d5c44523644c3a64b8d"),
    (2, 4, 0, 1, "b6f17ddba005849049417a1a1f829bb8a22ff4b1f860c04aa462d538c9681eef")])
def test_fp16_iterates_keep_their_roundings(solver, nr, march, tiles, digest):
    import paper_1211_0126_amd as tq
    dims = (8, 8, 8, 16)
    ctx = tq.tm_create(dims, 0.1632, 0.004, -1)
    tq.tm_gauge_load(ctx, make_gauge(dims, 0.25, 9))
    tq.tm_set_lane_rhs(ctx, tq.PREC_F16, nr)
    tq.tm_set_march(ctx, tq.PREC_F16, march)
    tq.tm_set_eo_tiles(ctx, tq.PREC_F16, tiles)
    p = tq.solve_params(prec=tq.PREC_F16, tol=0.0, max_iter=3, rhs_block=4, solver=solver, out_prec=tq.PREC_F32,
                        true_resid=0)
    x, _, _ = tq.tsm_solve_batch(ctx, p, 29, [0, 1, 2, 3])
    got = hashlib.sha256(x.cpu().numpy().tobytes()).hexdigest()
    ctx.close()
    assert got == digest
