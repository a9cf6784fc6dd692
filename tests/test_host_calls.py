"""Host code of the library on the CPU (see standin.py): what a call launches,
where it stops and what it leaves behind."""

from standin import run

# FP16 LP solves in blocks of 16, HP solves in blocks of 8 that keep their
# directions where they have room
SOLVES = """
tq = s.tq
dims = (8, 8, 8, 8)
large = (16, 16, 16, 8)  # where 16 sources keep their directions on the whole lattice
lp = tq.solve_params(prec=tq.PREC_F16, tol=1e-2, rhs_block=16, solver=tq.SOLVER_CG_EO, true_resid=0)
hp = tq.solve_params(prec=tq.PREC_F16, tol=1e-10, rhs_block=8, solver=tq.SOLVER_CG_EO, reliable=1, delta=3e-3)
whole = tq.solve_params(prec=tq.PREC_F16, tol=1e-2, rhs_block=16, solver=tq.SOLVER_CG, true_resid=0)

def named(launches, *parts):
    return [n for n, _ in launches if all(p in n for p in parts)]

def used(c):
    u = c.workspace_usage()
    return u["persistent"] + u["peak_scratch"]
"""


def test_a_call_without_room_for_directions_does_its_work_once(tmp_path):
    """The workspace that a call used with its directions kept, and 1 MiB less:
    each block of sources is prepared and solved once, in the first call and in
    the second, and without the room x is updated in every iteration."""
    run(tmp_path, SOLVES + """
calls = [(lambda c: tq.tsm_loops(c, 7, 8, 24, lp, hp, [[0, 0, 0]]), 4, "k_ring_rel_flush", dims),
         (lambda c: tq.tsm_solve_batch(c, hp, 7, list(range(8)), want_solutions=False), 1, "k_ring_rel_flush", dims),
         (lambda c: tq.tsm_solve_batch(c, whole, 7, list(range(16)), want_solutions=False), 1, "k_eo_xflush", large)]
for call, blocks, kept, dims in calls:
    size = 1 << 30
    for room in (True, True, False):
        c = s.context(dims, size)
        for _ in range(2):
            call(c)
            got = s.launches()
            assert len(named(got, "k_scal_init")) == blocks, (kept, room, len(named(got, "k_scal_init")))
            hp_kept = [n for n in named(got, kept) if "SF16" in n]
            assert bool(hp_kept) == room, (kept, room)
        size = used(c) if room and size == 1 << 30 else used(c) - (1 << 20)
        c.close()
""")


def test_directions_fit_the_workspace_of_the_fields(tmp_path):
    """tm_workspace_bytes asks for no room for directions (FP16 fields with
    reliable updates are smaller than FP32 ones, and so is their workspace, at
    every size), and yet the solves that it was asked for keep theirs in it."""
    run(tmp_path, SOLVES + """
import copy
for d in ((4, 4, 4, 4), dims, (32, 32, 32, 64)):
    for p in (hp, whole):
        wide = copy.copy(p)
        wide.prec = tq.PREC_F32
        a, b = (tq.tm_workspace_bytes(d, caps_=tq.caps([q], max_sources=32, max_mom=1)) for q in (p, wide))
        assert a < b, (d, a, b)
for d in (large, (16, 16, 12, 12)):
    for call, solves, kept in [
            (lambda c: tq.tsm_loops(c, 7, 8, 24, lp, hp, [[0, 0, 0]]), [lp, hp], "k_ring_rel_flush"),
            (lambda c: tq.tsm_loops(c, 7, 8, 24, whole, hp, [[0, 0, 0]]), [whole, hp], "k_ring_rel_flush"),
            (lambda c: tq.tsm_loops(c, 7, 0, 24, whole, whole, [[0, 0, 0]]), [whole], "k_eo_xflush"),
            (lambda c: tq.tsm_solve_batch(c, hp, 7, list(range(8)), want_solutions=False), [hp], "k_ring_rel_flush"),
            (lambda c: tq.tsm_solve_batch(c, whole, 7, list(range(32)), want_solutions=False), [whole], "k_eo_xflush")]:
        c = s.context(d, tq.tm_workspace_bytes(d, caps_=tq.caps(solves, max_sources=32, max_mom=1)))
        call(c)
        assert named(s.launches(), kept), (d, kept)
        c.close()
""")


def test_large_results_with_another_device_current(tmp_path):
    """A context on device 1 called with device 0 current: a result of 8 MiB
    reaches the host, and the caller's device is left as it was."""
    run(tmp_path, """
import ctypes
import numpy as np
tq = s.tq
dims = (8, 8, 8, 64)
c = s.context(dims, tq.tm_workspace_bytes(dims, caps_=tq.caps([], max_sources=1, all_mom_sources=1)), device=1)
s.hip.hipSetDevice(0)
sol = np.zeros(c.V * 24)
out = np.ones((1, 16, c.V), dtype=np.complex128)
ids = np.zeros(1, dtype=np.uint64)
rc = s.lib.tsm_contract(c.h, 31, 1, ids.ctypes.data_as(ctypes.c_void_p), sol.ctypes.data_as(ctypes.c_void_p),
                        tq.binding.ALL_MOMENTA, None, out.ctypes.data_as(ctypes.c_void_p))
assert rc == 0, s.lib.tm_last_error(c.h)
assert out.nbytes == 8 << 20 and not out.any()
assert s.hip.standin_device() == 0
c.close()
""")


def test_small_solves_take_one_source_per_lane(tmp_path):
    """Where the CG steps give each direction a wave, a lane width that is set
    neither fills a block up with further sources nor is timed by the tuners
    again (each candidate is 3 x 2 solves); tiles and marching keep theirs."""
    run(tmp_path, """
tq = s.tq
dims = (8, 8, 8, 8)
c = s.context(dims, 1 << 30)
groups = {tq.SOLVER_CG: 64, tq.SOLVER_CG_EO: 32}
for solver in groups:
    for prec in (tq.PREC_F32, tq.PREC_F16):
        tq.tm_set_lane_rhs(c, prec, 4)
        p = tq.solve_params(prec=prec, tol=1e-2, rhs_block=4, solver=solver, true_resid=0)
        for n in (1, 3, 4, 5):
            tq.tsm_solve_batch(c, p, 7, list(range(n)), want_solutions=False)
            grids = {g[0] for k, g in s.launches() if "k_quad_mp" in k}
            want = {groups[solver] * (1 if n == 1 else min(n, 4))} | ({groups[solver]} if n == 5 else set())
            assert grids == want, (solver, prec, n, grids)
tq.tm_set_eo_tiles(c, tq.PREC_F16, 1)
tq.tm_set_march(c, tq.PREC_F32, 4)
tq.tm_set_lane_rhs(c, tq.PREC_F32, 2)
tq.tm_set_lane_rhs(c, tq.PREC_F16, 2)
for prec, solver, kernel in ((tq.PREC_F16, tq.SOLVER_CG_EO, "k_eot_mp<false, tmq::SF16, 2>"),
                             (tq.PREC_F32, tq.SOLVER_CG, "k_tm_mp<float, tmq::SF32, tmq::GF32, 2>")):
    p = tq.solve_params(prec=prec, tol=1e-2, rhs_block=4, solver=solver, true_resid=0)
    tq.tsm_solve_batch(c, p, 7, [0], want_solutions=False)
    assert any(kernel in k for k, _ in s.launches()), kernel
tq.tm_autotune_cg(c, tq.PREC_BF16, 8)
assert sum("k_scal_init" in k for k, _ in s.launches()) == 6 * 6
tq.binding_tuning.tm_autotune_eo(c, tq.PREC_BF16, 8)
assert sum("k_scal_init" in k for k, _ in s.launches()) == 4 * 6
c.close()
""")


def test_pieces_of_large_results(tmp_path):
    """A result into pinned memory is one copy, as is one below 6 MiB into
    pageable memory; larger ones go in pieces through the pinned slots."""
    run(tmp_path, """
import ctypes
import numpy as np
tq = s.tq
for lt, pageable in ((32, [4 << 20]), (48, [512 << 10] * 12), (64, [512 << 10] * 16)):
    dims = (8, 8, 8, lt)
    c = s.context(dims, tq.tm_workspace_bytes(dims, caps_=tq.caps([], max_sources=1, all_mom_sources=1)))
    sol = np.zeros(c.V * 24)
    ids = np.zeros(1, dtype=np.uint64)
    pinned = ctypes.c_void_p()
    assert s.hip.hipHostMalloc(ctypes.byref(pinned), ctypes.c_size_t(16 * 16 * c.V), 0) == 0
    page = np.ones(16 * c.V, dtype=np.complex128)
    for out, pieces in ((pinned, [page.nbytes]), (page.ctypes.data_as(ctypes.c_void_p), pageable)):
        s.launches()
        rc = s.lib.tsm_contract(c.h, 31, 1, ids.ctypes.data_as(ctypes.c_void_p), sol.ctypes.data_as(ctypes.c_void_p),
                                tq.binding.ALL_MOMENTA, None, out)
        assert rc == 0, s.lib.tm_last_error(c.h)
        got = [g[0] for k, g in s.launches() if k == "copy"]
        assert got == pieces, got
    assert not page.any()
    c.close()
""")


def test_small_whole_lattice_solves_update_x(tmp_path):
    """16-bit solves on the whole lattice keep their directions from 4e5 sites
    times sources on (marching from 1e5), block by block, with one workspace."""
    run(tmp_path, SOLVES + """
size = tq.tm_workspace_bytes(large, caps_=tq.caps([whole], max_sources=32, max_mom=1))
c = s.context(large, size)
for n, march, kept in ((16, 0, 1), (12, 0, 0), (17, 0, 1), (4, 8, 1), (3, 8, 0)):
    tq.tm_set_march(c, tq.PREC_F16, march)
    tq.tm_set_lane_rhs(c, tq.PREC_F16, 1 if march else 0)
    tq.tsm_solve_batch(c, whole, 7, list(range(n)), want_solutions=False)
    assert len(named(s.launches(), "k_eo_xflush")) == kept, (n, march)
c.close()
""")


def test_marching_needs_a_lane_width(tmp_path):
    """A set marching length is used with a set width of 1 or 2, or where the
    block is no multiple of four sources (and in FP64, which has one per lane);
    a block of 16 without a width runs a lane per site."""
    run(tmp_path, """
tq = s.tq
c = s.context((8, 8, 8, 16), 1 << 30)
for prec in (tq.PREC_F64, tq.PREC_F32, tq.PREC_F16):
    tq.tm_set_march(c, prec, 8)
    for nr, block, marches in ((0, 16, prec == tq.PREC_F64), (0, 6, True), (0, 5, True), (1, 16, True), (2, 16, True),
                               (4, 16, prec == tq.PREC_F64)):
        tq.tm_set_lane_rhs(c, prec, nr)
        p = tq.solve_params(prec=prec, tol=1e-2, rhs_block=block, true_resid=0)
        tq.tsm_solve_batch(c, p, 7, list(range(2)), want_solutions=False)
        assert any("k_tm_mp" in k for k, _ in s.launches()) == marches, (prec, nr, block)
c.close()
""")
