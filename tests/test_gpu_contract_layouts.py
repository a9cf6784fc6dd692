"""Contraction of canonical solutions: read in place where they are 16-byte
aligned, through the native layout otherwise (8-byte aligned callers of the C
ABI).  Each loop form and the transform to all momenta, on lattices whose rows
leave part of a wave and of a block idle, against the FP64 oracle (1e-10 of
the largest loop, the bound of the other loop tests) and each other."""

import ctypes

import numpy as np
import pytest

from lattice_inputs import make_gauge, random_spinor
from lattice_inputs.workloads import momenta_27

pytestmark = pytest.mark.gpu

KAPPA, MU = 0.1632, 0.004


@pytest.mark.parametrize("dims", [(3, 5, 2, 4), (7, 4, 5, 3), (10, 6, 3, 5), (32, 2, 3, 2), (130, 2, 2, 3)])
@pytest.mark.parametrize("est", [0, 1, 2, 3])
def test_aligned_and_unaligned_solutions(orc, dims, est):
    import torch
    import paper_1211_0126_amd as tq
    U = make_gauge(dims, 0.25, 9)
    ctx = tq.tm_create(dims, KAPPA, MU, -1)
    tq.tm_gauge_load(ctx, U)
    n, ids, mom = 3, [4, 0, 9], momenta_27()[[0, 5, 13, 22]]
    s = random_spinor(dims, 21, n)
    sol = torch.from_numpy(s).cuda()
    got = tq.tsm_contract(ctx, 31, ids, sol, mom, estimator=est)
    off = torch.empty(2 * sol.numel() + 1, dtype=torch.float64, device="cuda")[1:]
    off.copy_(torch.view_as_real(sol).reshape(-1))
    other = np.zeros_like(got)
    mm = np.ascontiguousarray(mom, dtype=np.int32)
    ida = np.asarray(ids, dtype=np.uint64)
    rc = ctx.lib.tsm_contract_est(ctx.h, est, 31, n, ida.ctypes.data_as(ctypes.c_void_p), ctypes.c_void_p(off.data_ptr()),
                                  len(mom), mm.ctypes.data_as(ctypes.c_void_p), other.ctypes.data_as(ctypes.c_void_p))
    assert rc == 0 and off.data_ptr() % 16 == 8
    scale = np.max(np.abs(got))
    assert np.max(np.abs(got - other)) <= 1e-13 * scale
    for i, j in enumerate(ids):
        eta = orc.noise_z4(dims, 31, j)
        if est == 3:
            ref = orc.loops_deriv(dims, -1, U, eta, s[i], mom)
        else:
            ref = orc.loops_est(dims, -1, KAPPA, MU, U, est, s[i], mom, eta=eta)
        assert np.max(np.abs(got[i] - ref)) < 1e-10 * max(scale, np.max(np.abs(ref)))
    ctx.close()


@pytest.mark.parametrize("dims,n", [((8, 8, 8, 16), 1), ((8, 8, 8, 32), 1), ((9, 8, 8, 31), 3), ((16, 16, 16, 32), 1)])
def test_large_results_reach_the_host(orc, dims, n):
    """All momenta: 2 MiB (one copy), 4 MiB, 13.0 MiB in half-MiB pieces with a
    short last one, and 32 MiB; the sum over momenta of a loop is the volume
    times its value at the origin."""
    import torch
    import paper_1211_0126_amd as tq
    ctx = tq.tm_create(dims, KAPPA, MU, -1, caps=tq.caps([], max_sources=n, all_mom_sources=n))
    tq.tm_gauge_load(ctx, make_gauge(dims, 0.25, 9))
    s = random_spinor(dims, 21, n)
    sol = torch.from_numpy(s).cuda()
    got = tq.tsm_contract(ctx, 31, list(range(n)), sol, None)
    again = tq.tsm_contract(ctx, 31, list(range(n)), sol, None)
    ctx.close()
    assert np.array_equal(got, again)
    V3 = dims[0] * dims[1] * dims[2]
    for j in range(n):
        eta = orc.noise_z4(dims, 31, j).reshape(dims[3], V3, 12)
        at0 = np.sum(np.conj(eta[:, 0]) * s[j].reshape(dims[3], V3, 12)[:, 0], axis=1)
        total = got[j][0].sum(axis=0) / V3
        assert np.max(np.abs(total - at0)) < 1e-11 * np.max(np.abs(got[j]))
        # p = 0 against the direct sum
        ref = np.sum(np.conj(eta) * s[j].reshape(dims[3], V3, 12), axis=(1, 2))
        assert np.max(np.abs(got[j][0][0] - ref)) < 1e-11 * np.max(np.abs(ref))
