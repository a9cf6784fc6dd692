"""The time-boundary sign of a transport layer is that of its transported
spinors, bit for bit: one layer that passes a single time path through, with
antiperiodic against periodic time."""

import numpy as np
import pytest

from lattice_inputs import make_gauge, random_spinor

pytestmark = pytest.mark.gpu


def test_antiperiodic_layer_is_the_negative_across_the_boundary():
    import torch
    import paper_1211_0126_amd as tq
    dims = (32, 32, 32, 2)
    U = make_gauge(dims, 0.25, 17)
    x = torch.from_numpy(random_spinor(dims, 5, 8)).cuda()
    half = dims[0] * dims[1] * dims[2]
    out = {}
    for t_bc in (1, -1):
        ctx = tq.tm_create(dims, 0.1632, 0.004, t_bc, caps=tq.caps([], field_rhs=8))
        tq.tm_gauge_load(ctx, U)
        for path in (7, 8):  # x + t, x - t
            w = np.zeros((9, 4, 4), dtype=np.complex128)
            w[path] = np.eye(4)
            tq.tm_precond_set(ctx, [1, 1], w.reshape(-1))
            out[path, t_bc] = tq.tm_precond_apply(ctx, x)
        ctx.close()
    for path, wrapped in ((7, slice(half, None)), (8, slice(0, half))):
        p, m = out[path, 1], out[path, -1]
        sign = torch.ones(2 * half, 1, 1, dtype=torch.float64, device="cuda")
        sign[wrapped] = -1
        assert torch.equal(m, sign * p), int((m != sign * p).sum())
