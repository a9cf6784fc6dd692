"""One-derivative loops of FP32 solutions against the FP64 contraction of the
same solutions: no further off than the form with four transports per link,
measured on these inputs, was."""

import numpy as np
import pytest

from lattice_inputs import make_gauge
from lattice_inputs.workloads import momenta_27

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,bound", [((8, 8, 8, 16), 6.9e-8), ((16, 16, 16, 32), 3.9e-8)])
def test_fp32_loops_are_as_close_to_fp64(dims, bound):
    import paper_1211_0126_amd as tq
    ctx = tq.tm_create(dims, 0.1632, 0.004, -1)
    tq.tm_gauge_load(ctx, make_gauge(dims, 0.25, 9))
    lp = tq.solve_params(prec=tq.PREC_F32, tol=1e-2, rhs_block=16, true_resid=0)
    mom, ids = momenta_27(), list(range(16))
    got = tq.tsm_loops(ctx, 7, 0, 16, lp, lp, mom, per_source=True, estimator=tq.LOOP_DERIVATIVE)["per_source"]
    sol, _, _ = tq.tsm_solve_batch(ctx, lp, 7, ids)
    ref = tq.tsm_contract(ctx, 7, ids, sol, mom, estimator=tq.LOOP_DERIVATIVE)
    ctx.close()
    got = np.asarray(got)[:, 0].reshape(ref.shape)
    assert np.linalg.norm(got - ref) < bound * np.linalg.norm(ref)
