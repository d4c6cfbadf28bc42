"""The preconditioner on batches of several grids, on both sides of the plane
sizes at which its in-plane operator changes kernels, against the float64 oracle
with the tolerances of the parity tests."""

import numpy as np
import pytest

from oracle import precond as PC
from paper_0904_1543_amd import inputs, ops
from parity_helpers import TOL, assert_close

pytestmark = pytest.mark.gpu

HG = (0.8, 1.0, 0.9)
DIMS = {
    "64": [(32, 20, 3), (12, 32, 5), (7, 9, 2)],            # planes of up to 64 x 64
    "66": [(33, 20, 3), (12, 32, 5), (7, 9, 2)],            # ... one row longer
    "tall": [(20, 33, 3), (12, 32, 5), (7, 9, 2)],
    "112": [(56, 41, 2), (12, 56, 3), (33, 2, 4)],          # 49 tiles of 16 x 16; float32: 7 items
    "114": [(57, 49, 2), (12, 57, 3), (33, 2, 4)],          # 64 tiles
    "96": [(48, 48, 2), (16, 40, 3), (2, 3, 49)],           # float32: 5 items
    "128": [(64, 64, 2), (40, 12, 3), (9, 8, 5)],
}


@pytest.mark.parametrize("case", list(DIMS))
@pytest.mark.parametrize("prec", ["f64", "f32", "f32c"])
def test_uneven_planes(case, prec):
    dims, tol = DIMS[case], TOL[prec]
    C = inputs.coefficients(inputs.rng_for(230), dims)
    eps = np.array([-0.2, -0.6, -1.0])
    plan = ops.Plan(dims, prec=prec, shared_v=False, hgrid=HG)
    g = plan.pack(C)
    for iters in (1, 3):
        x, res = plan.precondition(g, eps, iters, residuals=True)
        want = [PC.pcg(C[b], eps[b], iters, HG) for b in range(3)]
        assert_close(plan.unpack(x), [w[0] for w in want], tol, f"{iters} steps")
        assert_close(res.cpu().numpy(), np.array([w[1] for w in want]), tol, f"residuals, {iters} steps")
