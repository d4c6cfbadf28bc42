"""The plain-float32 preconditioner keeps its CG arithmetic in float64: the
vectors p, q = Kin p, r are stored as float32, everything between them is
float64, the shift q - eps p with the float64 eps included.

With |eps| far above the kinetic operator the solution is all but found by the
first step, and what is left of the residual is the rounding of the stored
vectors: |r1| is about 2^-24 |g|.  A second rounding of that size (the shift in
float32, or eps itself) changes the residual norm by tens of percent.  The
steps are emulated here with the same stored roundings."""

import numpy as np
import pytest

from oracle import precond as PC
from paper_0904_1543_amd import inputs, ops
from parity_helpers import assert_scalar

pytestmark = pytest.mark.gpu

EPS = (-(2.0 ** 25 + 1.9), -(2.0 ** 27 + 7.8))      # all but half way between float32 values


def _f32(x):
    return x.astype(np.float32).astype(np.float64)


def _emulate(g, eps, iters):
    inv = 1.0 / PC.helmholtz_diagonal(g.shape, eps)
    r = _f32(g)
    p = _f32(r * inv)
    rz = np.sum(r * (r * inv))
    for _ in range(iters):
        q = PC.helmholtz(p, 0.0)
        pq = np.sum(p * q) - eps * np.sum(p * p)
        alpha = rz / pq
        new = r - alpha * (_f32(q) - eps * p)
        rz, old = np.sum(new * (new * inv)), rz
        r = _f32(new)
        p = _f32(r * inv + rz / old * p)
    return np.linalg.norm(new)


@pytest.mark.parametrize("dims", [(8, 6, 5), (17, 18, 20)])
@pytest.mark.parametrize("form", [None, "passes"], ids=["plane", "passes"])
def test_shift_in_float64(dims, form):
    cs = inputs.random_case(180, 2, dims)
    plan = ops.Plan(cs["dims"], prec="f32")
    # One step: q comes from float32 passes, whose error of at most 60 roundings
    # of values below 30 |p| is 2e-4 / |eps| |g|, against |r1| of at least
    # 1e-8 |g|: below 1e-3.  Two steps: the rounding pattern of the second
    # direction is its own, the norm of N >= 1900 such roundings agrees to
    # 5 / sqrt(2 N) = 8% within five standard deviations.
    for iters, tol in ((1, 1e-3), (2, 0.1)):
        _, res = plan.precondition(plan.pack(cs["C"]), EPS, iters, form=form, residuals=True)
        for b, eps in enumerate(EPS):
            assert_scalar(res[b].item(), _emulate(cs["C"][b], eps, iters), tol,
                          f"residual after {iters} steps, eps = {eps}")
