"""Compensated plans on both sides of the longest rows that the plane kernel
takes (128 values): the variant and the preconditioner's form keep
their numbers; beyond it the exact digit products run.  Against the float64
oracle with the tolerance of the parity tests."""

import numpy as np
import pytest

from oracle import precond as PR
from oracle import wavelet as W
from paper_0904_1543_amd import inputs, lib, ops
from parity_helpers import TOL, assert_close, assert_scalar

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(64, 32, 8), (72, 32, 8), (32, 72, 8), (8, 8, 72)])
def test_float_pairs_by_plane_length(dims):
    cs = inputs.random_case(99, 3, dims, potential="gauss16")
    C, V, occ, tol = cs["C"], cs["V"], np.array([2.0, 1.0, 0.5]), TOL["f32c"]
    plan = ops.Plan(cs["dims"], prec="f32c", occ=occ)
    assert plan.query(lib.WVL_Q_VARIANT) == 3 and plan.query(lib.WVL_Q_PRECOND_FORM) == 2
    assert plan.query(lib.WVL_Q_FUSED_Z) == (1 if dims[0] <= 64 else 0)
    ref = W.local_hpsi(C, V, occ)
    c, Vt = plan.pack(C), plan.pack_potential(V)
    r = plan.local_hpsi(c, Vt)
    assert_close(plan.unpack(r["hpsi"]), list(ref["hpsi"]), tol, "hpsi")
    assert_close(r["rho"].cpu().numpy(), ref["rho"].ravel(), tol, "rho")
    e = r["energies"].cpu().numpy()
    assert_scalar(e[0], ref["e_loc"], tol, "E_loc")
    assert_scalar(e[1], ref["e_kin"], tol, "E_kin")
    g = plan.energy_gradient(c, Vt)
    assert_close(plan.unpack(g), [2.0 * f * h for f, h in zip(occ, ref["hpsi"])], tol, "gradient")
    eps = np.array([-0.2, -0.6, -1.0])
    x = plan.unpack(plan.precondition(c, eps, 3))
    assert_close(x, [PR.pcg(C[b], eps[b], 3)[0] for b in range(3)], tol, "preconditioner")
    plan.local_hpsi(c, Vt, out=c)
    assert_close(plan.unpack(c), list(ref["hpsi"]), tol, "in place")
