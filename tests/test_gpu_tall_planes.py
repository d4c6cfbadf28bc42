"""Planes with columns of more than 128 values and short rows, which the plane
kernel holds while its buffers fit the LDS, against the float64 oracle with the
tolerances of the parity tests."""

import numpy as np
import pytest

from oracle import precond as PC
from oracle import wavelet as W
from paper_0904_1543_amd import inputs, ops
from parity_helpers import TOL, assert_close, assert_scalar

pytestmark = pytest.mark.gpu

HG = (0.8, 1.0, 0.9)


# two buffers (rows of up to 32 and 64 values), one, and too tall for any in float64
@pytest.mark.parametrize("dims", [(2, 150, 2), (12, 80, 3), (30, 76, 2), (40, 77, 2), (40, 100, 2)])
@pytest.mark.parametrize("prec", ["f64", "f32", "f32c"])
def test_tall_planes(dims, prec):
    cs = inputs.random_case(240, 3, dims, potential="gauss16")
    occ = np.array([2.0, 0.5, 1.25])
    C, V, tol = cs["C"], cs["V"], TOL[prec]
    plan = ops.Plan(cs["dims"], prec=prec, hgrid=HG, occ=occ)
    c, Vt = plan.pack(C), plan.pack_potential(V)
    ref = W.local_hpsi(C, V, occ, hgrid=HG)
    r = plan.local_hpsi(c, Vt, per_orbital=True)
    assert_close(plan.unpack(r["hpsi"]), list(ref["hpsi"]), tol, "hpsi")
    assert_close(r["rho"].cpu().numpy(), ref["rho"].ravel(), tol, "rho")
    assert_scalar(r["energies"][0].item(), ref["e_loc"], tol, "E_loc")
    assert_scalar(r["energies"][1].item(), ref["e_kin"], tol, "E_kin")
    assert_close(plan.local_density(c).cpu().numpy(), ref["rho"].ravel(), tol, "density")
    g = plan.energy_gradient(c, Vt)
    assert_close(plan.unpack(g), [2.0 * f * h for f, h in zip(occ, ref["hpsi"])], tol, "gradient")
    eps = np.array([-0.2, -0.7, -1.0])
    x = plan.unpack(plan.precondition(c, eps, 2))
    assert_close(x, [PC.pcg(C[b], eps[b], 2, hgrid=HG)[0] for b in range(3)], tol, "preconditioner")
