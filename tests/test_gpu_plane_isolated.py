"""The plane kernel with isolated axes, whose lines hold m coefficients and
m + 29 real-space values, at the edges of its launch shapes (real-space rows
of up to 32, 64, 80, 96 and 128 values; the first size past the last shape,
which the axis passes take), for both condition sets, against the float64
oracle with the tolerances of the parity tests."""

import numpy as np
import pytest

from oracle import boundary as BC
from oracle import precond as PC
from paper_0904_1543_amd import inputs, ops
from parity_helpers import TOL, assert_close, assert_scalar

pytestmark = pytest.mark.gpu

HG = (0.8, 1.0, 0.9)
SHAPES = [(2, 2, 2), (2, 3, 2), (17, 2, 3), (18, 17, 2), (17, 18, 2), (25, 26, 2), (26, 25, 2),
          (33, 4, 2), (4, 33, 2), (34, 33, 2), (49, 2, 2), (49, 49, 2), (50, 49, 2), (5, 50, 2),
          (3, 64, 2)]


@pytest.mark.parametrize("dims", SHAPES)
@pytest.mark.parametrize("bc", ["free", "surface"])
@pytest.mark.parametrize("prec", ["f64", "f32", "f32c"])
def test_isolated_plane_shapes(dims, bc, prec):
    cs, occ, tol = inputs.random_case(95, 2, dims), np.array([2.0, 0.75]), TOL[prec]
    V = inputs.potential_gauss(inputs.rng_for(96), BC.real_space_shape(dims, bc))
    C = cs["C"]
    plan = ops.Plan(cs["dims"], prec=prec, hgrid=HG, occ=occ, bc=bc)
    c, Vt = plan.pack(C), plan.pack_potential(V)
    ref = BC.local_hpsi(C, V, occ, bc, HG)
    r = plan.local_hpsi(c, Vt, per_orbital=True)
    assert_close(plan.unpack(r["hpsi"]), ref["hpsi"], tol, "hpsi")
    assert_close(r["rho"].cpu().numpy(), ref["rho"].ravel(), tol, "rho")
    e, eo = r["energies"].cpu().numpy(), r["e_orb"].cpu().numpy()
    assert_scalar(e[0], ref["e_loc"], tol, "E_loc")
    assert_scalar(e[1], ref["e_kin"], tol, "E_kin")
    assert_close(eo[:2], ref["e_loc_orb"], tol, "e_pot per orbital")
    assert_close(eo[2:], ref["e_kin_orb"], tol, "e_kin per orbital")
    rho = plan.local_density(c)
    rho = plan.local_density(c, rho=rho, accumulate=True)
    assert_close(rho.cpu().numpy(), 2.0 * ref["rho"].ravel(), tol, "density, twice")
    g = plan.energy_gradient(c, Vt)
    assert_close(plan.unpack(g), [2.0 * f * h for f, h in zip(occ, ref["hpsi"])], tol, "gradient")
    eps = np.array([-0.3, -0.9])
    x = plan.unpack(plan.precondition(c, eps, 2))
    assert_close(x, [PC.pcg(C[b], eps[b], 2, HG, bc=bc)[0] for b in range(2)], tol, "preconditioner")
