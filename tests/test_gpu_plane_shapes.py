"""The plane kernel at the edges of its launch shapes (rows of up to 32, 64,
80, 96 and 128 values; two plane buffers or one; short lines that wrap more
than once; segments and groups of lines that do not fill a wave), against the
float64 oracle with the tolerances of the parity tests: local H*psi with
density and energies, the density alone, the occupation-weighted gradient and
the preconditioner's operator, and one uneven batch that mixes every shape."""

import numpy as np
import pytest

from oracle import precond as PR
from oracle import wavelet as W
from paper_0904_1543_amd import inputs, ops
from parity_helpers import TOL, assert_close, assert_scalar

pytestmark = pytest.mark.gpu

HG = (0.8, 1.0, 0.9)      # keeps float pairs off the exact digit products
SHAPES = [(2, 2, 2), (16, 17, 2), (17, 16, 2), (32, 5, 3), (33, 40, 2), (40, 33, 2), (41, 48, 2),
          (48, 41, 2), (49, 20, 2), (2, 64, 2), (64, 2, 2), (64, 64, 2)]


@pytest.mark.parametrize("dims", SHAPES)
@pytest.mark.parametrize("prec", ["f64", "f32", "f32c"])
def test_plane_shapes(dims, prec):
    cs = inputs.random_case(90, 3, dims, potential="gauss16")
    occ = np.array([2.0, 0.5, 1.25])
    C, V, tol = cs["C"], cs["V"], TOL[prec]
    plan = ops.Plan(cs["dims"], prec=prec, hgrid=HG, occ=occ)
    c, Vt = plan.pack(C), plan.pack_potential(V)
    ref = W.local_hpsi(C, V, occ, hgrid=HG)
    r = plan.local_hpsi(c, Vt, per_orbital=True)
    assert_close(plan.unpack(r["hpsi"]), list(ref["hpsi"]), tol, "hpsi")
    assert_close(r["rho"].cpu().numpy(), ref["rho"].ravel(), tol, "rho")
    e, eo = r["energies"].cpu().numpy(), r["e_orb"].cpu().numpy()
    assert_scalar(e[0], ref["e_loc"], tol, "E_loc")
    assert_scalar(e[1], ref["e_kin"], tol, "E_kin")
    assert_close(eo[:3], ref["e_loc_orb"], tol, "e_pot per orbital")
    assert_close(eo[3:], ref["e_kin_orb"], tol, "e_kin per orbital")
    rho = plan.local_density(c)
    rho = plan.local_density(c, rho=rho, accumulate=True)
    assert_close(rho.cpu().numpy(), 2.0 * ref["rho"].ravel(), tol, "density, twice")
    g = plan.energy_gradient(c, Vt)
    assert_close(plan.unpack(g), [2.0 * f * h for f, h in zip(occ, ref["hpsi"])], tol, "gradient")
    eps = np.array([-0.2, -0.7, -1.0])
    x = plan.unpack(plan.precondition(c, eps, 2))
    assert_close(x, [PR.pcg(C[b], eps[b], 2, hgrid=HG)[0] for b in range(3)], tol, "preconditioner")


@pytest.mark.parametrize("prec", ["f64", "f32", "f32c"])
@pytest.mark.parametrize("persistent", [False, True])
def test_uneven_batch_of_every_shape(prec, persistent):
    dims = [(4, 5, 3), (64, 60, 2), (17, 16, 2), (41, 33, 2), (33, 12, 2), (48, 48, 2), (3, 61, 2),
            (16, 2, 4)]
    rng = inputs.rng_for(91)
    C = inputs.coefficients(rng, dims)
    V = [inputs.potential_gauss(rng, inputs.fine_shape(d)) for d in dims]
    plan = ops.Plan(dims, prec=prec, shared_v=False, persistent=persistent)
    c, Vt = plan.pack(C), plan.pack_potential(V)
    ref = W.local_hpsi(C, V, plan.occ, shared_v=False)
    r = plan.local_hpsi(c, Vt, per_orbital=True)
    eo = r["e_orb"].cpu().numpy()
    for b, got in enumerate(plan.unpack(r["hpsi"])):
        assert_close(got, ref["hpsi"][b], TOL[prec], f"orbital {b}")
    assert_close(eo[:len(dims)], ref["e_loc_orb"], TOL[prec], "e_pot per orbital")
    assert_close(eo[len(dims):], ref["e_kin_orb"], TOL[prec], "e_kin per orbital")
