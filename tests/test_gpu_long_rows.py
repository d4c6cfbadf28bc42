"""Planes whose rows are longer than the 128 values that the plane kernel of
wave-owned lines takes, outside the exact digit products: the workgroup-wide
in-plane kernels (local H*psi and the preconditioner's operator; matrix cores
and vector FMA) and the CG branch that goes with them, against the float64
oracle with the tolerances of the parity tests.  Shared potential with G > 1
density groups and a ragged last group; one potential per orbital, ordinary and
persistent; density, weighted gradient, in place, preconditioner."""

import numpy as np
import pytest

from oracle import precond as PC
from oracle import wavelet as W
from paper_0904_1543_amd import inputs, lib, ops
from parity_helpers import TOL, assert_close, assert_scalar

pytestmark = pytest.mark.gpu

HG = (0.8, 1.0, 0.9)
FORMS = ["f64", "f64_vector", "f32", "f32c"]


def _form(form, monkeypatch):
    if form == "f64_vector":
        monkeypatch.setenv("WVL_XY_VECTOR", "1")
    return form.split("_")[0]


@pytest.mark.parametrize("dims", [(72, 10, 5), (66, 7, 9), (66, 2, 2), (72, 40, 2), (100, 25, 3)])
@pytest.mark.parametrize("form", FORMS)
def test_shared_potential(dims, form, monkeypatch):
    prec = _form(form, monkeypatch)
    cs = inputs.random_case(210, 3, dims, potential="gauss16")
    occ = np.array([2.0, 0.5, 1.25])
    C, V, tol = cs["C"], cs["V"], TOL[prec]
    plan = ops.Plan(cs["dims"], prec=prec, hgrid=HG, occ=occ)
    assert plan.query(lib.WVL_Q_VARIANT) == (2 if form == "f64" else 1)
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
    assert plan.query(lib.WVL_Q_PRECOND_FORM) == 1
    for iters in (1, 3):
        x, res = plan.precondition(c, eps, iters, residuals=True)
        want = [PC.pcg(C[b], eps[b], iters, hgrid=HG) for b in range(3)]
        assert_close(plan.unpack(x), [w[0] for w in want], tol, f"preconditioner, {iters} steps")
        assert_close(res.cpu().numpy(), np.array([w[1] for w in want]), tol, "residuals")
    plan.local_hpsi(c, Vt, out=c)
    assert_close(plan.unpack(c), list(ref["hpsi"]), tol, "in place")


@pytest.mark.parametrize("form", FORMS)
def test_density_groups(form, monkeypatch):
    prec = _form(form, monkeypatch)
    norb, dims = 131, (66, 3, 8)
    cs = inputs.random_case(211, norb, dims, potential="gauss16")
    tol = TOL[prec]
    plan = ops.Plan(cs["dims"], prec=prec, hgrid=HG)
    assert plan.query(lib.WVL_Q_GROUP) == 2
    ref = W.local_hpsi(cs["C"], cs["V"], cs["occ"], hgrid=HG)
    r = plan.local_hpsi(plan.pack(cs["C"]), plan.pack_potential(cs["V"]), per_orbital=True)
    assert_close(r["rho"].cpu().numpy(), ref["rho"].ravel(), tol, "rho")
    assert_close(plan.unpack(r["hpsi"]), list(ref["hpsi"]), tol, "hpsi")
    assert_scalar(r["energies"][0].item(), ref["e_loc"], tol, "E_loc")
    eo = r["e_orb"].cpu().numpy()
    assert_close(eo[:norb], ref["e_loc_orb"], tol, "e_pot per orbital")
    assert_close(eo[norb:], ref["e_kin_orb"], tol, "e_kin per orbital")


@pytest.mark.parametrize("persistent", [False, True])
@pytest.mark.parametrize("form", FORMS)
def test_uneven_batch_with_a_long_plane(form, persistent, monkeypatch):
    """One plane too long for the other kernel: every orbital runs here."""
    prec = _form(form, monkeypatch)
    dims = [(4, 5, 3), (72, 10, 5), (20, 18, 6), (66, 7, 9), (16, 2, 4)]
    rng = inputs.rng_for(212)
    C = inputs.coefficients(rng, dims)
    V = [inputs.potential_gauss(rng, inputs.fine_shape(d)) for d in dims]
    plan = ops.Plan(dims, prec=prec, shared_v=False, persistent=persistent, hgrid=HG)
    ref = W.local_hpsi(C, V, plan.occ, shared_v=False, hgrid=HG)
    c = plan.pack(C)
    r = plan.local_hpsi(c, plan.pack_potential(V), per_orbital=True)
    eo = r["e_orb"].cpu().numpy()
    for b, got in enumerate(plan.unpack(r["hpsi"])):
        assert_close(got, ref["hpsi"][b], TOL[prec], f"orbital {b}")
    assert_close(eo[:len(dims)], ref["e_loc_orb"], TOL[prec], "e_pot per orbital")
    assert_close(eo[len(dims):], ref["e_kin_orb"], TOL[prec], "e_kin per orbital")
    eps = -rng.uniform(0.1, 1.0, len(dims))
    x = plan.unpack(plan.precondition(c, eps, 3))
    assert_close(x, [PC.pcg(C[b], eps[b], 3, HG)[0] for b in range(len(dims))], TOL[prec],
                 "preconditioner")
