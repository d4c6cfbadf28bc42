"""The last z step as one launch and as two (WVL_NO_ZFUSE, or in place).  In
float64 and float32 the results are equal bit for bit.  For float pairs the two
launches round K_z c + kxy to a pair in between, the fused one keeps it in
float64: equal to the tolerance of the compensated form; density and potential
energies, which come before that step, are equal bit for bit, and so are two
fused runs."""

import pytest
import torch

from oracle import wavelet as W
from paper_0904_1543_amd import inputs, lib, ops
from parity_helpers import TOL, assert_close, assert_scalar

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(16, 16, 16), (8, 24, 40), (48, 48, 8)])
def test_fused_and_two_pass_form(dims, monkeypatch):
    tol = TOL["f32c"]
    cs = inputs.random_case(220, 3, dims, potential="gauss16")
    fused = ops.Plan(cs["dims"], prec="f32c")
    monkeypatch.setenv("WVL_NO_ZFUSE", "1")
    two = ops.Plan(cs["dims"], prec="f32c")
    for plan, f in ((fused, 1), (two, 0)):
        assert plan.query(lib.WVL_Q_VARIANT) == 3 and plan.query(lib.WVL_Q_FUSED_Z) == f
    c, V = fused.pack(cs["C"]), fused.pack_potential(cs["V"])
    a, b = fused.local_hpsi(c, V, per_orbital=True), two.local_hpsi(c, V, per_orbital=True)
    again = fused.local_hpsi(c, V, per_orbital=True)
    for k in ("hpsi", "rho", "energies", "e_orb"):
        assert torch.equal(a[k], again[k]), k
    assert torch.equal(a["rho"], b["rho"]) and torch.equal(a["e_orb"][:3], b["e_orb"][:3])
    ref = W.local_hpsi(cs["C"], cs["V"], cs["occ"])
    inplace = c.clone()
    fused.local_hpsi(inplace, V, out=inplace)
    for what, h in (("fused", a["hpsi"]), ("two passes", b["hpsi"]), ("in place", inplace)):
        assert_close(fused.unpack(h), list(ref["hpsi"]), tol, what)
    assert torch.equal(inplace, b["hpsi"])      # in place: the two passes
    for r in (a, b):
        assert_scalar(r["energies"][1].item(), ref["e_kin"], tol, "E_kin")


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n3", [20, 32, 60, 73])
def test_bitwise_equal_in_both_kinds_of_z_pass(prec, n3, monkeypatch):
    """float64 and float32 keep the association of the two passes, with whole
    lines in LDS and strided."""
    cs = inputs.random_case(221, 3, (9, 7, n3), potential="gauss16")
    fused = ops.Plan(cs["dims"], prec=prec)
    monkeypatch.setenv("WVL_NO_ZFUSE", "1")
    two = ops.Plan(cs["dims"], prec=prec)
    assert fused.query(lib.WVL_Q_FUSED_Z) == 1 and two.query(lib.WVL_Q_FUSED_Z) == 0
    c, V = fused.pack(cs["C"]), fused.pack_potential(cs["V"])
    a = fused.local_hpsi(c, V, pot_scale=0.7, kin_scale=1.3, per_orbital=True)
    b = two.local_hpsi(c, V, pot_scale=0.7, kin_scale=1.3, per_orbital=True)
    for k in ("hpsi", "rho", "energies", "e_orb"):
        assert torch.equal(a[k], b[k]), k
    fused.local_hpsi(c, V, pot_scale=0.7, kin_scale=1.3, out=c)
    assert torch.equal(c, b["hpsi"])
