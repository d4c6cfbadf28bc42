"""The z passes where their launches change form, against the float64 oracle
with the tolerances of the parity tests: lines cut into segments (one orbital;
segments that do not divide the line; whole lines for many orbitals), the
preconditioner's direction update inside the z pass over the same batches, and
float64 batch arrays larger than the last cache, whose results bypass it."""

import numpy as np
import pytest

from oracle import precond as PR
from oracle import wavelet as W
from paper_0904_1543_amd import inputs, ops
from parity_helpers import TOL, assert_close, assert_scalar

pytestmark = pytest.mark.gpu

HG = (0.8, 1.0, 0.9)


def _check(prec, norb, dims, some, iters, seed):
    cs, tol = inputs.random_case(seed, norb, dims), TOL[prec]
    C, V = cs["C"], cs["V"]
    eps = -np.linspace(0.2, 1.0, norb)
    plan = ops.Plan(cs["dims"], prec=prec, hgrid=HG)
    c, Vt = plan.pack(C), plan.pack_potential(V)
    r = plan.local_hpsi(c, Vt, per_orbital=True)
    got, eo = plan.unpack(r["hpsi"]), r["e_orb"].cpu().numpy()
    ref = W.local_hpsi(C[some], V, np.ones(len(some)), hgrid=HG)
    x = plan.unpack(plan.precondition(c, eps, iters))
    for k, b in enumerate(some):
        assert_close(got[b], ref["hpsi"][k], tol, f"hpsi {b}")
        assert_scalar(eo[norb + b], ref["e_kin_orb"][k], tol, f"e_kin {b}")
        assert_close(x[b], PR.pcg(C[b], eps[b], iters, hgrid=HG)[0], tol, f"preconditioner {b}")


# planes of four blocks of lines, 18 values along z: segments of 4 (one orbital;
# 24: the last holds 2), 6 (60) and whole lines (130)
@pytest.mark.parametrize("norb", [1, 24, 60, 130])
@pytest.mark.parametrize("prec", ["f64", "f32", "f32c"])
def test_segments_of_lines(prec, norb):
    _check(prec, norb, (16, 16, 9), sorted({0, norb // 2, norb - 1}), 3, 97)


def test_batch_larger_than_the_last_cache():
    """320 orbitals of 0.86 MB each."""
    _check("f64", 320, (24, 20, 28), [0, 160, 319], 3, 98)
