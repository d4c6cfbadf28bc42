"""The z passes where their launches change form, against the float64 oracle
with the tolerances of the parity tests (local H*psi, kinetic energies and the
preconditioner): the edges of the shapes that hold whole lines in LDS, batches
of mixed shapes, the strided passes of longer lines with the lines whole or cut
into segments, and float64 batch arrays larger than the last cache, whose
results bypass it."""

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


# lines of 4 .. 144 values in LDS; longer ones strided
@pytest.mark.parametrize("n3", [2, 3, 16, 17, 32, 33, 40, 41, 48, 49, 60, 61, 72, 73])
@pytest.mark.parametrize("prec", ["f64", "f32", "f32c"])
def test_line_lengths(prec, n3):
    _check(prec, 3, (3, 7, n3), [0, 2], 3, 96)


# 73: strided; one block of 256 lines an orbital, 146 values a line: segments of
# 4 (one orbital), 8 (24), 18 (60: each time the last holds 2) and whole lines
# (520); 9: four tiles of 64 lines in LDS
@pytest.mark.parametrize("norb,dims", [(1, (8, 8, 73)), (24, (8, 8, 73)), (60, (8, 8, 73)),
                                       (520, (8, 8, 73)), (1, (16, 16, 9)), (130, (16, 16, 9))])
@pytest.mark.parametrize("prec", ["f64", "f32", "f32c"])
def test_segments_of_lines(prec, norb, dims):
    _check(prec, norb, dims, sorted({0, norb // 2, norb - 1}), 3, 97)


# 100 planes of 2304..4096 values: one launch per shape; 9 of them: one launch
@pytest.mark.parametrize("norb", [9, 100])
@pytest.mark.parametrize("prec", ["f64", "f32c"])
def test_mixed_line_lengths(prec, norb):
    n3 = [60, 16, 33, 41, 48, 2, 17, 72, 32]
    dims = [(24 + 4 * (b % 3), 32 - b % 2, n3[b % 9]) for b in range(norb)]
    rng = inputs.rng_for(94)
    C = inputs.coefficients(rng, dims)
    V = [inputs.potential_gauss(rng, inputs.fine_shape(d)) for d in dims]
    some = list(range(9))
    plan = ops.Plan(dims, prec=prec, hgrid=HG, shared_v=False)
    c, Vt = plan.pack(C), plan.pack_potential(V)
    r = plan.local_hpsi(c, Vt, per_orbital=True)
    got, eo = plan.unpack(r["hpsi"]), r["e_orb"].cpu().numpy()
    ref = W.local_hpsi([C[b] for b in some], [V[b] for b in some], np.ones(9), hgrid=HG, shared_v=False)
    eps = -np.linspace(0.2, 1.0, norb)
    x = plan.unpack(plan.precondition(c, eps, 3))
    for b in some:
        assert_close(got[b], ref["hpsi"][b], TOL[prec], f"hpsi {b}")
        assert_scalar(eo[norb + b], ref["e_kin_orb"][b], TOL[prec], f"e_kin {b}")
        assert_close(x[b], PR.pcg(C[b], eps[b], 3, hgrid=HG)[0], TOL[prec], f"preconditioner {b}")


def test_batch_larger_than_the_last_cache():
    """320 orbitals of 0.86 MB each."""
    _check("f64", 320, (24, 20, 28), [0, 160, 319], 3, 98)
