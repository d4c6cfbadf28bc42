"""z passes of batches of several line lengths, which hold whole lines in LDS at
every length that has a shape (uniform batches of float64 and float32 take the
strided passes at some of them): the edges of the shapes, against the float64
oracle with the tolerances of the parity tests."""

import numpy as np
import pytest

from oracle import precond as PR
from oracle import wavelet as W
from paper_0904_1543_amd import inputs, ops
from parity_helpers import TOL, assert_close, assert_scalar

pytestmark = pytest.mark.gpu

HG = (0.8, 1.0, 0.9)


@pytest.mark.parametrize("n3", [3, 16, 17, 32, 33, 40, 41, 48, 49, 60, 61, 72, 73])
@pytest.mark.parametrize("prec", ["f64", "f32", "f32c"])
def test_two_lengths(prec, n3):
    dims, tol = [(3, 7, n3), (5, 4, 2), (3, 7, n3)], TOL[prec]
    rng = inputs.rng_for(99)
    C = inputs.coefficients(rng, dims)
    V = [inputs.potential_gauss(rng, inputs.fine_shape(d)) for d in dims]
    eps = -np.linspace(0.2, 1.0, 3)
    plan = ops.Plan(dims, prec=prec, hgrid=HG, shared_v=False)
    c = plan.pack(C)
    r = plan.local_hpsi(c, plan.pack_potential(V), per_orbital=True)
    got, eo = plan.unpack(r["hpsi"]), r["e_orb"].cpu().numpy()
    ref = W.local_hpsi(C, V, np.ones(3), hgrid=HG, shared_v=False)
    x = plan.unpack(plan.precondition(c, eps, 3))
    for b in range(3):
        assert_close(got[b], ref["hpsi"][b], tol, f"hpsi {b}")
        assert_scalar(eo[3 + b], ref["e_kin_orb"][b], tol, f"e_kin {b}")
        assert_close(x[b], PR.pcg(C[b], eps[b], 3, hgrid=HG)[0], tol, f"preconditioner {b}")
