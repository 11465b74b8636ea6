"""Power iteration with one application and normalisation a launch (mode 0 of the
term fusion, grids of 2^28 points, and vectors out of the pipeline's range):
caps on either side of a chunk's end (64 iterations, then 128), converged and
capped runs, against the oracle and the pipeline.  Tolerance: lambda is a ratio
of norms of vectors a few hundred roundings from the oracle's: 1e-12."""
import pytest

import workloads as W
from gpu_util import make_pair
from oracle import bounds
from oracle import operator as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap", [1, 2, 63, 64, 65, 193])
@pytest.mark.parametrize("nx,ny,bc,storage,field", [(48, 48, O.DIRICHLET, 0, False), (33, 45, O.PERIODIC, 0, True),
                                                    (226, 30, O.PERIODIC, 1, False)])
def test_power_iteration_one_application_a_launch(nx, ny, bc, storage, field, cap):
    import paper_2307_12276_amd as A
    Dxx, Dxy, Dyy, ax, ay = W.random_fields(nx, ny, seed=nx, field_advection=field)
    oop, gop = make_pair(Dxx, Dxy, Dyy, ax, ay, 1.0 / nx, 0.8 / ny, bc, storage)
    for rtol in (1e-13, 3e-3):
        lam, itso, _ = bounds.power_iteration(lambda x: O.apply(oop, x), oop.shape, 5, cap, rtol)
        for mode in (0, 1):
            gop.set_term_fusion(mode)
            a, its = gop.spectral_bound(A.BOUND_POWER, max_iter=cap, rtol=rtol, seed=5)
            assert its == itso
            assert gop.last_power_estimate() == pytest.approx(lam, rel=1e-12)
            assert a == pytest.approx(-min(bounds.SAFETY * lam, abs(bounds.gershgorin(oop))), rel=1e-12)
