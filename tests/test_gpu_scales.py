"""Sweeps whose vectors leave the range in which squares of FP64 numbers are
finite: the codes, substeps and values of one-term launches."""
import pytest

import paper_2307_12276_amd as A
import workloads as W
from gpu_util import make_pair, rel, to_dev, to_np
from oracle import bounds
from oracle import operator as O

pytestmark = pytest.mark.gpu


# (tiles in registers; the pipeline)
@pytest.mark.parametrize("nx,ny,frac", [(48, 32, 0.76), (520, 260, 0.84)])
def test_interval_too_small_takes_substeps(nx, ny, frac):
    """A set interval that leaves out part of the spectrum: y grows past 1e155
    within the cap of 500 terms while d y stays finite in the norms, so the sweep
    ends at the cap and the step is taken in substeps; it does not overflow.
    Each result meets tol = 1e-10, so two of them agree to 1e-9."""
    Dxx, Dxy, Dyy, ax, ay = W.random_fields(nx, ny, seed=nx, field_advection=False)
    oop, gop = make_pair(Dxx, Dxy, Dyy, ax, ay, 1.0 / nx, 0.8 / ny, O.DIRICHLET, 0)
    alpha = bounds.gershgorin(oop)
    gop.set_bound(frac * alpha)
    v = to_dev(W.random_vector((ny, nx), 13))
    dt = 100.0 / abs(alpha)
    got = {}
    for mode in (0, 1):
        gop.set_term_fusion(mode)
        for step in ("phi", "midpoint"):
            u = v.clone()
            st = gop.leja_phi(1, dt, v, u, 1e-10) if step == "phi" else gop.midpoint_step(u, None, dt, 1e-10)
            got[mode, step] = to_np(u), st["substeps"]
    u = v.clone()
    st = A.Batch([gop]).midpoint_step([u], None, dt, 1e-10)
    got["batch", "midpoint"] = to_np(u), st[0]["substeps"]
    for (mode, step), (x, substeps) in got.items():
        want, K = got[0, step]
        assert K > 1 and substeps == K
        assert rel(x, want) <= 1e-9
