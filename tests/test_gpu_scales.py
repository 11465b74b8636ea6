"""Sweeps and power iterations whose vectors leave the range in which squares
of FP64 numbers are finite and nonzero: the codes, counts and values of one-term
launches and of the oracle."""
import numpy as np
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


HOT = {"hot-spot": (1e-10, 3.0), "nilpotent": (0.0, 3.0)}


@pytest.mark.parametrize("name", sorted(HOT))
def test_power_iteration_on_a_hot_spot(name):
    """Advection at one node, 1e10 times the diffusion (or without any): the
    Gershgorin bound is 1e5 times the norms' growth, so vectors scaled by it
    vanish; the iteration itself converges, or finds lambda = 0."""
    nx, ny = 48, 40
    eps, hot = HOT[name]
    one, ax, ay = np.ones((ny, nx)), np.full((ny, nx), eps), np.full((ny, nx), eps)
    ax[20, 20], ay[20, 20] = hot, -2.0
    oop, gop = make_pair(eps * one, 0.0 * one, eps * one, ax, ay, 1.0 / nx, 1.0 / ny, O.PERIODIC, 0)
    lam, its, _ = bounds.power_iteration(lambda x: O.apply(oop, x), oop.shape, 5, 2000, 1e-3)
    if lam == 0.0:
        with pytest.raises(A.AdlError) as e:
            gop.spectral_bound(A.BOUND_POWER, max_iter=2000, rtol=1e-3, seed=5)
        assert e.value.code == A.EBOUND
        return
    # (a few thousand ratios of norms of vectors with two separate scales; the
    # stopping test's outcome flips within rounding of rtol: lambda to rtol)
    gop.spectral_bound(A.BOUND_POWER, max_iter=2000, rtol=1e-3, seed=5)
    assert gop.last_power_estimate() == pytest.approx(lam, rel=2e-3)


@pytest.mark.parametrize("scale", [1e-170, 1e-100, 1e100, 1e160])
def test_power_iteration_at_extreme_scales(scale):
    """Coefficients whose squared norms underflow or overflow are refused as
    ever, others give the scaled estimate."""
    nx, ny = 48, 40
    Dxx, Dxy, Dyy, ax, ay = W.random_fields(nx, ny, seed=nx, field_advection=False)
    s = scale
    oop, gop = make_pair(Dxx * s, Dxy * s, Dyy * s, ax * s, ay * s, 1.0 / nx, 0.8 / ny, O.PERIODIC, 0)
    if not 1e-150 < scale < 1e150:
        with pytest.raises(A.AdlError) as e:
            gop.spectral_bound(A.BOUND_POWER, max_iter=2000, rtol=1e-3, seed=5)
        assert e.value.code == (A.EBOUND if scale < 1.0 else A.ENAN)
        return
    lam, its, _ = bounds.power_iteration(lambda x: O.apply(oop, x), oop.shape, 5, 2000, 1e-3)
    _, k = gop.spectral_bound(A.BOUND_POWER, max_iter=2000, rtol=1e-3, seed=5)
    assert k == its and gop.last_power_estimate() == pytest.approx(lam, rel=1e-12)
