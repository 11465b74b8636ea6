"""The pipeline kernel (the default mode: seven Newton terms per launch, the
stage vector in the first launch) against one-term launches of the same sweep,
at the edges of its strips (112 own columns, two columns per lane) and runs of
rows, and of the tiles that small grids take (50 x 10 own points), and against one-term launches' degrees.

Tolerance: both orders of summation stay within a few 1e-15 of the exact
Newton sum per term taken, so 4e-15 per term (at least 1e-13); Newton vectors
stored as floats round at 6e-8 per term with cancelling signs: 1e-5.  Each is
relative to the largest partial sum: a phi evaluation's is its result's size, a
midpoint step's passes through A u, whose sums are hundreds of times the step's
result on random fields (16 x 12, Dirichlet: 5100 times, where one-term
launches are 1.1e-11 from the 80-bit sum and the pipeline 7.3e-12)."""
import numpy as np
import pytest

import paper_2307_12276_amd as A
import workloads as W
from gpu_util import make_pair, to_dev, to_np
from oracle import bounds
from oracle import operator as O

pytestmark = pytest.mark.gpu

SHAPES = [
    (16, 12),      # a fraction of one tile (50 x 10 points)
    (50, 10),      # one whole tile
    (51, 11),      # ... and one column and one row more
    (250, 510),    # 255 tiles, the most
    (250, 511),    # one row more: the pipeline
    (33, 45),      # odd width: columns loaded one by one
    (112, 3),      # one whole strip, three rows
    (113, 40),     # ... and one column more
    (224, 50),     # two whole strips
    (250, 7),      # fewer rows than a launch's stages on either side
    (1001, 300),   # nine strips, the last one with 105 columns
    (40, 10300),   # more rows than 255 blocks take one by one: two blocks per CU
]


def step_peak(oop, alpha, dt, m, v, S):
    """Norm of the largest partial sum of dt phi_1(dt A)(A v + S)."""
    xi, d = A.leja_points(m + 1), A.newton_coefficients(1, alpha, dt, m + 1)
    y = O.apply(oop, v) + S
    p, peak = d[0] * y, 0.0
    for k in range(m):
        y = (O.apply(oop, y) - (alpha / 2.0 - alpha / 4.0 * xi[k]) * y) / (-alpha / 4.0)
        p += d[k + 1] * y
        peak = max(peak, float(np.linalg.norm(p)))
    return dt * peak


@pytest.mark.parametrize("bc", [O.PERIODIC, O.DIRICHLET])
@pytest.mark.parametrize("storage,field", [(0, False), (0, True), (1, False), (2, True)])
@pytest.mark.parametrize("nx,ny", SHAPES)
def test_pipeline_matches_one_term_launches(nx, ny, storage, field, bc):
    import torch
    Dxx, Dxy, Dyy, ax, ay = W.random_fields(nx, ny, seed=nx + ny, field_advection=field)
    oop, gop = make_pair(Dxx, Dxy, Dyy, ax, ay, 1.0 / nx, 0.8 / ny, bc, storage)
    alpha = bounds.gershgorin(oop)
    gop.set_bound(alpha)
    # an unaligned v (its base 8 bytes past a 16-byte boundary) beside aligned vectors
    flat = torch.zeros(nx * ny + 1, dtype=torch.float64, device="cuda")
    odd = flat[1:].view(ny, nx)
    v0, S0 = W.random_vector((ny, nx), 13), W.random_vector((ny, nx), 3)
    v, S = to_dev(v0), to_dev(S0)
    odd.copy_(v)
    dt = 300.0 / abs(alpha)
    got = {}
    for mode in (0, 1):
        gop.set_term_fusion(mode)
        out = []
        for mult in (3.0, 40.0, 300.0):
            # twice: a plan's first sweep guesses its degree and stops inside a
            # launch by replay, the second one has stored p there
            for vec in (v, v, odd):
                o = torch.full_like(v, float("nan"))
                st = gop.leja_phi(1, mult / abs(alpha), vec, o, 1e-10)
                out.append((to_np(o), st["max_degree"], 0.0))
        peak = step_peak(oop, alpha, dt, out[-1][1], v0, S0)
        for step in (lambda u: gop.midpoint_step(u, S, dt, 1e-10), lambda u: gop.midpoint_step(u, None, dt, 1e-10),
                     lambda u: gop.quad2_step(u, S, 2 * S, 1 / 3, 2 / 3, dt, 1e-10)):
            u = v.clone()
            st = step(u)
            out.append((to_np(u), st["matvecs"], peak))
        got[mode] = out
    for (a, da, _), (b, db, peak) in zip(got[1], got[0]):
        assert da == db
        tol = 1e-5 if storage == 2 else max(1e-13, 4e-15 * db)
        assert np.isfinite(a).all()
        assert np.linalg.norm(a - b) <= tol * max(np.linalg.norm(b), peak)


@pytest.mark.parametrize("bc", [O.PERIODIC, O.DIRICHLET])
def test_two_sweeps_with_substeps_keep_the_first_result(bc):
    """Two-sweep quadrature steps in several substeps: the second evaluation's
    sweeps must leave the vector that holds the first one's result alone."""
    nx, ny = 64, 48
    Dxx, Dxy, Dyy, ax, ay = W.random_fields(nx, ny, seed=3, field_advection=False)
    oop, gop = make_pair(Dxx, Dxy, Dyy, ax, ay, 1.0 / nx, 0.8 / ny, bc, 0)
    alpha = bounds.gershgorin(oop)
    gop.set_bound(alpha)
    gop.set_limits(500, 20.0)
    gop.set_quad2_mode(A.QUAD2_TWO_SWEEP)
    u0, S0 = W.random_vector((ny, nx), 13), W.random_vector((ny, nx), 3)
    S = to_dev(S0)
    dt = 70.0 / abs(alpha)
    got = {}
    for mode in (0, 1):
        gop.set_term_fusion(mode)
        u, mv = to_dev(u0), []
        for _ in range(3):
            mv.append(gop.quad2_step(u, S, 3 * S, 1 / 3, 2 / 3, dt, 1e-10)["matvecs"])
        got[mode] = to_np(u), mv
    # (three steps of two evaluations whose partial sums are up to 20 / 2 times
    # their results, rho h = 20: 4e-15 per term of each)
    a, b = got[1][0], got[0][0]
    assert got[0][1] == got[1][1]
    assert np.linalg.norm(a - b) <= 10 * 4e-15 * sum(got[0][1]) * np.linalg.norm(b)
