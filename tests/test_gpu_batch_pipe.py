"""Batched bins on the pipeline kernel (the default of eager steps) against the
same steps of each bin alone: the first step of a batch (guessed degrees, so
replays and added launches), steps after it (planned), a larger and a smaller
step size, bins without a source beside bins with one, a bin at rest, sizes at
the edges of strips (112 columns) and runs (16 rows and multiples).  Graph
steps keep the tile kernels: both on one batch.

Tolerance: both are the same Newton sums but for the grouping of the norms, so
the same degrees, and u to 1e-13 of itself (a step of at most 60 terms)."""
import numpy as np
import pytest

import workloads as W
from gpu_util import make_pair, rel, to_dev, to_np
from oracle import bounds
from oracle import operator as O

pytestmark = pytest.mark.gpu

CASES = {
    "even-fp32": ([(128, 64), (112, 16), (114, 17), (256, 200), (64, 300), (224, 48)], 1, False),
    "odd-fp64": ([(113, 65), (97, 15), (33, 20), (225, 130), (16, 12)], 0, False),
    "even-field": ([(128, 45), (130, 70), (256, 33), (16, 16)], 0, True),
    "one-bin": ([(112, 33)], 0, False),
}


@pytest.mark.parametrize("bc", [O.PERIODIC, O.DIRICHLET])
@pytest.mark.parametrize("name", sorted(CASES))
def test_batched_steps_equal_single_steps(name, bc):
    import torch
    import paper_2307_12276_amd as A
    shapes, storage, field = CASES[name]
    ops, alone, us, vs, Ss, scale = [], [], [], [], [], []
    for i, (nx, ny) in enumerate(shapes):
        X, Y, hx, hy = W.grid_2d(nx, ny, bc)
        Dxx, Dxy, Dyy = W.tensor_from_direction(*W.circular_direction(X, Y), 0.1 * 2.0 ** i, 0.01)
        ax, ay = (0.3 * np.cos(6.0 * Y), 0.2 * np.sin(6.0 * X)) if field else (0.2, 0.1)
        for dst in (ops, alone):
            oop, op = make_pair(Dxx, Dxy, Dyy, ax, ay, hx, hy, bc, storage)
            op.set_bound(bounds.gershgorin(oop))
            dst.append(op)
        scale.append(abs(bounds.gershgorin(oop)))
        u = 0.0 * X if i == 2 else W.gaussian(X, Y, 0.4, 0.45, 0.1)
        us.append(to_dev(u))
        vs.append(to_dev(u))
        Ss.append(to_dev(W.gaussian(X, Y, 0.6, 0.5, 0.1)) if i % 2 == 0 and i != 2 else None)
    batch = A.Batch(ops)
    big = 150.0 / max(scale)
    for dt in (big, big, big, 4.0 * big, 0.1 * big, 0.1 * big):
        got = batch.midpoint_step(us, Ss, dt, 1e-10)
        for u, v, S, op, st in zip(us, vs, Ss, alone, got):
            want = op.midpoint_step(v, S, dt, 1e-10)
            assert st["matvecs"] == want["matvecs"] and st["fallback"] == 0
            a, b = to_np(u), to_np(v)
            assert np.isfinite(a).all() and (rel(a, b) <= 1e-13 if np.any(b) else not np.any(a))
            v.copy_(u)


def test_graph_and_eager_steps_of_one_batch():
    """Graph steps (tiles) before, between and after eager ones (pipeline) of
    the same batch, and the autotuner before both: u as by the bins alone."""
    import torch
    import paper_2307_12276_amd as A
    ops, alone, us, vs, Ss = [], [], [], [], []
    for i, (nx, ny) in enumerate([(128, 64), (256, 100), (192, 40)]):
        X, Y, hx, hy = W.grid_2d(nx, ny, O.DIRICHLET)
        D = W.tensor_from_direction(*W.circular_direction(X, Y), 1.0, 0.01)
        for dst in (ops, alone):
            oop, op = make_pair(*D, 0.2, 0.1, hx, hy, O.DIRICHLET, 1)
            op.set_bound(bounds.gershgorin(oop))
            dst.append(op)
        us.append(to_dev(W.gaussian(X, Y, 0.4, 0.45, 0.1)))
        vs.append(us[-1].clone())
        Ss.append(to_dev(W.gaussian(X, Y, 0.6, 0.5, 0.1)) if i != 1 else None)
    dt = 150.0 / abs(bounds.gershgorin(oop)) * 0.1
    batch = A.Batch(ops)
    batch.autotune(us, Ss, dt, 1e-10, candidates=(8, 16))
    for use_graph in (True, False, True, False, False):
        batch.midpoint_step(us, Ss, dt, 1e-10, use_graph=use_graph)
        for u, v, S, op in zip(us, vs, Ss, alone):
            op.midpoint_step(v, S, dt, 1e-10)
            # (a graph step rebuilds p at the stop from the last y: 1e-12)
            assert rel(to_np(u), to_np(v)) <= 1e-12
            v.copy_(u)
