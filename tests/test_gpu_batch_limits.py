"""Batched eager steps whose bins' degree caps change between steps, with u, S,
dt and tol unchanged: the same degrees and u as by the bins alone.

Tolerance: both are the same Newton sums but for the grouping of the norms: u
to 1e-13 of itself (a step of at most 60 terms)."""
import numpy as np
import pytest

import workloads as W
from gpu_util import make_pair, rel, to_dev, to_np
from oracle import bounds
from oracle import operator as O

pytestmark = pytest.mark.gpu


def bins(shapes, bc=O.DIRICHLET, storage=1):
    """(ops of a batch, the same ops alone, u of each, sources, a dt of rho dt =
    150 in the stiffest bin)."""
    ops, alone, us, vs, Ss, scale = [], [], [], [], [], []
    for i, (nx, ny) in enumerate(shapes):
        X, Y, hx, hy = W.grid_2d(nx, ny, bc)
        D = W.tensor_from_direction(*W.circular_direction(X, Y), 1.0, 0.01)
        for dst in (ops, alone):
            oop, op = make_pair(*D, 0.2, 0.1, hx, hy, bc, storage)
            op.set_bound(bounds.gershgorin(oop))
            dst.append(op)
        scale.append(abs(bounds.gershgorin(oop)))
        us.append(to_dev(W.gaussian(X, Y, 0.4, 0.45, 0.1)))
        vs.append(us[-1].clone())
        Ss.append(to_dev(W.gaussian(X, Y, 0.6, 0.5, 0.1)) if i % 2 else None)
    return ops, alone, us, vs, Ss, 150.0 / max(scale)


def steps_agree(batch, alone, us, vs, Ss, dt, n=2):
    for _ in range(n):
        got = batch.midpoint_step(us, Ss, dt, 1e-10)
        for u, v, S, op, st in zip(us, vs, Ss, alone, got):
            want = op.midpoint_step(v, S, dt, 1e-10)
            assert (st["matvecs"], st["substeps"]) == (want["matvecs"], want["substeps"])
            assert rel(to_np(u), to_np(v)) <= 1e-13
            v.copy_(u)


@pytest.mark.parametrize("use_graph", [False, True])
def test_cap_raised_between_steps(use_graph):
    """A cap of 20 terms, too few (those bins take substeps), then 500: the
    coefficients past the 20th must reach the device with the new cap.  With
    a graph step before either."""
    import paper_2307_12276_amd as A
    ops, alone, us, vs, Ss, dt = bins([(128, 64), (112, 40), (64, 64)])
    batch = A.Batch(ops)
    for cap in (20, 500):
        for op in ops + alone:
            op.set_limits(cap, 1600.0)
        if use_graph:
            batch.midpoint_step(us, Ss, dt, 1e-10, use_graph=True)
            for u, v, S, op in zip(us, vs, Ss, alone):
                op.midpoint_step(v, S, dt, 1e-10)
                assert rel(to_np(u), to_np(v)) <= 1e-12
                v.copy_(u)
        steps_agree(batch, alone, us, vs, Ss, dt)
