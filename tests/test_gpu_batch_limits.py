"""Batched eager steps whose bins' degree caps change between steps, with u, S,
dt and tol unchanged: the same degrees and u as by the bins alone.

Tolerance: both are the same Newton sums of at most 60 terms, in another order
of rounding: 1e-13 of the largest partial sum, which is no more than the
result's size where u is smooth, and 185 times it in the first step from a
random u (52 x 42 points)."""
import numpy as np
import pytest

import paper_2307_12276_amd as A

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
            op.oracle = oop
            dst.append(op)
        scale.append(abs(bounds.gershgorin(oop)))
        us.append(to_dev(W.gaussian(X, Y, 0.4, 0.45, 0.1)))
        vs.append(us[-1].clone())
        Ss.append(to_dev(W.gaussian(X, Y, 0.6, 0.5, 0.1)) if i % 2 else None)
    return ops, alone, us, vs, Ss, 150.0 / max(scale)


def step_peak(op, dt, u, S, m=60):
    """Norm of the largest partial sum of dt phi_1(dt A)(A u + S)."""
    alpha = bounds.gershgorin(op.oracle)
    xi, d = A.leja_points(m + 1), A.newton_coefficients(1, alpha, dt, m + 1)
    y = O.apply(op.oracle, u) + S
    p, peak = d[0] * y, 0.0
    for k in range(m):
        y = (O.apply(op.oracle, y) - (alpha / 2.0 - alpha / 4.0 * xi[k]) * y) / (-alpha / 4.0)
        p += d[k + 1] * y
        peak = max(peak, float(np.linalg.norm(p)))
    return dt * peak


def steps_agree(batch, alone, us, vs, Ss, dt, n=2, rough=None):
    """rough: the bin whose u is random."""
    for _ in range(n):
        got = batch.midpoint_step(us, Ss, dt, 1e-10)
        for i, (u, v, S, op, st) in enumerate(zip(us, vs, Ss, alone, got)):
            peak = step_peak(op, dt, to_np(v), 0.0 if S is None else to_np(S)) if i == rough else 0.0
            want = op.midpoint_step(v, S, dt, 1e-10)
            assert (st["matvecs"], st["substeps"]) == (want["matvecs"], want["substeps"])
            a, b = to_np(u), to_np(v)
            assert np.linalg.norm(a - b) <= 1e-13 * max(np.linalg.norm(b), peak)
            v.copy_(u)


@pytest.mark.parametrize("use_graph", [False, True])
def test_cap_raised_between_steps(use_graph):
    """A cap of 20 terms, too few (those bins take substeps), then 500: the
    coefficients past the 20th must reach the device with the new cap.  With
    a graph step before either."""
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


def test_cap_lowered_between_steps():
    """One bin of twenty ends at a cap of 20 from the first step on, another
    one's cap falls to 20 after steps of some 55 terms, and its u is replaced by
    one that takes more; too few of the bins change for that alone to plan the
    launches again.  Both bins take substeps then.  At a cap of 6 no substeps
    suffice: the batch refuses as the bin alone does, the others have advanced."""
    shapes = [(16 + 2 * i, 60 - i) for i in range(20)]
    ops, alone, us, vs, Ss, dt = bins(shapes)
    for op in (ops[19], alone[19]):
        op.set_limits(20, 1600.0)
    batch = A.Batch(ops)
    steps_agree(batch, alone, us, vs, Ss, dt)
    for cap in (20, 6, 500):
        for op in (ops[18], alone[18]):
            op.set_limits(cap, 1600.0)
        us[18].copy_(to_dev(W.random_vector(us[18].shape, 7)))
        vs[18].copy_(us[18])
        if cap > 6:
            steps_agree(batch, alone, us, vs, Ss, dt, rough=18)
            continue
        with pytest.raises(A.AdlError) as e:
            batch.midpoint_step(us, Ss, dt, 1e-10)
        assert e.value.code == A.ENOCONV
        for i, (u, v, S, op) in enumerate(zip(us, vs, Ss, alone)):
            if i == 18:
                with pytest.raises(A.AdlError) as e:
                    op.midpoint_step(v, S, dt, 1e-10)
                assert e.value.code == A.ENOCONV
            else:
                op.midpoint_step(v, S, dt, 1e-10)
            assert rel(to_np(u), to_np(v)) <= 1e-13


def test_tile_rows_set_right_after_steps_on_a_side_stream():
    """Steps on a stream of the caller's, each with another dt (so that its
    sweeps stop away from the expected degrees and are replayed), and the tile
    tables written anew as soon as a step returns: a step has read them all by
    then."""
    import torch
    ops, alone, us, vs, Ss, dt = bins([(512, 500), (256, 300), (384, 260), (128, 700)])
    batch = A.Batch(ops, tile_rows=3)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for i, rows in enumerate((64, 1, 33, 2, 100, 5)):
            got = batch.midpoint_step(us, Ss, dt * 0.8 ** i, 1e-10)
            batch.set_tile_rows(rows)
            for u, v, S, op, st in zip(us, vs, Ss, alone, got):
                want = op.midpoint_step(v, S, dt * 0.8 ** i, 1e-10)
                assert st["matvecs"] == want["matvecs"]
                assert rel(to_np(u), to_np(v)) <= 1e-13
                v.copy_(u)


@pytest.mark.parametrize("shapes", [[(128, 64), (256, 40)], [(113, 33), (64, 50)]])
def test_mode_set_and_reset(shapes):
    """Modes of the term fusion between steps of one batch, eager and as a graph,
    and back to the default: bitwise the pipeline's steps then."""
    ops, alone, us, vs, Ss, dt = bins(shapes)
    batch, plain = A.Batch(ops), A.Batch(alone)
    for mode in (None, False, None, 3 if shapes[0][0] == 128 else True, None):
        if mode is None:
            batch.reset_term_fusion()
        else:
            batch.set_term_fusion(mode)
        for use_graph in (False, True, False):
            batch.midpoint_step(us, Ss, dt, 1e-10, use_graph=use_graph)
            plain.midpoint_step(vs, Ss, dt, 1e-10)
            for u, v in zip(us, vs):
                a, b = to_np(u), to_np(v)
                if mode is None and not use_graph:
                    assert np.array_equal(a, b)
                assert rel(a, b) <= 1e-12
                u.copy_(v)
