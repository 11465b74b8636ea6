"""Calls on a stream of the caller's, whose inputs an unfinished launch of that
stream is still writing and whose results its next launch reads, without a
synchronisation: bitwise what the default stream gives.  Sizes on either side
of the rule between tiles and the pipeline."""
import pytest

import paper_2307_12276_amd as A
import workloads as W
from gpu_util import make_pair, to_dev
from oracle import bounds
from oracle import operator as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,storage", [(64, 48, 0), (520, 260, 1), (520, 260, 2)])
def test_calls_on_a_side_stream(nx, ny, storage):
    import torch
    Dxx, Dxy, Dyy, ax, ay = W.random_fields(nx, ny, seed=nx, field_advection=False)
    oop, gop = make_pair(Dxx, Dxy, Dyy, ax, ay, 1.0 / nx, 0.8 / ny, O.DIRICHLET, storage)
    alpha = bounds.gershgorin(oop)
    dt = 200.0 / abs(alpha)
    v, S = to_dev(W.random_vector((ny, nx), 13)), to_dev(W.random_vector((ny, nx), 3))
    busy = torch.rand(4096, 4096, device="cuda")
    batch = A.Batch([gop]) if storage < 2 else None

    def calls(delay):
        out = []
        gop.set_bound(alpha)
        for step in (lambda u: gop.midpoint_step(u, S, dt, 1e-10), lambda u: gop.quad2_step(u, S, 2 * S, .25, .75, dt, 1e-10),
                     lambda u: gop.leja_phi(0, dt, v, u, 1e-10),
                     lambda u: batch and batch.midpoint_step([u], [S], dt, 1e-10)):
            for _ in range(3):
                u = torch.empty_like(v)
                w = busy
                for _ in range(8 * delay):
                    w = torch.relu(w @ busy)
                u.copy_(v)
                step(u)
                out.append(u * 2.0)
        out.append(gop.spectral_bound(A.BOUND_POWER, max_iter=200, rtol=1e-6, seed=3))
        return out

    want = calls(0)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        got = calls(1)
    side.synchronize()
    for a, b in zip(got[:-1], want[:-1]):
        assert torch.equal(a, b)
    assert got[-1] == want[-1]
