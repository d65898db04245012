"""GPU tests of the serving loop on streams of a single size: QPs of a bucket
whose launch is in flight start on an idle lane instead of waiting for it.

Every request holds the same QP and a launch runs it to the end, so all of them
take the same time on the device and their completion times tell whether they
ran side by side."""
import time

import numpy as np
import pytest

import qpgen

import parity as pt

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _alone(srv, args, count=3):
    """Fastest of a few solves on an idle server (s), and the last result."""
    res = [srv.wait(srv.submit(*args)) for _ in range(count)]
    return min(r["t_done"] - r["t_submit"] for r in res), res[-1]


def _same(a, b):
    assert a["status"] == b["status"] and a["iters"] == b["iters"]
    for k in ("x", "y", "z", "s"):
        assert np.array_equal(a[k], b[k]), k


def test_arrival_while_its_bucket_is_in_flight():
    # a second request that arrives a quarter of the way into the first one's
    # launch ends a quarter of a solve after it; held back it would end a
    # whole solve after it
    import paper_2605_17913_amd as qpx
    pt.dev()
    P = qpgen.random_feasible(1, 256, 512, 25, seed=11)
    args = (P.Q[0], P.q[0], P.A[0], P.b[0], P.G[0], P.h[0])
    with qpx.Server(max_slots=8, iters_per_step=100) as srv:
        T, ref = _alone(srv, args)
        assert pt.outcome(ref["status"]) == 0
        gaps = []
        for _ in range(5):
            first = srv.submit(*args)
            time.sleep(T / 4)
            second = srv.submit(*args)
            a, b = srv.wait(first), srv.wait(second)
            _same(a, ref)
            _same(b, ref)
            gaps.append((b["t_done"] - a["t_done"]) / T)
    print(f"n=256 alone {T * 1e3:.2f} ms, gaps {['%.2f' % g for g in gaps]}", flush=True)
    assert sorted(gaps)[2] < 0.7, gaps


def test_requests_beyond_the_staging_buffer():
    # m far above 2 n_max: a lane's staging buffer (one iterate of n_max
    # variables and 4096 rows, 8320 floats here) holds two iterates of 3024
    # floats, so six requests need at least three launches
    import paper_2605_17913_amd as qpx
    d = pt.dev()
    n, m, p = 24, 1500, 0
    P = qpgen.random_feasible(1, n, m, p, seed=12)
    args = (P.Q[0], P.q[0], None, None, P.G[0], P.h[0])
    sol = pt.npd(qpx.solve(*[None if a.shape[1] == 0 else torch.from_numpy(a).to(d)
                             for a in P.arrays()]))
    with qpx.Server(max_slots=8, iters_per_step=100, n_max=32) as srv:
        T, ref = _alone(srv, args)
        assert pt.outcome(ref["status"]) == 0
        for k in ("x", "z", "s"):
            assert np.array_equal(sol[k][0], ref[k]), k
        spans = []
        for _ in range(5):
            res = [srv.wait(t) for t in [srv.submit(*args) for _ in range(6)]]
            for r in res:
                _same(r, ref)
            spans.append((max(r["t_done"] for r in res) - min(r["t_done"] for r in res)) / T)
    print(f"n={n} m={m} alone {T * 1e3:.2f} ms, spans {['%.2f' % s for s in spans]}", flush=True)
    # the requests are submitted within a fraction of T; one launch after
    # another they end over more than two of them
    assert sorted(spans)[2] < 1.5, spans
