"""Systems of 257 rows with the factor in LDS: 512 threads and 8 rows per lane.

Few inequality rows and many equalities leave room for the factor of 257 rows
in LDS, the only size at which a right-hand side of the LDS solves is shared by
several waves (four), which pass each block's values on through two buffers
taken in turn.  Solution, relaxed point and gradients against the float64
oracle with the tolerances of tests/parity.py; and 300 copies of a QP, which
fill every CU, agree bit for bit (values read from a buffer that its next owner
had already written would differ between copies)."""
import numpy as np
import pytest

import qpgen
from oracle import implicit, gradients

import parity as pt

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

KR = 1e-3


def _plan(n, m, p):
    import paper_2605_17913_amd as qpx
    pl = qpx.plan(n, m, p)
    assert pl["threads"] == 512 and pl["factor_in_lds"] and n + pl["kb"] + p == 257, pl


@pytest.mark.parametrize("shape", [(164, 3, 90), (168, 1, 88)], ids=lambda s: "n%d_m%d_p%d" % s)
def test_four_waves_per_right_hand_side_vs_oracle(shape):
    import paper_2605_17913_amd as qpx
    n, m, p = shape
    _plan(n, m, p)
    print(f"257 rows in LDS: n={n} m={m} p={p} B=3", flush=True)
    P = qpgen.random_feasible(3, n, m, p, seed=n + m + p)
    Td = pt.to_dev(P)
    sol = qpx.solve(*Td)
    gx = qpgen.upstream(P.B, n, seed=3)
    g = qpx.backward(*Td, sol, torch.from_numpy(gx).to(Td[0].device), kappa_relax=KR, relaxed=True)
    torch.cuda.synchronize()
    sol, g = pt.npd(sol), pt.npd(g)
    assert np.all(pt.outcome(sol["status"]) == 0), sol["status"]
    assert np.all(pt.outcome(g["relaxed"]["status"]) == 0), g["relaxed"]["status"]
    for i in range(P.B):
        r = implicit.solve_qp(*P.one(i), tol=1e-11, max_iter=200)
        assert r.status == implicit.CONVERGED
        pt.check_point(f"{shape} QP {i}", P, i, sol, r)
        ref, _ = gradients.grad_at_relaxed(*P.one(i), KR, gx[i].astype(np.float64))
        pt.check_grads(f"{shape} QP {i}", g, i, ref)


@pytest.mark.parametrize("shape", [(128, 2, 127), (164, 3, 90)], ids=lambda s: "n%d_m%d_p%d" % s)
def test_copies_agree_bit_for_bit(shape):
    import paper_2605_17913_amd as qpx
    n, m, p = shape
    _plan(n, m, p)
    B = 300
    print(f"257 rows in LDS: n={n} m={m} p={p}, {B} copies", flush=True)
    P = qpgen.random_feasible(1, n, m, p, seed=5)
    Td = [a.expand(B, *a.shape[1:]).contiguous() for a in pt.to_dev(P)]
    sol = qpx.solve(*Td)
    gx = torch.from_numpy(qpgen.upstream(1, n, seed=3)).to(Td[0].device).expand(B, n)
    g = qpx.backward(*Td, sol, gx, kappa_relax=KR)
    torch.cuda.synchronize()
    for what, d in (("sol", sol), ("grad", g)):
        for k, v in d.items():
            v = v.cpu().numpy()
            assert np.array_equal(v, np.broadcast_to(v[:1], v.shape), equal_nan=True), (what, k)
