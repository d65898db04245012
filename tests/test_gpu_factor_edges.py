"""Edges of the factorisation, the triangular solves and the matrix-core
assembly against float64.

Without inequalities the bordered system has exactly n + p rows, and the answer
is one factorisation, one solve and its refinement: sizes around whole 16-row
blocks, and around the number of blocks that a workgroup's waves hold at once
(3 per wave and the diagonal block: 112 rows at 128 threads, 208 at 256, 400
at 512), above which further blocks replay the panel; above 512 rows each lane
holds two rows of the solves.  Q = M M' / n + I, so cond(K) stays below a few
hundred and float32 with refinement is within tests/parity.py's bound on x
(1e-4) by two orders.  Then the assembly with more columns than a wave loads
ahead and more tiles than one pass takes, and degenerate QPs, whose border
pivots need regularisation in whole, mixed and partial panels.
"""
import numpy as np
import pytest

import qpgen
from oracle import implicit

import parity as pt

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ROWS = [(None, r) for r in (2, 15, 16, 17, 32, 33, 63, 64, 65, 128, 129, 256, 257, 512, 513, 1024)]
ROWS += [(128, r) for r in (112, 113, 129)] + [(256, r) for r in (208, 209, 257)]
ROWS += [(512, r) for r in (17, 400, 401, 640)]


@pytest.mark.parametrize("block,rows", ROWS)
def test_equality_only_rows(block, rows):
    import paper_2605_17913_amd as qpx
    p = rows // 4
    n = rows - p
    print(f"equality-only QPs: {rows} rows (n={n} p={p}), block={block}", flush=True)
    rng = np.random.default_rng(rows)
    M = rng.standard_normal((2, n, n))
    Q = (M @ np.swapaxes(M, 1, 2) / n + np.eye(n)).astype(np.float32)
    q, A, b = (rng.standard_normal(s).astype(np.float32) for s in ((2, n), (2, p, n), (2, p)))
    T = lambda a: torch.from_numpy(a).to(pt.dev())
    kw = {} if block is None else {"block": block}
    sol = pt.npd(qpx.solve(T(Q), T(q), T(A) if p else None, T(b) if p else None, None, None, **kw))
    assert np.all(pt.outcome(sol["status"]) == 0), sol["status"]
    for i in range(2):
        K = np.zeros((rows, rows))
        K[:n, :n] = Q[i]
        K[:n, n:], K[n:, :n] = A[i].T, A[i]
        ref = np.linalg.solve(K, np.concatenate([-q[i], b[i]]).astype(np.float64))
        pt.check_x(f"{rows} rows QP {i}", sol["x"][i], ref[:n])


ASSEMBLY = [(100, 128), (130, 256), (130, 512), (272, 512)]


@pytest.mark.parametrize("mode", ["mfma_fp32", "bf16x3"])
@pytest.mark.parametrize("n,block", ASSEMBLY)
def test_matrix_core_assembly_edges(n, block, mode):
    import paper_2605_17913_amd as qpx
    m, p = 2 * n + 9, 3  # a last chunk of rows that is not whole
    print(f"assembly {mode}: n={n} m={m} p={p} block={block}", flush=True)
    P = qpgen.random_feasible(2, n, m, p, seed=n)
    sol = pt.npd(qpx.solve(*pt.to_dev(P), block=block, assembly=mode))
    assert np.all(pt.outcome(sol["status"]) == 0), sol["status"]
    r = implicit.solve_qp(*P.one(0), tol=1e-10, max_iter=200)
    assert r.status == implicit.CONVERGED
    pt.check_point(f"n={n} {mode} QP 0", P, 0, sol, r)


@pytest.mark.parametrize("n", [24, 40, 72, 128])
def test_degenerate_qps(n):
    import paper_2605_17913_amd as qpx
    print(f"degenerate QPs: n={n}", flush=True)
    P = qpgen.ill_conditioned(8, n, 2 * n, n // 8, seed=n)
    sol = pt.npd(qpx.solve(*pt.to_dev(P), tol=1e-6))
    assert np.all(pt.outcome(sol["status"]) == 0), sol["status"]
    for i in range(P.B):
        pt.check_x(f"n={n} QP {i}", sol["x"][i], P.extra["x_star"][i])
