"""One-shape launches at one knot per lane group run with the wavefronts their
longest horizon needs. A solve must not depend on that: the same solves next to
one at the full horizon (full workgroups) give the same bits.
"""
import numpy as np
import pytest

import workload as w

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

import paper_2510_07625_amd as g  # noqa: E402


def run(solves, params, its=2):
    b = g.Batch.from_solves(solves, params)
    xs, goal, X, U = g.pack_inputs(solves)
    st = b.stats_buffer(its)
    b.step(xs, goal, X, U, its, st)
    out = X.cpu().numpy(), U.cpu().numpy(), g.Batch.decode_stats(st, b.M, its)
    b.close()
    return out


# One wavefront, one and two lane groups into the next one, both sides of 256
# threads (two workgroups per CU), more solves than one round of them; 16 step
# candidates need more threads than 3 DoF lane groups at N = 9.
@pytest.mark.parametrize("n,N,M,f64,n_alpha,task", [
    (6, 2, 3, 1, 8, 0), (7, 4, 3, 1, 8, 0), (7, 5, 3, 1, 8, 0), (6, 16, 600, 1, 8, 0), (7, 17, 3, 1, 16, 0),
    (3, 9, 3, 1, 16, 0), (3, 32, 520, 1, 8, 0), (7, 8, 3, 0, 8, 0), (6, 16, 3, 0, 1, 0), (7, 5, 3, 1, 8, 1)])
def test_solve_does_not_depend_on_the_workgroup(n, N, M, f64, n_alpha, task):
    print(f"[gpu-case] block threads n={n} N={N} M={M} f64={f64} n_alpha={n_alpha} task={task}", flush=True)
    batch = w.figure8_batch if task else w.chain_batch
    p = g.Params(schur_fp64=f64, n_alpha=n_alpha, sqp_iters=2)
    solves = batch(31, M, n=n, N=N)
    long = batch(32, 1, n=n, N=64 if n == 3 else 32)
    X, U, st = run(solves, p)
    Xl, Ul, stl = run(solves + long, p)
    nx = 2 * n
    np.testing.assert_array_equal(X.reshape(M, N, nx), Xl[:M].reshape(M, -1, nx)[:, :N])
    np.testing.assert_array_equal(U.reshape(M, N - 1, n), Ul[:M].reshape(M, -1, n)[:, :N - 1])
    np.testing.assert_array_equal(st, stl[:M])
    assert np.isfinite(X).all() and np.isfinite(U).all()
