"""PCG tolerances far below rounding (any positive tolerance is taken). The loops
that form u = P r from the residual itself drive r^T P r down to the end of FP64's
range; the multipliers have long converged by then and have to stay so, with the
status saying that the tolerance was not reached. Against the exact step of the
oracle at the trajectory bar (FP32 results)."""
import numpy as np
import pytest

import oracle
import workload as w

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

import paper_2510_07625_amd as g  # noqa: E402


# Four knots per lane group on one workgroup (its cap N nx is far enough on these
# well-conditioned systems); tip tracking at one knot per lane group.
@pytest.mark.parametrize("kind,n,N,cap", [("linear", 7, 65, 0), ("linear", 6, 128, 0), ("linear", 7, 100, 4000),
                                          ("tip", 6, 16, 700), ("tip", 3, 8, 180), ("tip", 3, 8, 4000)])
def test_a_tolerance_that_cannot_be_reached(kind, n, N, cap):
    print(f"[gpu-case] tight {kind} n={n} N={N} cap={cap}", flush=True)
    make = w.double_integrator_solve if kind == "linear" else w.figure8_solve
    solves = [make(1, i, n=n, N=N) for i in range(2)]
    b = g.Batch.from_solves(solves, g.Params(sqp_iters=1, pcg_tol=1e-200, pcg_max_iter=cap))
    b.set_split(1)
    xs, goal, X, U = g.pack_inputs(solves)
    buf = b.stats_buffer(1)
    b.step(xs, goal, X, U, 1, buf)
    st = g.Batch.decode_stats(buf, 2, 1)
    X, U = X.cpu().numpy(), U.cpu().numpy()
    lam = b.get_multipliers().cpu().numpy()
    b.close()
    assert np.isfinite(lam).all()
    for i, s in enumerate(solves):
        ref = oracle.sqp(s, oracle.Params(sqp_iters=1, kkt_mode=2), alpha_replay=[float(st["alpha"][i, 0])])
        err = max(np.abs(X[i] - ref.X).max() / np.abs(ref.X).max(), np.abs(U[i] - ref.U).max() / np.abs(ref.U).max())
        print(i, int(st["pcg_iters"][i, 0]), int(st["status"][i, 0]), f"{err:.1e}")
        assert int(st["status"][i, 0]) & g.ST_PCG_MAXITER and not int(st["status"][i, 0]) & g.ST_NONFINITE
        assert st["alpha"][i, 0] > 0.0
        assert err <= 1e-4


def test_nothing_left_to_solve_counts_as_reached():
    # At rest on the goal gamma~ and its norm are exactly zero.
    print("[gpu-case] tight zero", flush=True)
    s = w.double_integrator_solve(2, 0, n=7, N=65)
    b = g.Batch.from_solves([s], g.Params(sqp_iters=1, pcg_tol=1e-200))
    b.set_split(1)
    xs, goal, X, U = (t.zero_() for t in g.pack_inputs([s]))
    buf = b.stats_buffer(1)
    b.step(xs, goal, X, U, 1, buf)
    st = g.Batch.decode_stats(buf, 1, 1)[0, 0]
    b.close()
    assert int(st["pcg_iters"]) == 0 and not int(st["status"]) & (g.ST_PCG_MAXITER | g.ST_NONFINITE)
    assert float(X.abs().max()) == 0.0 and float(U.abs().max()) == 0.0
