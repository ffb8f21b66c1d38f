"""A launch context's kernel reads its pinned inputs and writes x_1, u_0 and the
statistics to pinned memory itself: over changed slots, requests and inputs they
equal rows 1 and 0 of the launch's trajectories and the results of a plain serving
step on device arrays, bit for bit.
"""
import numpy as np
import pytest

import workload as w

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

import paper_2510_07625_amd as g  # noqa: E402


@pytest.mark.parametrize("n,N", [(3, 2), (7, 32), (6, 40)])
def test_context_outputs_are_the_launchs(n, N):
    print(f"[gpu-case] serve context n={n} N={N}", flush=True)
    M, its = 5, 2
    solves = w.chain_batch(41, M, n=n, N=N)
    xs, goal, X0, U0 = g.pack_inputs(solves)
    h_xs, h_goal = xs.cpu().numpy(), goal.cpu().numpy()
    a, b = (g.Batch.from_solves(solves, g.Params(sqp_iters=its)) for _ in range(2))
    for q in (a, b):
        q.set_trajectories(X0, U0)
    torch.cuda.synchronize()
    ctx = g.ServeContext(a, capacity=M, n_iters=its)
    for turn, slots in enumerate(([4, 1, 3], [0], [2, 0, 1, 4, 3])):
        R = len(slots)
        shift = turn % 2
        ctx.slots[:R] = slots
        ctx.xs[:R] = h_xs[slots] + np.float32(0.01 * turn)
        ctx.goal[:R] = h_goal[slots]
        ctx.submit(R, shift=shift)
        while not ctx.done():
            pass
        X, U = ctx.trajectories()
        np.testing.assert_array_equal(ctx.x1[:R], X[:R, 1])
        np.testing.assert_array_equal(ctx.u0[:R], U[:R, 0])
        d = lambda v: torch.from_numpy(np.array(v)).cuda()
        st = b.stats_buffer(its)
        Xb, Ub = torch.zeros((R, N, 2 * n), device="cuda"), torch.zeros((R, N - 1, n), device="cuda")
        b.serve_step(d(np.asarray(slots, np.int32)), d(ctx.xs[:R]), d(ctx.goal[:R]), n_iters=its, shift=shift, Xout=Xb,
                     Uout=Ub, d_stats=st)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(X, Xb.cpu().numpy())
        np.testing.assert_array_equal(U, Ub.cpu().numpy())
        its_b = g.Batch.decode_stats(st, b.M, its)["pcg_iters"][:R]
        np.testing.assert_array_equal(ctx.stats[:R]["pcg_iters"], its_b)
    ctx.close()
    a.close()
    b.close()
