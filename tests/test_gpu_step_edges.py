"""SQP steps at the edges of the PCG's work split: the same shapes as the stage tests on
caller-given QP data, but with the Euler step's operators, which those never enter
([I, hI] joint rows of A as one entry per lane; with four knots per lane group the
velocity rows in LDS). Against the oracle replaying the accepted steps with exact QP
solves, at the bar of the trajectory tests (1e-4, PCG tolerance 1e-7)."""
import numpy as np
import pytest

import oracle
import workload as w

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

import paper_2510_07625_amd as g  # noqa: E402

PARAMS = g.Params(sqp_iters=2, pcg_tol=1e-7)


def _check(solves, split, sampled=None):
    b = g.Batch.from_solves(solves, PARAMS)
    b.set_split(split)
    xs, goal, X, U = g.pack_inputs(solves)
    buf = b.stats_buffer(2)
    b.step(xs, goal, X, U, 2, buf)
    st = g.Batch.decode_stats(buf, len(solves), 2)
    X, U = X.cpu().numpy(), U.cpu().numpy()
    lam = b.get_multipliers().cpu().numpy()
    b.close()
    assert not (st["status"] & (g.ST_PCG_MAXITER | g.ST_NONFINITE | g.ST_EXCHANGE)).any(), st["status"]
    for i in sampled or range(len(solves)):
        s = solves[i]
        ref = oracle.sqp(s, oracle.Params(sqp_iters=2, kkt_mode=2), alpha_replay=st["alpha"][i].astype(np.float64))
        ex = np.abs(X[i] - ref.X).max() / np.abs(ref.X).max()
        eu = np.abs(U[i] - ref.U).max() / np.abs(ref.U).max()
        print(f"solve {i}: X {ex:.1e} U {eu:.1e} its {st['pcg_iters'][i]}")
        assert ex <= 1e-4 and eu <= 1e-4, (i, ex, eu)
    return lam


# 6-7 DoF: 4 knots per wavefront, 32 per pass over the lane groups, one or two passes,
# up to four with N > 64 (on one workgroup); 3 DoF: 8 per wavefront, 64 per pass.
@pytest.mark.parametrize("n,N", [(7, 2), (7, 4), (7, 5), (6, 17), (7, 29), (7, 31), (7, 32), (7, 33), (6, 36), (7, 37),
                                 (7, 63), (6, 64), (3, 2), (3, 7), (3, 9), (3, 63), (3, 64), (3, 65), (3, 73), (3, 128),
                                 (7, 65), (6, 96), (6, 97), (6, 101), (7, 127), (6, 128), (7, 128)])
def test_step_on_one_workgroup(n, N):
    print(f"[gpu-case] step edges n={n} N={N}", flush=True)
    _check([w.chain_solve(51, i, n=n, N=N) for i in range(3)], split=1)


# Two workgroups per solve (80 solves: four each do not fit): a second part of one knot, of
# a full first pass, and of one knot more.
@pytest.mark.parametrize("n,N", [(7, 65), (6, 96), (7, 97)])
def test_step_on_two_workgroups(n, N):
    print(f"[gpu-case] step edges two parts n={n} N={N}", flush=True)
    solves = [w.chain_solve(53, i % 4, n=n, N=N) for i in range(80)]
    lam = _check(solves, split=4, sampled=(0, 1, 2, 3, 79))
    one = _check(solves[:4], split=1)
    assert not np.array_equal(lam[:4], one), "the split path did not run"
