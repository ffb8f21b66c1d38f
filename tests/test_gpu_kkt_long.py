"""Caller-given QP data of long solves (6-7 DoF, N > 64): a batch of mixed shapes, whose
long solves run kernels of their own, against the oracle's exact solve at the bar of
the KKT parity test, and the time of an iteration next to a shorter horizon's."""
import numpy as np
import pytest

import oracle
import workload as w

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

import paper_2510_07625_amd as g  # noqa: E402


@pytest.mark.parametrize("dispatch", [g.DISPATCH_AUTO, g.DISPATCH_GROUPED, g.DISPATCH_MIXED])
def test_mixed_shapes_with_long_horizons(dispatch):
    print(f"[gpu-case] kkt mixed shapes dispatch={dispatch}", flush=True)
    shapes = [(7, 128), (6, 100), (3, 16), (7, 32), (6, 65), (3, 128), (7, 50)]
    solves = [w.chain_solve(71, i, n=n, N=N) for i, (n, N) in enumerate(shapes)]
    M, N_max, nx_max, nu_max = len(solves), 128, 14, 7
    rng = np.random.default_rng(4)
    arr = dict(A=np.zeros((M, N_max - 1, nx_max, nx_max), np.float32), B=np.zeros((M, N_max - 1, nx_max, nu_max), np.float32),
               e=np.zeros((M, N_max - 1, nx_max), np.float32), q=np.zeros((M, N_max, nx_max), np.float32),
               r=np.zeros((M, N_max - 1, nu_max), np.float32), c0=np.zeros((M, nx_max), np.float32))
    data = []
    for i, s in enumerate(solves):
        d = {k: np.asarray(v, np.float64) for k, v in oracle.lq(s, s.X0, s.U0).items()}
        d["A"] = d["A"] + 0.02 * rng.normal(size=d["A"].shape)
        d = {k: d[k].astype(np.float32) for k in arr}
        for k, v in d.items():
            arr[k][(i,) + tuple(slice(0, m) for m in v.shape)] = v
        data.append({k: v.astype(np.float64) for k, v in d.items()})
    b = g.Batch.from_solves(solves, g.Params(pcg_tol=1e-9))
    b.set_dispatch(dispatch)
    dX, dU, lam, _ = (t.cpu().numpy() for t in b.debug_kkt(*(torch.from_numpy(arr[k]).cuda()
                                                            for k in ("A", "B", "e", "q", "r", "c0"))))
    b.close()
    for i, s in enumerate(solves):
        n, N, c = s.n, s.N, data[i]
        Qh = np.tile(s.Qd, (N, 1))
        Qh[-1] = s.QNd
        rX, rU, rl, _ = oracle.kkt_from_lq(c["A"], c["B"], c["e"], c["q"], c["r"], c["c0"], Qh, s.Rd, mode=2)
        ref = np.concatenate([rX.ravel(), rU.ravel()])
        got = np.concatenate([dX[i, :N, :2 * n].ravel(), dU[i, :N - 1, :n].ravel()])
        assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max(), (i, n, N)
        assert np.abs(lam[i, :N, :2 * n] - rl).max() <= 1e-5 * np.abs(rl).max(), (i, n, N)


def test_an_iteration_of_a_long_horizon_costs_in_proportion():
    # N = 128 holds four knots per lane group where N = 64 holds two, and reads the A blocks where
    # they are used: a few times the cost per PCG iteration, not the serial reads of every entry.
    def us(N):
        print(f"[gpu-case] kkt time N={N}", flush=True)
        solves = w.chain_batch(73, 16, n=7, N=N)
        b = g.Batch.from_solves(solves, g.Params())
        xs, goal, X, U = g.pack_inputs(solves)
        A, B, e = b.debug_lq(xs, goal, X, U)
        torch.manual_seed(0)
        q, r, c0 = (torch.randn(s, device="cuda") for s in ((16, N, 14), (16, N - 1, 7), (16, 14)))
        t = []
        for _ in range(8):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            e0.record()
            out = b.debug_kkt(A, B, e, q, r, c0)
            torch.cuda.synchronize()
            e1.record()
            e1.synchronize()
            t.append(e0.elapsed_time(e1) * 1e3)
        b.close()
        return float(np.median(t[2:])) / int(out[3].max())

    short, long = us(64), us(128)
    print(f"us per iteration: N = 64 {short:.2f}, N = 128 {long:.2f}")
    assert long <= 8.0 * short, (short, long)
