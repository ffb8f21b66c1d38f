"""The PCG at the edges of its work split: wavefronts without knots, lane groups
without knots inside a wavefront, and second knots that only some wavefronts
hold. The KKT solve on identical QP data against the oracle's exact solve, with
the bar of the KKT parity test (1e-5 at PCG tolerance 1e-9), and the bitwise
independence of a solve from the batch it runs in.
"""
import numpy as np
import pytest

import oracle
import workload as w

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

import paper_2510_07625_amd as g  # noqa: E402


# 6-7 DoF: 4 knots per wavefront, 32 per pass over the lane groups, one or two
# passes, up to four passes with the A blocks' velocity rows in LDS; 3 DoF: 8 per
# wavefront, 64 per pass. general: joint rows of A other than [I, hI], which the
# Euler step never gives but a caller may.
@pytest.mark.parametrize("n,N,general", [(7, 4, 0), (7, 5, 0), (6, 17, 0), (7, 29, 0), (7, 31, 0), (6, 36, 0),
                                         (7, 37, 0), (7, 63, 0), (3, 7, 0), (3, 9, 0), (3, 63, 0), (3, 65, 0),
                                         (3, 73, 0), (3, 128, 0), (7, 65, 0), (6, 97, 0), (6, 101, 0), (7, 127, 0),
                                         (6, 128, 0), (7, 32, 1), (6, 64, 1), (7, 100, 1), (6, 128, 1)])
def test_kkt_at_the_edges_of_the_split(n, N, general):
    print(f"[gpu-case] pcg edges n={n} N={N} general={general}", flush=True)
    solves = [w.chain_solve(51, i, n=n, N=N) for i in range(3)]
    nx = 2 * n
    data = [oracle.lq(s, s.X0, s.U0) for s in solves]
    if general:
        rng = np.random.default_rng(5)
        for d in data:
            d["A"] = d["A"] + 0.02 * rng.normal(size=d["A"].shape)
    f32 = [{k: np.asarray(v, np.float32).astype(np.float64) for k, v in d.items()} for d in data]
    b = g.Batch.from_solves(solves, g.Params(pcg_tol=1e-9))
    dev = lambda k: torch.from_numpy(np.stack([c[k] for c in f32]).astype(np.float32)).cuda()
    dX, dU, lam, its = b.debug_kkt(*(dev(k) for k in ("A", "B", "e", "q", "r", "c0")))
    dX, dU, lam = (t.cpu().numpy() for t in (dX, dU, lam))
    b.close()
    for i, s in enumerate(solves):
        c = f32[i]
        Qh = np.tile(s.Qd, (N, 1))
        Qh[-1] = s.QNd
        rX, rU, rl, _ = oracle.kkt_from_lq(c["A"], c["B"], c["e"], c["q"], c["r"], c["c0"], Qh, s.Rd, mode=2)
        ref = np.concatenate([rX.ravel(), rU.ravel()])
        got = np.concatenate([dX[i].ravel(), dU[i].ravel()])
        err = np.abs(got - ref).max() / np.abs(ref).max()
        el = np.abs(lam[i].reshape(N, nx) - rl).max() / np.abs(rl).max()
        print(f"solve {i}: dZ {err:.2e} lambda {el:.2e} its {int(its[i])}")
        assert err <= 1e-5 and el <= 1e-5, (i, err, el)
        # Alone in its batch: the same bits.
        one = g.Batch.from_solves([s], g.Params(pcg_tol=1e-9))
        oX, _, ol, _ = one.debug_kkt(*(dev(k)[i:i + 1].contiguous() for k in ("A", "B", "e", "q", "r", "c0")))
        np.testing.assert_array_equal(oX.cpu().numpy()[0], dX[i])
        np.testing.assert_array_equal(ol.cpu().numpy()[0], lam[i])
        one.close()
