"""The plant's lane groups: wavefronts that hold robots of different DoF and model,
a last wavefront that is not full, tip forces, an update in place, and the
status of a slot out of range and of a non-finite state, each next to instances
that have to be left as they are. Against the oracle's RK4 at the bars of the
plant's parity test (FP32 states)."""
import dataclasses

import numpy as np
import pytest

import oracle
import workload as w

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

import paper_2510_07625_amd as g  # noqa: E402


@pytest.mark.parametrize("M,force", [(1, False), (5, True), (11, False), (16, True)])
def test_mixed_groups_match_the_oracle(M, force):
    print(f"[gpu-case] plant groups M={M} force={force}", flush=True)
    dofs = [(7, 3, 6, 3), (3, 7, 7, 6)]
    solves = []
    for i in range(M):
        n = dofs[(i // 4) % 2][i % 4]
        linear = i % 5 == 4
        solves.append(w.double_integrator_solve(61, i, n=n, N=8) if linear else w.chain_solve(61, i, n=n, N=8))
    b = g.Batch.from_solves(solves, g.Params(sqp_iters=1))
    rng = np.random.default_rng(7)
    x = np.zeros((M, b.nx_max), np.float32)
    tau = np.zeros((M, b.nu_max), np.float32)
    fe = np.zeros((M, 3), np.float32)
    for i, s in enumerate(solves):
        x[i, :2 * s.n] = rng.uniform(-1, 1, 2 * s.n)
        tau[i, :s.n] = rng.normal(0, 3, s.n)
        fe[i] = rng.normal(0, 10, 3)
    xd = torch.from_numpy(x).cuda()
    status = torch.full((M,), -1, dtype=torch.int32, device="cuda")
    out = b.plant_step(xd, torch.from_numpy(tau).cuda(), h=0.01, substeps=3, xn=xd, status=status,
                       fext=torch.from_numpy(fe).cuda() if force else None)
    xn = out.cpu().numpy()
    assert (status.cpu().numpy() == 0).all()
    for i, s in enumerate(solves):
        if force and s.model == 0:
            s = dataclasses.replace(s, fext=tuple(float(v) for v in fe[i]))
        ref = oracle.plant_rk4(s, x[i, :2 * s.n].astype(np.float64), tau[i, :s.n].astype(np.float64), 0.01, 3)
        np.testing.assert_allclose(xn[i, :2 * s.n], ref, rtol=2e-6, atol=2e-6)
        np.testing.assert_array_equal(xn[i, 2 * s.n:], x[i, 2 * s.n:])
    b.close()


def test_bad_instances_are_reported_alone():
    print("[gpu-case] plant bad instances", flush=True)
    solves = [w.chain_solve(63, i, n=7, N=8) for i in range(6)]
    b = g.Batch.from_solves(solves, g.Params(sqp_iters=1))
    rng = np.random.default_rng(9)
    x = rng.uniform(-1, 1, (6, 14)).astype(np.float32)
    tau = rng.normal(0, 3, (6, 7)).astype(np.float32)
    slots = np.arange(6, dtype=np.int32)
    dev = lambda a: torch.from_numpy(a).cuda()
    good = b.plant_step(dev(x), dev(tau), substeps=2, slots=dev(slots)).cpu().numpy()
    x[1, 3] = np.nan
    slots[4] = 6
    xn = torch.full((6, 14), 5.0, dtype=torch.float32, device="cuda")
    status = torch.full((6,), -1, dtype=torch.int32, device="cuda")
    out = b.plant_step(dev(x), dev(tau), substeps=2, slots=dev(slots), xn=xn, status=status).cpu().numpy()
    assert status.cpu().numpy().tolist() == [0, g.ST_NONFINITE, 0, 0, g.ST_NONFINITE, 0]
    for i in (0, 2, 3, 5):
        np.testing.assert_array_equal(out[i], good[i])
    assert (out[4] == 5.0).all()
    b.close()
