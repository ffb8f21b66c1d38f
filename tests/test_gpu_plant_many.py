"""The plant of many instances: one thread per instance from 8193 on (3 DoF: 4097), where
16-lane groups would queue for the device. Both sides of that count against the oracle's RK4
at the bars of the plant's parity test (FP32 states), with robots of different DoF
and model, tip forces, an update in place and instances that cannot be stepped; and
the time of many instances against few."""
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


@pytest.mark.parametrize("M,force,dofs", [(8192, True, (7, 3, 6)), (8193, False, (7, 3, 6)), (8193, True, (7, 3, 6)),
                                          (8257, True, (6, 3, 6)), (4096, True, (3,)), (4097, True, (3,))])
def test_both_sides_of_the_count_match_the_oracle(M, force, dofs):
    print(f"[gpu-case] plant many M={M} force={force} dofs={dofs}", flush=True)
    kinds = [w.double_integrator_solve(65, i, n=n, N=2) if i % 4 == 3 else w.chain_solve(65, i, n=n, N=2)
             for i, n in enumerate((dofs * 9)[:9])]
    solves = [kinds[i % len(kinds)] for i in range(M)]
    b = g.Batch.from_solves(solves, g.Params(sqp_iters=1))
    rng = np.random.default_rng(3)
    x = rng.uniform(-1, 1, (M, b.nx_max)).astype(np.float32)
    tau = rng.normal(0, 3, (M, b.nu_max)).astype(np.float32)
    fe = rng.normal(0, 10, (M, 3)).astype(np.float32)
    slots = np.arange(M, dtype=np.int32)
    slots[5], slots[M - 2] = M, -1       # out of range: left as they are
    x[M - 3, 1] = np.nan
    dev = lambda a: torch.from_numpy(a.copy()).cuda()
    xd, status = dev(x), torch.full((M,), -1, dtype=torch.int32, device="cuda")
    b.plant_step(xd, dev(tau), h=0.01, substeps=3, slots=dev(slots), xn=xd, status=status, fext=dev(fe) if force else None)
    xn, status = xd.cpu().numpy(), status.cpu().numpy()
    b.close()
    bad = {5, M - 2, M - 3}
    assert set(np.flatnonzero(status)) == bad and all(status[i] == g.ST_NONFINITE for i in bad)
    for i in sorted(bad - {M - 3}):
        np.testing.assert_array_equal(xn[i], x[i])
    for i in sorted(set(range(0, 20)) | set(range(M - 20, M)) | set(range(64, M, 509))):
        s = solves[i]
        np.testing.assert_array_equal(xn[i, 2 * s.n:], x[i, 2 * s.n:])
        if i in bad:
            continue
        if force and s.model == 0:
            s = dataclasses.replace(s, fext=tuple(float(v) for v in fe[i]))
        ref = oracle.plant_rk4(s, x[i, :2 * s.n].astype(np.float64), tau[i, :s.n].astype(np.float64), 0.01, 3)
        np.testing.assert_allclose(xn[i, :2 * s.n], ref, rtol=2e-6, atol=2e-6)


def test_many_instances_cost_little_more_than_a_few():
    # One thread each, 32768 instances are 512 wavefronts: half the device's SIMDs, so the latency of
    # one instance (about twice a lane group's); as lane groups they would be eight rounds of it.
    def ms(M):
        print(f"[gpu-case] plant time M={M}", flush=True)
        one = [w.chain_solve(66, i, n=7, N=2) for i in range(16)]
        b = g.Batch.from_solves([one[i % 16] for i in range(M)], g.Params(sqp_iters=1))
        x = torch.zeros((M, 14), device="cuda")
        tau, xn = torch.zeros((M, 7), device="cuda"), torch.empty_like(x)
        t = []
        for _ in range(12):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            b.plant_step(x, tau, h=0.01, substeps=10, xn=xn, stream=torch.cuda.current_stream())
            e1.record()
            torch.cuda.synchronize()
            t.append(e0.elapsed_time(e1))
        b.close()
        return float(np.median(t[2:]))

    few, many = ms(1024), ms(32768)
    print(f"1024: {few * 1e3:.0f} us, 32768: {many * 1e3:.0f} us")
    assert many <= 5.0 * few, (few, many)
