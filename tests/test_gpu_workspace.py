"""Device memory of a batch: with FP64 Schur rows only A and B of a solve may need
the workspace (once, also where a long solve can split), next to its multipliers and
resident trajectories."""
import pytest

import workload as w

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("no GPU", allow_module_level=True)

import paper_2510_07625_amd as g  # noqa: E402


@pytest.mark.parametrize("n,N", [(6, 128), (7, 64)])
def test_no_dead_workspace_with_fp64_schur_rows(n, N):
    print(f"[gpu-case] workspace n={n} N={N}", flush=True)
    M, nx, nu = 512, 2 * n, n
    solves = [w.chain_solve(3, i % 8, n=n, N=N) for i in range(M)]
    g.Batch.from_solves(solves[:1]).close()   # (what the runtime allocates once)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    b = g.Batch.from_solves(solves)
    used = before - torch.cuda.mem_get_info()[0]
    b.close()
    need = M * ((N - 1) * (nx * nx + nx * nu) * 4 + N * nx * 8 + (N * nx + (N - 1) * nu) * 4)
    xch = M * 4 * (8 * 104 + 1024) * 8 if N > 64 else 0   # the parts' exchange words
    print(f"used {used >> 20} MiB, {need >> 20} needed, {xch >> 20} exchange")
    assert used <= 1.1 * (need + xch) + (32 << 20)   # (allocation granules)
