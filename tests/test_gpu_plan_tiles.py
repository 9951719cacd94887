"""Plans on maps with tiles (wide queries run tiled, the others on the persistent
workers) give the plain kernel's bits, by graph and by plain launches, replayed with
other work between, for batches without, with some and with only wide queries, and in
several rounds."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a HIP device")]


def queries(n, count, seed, lo, hi):
    rng = np.random.default_rng(seed)
    q = np.empty((count, 6), np.float32)
    q[:, :2] = rng.uniform(0, n, (count, 2))
    q[:, 2:4] = np.exp(rng.uniform(np.log(lo), np.log(hi), (count, 1)))
    r, t = 0.3 * np.sqrt(rng.uniform(size=count)), rng.uniform(0, 2 * np.pi, count)
    q[:, 4], q[:, 5] = r * np.cos(t), r * np.sin(t)
    return q


@pytest.fixture(scope="module")
def hier():
    import torch
    import workloads
    import paper_2505_08985_amd as P
    nrm = workloads.make_map("scratched", 1024, 43, scratches=1200, flakes=3000)
    return P.build_hierarchy(P.build_mesh(torch.from_numpy(nrm).cuda()), cluster=True)


@pytest.mark.parametrize("use_graph", [0, 1])
@pytest.mark.parametrize("chunk", [None, 700])
@pytest.mark.parametrize("tau", [0.0, 1e-3])
def test_plan_tiles_equal_plain(hier, monkeypatch, tau, chunk, use_graph):
    import torch
    import paper_2505_08985_amd as P
    batches = [torch.from_numpy(queries(1024, c, k, lo, hi)).cuda()
               for k, (c, lo, hi) in enumerate([(3001, 2.0, 600.0), (1, 300.0, 301.0), (2000, 1.0, 40.0),
                                                (1500, 100.0, 900.0), (3, 2.0, 3.0)])]
    want = [P.eval_batch(hier, q, tau=tau, input_order=True) for q in batches]
    if chunk:
        monkeypatch.setenv("PNDF_LAUNCH_CHUNK", str(chunk))
    plan = P.Plan(hier, 3001, tau=tau, tuning=dict(blocks_per_cu=2, split_level=3, queue_factor=16, use_graph=use_graph))
    for _ in range(3):
        for q, w in zip(batches, want):
            got = plan.eval(q)
            noise = torch.randn(1 << 18, device="cuda").sum()
            torch.cuda.synchronize()
            assert plan.stats()["error"] == 0
            assert torch.equal(got.view(torch.int32), w.view(torch.int32))
            del noise
    plan.close()
