"""Tiled evaluation of wide footprints: on maps with tiles an ordered batch (wide
queries descend to the tiles, which are evaluated tile by tile) gives the bits of the
same batch in input order (every query as a whole), for narrow, wide and invalid
queries, every footprint kernel, and when rounds are short and the items do not fit."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a HIP device")]


def queries(n, count, seed, lo, hi):
    rng = np.random.default_rng(seed)
    q = np.empty((count, 6), np.float32)
    q[:, :2] = rng.uniform(-n, 2 * n, (count, 2))
    q[:, 2] = np.exp(rng.uniform(np.log(lo), np.log(hi), count))
    q[:, 3] = q[:, 2] * np.exp(rng.uniform(-0.7, 0.7, count))
    r, t = 0.3 * np.sqrt(rng.uniform(size=count)), rng.uniform(0, 2 * np.pi, count)
    q[:, 4], q[:, 5] = r * np.cos(t), r * np.sin(t)
    return q


@pytest.fixture(scope="module", params=["powerlaw", "scratched"])
def hier(request):
    import torch
    import workloads
    import paper_2505_08985_amd as P
    kw = {} if request.param == "powerlaw" else dict(scratches=1200, flakes=3000)
    nrm = workloads.make_map(request.param, 1024, 41, **kw)
    return P.build_hierarchy(P.build_mesh(torch.from_numpy(nrm).cuda()), cluster=True)


# (no wide query; the threshold sigma = 256 / 3 between both; all wide, up to 4 maps)
@pytest.mark.parametrize("lo,hi,count", [(0.5, 20.0, 4096), (60.0, 110.0, 4200), (90.0, 1300.0, 4097)])
@pytest.mark.parametrize("tau", [0.0, 1e-4, 3e-2])
def test_tiles_change_no_bit(hier, tau, lo, hi, count):
    import torch
    import paper_2505_08985_amd as P
    q = queries(1024, count, 5, lo, hi)
    q[7, 2] = np.nan
    q[8, 2] = -1.0
    q[9, 0] = np.inf
    q[10, 2:4] = 3e7
    q[11, :2] = 2e7
    tq = torch.from_numpy(q).cuda()
    a = P.eval_batch(hier, tq, tau=tau)
    b = P.eval_batch(hier, tq, tau=tau, input_order=True)
    assert torch.equal(a.view(torch.int32), b.view(torch.int32))
    assert bool((a > 0).any()) and int(torch.isnan(a).sum()) == 5


@pytest.mark.parametrize("kernel", ["disk", "box"])
@pytest.mark.parametrize("tau", [0.0, 1e-3])
def test_tiles_footprint_kernels(hier, kernel, tau):
    import torch
    import paper_2505_08985_amd as P
    tq = torch.from_numpy(queries(1024, 4099, 9, 20.0, 700.0)).cuda()
    a = P.eval_batch(hier, tq, tau=tau, kernel=kernel, sigma_to_r=1.5)
    b = P.eval_batch(hier, tq, tau=tau, kernel=kernel, sigma_to_r=1.5, input_order=True)
    assert torch.equal(a.view(torch.int32), b.view(torch.int32))


# rounds of 1000 queries; rounds of 8, whose segments (4 items) a query's items overflow
@pytest.mark.parametrize("chunk,count", [(1000, 4500), (8, 4096)])
@pytest.mark.parametrize("tau", [0.0, 1e-4])
def test_tiles_rounds_and_overflow(hier, monkeypatch, tau, chunk, count):
    import torch
    import paper_2505_08985_amd as P
    q = queries(1024, count, 13, 1.0, 20.0)
    q[::7] = queries(1024, len(q[::7]), 15, 90.0, 500.0)
    tq = torch.from_numpy(q).cuda()
    b = P.eval_batch(hier, tq, tau=tau, input_order=True)
    monkeypatch.setenv("PNDF_LAUNCH_CHUNK", str(chunk))
    for _ in range(2):
        a = P.eval_batch(hier, tq, tau=tau)
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))


# the shortest rounds, with every query wide: none may be left over
@pytest.mark.parametrize("chunk", [1, 2, 3])
@pytest.mark.parametrize("plan", [False, True])
def test_tiles_shortest_rounds(hier, monkeypatch, plan, chunk):
    import torch
    import paper_2505_08985_amd as P
    count = 4096 if not plan else 101
    tq = torch.from_numpy(queries(1024, count, 19, 130.0, 300.0)).cuda()
    b = P.eval_batch(hier, tq, tau=1e-2, input_order=True)
    assert not bool(torch.isnan(b).any())
    out = torch.full((count,), float("nan"), device="cuda")
    monkeypatch.setenv("PNDF_LAUNCH_CHUNK", str(chunk))
    if plan:
        p = P.Plan(hier, count, tau=1e-2)
        p.eval(tq, out=out)
        assert p.stats()["error"] == 0
        p.close()
    else:
        P.eval_batch(hier, tq, tau=1e-2, out=out)
    assert torch.equal(out.view(torch.int32), b.view(torch.int32))


# the sizes up to which one workgroup orders a batch, in calls and in plans, with
# launches that end among the narrow and among the wide queries
@pytest.mark.parametrize("count", [4096, 8191, 8192, 8193])
@pytest.mark.parametrize("chunk", [None, 3000])
def test_order_sizes(hier, monkeypatch, chunk, count):
    import torch
    import paper_2505_08985_amd as P
    q = queries(1024, count, 23, 0.5, 30.0)
    q[::3] = queries(1024, len(q[::3]), 25, 90.0, 400.0)
    q[5, 0] = np.nan
    tq = torch.from_numpy(q).cuda()
    b = P.eval_batch(hier, tq, tau=1e-3, input_order=True)
    if chunk:
        monkeypatch.setenv("PNDF_LAUNCH_CHUNK", str(chunk))
    out = torch.full((count,), 7.0, device="cuda")
    P.eval_batch(hier, tq, tau=1e-3, out=out)
    assert torch.equal(out.view(torch.int32), b.view(torch.int32))
    for use_graph in (0, 1):
        p = P.Plan(hier, count, tau=1e-3, tuning=dict(blocks_per_cu=2, split_level=3, queue_factor=16, use_graph=use_graph))
        for k in (count, 100, count):
            out.fill_(7.0)
            p.eval(tq[:k], out=out[:k])
            assert p.stats()["error"] == 0
            assert torch.equal(out[:k].view(torch.int32), b[:k].view(torch.int32))
        p.close()


# mixed batches whose wide queries the cut makes light (a smooth map) or leaves heavy
@pytest.mark.parametrize("count", [6000, 9000, 40000])
@pytest.mark.parametrize("tau", [1e-4, 1e-3, 3e-2])
def test_light_queries(hier, tau, count):
    import torch
    import paper_2505_08985_amd as P
    q = queries(1024, count, 27, 30.0, 1000.0)
    q[::5] = queries(1024, len(q[::5]), 29, 1.0, 8.0)
    q[11, 3] = np.inf
    tq = torch.from_numpy(q).cuda()
    b = P.eval_batch(hier, tq, tau=tau, input_order=True)
    out = torch.full((count,), 7.0, device="cuda")
    P.eval_batch(hier, tq, tau=tau, out=out)
    assert torch.equal(out.view(torch.int32), b.view(torch.int32))
    p = P.Plan(hier, count, tau=tau)
    assert torch.equal(p.eval(tq).view(torch.int32), b.view(torch.int32)) and p.stats()["error"] == 0
    p.close()


def test_light_queries_are_not_slower_by_tiles():
    """A mixed batch on a smooth map under the cut against the same queries as wholes in input
    order: 0.8 of the time; with every wide query run tiled 1.3 times."""
    import time
    import torch
    import workloads
    import paper_2505_08985_amd as P
    h = P.build_hierarchy(P.build_mesh(torch.from_numpy(workloads.make_map("powerlaw", 2048, 41)).cuda()), cluster=True)
    q = torch.from_numpy(queries(2048, 131072, 5, 1.0, 2048.0)).cuda()

    def best(order):
        t = []
        for _ in range(6):
            torch.cuda.synchronize()
            a = time.perf_counter()
            for _ in range(3):
                P.eval_batch(h, q, tau=1e-3, input_order=order)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - a)
        return min(t) / 3

    tiled, whole = best(False), best(True)
    print("ordered %.2f ms, in input order %.2f ms" % (tiled * 1e3, whole * 1e3))
    assert tiled < 1.15 * whole
