"""Small batches, several wavefronts per query: the bits of the one-wavefront kernel
(eval_counts runs it) at the batch sizes where the number of waves changes, for
footprints from a fraction of a cell to several maps, tiny maps, the cut's entry
levels and every footprint kernel."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a HIP device")]


def queries(n, count, seed, aniso):
    rng = np.random.default_rng(seed)
    q = np.empty((count, 6), np.float32)
    q[:, :2] = rng.uniform(-2 * n, 2 * n, (count, 2))
    q[:, 2] = np.exp(rng.uniform(np.log(0.05), np.log(1.5 * n), count))
    q[:, 3] = q[:, 2] * np.exp(rng.uniform(-aniso, aniso, count))
    r, t = 0.3 * np.sqrt(rng.uniform(size=count)), rng.uniform(0, 2 * np.pi, count)
    q[:, 4], q[:, 5] = r * np.cos(t), r * np.sin(t)
    # half-widths around the rule that leaves a query to one wave, centres on cell edges
    q[::11, 2:4] = np.float32(16.0 / 3.0)
    q[1::11, 2:4] = np.nextafter(np.float32(16.0 / 3.0), np.float32(99))
    q[2::13, :2] = np.round(q[2::13, :2])
    if count > 5:
        q[3, 2], q[4, 0], q[5, 4] = -1.0, np.inf, np.nan
    return q


@pytest.fixture(scope="module", params=[("powerlaw", 2), ("powerlaw", 16), ("powerlaw", 128), ("scratched", 512)])
def hier(request):
    import torch
    import workloads
    import paper_2505_08985_amd as P
    kind, n = request.param
    kw = dict(scratches=300, flakes=800) if kind == "scratched" else {}
    nrm = workloads.make_map(kind, n, 47, **kw)
    return P.build_hierarchy(P.build_mesh(torch.from_numpy(nrm).cuda()), cluster=True)


@pytest.mark.parametrize("nq", [1, 7, 256, 257, 1024, 1025])
@pytest.mark.parametrize("tau", [0.0, 1e-4, 3e-2, 10.0])
def test_split_changes_no_bit(hier, tau, nq):
    import torch
    import paper_2505_08985_amd as P
    for aniso in (0.0, 1.5):
        q = torch.from_numpy(queries(hier.n, nq, 3, aniso)).cuda()
        want, _ = P.eval_counts(hier, q, tau=tau)
        for f in (P.eval_batch, P.eval_batch_noalloc):
            got = f(hier, q, tau=tau)
            assert torch.equal(got.view(torch.int32), want.view(torch.int32))


@pytest.mark.parametrize("kernel", ["disk", "box"])
def test_split_footprint_kernels(hier, kernel):
    import torch
    import paper_2505_08985_amd as P
    q = torch.from_numpy(queries(hier.n, 200, 5, 1.0)).cuda()
    for tau in (0.0, 1e-3):
        want, _ = P.eval_counts(hier, q, tau=tau, kernel=kernel, sigma_to_r=1.5)
        got = P.eval_batch(hier, q, tau=tau, kernel=kernel, sigma_to_r=1.5)
        assert torch.equal(got.view(torch.int32), want.view(torch.int32))


@pytest.mark.parametrize("nq", [16, 256, 1000])
def test_split_largest_map(nq):
    """The deepest lists: sixteen and four waves of them in a workgroup's LDS."""
    import torch
    import paper_2505_08985_amd as P
    g = torch.Generator(device="cuda").manual_seed(5)
    k = torch.arange(8192, device="cuda") * (2 * np.pi / 8192)
    nrm = 0.05 * torch.randn(8192, 8192, 2, generator=g, device="cuda")
    nrm[..., 0] += 0.3 * torch.sin(3 * k)[None, :]
    nrm[..., 1] += 0.3 * torch.cos(2 * k)[:, None]
    hier = P.build_hierarchy(P.build_mesh(nrm.clamp_(-0.6, 0.6)), cluster=True)
    q = torch.from_numpy(queries(8192, nq, 7, 0.5)).cuda()
    q[:, 2:4] = q[:, 2:4].clamp(max=400.0)
    for tau in (0.0, 1e-3):
        want, _ = P.eval_counts(hier, q, tau=tau)
        got = P.eval_batch(hier, q, tau=tau)
        assert torch.equal(got.view(torch.int32), want.view(torch.int32))
        assert bool((got > 0).any())
