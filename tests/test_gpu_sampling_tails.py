"""The Gaussian draw's table against the FP64 oracle where its pieces meet: supports of
0.3 to 9 sigma (bounds inside the table, beyond its end and cut to cells), uniforms
from 1e-12 (tails, which take the library's functions) through both sides of that
rule and of the median.  u agrees to 1e-9: the conditioning of the quantile at
1 - 1e-6 leaves 2e-11 sigma of FP64's rounding of the probability."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a HIP device")]


@pytest.mark.parametrize("s2r", [0.3, 1.0, 3.0, 5.5, 9.0])
@pytest.mark.parametrize("sigma", [0.05, 0.6, 3.0, 9.0])
def test_gaussian_draw_tails(oracle_mod, s2r, sigma):
    import torch
    import workloads
    import paper_2505_08985_amd as P
    nrm = workloads.make_map("powerlaw", 64, 7)
    hier = P.build_hierarchy(P.build_mesh(torch.from_numpy(nrm).cuda()), cluster=False)
    rng = np.random.default_rng(11)
    lo = np.concatenate([10.0 ** rng.uniform(-12, -0.3, 400), 1.1e-5 * (1 + 1e-3 * rng.uniform(-1, 1, 60)),
                         0.5 + rng.uniform(-1e-9, 1e-9, 40)])
    x = np.concatenate([lo, 1.0 - np.maximum(lo, 1e-6), rng.uniform(0, 1, 500), [0.0, 0.5, 0.25, 1.0 - 1e-6]])
    xi = np.stack([x, rng.permutation(x)], axis=1)
    q = np.zeros((len(x), 6), np.float32)
    q[:, :2] = rng.uniform(0, 64, (len(x), 2))
    q[:, 2] = sigma * np.exp(rng.uniform(-0.2, 0.2, len(x)))
    q[:, 3] = sigma * np.exp(rng.uniform(-0.2, 0.2, len(x)))
    _, tri, u = P.sample_batch(hier, torch.from_numpy(q).cuda(), torch.from_numpy(xi[None]).cuda(), sigma_to_r=s2r, u=True)
    ref = oracle_mod.sample(nrm, q, xi, sigma_to_r=s2r)
    np.testing.assert_allclose(u.cpu().numpy(), ref["u"], rtol=1e-9, atol=1e-9)
    ok = (ref["flags"] & 2) == 0
    assert ok.mean() > 0.5
    np.testing.assert_array_equal(tri.cpu().numpy().view(np.uint64)[ok], ref["tri"][ok])


@pytest.mark.parametrize("sigma", [0.6, 9.0, 300.0])
def test_gaussian_draw_centre(oracle_mod, sigma):
    """Away from the tails (|z| < 3): both sides' probabilities are within 4e-15 (the table's
    relative error of 3e-15 at 1/2, two roundings), which the quantile's slope 1 / phi(z) turns into
    u's error; 1e-13 for the roundings of u itself."""
    import torch
    import workloads
    import paper_2505_08985_amd as P
    nrm = workloads.make_map("powerlaw", 64, 7)
    hier = P.build_hierarchy(P.build_mesh(torch.from_numpy(nrm).cuda()), cluster=False)
    rng = np.random.default_rng(13)
    xi = rng.uniform(0.002, 0.998, (4000, 2))
    q = np.zeros((4000, 6), np.float32)
    q[:, :2] = rng.uniform(0, 64, (4000, 2))
    q[:, 2:4] = sigma * np.exp(rng.uniform(-0.2, 0.2, (4000, 2)))
    _, _, u = P.sample_batch(hier, torch.from_numpy(q).cuda(), torch.from_numpy(xi[None]).cuda(), u=True)
    ref = oracle_mod.sample(nrm, q, xi)["u"]
    z = (ref - q[:, :2]) / q[:, 2:4]
    assert np.abs(z).max() < 3.5
    tol = 2 * 4e-15 * np.sqrt(2 * np.pi) * np.exp(0.5 * z * z) * q[:, 2:4] + 1e-13 * np.maximum(1.0, q[:, 2:4] / 64)
    err = np.abs(u.cpu().numpy() - ref)
    assert (err <= tol).all(), float((err / tol).max())
