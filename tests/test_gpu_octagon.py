"""Octagon pruning (bounds of x, y, x + y, x - y per node) never drops a hit: on maps
whose normals lie along slanted lines, where the diagonal bounds are as thin as a
single half-precision value, the descent finds exactly the hits of the brute force,
for query normals on those lines, at vertices and at both zeros."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a HIP device")]


def slanted_map(n, kind, seed):
    """Normals on the 1/128 lattice along a slanted line (diag, anti), around zero
    (zero), or off the lattice (free): lattice offsets and edge functions are exact."""
    rng = np.random.default_rng(seed)
    t = rng.integers(-24, 25, (n, n))
    w = rng.integers(-1, 2, (n, n))
    if kind == "diag":
        x, y = t, t + w
    elif kind == "anti":
        x, y = t, -t + w
    elif kind == "zero":
        x, y = rng.integers(-1, 2, (n, n)), rng.integers(-1, 2, (n, n))
    else:
        x = rng.normal(0.0, 20.0, (n, n))
        y = 0.7 * x + rng.normal(0.0, 0.4, (n, n))
    return (np.stack([x, y], -1) / 128.0).astype(np.float32)


@pytest.mark.parametrize("kind", ["diag", "anti", "zero", "free"])
@pytest.mark.parametrize("n", [2, 8, 64])
def test_octagons_drop_no_hit(kind, n):
    import torch
    import paper_2505_08985_amd as P
    rng = np.random.default_rng(7)
    nrm = slanted_map(n, kind, 3)
    nq = 600
    q = np.empty((nq, 6), np.float32)
    q[:, :2] = rng.uniform(0, n, (nq, 2))
    q[:, 2:4] = np.exp(rng.uniform(np.log(0.3), np.log(n), (nq, 2)))
    i, j = rng.integers(0, n, nq), rng.integers(0, n, nq)
    q[:, 4:] = nrm[j, i]                                              # at vertices
    q[::3, 4:] = 0.5 * (nrm[j, i] + nrm[j, (i + 1) % n])[::3]         # edge midpoints
    q[1::3, 4:] += rng.integers(-2, 3, (len(q[1::3]), 2)).astype(np.float32) / 256.0
    q[:8, 4:] = [[0.0, 0.0], [-0.0, 0.0], [0.0, -0.0], [-0.0, -0.0],
                 [2.0 ** -11, -2.0 ** -11], [-2.0 ** -30, 0.0], [0.0, 2.0 ** -30], [2.0 ** -30, -2.0 ** -30]]
    mesh = P.build_mesh(torch.from_numpy(nrm).cuda())
    hier = P.build_hierarchy(mesh, cluster=True)
    tq = torch.from_numpy(q).cuda()
    plain, c = P.eval_counts(hier, tq, algo="plain")
    brute, cb = P.eval_counts(hier, tq, algo="brute")
    np.testing.assert_array_equal(c.cpu().numpy()[:, 3], cb.cpu().numpy()[:, 3])
    np.testing.assert_array_equal(plain.cpu().numpy().view(np.uint32), brute.cpu().numpy().view(np.uint32))
    assert cb.cpu().numpy()[:, 3].sum() > 0
