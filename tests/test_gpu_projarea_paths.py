"""The projected area's paths against the FP64 oracle: the batch sizes at which eight,
four and one wavefronts share a query and at which the batch is ordered, and the
footprints at which the table of axis factors stops fitting, on a map whose edges are
short, one whose edges need the long form and one with clamped triangles.  All paths
evaluate the same sum in FP64 and round it once to float32, so they agree with the
oracle to 1e-5 relative plus 1e-9 absolute like the whole entry point."""
import numpy as np
import pytest

from conftest import gpu_available
from test_gpu_projarea import ATOL, MAPS, RTOL, announce, build, queries, to_dev

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a HIP device")]


@pytest.fixture(scope="module")
def P():
    import paper_2505_08985_amd as P
    return P


def check(P, oracle_mod, nrm, q, kernel, sub):
    s2r = 3.0 if kernel == "gaussian" else 1.5
    _, hier = build(P, nrm)
    got = P.projected_area(hier, to_dev(q), sigma_to_r=s2r, kernel=kernel).cpu().numpy().astype(np.float64)
    # (a direction within 1e-4 of the horizon may round to a norm above 1: invalid)
    wide = (q[:, 4:6].astype(np.float64) ** 2).sum(1) > 1.0
    assert np.array_equal(np.isnan(got), wide)
    sub = sub[~wide[sub]]
    ref = oracle_mod.projected_area(nrm, q[sub], sigma_to_r=s2r, kernel=kernel)
    err = np.abs(got[sub] - ref)
    assert (err <= RTOL * np.abs(ref) + ATOL).all(), float((err / (np.abs(ref) + ATOL)).max())
    assert (ref > 0).any()


@pytest.mark.parametrize("nq", [1, 21, 512, 513, 4096, 4097])
@pytest.mark.parametrize("name", ["powerlaw128", "steep16", "flatpatch32"])
def test_batch_sizes(P, oracle_mod, name, nq):
    announce("projected area %s, %d queries" % (name, nq))
    nrm = MAPS[name]()
    q = queries(nrm.shape[0], max(nq, 16), 60 + nq, 0.3, 5.0)[-nq:]
    sub = np.unique(np.concatenate([np.arange(min(nq, 100)), np.arange(max(0, nq - 100), nq)]))
    check(P, oracle_mod, nrm, q, "gaussian", sub)


@pytest.mark.parametrize("kernel,sigma", [("gaussian", 26.5), ("box", 53.0)])
def test_axis_table_limit(P, oracle_mod, kernel, sigma):
    """Columns plus rows from below 320 to above it, one axis wider than the map too."""
    announce("projected area axis table %s" % kernel)
    nrm = __import__("workloads").make_map("powerlaw", 256, 7)
    q = queries(256, 24, 71, 1.0, 1.0)
    q[:, 2] = q[:, 3] = sigma * np.linspace(0.97, 1.03, 24)
    q[20:, 2] *= 2.0
    q[20:, 3] *= np.array([0.2, 0.3, 0.4, 0.5], np.float32)
    check(P, oracle_mod, nrm, q, kernel, np.arange(24))
