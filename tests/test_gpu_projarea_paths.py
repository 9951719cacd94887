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


def patched(kind, n=64, seed=5):
    """Maps of clamped cells: constant; constant patches; single triangles clamped beside
    regular ones (three of a cell's corners on a line)."""
    rng = np.random.default_rng(seed)
    if kind == "constant":
        return np.full((n, n, 2), (0.3, -0.2), np.float32)
    if kind == "patches":
        r = rng.uniform(-0.6, 0.6, (n // 4, n // 4, 2)).astype(np.float32)
        return np.repeat(np.repeat(r, 4, 0), 4, 1)
    nrm = rng.uniform(-0.6, 0.6, (n, n, 2)).astype(np.float32)
    nrm[::3, 1::3] = nrm[::3, ::3][:, :nrm[::3, 1::3].shape[1]]
    nrm[2::4, 2::4] = 0.97 * nrm[2::4, 2::4] / np.linalg.norm(nrm[2::4, 2::4], axis=-1, keepdims=True)
    return nrm


@pytest.mark.parametrize("nq", [300, 3000, 6000])
@pytest.mark.parametrize("kind", ["constant", "patches", "single"])
def test_clamped_cells(P, oracle_mod, kind, nq):
    announce("projected area, clamped cells: %s, %d queries" % (kind, nq))
    q = queries(64, nq, 90 + nq, 0.3, 4.0)
    check(P, oracle_mod, patched(kind), q, "gaussian", np.arange(0, nq, max(1, nq // 200)))


def test_clamped_cells_are_not_slower(P):
    """A constant map, whose cells are all clamped, takes no longer than a power-law map (0.7 of
    the time; when all of its triangles were clipped, 2.4 times)."""
    import time
    import torch
    import workloads
    q = to_dev(queries(512, 65536, 97, 1.0, 4.0))

    def best(nrm):
        _, h = build(P, nrm)
        t = []
        for _ in range(8):
            torch.cuda.synchronize()
            a = time.perf_counter()
            for _ in range(4):
                P.projected_area(h, q)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - a)
        return min(t) / 4

    flat, rough = best(patched("constant", 512)), best(workloads.make_map("powerlaw", 512, 7))
    print("constant %.0f us, power law %.0f us" % (flat * 1e6, rough * 1e6))
    assert flat < rough
