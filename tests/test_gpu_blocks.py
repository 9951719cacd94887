"""Handles made from memory that earlier handles released: a map loaded over another's
memory gives what it gives in fresh memory, whatever the sizes, with several threads,
and when the earlier handle goes while its evaluation is still in flight."""
import threading

import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a HIP device")]


def a_map(n, seed):
    import torch
    rng = np.random.default_rng(seed)
    k = np.arange(n) * (2 * np.pi / n)
    f = rng.integers(1, 4, 2)
    x = 0.3 * np.sin(f[0] * k)[None, :] + rng.normal(0, 0.05, (n, n))
    y = 0.3 * np.cos(f[1] * k)[:, None] + rng.normal(0, 0.05, (n, n))
    return torch.from_numpy(np.stack([x, y], -1).astype(np.float32)).cuda()


def queries(n, count, seed):
    import torch
    rng = np.random.default_rng(seed)
    q = np.empty((count, 6), np.float32)
    q[:, :2] = rng.uniform(0, n, (count, 2))
    q[:, 2:4] = np.exp(rng.uniform(0, np.log(n / 2), (count, 2)))
    q[:, 4:] = rng.uniform(-0.3, 0.3, (count, 2))
    return torch.from_numpy(q).cuda()


def load(P, n, seed, cluster=True):
    return P.build_hierarchy(P.build_mesh(a_map(n, seed)), cluster)


def bits(t):
    return t.cpu().numpy().view(np.uint32)


def test_reloaded_maps_give_the_same():
    import paper_2505_08985_amd as P
    order = [(64, 1), (256, 2), (64, 3), (2, 4), (256, 5), (128, 6), (256, 2), (64, 1), (128, 6), (2, 4)]
    first = {}
    for n, seed in order + order[::-1]:
        for cluster in (True, False):
            h = load(P, n, seed, cluster)
            q = queries(n, 300, 9)
            got = [bits(P.eval_batch(h, q, tau=t)) for t in ((0.0, 1e-2) if cluster else (0.0,))]
            got += [bits(x) for x in P.hier_export_level(h, 1).values() if x is not None]
            h.mesh.close()
            h.close()
            for a, b in zip(first.setdefault((n, seed, cluster), got), got):
                np.testing.assert_array_equal(a, b)


def test_released_in_flight():
    import torch
    import paper_2505_08985_amd as P
    q = queries(256, 3000, 3)
    a = load(P, 256, 11)
    want = bits(P.eval_batch(a, q))
    for _ in range(5):
        got = P.eval_batch(a, q)
        a.mesh.close()
        a.close()                       # its memory may be the next map's
        load(P, 256, 12)
        np.testing.assert_array_equal(bits(got), want)
        a = load(P, 256, 11)
    torch.cuda.synchronize()


def test_threads_load_maps():
    import torch
    import paper_2505_08985_amd as P
    want = {s: bits(P.eval_batch(load(P, 128, s), queries(128, 200, s), tau=1e-3)) for s in range(4)}
    bad = []

    def work(s):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for _ in range(6):
                h = load(P, 128, s)
                if not np.array_equal(bits(P.eval_batch(h, queries(128, 200, s), tau=1e-3)), want[s]):
                    bad.append(s)
                h.mesh.close()
                h.close()

    ts = [threading.Thread(target=work, args=(s,)) for s in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
