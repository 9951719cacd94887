"""The calls' stream-ordered workspace: batches that overlap on several streams and
threads without a synchronisation get what each gets alone (bit for bit), and what the
library keeps is given back with the last handle."""
import subprocess
import sys
import threading

import numpy as np
import pytest

from conftest import gpu_available
from test_gpu_blocks import bits, load, queries

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a HIP device")]


@pytest.mark.parametrize("threads", [1, 3])
def test_overlapping_streams(threads):
    import torch
    import paper_2505_08985_amd as P
    h = load(P, 1024, 3, False)
    qs = [queries(1024, 4096 + 1500 * k, 20 + k) for k in range(4)]
    ref = []
    for q in qs:
        ref.append((bits(P.eval_batch(h, q)), bits(P.projected_area(h, q[:4500]))))
    torch.cuda.synchronize()
    bad = []

    def work(t):
        streams = [torch.cuda.Stream() for _ in range(2)]
        outs = []
        for r in range(6):
            k = (r + t) % len(qs)
            with torch.cuda.stream(streams[r % 2]):
                outs.append((k, P.eval_batch(h, qs[k]), P.projected_area(h, qs[k][:4500])))
        for s in streams:
            s.synchronize()
        for k, a, b in outs:
            if not (np.array_equal(bits(a), ref[k][0]) and np.array_equal(bits(b), ref[k][1])):
                bad.append((t, k))

    pool = [threading.Thread(target=work, args=(t,)) for t in range(threads)]
    for t in pool:
        t.start()
    for t in pool:
        t.join()
    assert not bad, bad


def test_given_back():
    """The workspace of 100000 queries on 16 tiles: 2 x 16 items of 8 bytes each and as
    many sorted (49 MiB), 48 bytes of sums and a query's setup of 100 or more (14 MiB)."""
    code = """
import sys; sys.path[:0] = ['tests', '.']
import torch, paper_2505_08985_amd as P
from test_gpu_blocks import load, queries
h = load(P, 1024, 3, False); q = queries(1024, 100000, 5)
q[:, 2:4] = q[:, 2:4].clamp(max=8.0)
P.eval_batch(h, q); torch.cuda.synchronize()
kept = torch.cuda.mem_get_info()[0]
h.mesh.close(); h.close(); torch.cuda.synchronize()
print((torch.cuda.mem_get_info()[0] - kept) >> 20)
"""
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    assert int(r.stdout.split()[-1]) >= 60, r.stdout
