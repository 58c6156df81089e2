"""Calls from several threads on one stream, which share the stream's temporary buffer: each holds it until
its last kernel is queued, so their kernels never mix on it. Sizes differ, so the buffer also grows between
calls. Sums of integers, exact in any order."""
import threading

import numpy as np
import pytest
import torch

import paper_2404_03019_amd as geot
from gpu_util import say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def problem(seed, n, R, nx, F):
    rng = np.random.default_rng(seed)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    row = np.sort(rng.integers(0, R, n)).astype(np.int64)
    return (up(rng.integers(-4, 5, (nx, F)).astype(np.float32)), up(rng.integers(0, nx, n).astype(np.int64)),
            up(rng.integers(0, 3, n).astype(np.float32)), up(row), R, up(rng.integers(-4, 5, (R, F)).astype(np.float32)))


def call(p):
    x, col, w, row, R, g = p
    out = geot.gather_scatter(x, col, w, row, R, "sum")
    gx, gw = geot.gather_scatter_backward(x, col, w, row, g, "sum")
    return out, gx, gw


@pytest.mark.parametrize("sizes", [((30_000, 900, 1100, 16), (60_000, 30_000, 700, 33), (5_000, 300, 4_000, 100))])
def test_threads_on_one_stream(sizes):
    problems = [problem(i, *s) for i, s in enumerate(sizes)]
    want = [call(p) for p in problems]
    torch.cuda.synchronize()
    geot.release_scratch()                  # the buffer grows again while the threads run
    say("threads on one stream")
    bad = []

    def work(k):
        for i in range(30):
            p = (k + i) % len(problems)
            if not all(torch.equal(a, b) for a, b in zip(call(problems[p]), want[p])):
                bad.append((k, i, p))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not bad, bad


@pytest.mark.parametrize("nx", [1, 255, 4096, 4097, 70_000, (1 << 23) + 5])
def test_direct_transposition_scan(nx):
    """Column starts of short edge lists: one tile of 4,096 columns, its edges, and more tiles than the blocks
    add up themselves (over 2,048)."""
    rng = np.random.default_rng(nx)
    n, R = 5000, 400
    col, row = rng.integers(0, nx, n).astype(np.int64), np.sort(rng.integers(0, R, n)).astype(np.int64)
    col[:40] = nx - 1
    w = rng.integers(1, 5, n).astype(np.float32)
    say(f"transposition scan nx={nx}")
    sc, rt, cf = (t.cpu().numpy() for t in geot.transpose_edges(*(torch.from_numpy(a).to(DEV) for a in (col, w, row)), nx, R))
    got = sorted(zip(sc.tolist(), rt.tolist(), cf.tolist()))
    assert np.array_equal(sc, np.sort(col)) and got == sorted(zip(col.tolist(), row.tolist(), w.tolist()))
