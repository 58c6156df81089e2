"""The segment gradients that read the ids, whose blocks take whole rows' vectors end to end: rows of one
vector up to several tiles of 1,024, widths that no vector divides (the last one overlaps), and addresses
that are aligned to elements only. Sum and recorded max are copies, so exact; mean is one rounded product."""
import numpy as np
import pytest
import torch

import paper_2404_03019_amd as geot
from gpu_util import say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("F", [1, 2, 3, 4, 5, 12, 47, 48, 100, 260, 1000, 4100, 8200])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("shift", [0, 1])
def test_flat_gradients(F, dtype, shift):
    rng = np.random.default_rng(F)
    n, S = (2053, 300) if F <= 260 else (37, 9)
    index = np.sort(rng.integers(0, S, n))
    i = torch.from_numpy(index).to(DEV)
    gflat = torch.randn(S * F + shift, device=DEV)
    g = gflat[shift:].view(S, F)
    buf = torch.full((n * F + shift + 64,), 7.0, dtype=dtype, device=DEV)
    out = buf[shift:shift + n * F].view(n, F)
    say(f"flat gradients F={F} {dtype} shift={shift}")
    counts = torch.bincount(i, minlength=S).clamp_(min=1).float()
    for idx in (i, i.int()):
        geot.segment_reduce_backward(g, idx, "sum", grad_src=out)
        assert torch.equal(out, g[i].to(dtype))
        geot.segment_reduce_backward(g, idx, "mean", grad_src=out)
        assert torch.equal(out, (g * (1.0 / counts)[:, None])[i].to(dtype))
        assert torch.all(buf[shift + n * F:] == 7.0) and torch.all(buf[:shift] == 7.0)
    rows = torch.from_numpy(rng.integers(0, n, (S, F)).astype(np.int32)).to(DEV)   # a recipient somewhere, or none
    arg = torch.where(torch.from_numpy(rng.random((S, F)) < 0.2).to(DEV), -1, rows)
    want = torch.where(arg[i] == torch.arange(n, device=DEV)[:, None], g[i], 0.0).to(dtype)
    assert torch.equal(geot.segment_reduce_backward_max_arg(g.contiguous(), i, arg, dtype), want)
    wrong = i.clone()
    wrong[0], wrong[-1] = -1, S + 3                        # out of range: zero rows
    geot.segment_reduce_backward(g, wrong, "sum", grad_src=out)
    assert torch.all(out[0] == 0) and torch.all(out[-1] == 0) and torch.equal(out[1:-1], g[i[1:-1]].to(dtype))


@pytest.mark.parametrize("F", [31, 32, 47, 48, 100])
@pytest.mark.parametrize("S", [60, 300])
def test_mean_of_short_and_long_segments(F, S):
    """The mean's two load orders (segments of 34 and of 7 rows, from 32 columns on), with ids out of range."""
    rng = np.random.default_rng(F + S)
    i = torch.from_numpy(np.sort(rng.integers(0, S, 2053))).to(DEV)
    i[0], i[-1] = -1, S + 3
    g = torch.randn(S, F, device=DEV)
    counts = torch.bincount(i[1:-1], minlength=S).clamp_(min=1).float()
    say(f"mean of segments F={F} S={S}")
    got = geot.segment_reduce_backward(g, i, "mean")
    assert torch.equal(got[1:-1], (g * (1.0 / counts)[:, None])[i[1:-1]])
    assert torch.all(got[0] == 0) and torch.all(got[-1] == 0)


def test_gradient_rows_beyond_the_cache():
    """More than 200 MB of gradient rows (with their recipients) in segments of a block's rows and more, which take
    the segments from the offsets: copies, so exact."""
    n, S, F = 1_700_000, 104_000, 256
    g = torch.Generator(device=DEV).manual_seed(1)
    i = torch.sort(torch.randint(0, S, (n,), device=DEV, generator=g)).values
    go = torch.randn(S, F, device=DEV, generator=g)
    arg = torch.randint(0, n, (S, F), device=DEV, generator=g, dtype=torch.int32)
    arg[i[::3]] = torch.arange(0, n, 3, device=DEV, dtype=torch.int32)[:, None]     # some recipients
    say("gradient rows beyond the cache")
    for idx in (i, i.int()):
        got = geot.segment_reduce_backward_max_arg(go, idx, arg, torch.float32)
        assert torch.equal(got, torch.where(arg[i] == torch.arange(n, device=DEV)[:, None], go[i], 0.0))
    del got
    big = torch.randn(2 * S, F, device=DEV, generator=g)
    j = torch.sort(torch.randint(0, 2 * S, (2 * n,), device=DEV, generator=g)).values
    assert torch.equal(geot.segment_reduce_backward(big, j, "sum"), big[j])


@pytest.mark.parametrize("op", ["sum", "max"])
def test_gradient_rows_beyond_the_cache_captured_first(op):
    """Captured on a stream that no call has run on: the ids' path, which takes no temporary memory."""
    n, S, F = 1_700_000 * (2 if op == "sum" else 1), 104_000 * (2 if op == "sum" else 1), 256
    g = torch.Generator(device=DEV).manual_seed(2)
    i = torch.sort(torch.randint(0, S, (n,), device=DEV, generator=g)).values
    go = torch.randn(S, F, device=DEV, generator=g)
    arg = torch.zeros(S, F, device=DEV, dtype=torch.int32)
    first = torch.searchsorted(i, torch.arange(S, device=DEV))
    arg[:] = first[:, None].int()
    out = torch.empty(n, F, device=DEV)

    def call():
        if op == "sum":
            geot.segment_reduce_backward(go, i, "sum", grad_src=out)
        else:
            out.copy_(geot.segment_reduce_backward_max_arg(go, i, arg, torch.float32))

    say(f"capture without a call before it, {op}")
    torch.cuda.synchronize()
    geot.release_scratch()
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=side):
        call()
    for _ in range(3):
        go.mul_(0.5)
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        want = go[i] if op == "sum" else torch.where((first[i] == torch.arange(n, device=DEV))[:, None], go[i], 0.0)
        assert torch.equal(out, want)
