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
