"""Segments that cross block edges, joined in one launch where the partials are few: segments that
reach into the next block, into a handful (a wave's walk) and into hundreds (the thread block's), with
the lowest row of equal maxima, empty segments, and rows of every vector width. Against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_03019_amd as geot
from gpu_util import compare, oracle_segment, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
NONE = 0xFFFFFFFF


def lengths(kind, S, rng):
    n = rng.integers(0, 9, S)
    if kind == "few":        # up to 12 blocks of 4 rows
        n[::7] = rng.integers(20, 48, n[::7].size)
    elif kind == "hub":      # one over hundreds of blocks, one at each end of the list
        n[S // 2], n[0], n[-1] = 2900, 700, 333
    return n


@pytest.mark.parametrize("F", [1, 2, 3, 4, 47, 64, 260])
@pytest.mark.parametrize("kind", ["next", "few", "hub"])
def test_join(kind, F):
    rng = np.random.default_rng(F)
    S = 900
    n = lengths(kind, S, rng)
    index = np.repeat(np.arange(S), n).astype(np.int64)
    src = rng.integers(-6, 7, (index.size, F)).astype(np.float32)   # exact sums; ties for the maxima
    s, i = torch.from_numpy(src).to(DEV), torch.from_numpy(index).to(DEV)
    for choice in (dict(family="ep", rows=1, lanes=64), dict(family="ep", rows=2), dict(family="ep", rows=3, lanes=4)):
        say(f"join {kind} F={F} {choice}")
        for op in ("sum", "mean", "max"):
            ref, terms = oracle_segment(src, index, S, op)
            compare(geot.segment_reduce(s, i, S, op, choice=choice).cpu().numpy(), ref, op, terms, f"{kind} {op}")
        out, arg = geot.segment_reduce_max_arg(s, i, S, choice=choice)
        ref = oracle.segment_reduce(src, index, S, "max")
        compare(out.cpu().numpy(), ref, "max", what=f"{kind} max with recipients")
        want = np.full((S, F), NONE, dtype=np.uint64)
        np.minimum.at(want, index, np.where(src == ref[index], np.arange(index.size, dtype=np.uint64)[:, None], np.uint64(NONE)))
        assert np.array_equal(arg.cpu().numpy().view(np.uint32), want.astype(np.uint32))


def test_join_special_values():
    """Infinities and NaN in segments that cross blocks: as the definition has them, NaN without a recipient."""
    rng = np.random.default_rng(5)
    S, F = 300, 8
    index = np.repeat(np.arange(S), 9).astype(np.int64)
    src = rng.standard_normal((index.size, F)).astype(np.float32)
    src[rng.random(src.shape) < 0.05] = -np.inf
    src[:90] = -np.inf                                      # maxima equal to the neutral value
    src[500, 2] = src[1200, 5] = np.nan
    src[1300, 1] = np.inf
    s, i = torch.from_numpy(src).to(DEV), torch.from_numpy(index).to(DEV)
    choice = dict(family="ep", rows=1, lanes=64)
    say("join, special values")
    ref = oracle.segment_reduce(src, index, S, "max")
    out, arg = geot.segment_reduce_max_arg(s, i, S, choice=choice)
    compare(out.cpu().numpy(), ref, "max", what="max")
    compare(geot.segment_reduce(s, i, S, "max", choice=choice).cpu().numpy(), ref, "max", what="plain max")
    want = np.full((S, F), NONE, dtype=np.uint64)
    np.minimum.at(want, index, np.where(src == ref[index], np.arange(index.size, dtype=np.uint64)[:, None], np.uint64(NONE)))
    assert np.array_equal(arg.cpu().numpy().view(np.uint32), want.astype(np.uint32))
