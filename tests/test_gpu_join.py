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


@pytest.mark.parametrize("F", [1, 4])
def test_join_by_the_block(F):
    """A segment over 1,500 blocks of 4 rows, more than a wave's turns reach over at rows of one vector
    (1,024 partials): the thread block's walk, with 512 groups."""
    rng = np.random.default_rng(F)
    S = 900
    n = rng.integers(0, 9, S)
    n[S // 2] = 6000
    index = np.repeat(np.arange(S), n).astype(np.int64)
    assert index.size <= S * 16 and index.size // 4 > 1024     # few enough rows a segment for the join
    src = rng.integers(-6, 7, (index.size, F)).astype(np.float32)
    s, i = torch.from_numpy(src).to(DEV), torch.from_numpy(index).to(DEV)
    choice = dict(family="ep", rows=1, lanes=64)
    say(f"join by the block F={F}")
    for op in ("sum", "mean", "max"):
        ref, terms = oracle_segment(src, index, S, op)
        compare(geot.segment_reduce(s, i, S, op, choice=choice).cpu().numpy(), ref, op, terms, op)
    out, arg = geot.segment_reduce_max_arg(s, i, S, choice=choice)
    ref = oracle.segment_reduce(src, index, S, "max")
    compare(out.cpu().numpy(), ref, "max", what="max with recipients")
    want = np.full((S, F), NONE, dtype=np.uint64)
    np.minimum.at(want, index, np.where(src == ref[index], np.arange(index.size, dtype=np.uint64)[:, None], np.uint64(NONE)))
    assert np.array_equal(arg.cpu().numpy().view(np.uint32), want.astype(np.uint32))


def test_join_sums_in_short_chains():
    """2,400 partials of 1 + 2^-16 in one segment, 300 for each of the block's 8 groups: in one chain every
    term past the 256th would lose its 2^-16 (2e-6 of the sum). Sums of 16 and sums of those are exact; what
    remains are the last three roundings, of 2^-24 each."""
    S, F, blocks = 700, 260, 2400
    index = torch.full((4 * blocks,), 5, device=DEV)
    src = torch.full((4 * blocks, F), 0.25 * (1 + 2.0 ** -16), device=DEV)
    assert 4 * blocks <= S * 16 and blocks * F * 4 <= 5 << 19
    say("join, short chains")
    out = geot.segment_reduce(src, index, S, "sum", choice=dict(family="ep", rows=1, lanes=64))
    want = blocks * (1 + 2.0 ** -16)
    assert float((out[5].double() - want).abs().max()) <= 3 * 2.0 ** -24 * want
    assert int((out != 0).any(1).sum()) == 1
