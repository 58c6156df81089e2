"""bf16 and fp16 rows of widths that no vector divides, which move in 8-, 4- and 2-element vectors
whose last one overlaps its neighbour, at any 2-byte aligned address; and the choices made for small and
large X. Against the oracle on the exactly widened values."""
import numpy as np
import pytest
import torch

import paper_2404_03019_amd as geot
from gpu_util import compare, oracle_gather, oracle_segment, say
from workloads import random_gather_problem, random_problem

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def stored(a, dtype, shift):
    """`a` on the GPU in 16 bits, `shift` elements past an aligned address, and its exact values."""
    flat = torch.zeros(a.size + shift, dtype=dtype, device=DEV)
    t = flat[shift:].view(a.shape)
    t.copy_(torch.from_numpy(a))
    return t, t.float().cpu().numpy()


@pytest.mark.parametrize("F", [1, 2, 3, 5, 7, 9, 15, 47, 100, 255, 259, 520])
@pytest.mark.parametrize("dtype,shift", [(torch.bfloat16, 0), (torch.float16, 0), (torch.float16, 1), (torch.bfloat16, 3)])
def test_segment_rows(dtype, shift, F):
    p = random_problem(F + 1, 5003, 400, F, "zipf", "normal", 0.1)
    s, wide = stored(p["src"], dtype, shift)
    i = torch.from_numpy(p["index"]).to(DEV)
    say(f"segment {dtype} F={F} shift={shift}")
    for op in ("sum", "mean", "max"):
        ref, terms = oracle_segment(wide, p["index"], 400, op)
        for idx in (i, i.int()):
            compare(geot.segment_reduce(s, idx, 400, op).cpu().numpy(), ref, op, terms, f"F={F} {op}")
        out, arg = geot.segment_reduce_max_arg(s, i, 400) if op == "max" else (None, None)
        if out is not None:
            compare(out.cpu().numpy(), ref, "max", what="max with recipients")
            a = arg.cpu().numpy().view(np.uint32).astype(np.int64)
            ok = a != 0xFFFFFFFF
            assert np.array_equal(wide[a[ok], np.nonzero(ok)[1]], ref[ok])


@pytest.mark.parametrize("F", [3, 7, 15, 47, 100, 259])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_gather_rows(dtype, F):
    g = random_gather_problem(F, 6007, 500, 700, F, "lognormal", "normal", True, 0.05)
    x, wide = stored(g["X"], dtype, 1)
    col, w, row = (torch.from_numpy(g[k]).to(DEV) for k in ("col", "weight", "index"))
    say(f"gather {dtype} F={F}")
    for op in ("sum", "mean", "max"):
        ref, terms = oracle_gather(wide, g["col"], g["weight"], g["index"], 500, op)
        got = geot.gather_scatter(x, col.int(), w, row.int(), 500, op)
        compare(got.cpu().numpy(), ref, op, terms, f"F={F} {op}")


@pytest.mark.parametrize("nnz,F,x_rows", [(40_000, 64, 3000), (40_000, 100, 3000), (300_000, 128, 140_000)])
def test_column_tiles_by_the_size_of_x(nnz, F, x_rows):
    """Whole rows and column tiles in sequence agree with the oracle where the rule chooses between them,
    and the workspace that the size query names is enough for either."""
    g = random_gather_problem(nnz, nnz, nnz // 20, x_rows, F, "poisson", "normal", True, 0.0)
    x, col, w, row = (torch.from_numpy(g[k]).to(DEV) for k in ("X", "col", "weight", "index"))
    R = nnz // 20
    say(f"tiles nnz={nnz} F={F} X rows={x_rows}")
    ref, terms = oracle_gather(g["X"], g["col"], g["weight"], g["index"], R, "sum")
    compare(geot.gather_scatter(x, col, w, row, R).cpu().numpy(), ref, "sum", terms, "pooled")
    ws = torch.empty(geot.workspace_size(nnz, R, F, "sum", gather=True), dtype=torch.uint8, device=DEV)
    compare(geot.gather_scatter_ws(x, col, w, row, R, "sum", ws).cpu().numpy(), ref, "sum", terms, "workspace")
    big = torch.zeros(200_000, F, device=DEV)
    big[:x_rows] = x
    compare(geot.gather_scatter_ws(big, col, w, row, R, "sum", ws).cpu().numpy(), ref, "sum", terms, "large X")


@pytest.mark.parametrize("nnz,F,x_rows,tiled", [(1_200_000, 128, 32_000, True), (600_000, 256, 50_000, True),
                                                (900_000, 160, 50_000, True), (1_200_000, 128, 7_000, False),
                                                (300_000, 128, 100_000, False), (900_000, 100, 100_000, False)])
def test_column_tiles_kept_where_their_slab_fits(nnz, F, x_rows, tiled):
    """X of 16 to 51 MB in tiles whose slabs the L2s hold keeps them; an X that fits one L2, few elements and
    tiles of idle lanes take whole rows. Same sums."""
    g = torch.Generator(device=DEV).manual_seed(nnz)
    R = nnz // 60
    row = torch.sort(torch.randint(0, R, (nnz,), device=DEV, generator=g)).values
    col = torch.randint(0, x_rows, (nnz,), device=DEV, generator=g)
    x = torch.randint(-4, 5, (x_rows, F), device=DEV, generator=g).float()   # integers: exact sums
    w = torch.randint(1, 3, (nnz,), device=DEV, generator=g).float()
    say(f"tiles kept nnz={nnz} F={F} X rows={x_rows}")
    got = geot.gather_scatter(x, col, w, row, R)
    used = geot.last_choice()["flags"] & 4
    assert torch.equal(got, torch.zeros(R, F, device=DEV).index_add_(0, row, x[col] * w[:, None]))
    assert bool(used) == tiled, geot.last_choice()
    plain = geot.last_choice()
    assert plain == geot.select(nnz, R, F, gather=True, x_rows=x_rows)     # what geot_select_gather says
    with_stats = geot.gather_scatter(x, col, w, row, R, stats=geot.index_stats(row, R))
    assert torch.equal(got, with_stats)
    assert tiled or not geot.last_choice()["flags"] & 4


@pytest.mark.parametrize("F,n,mean,rows", [(48, 900_000, 300, 48), (48, 900_000, 9, 32), (64, 900_000, 9, 16),
                                           (96, 700_000, 300, 64), (128, 300_000, 300, 32), (48, 60_000, 300, 16)])
def test_row_runs_follow_segment_length_and_grid(F, n, mean, rows):
    """Long segments take long row runs where the grid stays full; at most `rows` otherwise. Same sums."""
    p = random_problem(F + mean, n, n // mean, F, "poisson", "normal", 0.0)
    s, wide = stored(p["src"], torch.bfloat16, 0)
    i = torch.from_numpy(p["index"]).to(DEV)
    say(f"row runs F={F} n={n} mean={mean}")
    ref, terms = oracle_segment(wide, p["index"], n // mean, "sum")
    compare(geot.segment_reduce(s, i, n // mean, "sum").cpu().numpy(), ref, "sum", terms, f"F={F}")
    got = geot.last_choice()["rows"]
    assert got <= rows and (rows < 32 or got >= 32), got


@pytest.mark.parametrize("F,n,rows", [(64, 1_000_000, 16), (128, 1_000_000, 32), (256, 400_000, 32), (128, 60_000, 16)])
def test_row_runs_of_gathers(F, n, rows):
    """Gathers of more than 64 columns whose grid stays full keep runs of 32 edges or more."""
    g = torch.Generator(device=DEV).manual_seed(n)
    S, nx = n // 100, n // 8
    row = torch.sort(torch.randint(0, S, (n,), device=DEV, generator=g)).values
    col = torch.randint(0, nx, (n,), device=DEV, generator=g)
    x = torch.randint(-4, 5, (nx, F), device=DEV, generator=g).to(torch.bfloat16)   # integers: exact sums
    say(f"gather row runs F={F} n={n}")
    got = geot.gather_scatter(x, col, None, row, S)
    used = geot.last_choice()["rows"]
    assert torch.equal(got, torch.zeros(S, F, device=DEV).index_add_(0, row, x.float()[col]))
    assert used >= 32 if rows >= 32 else used <= rows, used
