"""Which kernel choice the gather over a kept graph's transposed list takes (host logic, no GPU): row runs by
the edges, the columns and how the destinations' edge counts spread; a program's own choice first."""
import pytest
import torch

from paper_2404_03019_amd import autograd as ga


def graph(n, num_nodes, heavy):
    g = ga.Graph(torch.zeros(0, dtype=torch.int64), torch.empty(n, dtype=torch.int64, device="meta"), num_nodes)
    g.stats = lambda: dict(mean_len=4.0, var_len=(33.0 if heavy else 31.0) ** 2)
    return g


FEW, MANY = 6_000, 600_000     # destinations: rows that fit the caches, and rows that do not


@pytest.mark.parametrize("n,F,nodes,heavy,rows", [
    ((1 << 20) - 1, 128, FEW, True, None), (1 << 20, 128, FEW, False, 128), (1 << 20, 64, FEW, False, 128),
    (1 << 20, 32, FEW, True, 64), (1 << 20, 128, MANY, False, 16), (1 << 20, 200, MANY, False, None),
    (1 << 20, 64, MANY, True, 128), (1 << 21, 64, MANY, True, 128), (1 << 25, 128, MANY, True, 256),
    (1 << 25, 128, MANY, False, 16), (1 << 25, 128, FEW, True, 128), (1 << 22, 16, MANY, True, 8),
    (1 << 18, 16, MANY, True, None), (1 << 22, 8, MANY, True, None), (1 << 20, 300, FEW, False, 128)])
def test_row_runs(n, F, nodes, heavy, rows):
    want = None if rows is None else dict(family="ep", rows=rows)
    assert graph(n, nodes, heavy).transposed_choice(F) == want


def test_a_programs_own_choice_comes_first():
    g = graph(1 << 25, MANY, False)
    assert g.gather_choice is None and ga.Graph.TRANSPOSED_GATHER == dict(family="ep", rows=256)
    g.gather_choice = dict(family="ep", rows=64)
    assert g.transposed_choice(128) == dict(family="ep", rows=64)
