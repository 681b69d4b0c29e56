"""Each kernel and each branch of a dispatch at the sizes where it can go
wrong (edges of tiles and groups, remainders, the smallest and the largest of
its range), against the oracle, bit for bit."""

import pytest

from paper_1905_11722_amd import workloads as W

from tests.test_gpu_parity import compare

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_11722_amd import rcdp
    rcdp.load_library()
    return rcdp


@pytest.mark.parametrize("nodes", [1, 2, 63, 64, 65, 128, 255, 256, 257, 300])
def test_optarg_table_list_lengths(rc, oracle_mod, nodes):
    """Whole-table optarg with predecessor lists up to and over one group of
    64 pairs and one round of four groups, rows up to and over 64 cells."""
    g = W.chain(nodes, seed=nodes, tmax=2, mmax=9)
    compare(rc, oracle_mod, g, "pruned", (3 * sum(g.M)) // 2, objectives=("tc",))


def test_optarg_table_long_rows_short_lists(rc, oracle_mod):
    """Rows of many cells with few predecessors: one thread per cell."""
    g = W.chain(5, seed=3, tmax=400000, mmax=9)
    fam = rc.Graph.create(g).build_family("pruned")
    assert fam.info["table_cells"] > 1 << 20 and fam.info["num_pairs"] < 64 * fam.info["num_sets"]
    compare(rc, oracle_mod, g, "pruned", (3 * sum(g.M)) // 2, objectives=("tc",))
