"""Workspace sizes do not fall when an argument grows, so that a workspace
queried for the largest call of a program serves all of its calls, whichever
way a size is computed."""
import itertools

import pytest

from paper_2512_00385_amd import ezsp

NS = [1, 2, 500, 100_000, 131_072, 131_073, 1_000_000, 3_000_000, 40_000_000]
QUERIES = {
    "ezsp_purity_workspace_size":
        (NS, [1, 2, 9000, 131_073, 1_048_576, 1_048_577, 9_000_000],
         [1, 2, 8, 63, 64, 65, 541, 2048, 2049, 100_000]),
    "ezsp_component_stats_workspace_size":
        (NS, [1, 2, 9000, 1_048_577, 9_000_000], [1, 3, 4, 16, 64]),
    "ezsp_edge_loss_workspace_size":
        (NS[:-1], [1, 7, 8, 15, 16, 31, 32, 64]),
    "ezsp_knn_workspace_size":
        (NS + [1 << 16, (1 << 16) + 1, 1 << 19, (1 << 19) + 1, 1 << 21,
               (1 << 21) + 1, 1 << 25, (1 << 25) + 1], [1, 4, 10, 24, 32]),
    "ezsp_grid_subsample_workspace_size": (NS,),
}


@pytest.mark.parametrize("name", QUERIES)
def test_sizes_grow(name):
    query = getattr(ezsp.load(), name)
    axes = [sorted(a) for a in QUERIES[name]]
    for at in itertools.product(*(range(len(a)) for a in axes)):
        here = query(*(a[i] for a, i in zip(axes, at)))
        assert here > 0
        for j, i in enumerate(at):
            if i + 1 < len(axes[j]):
                more = list(at)
                more[j] += 1
                assert query(*(a[m] for a, m in zip(axes, more))) >= here, \
                    (name, [a[m] for a, m in zip(axes, at)], j)
