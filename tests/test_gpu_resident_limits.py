"""Which refinements run their sweeps from LDS, seen by the number of launches that a call records: levels at the
most LDS bytes and one node past them, unit and given weights (which need more), both orders; weights set after the
plan was built, where a level of unit weights grows the weights' arrays.  The results equal the sweeps one at a time
bit for bit on either side."""
import numpy as np
import pytest

from tests.graph_nodes import nodes_of
from tests.test_gpu_resident import _check, _hypergraph, _sizes

pytestmark = pytest.mark.gpu

LDS = 160 * 1024


@pytest.fixture(scope="module")
def H():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2103_09660_amd as H
    return H


def _lds_bytes(nodes, edges, nnz, order, weighted):
    """Rows (hyperedge rows twice in the Jacobi order), 16-bit lists that start at multiples of 4, weights of the node
    lists, 8 bytes per item, 4 per factor, 8: each from a multiple of 16."""
    parts = [4 * nodes, 4 * edges] + [4 * edges] * (order == "jacobi")
    parts += [2 * (nnz + 3 * edges), 2 * (nnz + 3 * nodes)] + [4 * (nnz + 3 * nodes)] * weighted
    parts += [8 * (nodes + edges), 4 * (nodes + edges), 8]
    return sum((p + 15) // 16 * 16 for p in parts)


def _launches(plan, sweeps):
    import torch
    z = torch.zeros(plan.rows(plan.n_levels - 1), plan.d, dtype=plan.torch_dtype, device="cuda")
    return nodes_of(lambda: plan.refine(z, sweeps, 0.6))


@pytest.mark.parametrize("order", ["jacobi", "edge_first"])
@pytest.mark.parametrize("weighted", [False, True])
def test_at_the_limit(H, order, weighted):
    def total(n):
        return _lds_bytes(n, 1, 4, order, weighted)
    most = max(n for n in range(1000, 9000) if total(n) <= LDS)
    assert LDS - total(most) < 64 < total(most + 8) - LDS + 64
    for n in (most - 8, most - 1, most, most + 1, most + 8):
        print("resident limit", order, weighted, n, total(n), flush=True)
        hg = _hypergraph(n, n, [4], weighted)
        plan = H.Plan(H.Hierarchy.build(hg.n_nodes, hg.n_edges, hg.edge_ptr, hg.edge_idx, hg.edge_w, 0), 16, "f32",
                      options={"order": order})
        fits = total(n) <= LDS
        assert _launches(plan, [8]) == (1 if fits else 8 if order == "jacobi" else 16), n
        _check(H, plan, [8], f"{n} nodes")


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("order", ["jacobi", "edge_first"])
@pytest.mark.parametrize("dtype,d", [("f32", 32), ("f32", 40), ("bf16", 128)])
def test_weights_set_on_the_plan(H, dtype, d, order, weighted):
    import torch
    print("resident weights", dtype, d, order, weighted, flush=True)
    hg = _hypergraph(11, 1500, _sizes(12, 700), weighted)
    plan = H.Plan(H.Hierarchy.build(hg.n_nodes, hg.n_edges, hg.edge_ptr, hg.edge_idx, hg.edge_w, 2), d, dtype,
                  options={"order": order})
    g = torch.Generator("cuda").manual_seed(5)
    for what in ("as built", "one level's weights set", "all levels' weights set"):
        if what != "as built":
            for l in range(1 if what.startswith("one") else plan.n_levels):
                plan.set_edge_weights(l, torch.rand(plan.level_info(l)[1], device="cuda", generator=g) + 0.5)
        assert _launches(plan, [17, 16, 40]) == 3, what
        _check(H, plan, [17, 16, 40], what)
