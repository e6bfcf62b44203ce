"""Refinements of small levels, whose sweeps run many to a launch from LDS,
against the sweeps one at a time: the same sums in the same order, so the
embeddings and the residuals must be identical bit for bit.  Widths of 4, 8 and
16 lanes and one that is no power of two; both orders; unit and given weights;
rows on both tiers (a wavefront's, a workgroup's with one hub); nodes without
hyperedges; sweep counts that take one launch and several; a level at the most
LDS that such a launch takes and one just past it."""
import numpy as np
import pytest

from synth.hypergraph import Hypergraph

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2103_09660_amd as H
    return H


def _hypergraph(seed, n_nodes, sizes, weighted):
    rng = np.random.default_rng(seed)
    edges = [np.sort(rng.choice(n_nodes - 7, size=k, replace=False)) for k in sizes]   # the last 7 nodes have none
    if len(edges) > 300:
        edges[:300] = [np.unique(np.concatenate([[3], e])) for e in edges[:300]]        # a hub node
    ptr = np.concatenate([[0], np.cumsum([len(e) for e in edges])]).astype(np.int64)
    w = rng.uniform(0.1, 3.0, len(edges)).astype(np.float32) if weighted else None
    return Hypergraph(n_nodes, len(edges), ptr, np.concatenate(edges).astype(np.int32), w)


def _sizes(seed, n):
    rng = np.random.default_rng(seed)
    return [700, 300, 257, 256, 64, 65, 17, 16, 15] + list(rng.integers(1, 7, n))


def _check(H, plan, sweeps, what, seed=3):
    import torch
    g = torch.Generator().manual_seed(seed)
    zc = torch.randn(plan.rows(plan.n_levels - 1), plan.d, generator=g).to(plan.torch_dtype).cuda()
    z, res = zc, []
    top = plan.n_levels - 1
    for l in range(top, -1, -1):
        if sweeps[l] == 0 and l < top:
            z = plan.project(l, z)
        for k in range(sweeps[l]):
            r = torch.zeros(1, dtype=torch.float64, device="cuda")
            z = plan.sweep(l, z, 0.6, from_coarse=(k == 0 and l < top), resid=r)
            res.append(r.item())
    out, got, _ = plan.refine(zc, sweeps, 0.6, residuals=True)
    assert torch.equal(out, z), what
    assert got.cpu().tolist() == res, what
    assert torch.equal(plan.refine(zc, sweeps, 0.6)[0], z), what + " without residuals"


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("order", ["jacobi", "edge_first"])
@pytest.mark.parametrize("dtype,d", [("f32", 16), ("f32", 32), ("f32", 64), ("f32", 40), ("bf16", 32), ("bf16", 128),
                                     ("bf16", 104)])
def test_refine_equals_sweeps(H, dtype, d, order, weighted):
    import torch
    print("resident", dtype, d, order, weighted, flush=True)
    hg = _hypergraph(11, 1500, _sizes(12, 700), weighted)
    hier = H.Hierarchy.build(hg.n_nodes, hg.n_edges, hg.edge_ptr, hg.edge_idx, hg.edge_w, 2)
    plan = H.Plan(hier, d, dtype, options={"order": order})
    for sweeps in ([2, 2, 2], [1, 0, 5], [17, 16, 40]):
        _check(H, plan, sweeps, f"{sweeps}")
    # weights set on the plan afterwards
    n_e = plan.level_info(0)[1]
    plan.set_edge_weights(0, torch.rand(n_e, device="cuda") + 0.5)
    _check(H, plan, [3, 2, 0], "new weights")


@pytest.mark.parametrize("order,per_node", [("jacobi", 28), ("edge_first", 28)])
def test_at_the_lds_limit(H, order, per_node):
    """One hyperedge of 4 members over nodes of 16 + 12 bytes each: 28 n plus the
    hyperedge's few words is at the limit of 163,840 bytes around n = 5,849."""
    print("resident limit", order, flush=True)
    for n in (5820, 5843, 5846, 5847, 5848, 5849, 5850, 5851, 5900):
        hg = _hypergraph(n, n, [4], False)
        hier = H.Hierarchy.build(hg.n_nodes, hg.n_edges, hg.edge_ptr, hg.edge_idx, hg.edge_w, 0)
        _check(H, H.Plan(hier, 16, "f32", options={"order": order}), [4], f"{n} nodes")
