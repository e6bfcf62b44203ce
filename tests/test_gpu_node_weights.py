"""Node weight sums over lists of every length class (a few lanes, a wavefront, a
workgroup), at their edges, with node ids in order and a grid apart.  Whole
weights below 8 over rows of ones: the FP32 sums of a sweep are whole numbers
below 2^24, so exact, and with omega = 1 a node's new value is S_v * fl(1 / S_v):
1 within half a unit of the reciprocal and half of the product, 2^-23."""
import numpy as np
import pytest

from synth.hypergraph import Hypergraph

pytestmark = pytest.mark.gpu

DEGREES = [1, 2, 3, 4, 5, 8, 9, 63, 64, 65, 66, 2047, 2048, 2049, 5000]


@pytest.mark.parametrize("extra_nodes", [0, 3000])
def test_weighted_means_of_ones(extra_nodes):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2103_09660_amd as H
    print("node weights", extra_nodes, flush=True)
    rng = np.random.default_rng(6)
    n_e = max(DEGREES)
    degrees = DEGREES + [int(x) for x in rng.integers(1, 130, 200)] + [0] * extra_nodes   # (0: the value stays)
    members = [[] for _ in range(n_e)]
    for v, k in enumerate(degrees):
        for e in rng.choice(n_e, size=k, replace=False):
            members[e].append(v)
    ptr = np.concatenate([[0], np.cumsum([len(m) for m in members])]).astype(np.int64)
    w = rng.integers(1, 8, n_e).astype(np.float32)
    hg = Hypergraph(len(degrees), n_e, ptr, np.concatenate(members).astype(np.int32), w)
    hier = H.Hierarchy.build(hg.n_nodes, hg.n_edges, hg.edge_ptr, hg.edge_idx, hg.edge_w, 0)
    plan = H.Plan(hier, 8, "f32")
    z = torch.ones(plan.rows(0), 8, device="cuda")
    for new in (None, torch.as_tensor(rng.integers(1, 8, n_e).astype(np.float32)).cuda()):
        if new is not None:
            plan.set_edge_weights(0, new)
        out = plan.sweep(0, z, 1.0)
        assert (out - 1.0).abs().max().item() <= 2.0 ** -23
