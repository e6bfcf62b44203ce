"""Plan.sweeps and Plan.sweeps_adjoint, several sweeps of a level in one call,
against the same number of calls of one sweep: identical bit for bit, for
results kept and not kept, runs of one sweep and of several, small and larger
levels, and the first sweep from the coarser level; and against Plan.sweep and
Plan.sweep_adjoint, whose rows of more than a few neighbours are added in another
order: one rounding of the storage type per sweep and column apart at most, in
the norm (2^-23 or 2^-8 per sweep, seven sweeps; reverse in FP32)."""
import numpy as np
import pytest

from tests.cases import random_hypergraph

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2103_09660_amd as H
    return H


@pytest.mark.parametrize("nodes,edges", [(900, 500), (20000, 9000)])
@pytest.mark.parametrize("dtype,order", [("f32", "jacobi"), ("bf16", "jacobi"), ("f32", "edge_first")])
def test_sweeps_equal_single_calls(H, dtype, order, nodes, edges):
    import torch
    print("sweeps", dtype, order, nodes, flush=True)
    hg = random_hypergraph(4, nodes, edges, 1, 20, weighted=True)
    hier = H.Hierarchy.build(hg.n_nodes, hg.n_edges, hg.edge_ptr, hg.edge_idx, hg.edge_w, 1)
    plan = H.Plan(hier, 48, dtype, options={"order": order})
    g = torch.Generator().manual_seed(1)
    for from_coarse in (False, True):
        z0 = torch.randn(plan.rows(1 if from_coarse else 0), 48, generator=g).to(plan.torch_dtype).cuda()
        for keep in ([1], [0, 1], [0, 0, 1], [1, 1, 1], [0, 0, 0, 0, 1, 0, 1], [1, 0, 0, 1]):
            want, z, y = [], z0, z0
            for i, k in enumerate(keep):
                z = plan.sweeps(0, z, [1], 0.7, from_coarse=from_coarse and i == 0)[0]
                y = plan.sweep(0, y, 0.7, from_coarse=from_coarse and i == 0)
                if k:
                    want.append(z)
            got = plan.sweeps(0, z0, keep, 0.7, from_coarse=from_coarse)
            assert len(got) == len(want)
            assert all(torch.equal(a, b) for a, b in zip(got, want)), (from_coarse, keep)
            off = (z.double() - y.double()).norm() / y.double().norm()
            assert off.item() <= len(keep) * (2.0 ** -23 if dtype == "f32" else 2.0 ** -8), (from_coarse, keep)
    # reverse, with and without the weight gradient
    states = [torch.randn(plan.rows(0), 48, generator=g).to(plan.torch_dtype).cuda()]
    states += plan.sweeps(0, states[0], [True] * 4, 0.7)
    top = torch.randn(plan.rows(0), 48, generator=g).to(plan.torch_dtype).cuda()
    n_v, n_e, _ = plan.level_info(0)
    for n in (1, 2, 4):
        for grad in (False, True):
            acc = [[torch.zeros(m, device="cuda") if grad else None for m in (n_e, n_v)] for _ in range(2)]
            want = top
            for i in range(n, 0, -1):
                want = plan.sweeps_adjoint(0, want, states[i - 1:i + 1], 0.7, dw=acc[0][0], node_acc=acc[0][1])
            got = plan.sweeps_adjoint(0, top, states[:n + 1], 0.7, dw=acc[1][0], node_acc=acc[1][1])
            assert torch.equal(got, want), (n, grad)
            assert not grad or all(torch.equal(a, b) for a, b in zip(*acc)), n
    from paper_2103_09660_amd._lib import HNV_EINVAL, HnvError
    with pytest.raises(HnvError) as ei:
        plan.sweeps(0, states[0], [True], 1.5)
    assert ei.value.status == HNV_EINVAL
    with pytest.raises(ValueError):
        plan.sweeps(0, states[0], [True, False])
