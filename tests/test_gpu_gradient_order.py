"""The calls that serve gradients (sweeps, and the reverse sweeps) add each row in
an order that the level's tiers don't change: a plan with the default tiers and
one with lane groups of up to 64 neighbours and a wavefront per 512, which lay
their work out differently, give the same bits; rows on every edge of that order
(64, 512, 2,048 neighbours and beyond), against the oracle too; and the default
tiers are not the slower ones."""
import numpy as np
import pytest

from tests.cases import assert_close, both_hierarchies
from tests.test_gpu_long_rows import _hypergraph

pytestmark = pytest.mark.gpu

LENGTHS = [1, 4, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 66, 256, 257, 511, 512, 513, 1024, 1025, 1536, 2047, 2048,
           2049, 2050, 2112, 2113, 2560, 2561, 4097, 5000]
PLAIN = {"small_max": 64, "chunk": 512}


@pytest.fixture(scope="module")
def H():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2103_09660_amd as H
    return H


@pytest.mark.parametrize("n_nodes", [6000, 40000])
@pytest.mark.parametrize("dtype,d", [("f32", 8), ("f32", 16), ("f32", 64), ("f32", 256), ("bf16", 72)])
@pytest.mark.parametrize("order", ["jacobi", "edge_first"])
@pytest.mark.parametrize("build", ["host", "device"])
def test_bits_do_not_depend_on_the_tiers(H, n_nodes, dtype, d, order, build):
    import torch
    print("gradient order", n_nodes, dtype, d, order, build, flush=True)
    hg = _hypergraph(n_nodes, LENGTHS, [n for n in LENGTHS if n > 4], n_nodes + d)
    hier = H.Hierarchy.build(hg.n_nodes, hg.n_edges, hg.edge_ptr, hg.edge_idx, hg.edge_w, 1)
    plans = [H.Plan(hier, d, dtype, options=dict(o, order=order), build=build) for o in ({}, PLAIN)]
    g = torch.Generator().manual_seed(d)
    rows = plans[0].rows(0)

    def rand(n):
        return torch.randn(n, d, generator=g).to(plans[0].torch_dtype).cuda()

    for from_coarse in (False, True):
        z = rand(plans[0].rows(1) if from_coarse else rows)
        a, b = (p.sweeps(0, z, [True] * 3, 0.6, from_coarse=from_coarse) for p in plans)
        assert all(torch.equal(x, y) for x, y in zip(a, b)), f"sweeps, from_coarse {from_coarse}"
    states, top = [rand(rows)] + a, rand(rows)
    for split in (False, True):
        got = []
        for p in plans:
            dw, acc = torch.zeros(hg.n_edges, device="cuda"), torch.zeros(hg.n_nodes, device="cuda")
            got.append([p.sweep_adjoint(0, top, states[0], states[1], 0.6, dw=dw, node_acc=acc if split else None)])
            if split:
                got[-1].append(p.sweeps_adjoint(0, top, states, 0.6, dw=dw, node_acc=acc))
            got[-1] += [dw, acc]
        assert all(torch.equal(x, y) for x, y in zip(*got)), f"reverse, split {split}"


@pytest.mark.parametrize("n_nodes,d", [(6000, 8), (6000, 64), (40000, 32)])
@pytest.mark.parametrize("order", ["jacobi", "edge_first"])
def test_long_rows_against_the_oracle(oracle_mod, H, n_nodes, d, order):
    import torch
    print("gradient order, oracle", n_nodes, d, order, flush=True)
    hg = _hypergraph(n_nodes, LENGTHS, [n for n in LENGTHS if n > 4], n_nodes + d)
    levels, maps, hier = both_hierarchies(oracle_mod, H, hg, 1)
    plan = H.Plan(hier, d, "f32", options={"order": order})
    rng = np.random.default_rng(d)
    z, g = (rng.standard_normal((levels[0].rows, d)).astype(np.float32) for _ in range(2))
    kw = {"order": 0 if order == "jacobi" else 1}
    ref = oracle_mod.sweep(levels[0], z, 0.5, **kw)
    out = plan.sweeps(0, torch.as_tensor(z).cuda(), [True], 0.5)[0]
    assert_close(out.cpu().numpy(), ref, 1e-5, "sweeps")
    dw, acc = torch.zeros(hg.n_edges, device="cuda"), torch.zeros(hg.n_nodes, device="cuda")
    gz = plan.sweeps_adjoint(0, torch.as_tensor(g).cuda(), [torch.as_tensor(z).cuda(), out], 0.5, dw=dw, node_acc=acc)
    plan.weight_grad_finish(0, acc, dw)
    g_ref, w_ref = oracle_mod.sweep_vjp(levels[0], z, g, 0.5, **kw)
    assert_close(gz.cpu().numpy(), g_ref, 1e-4, "sweeps_adjoint")
    # singleton hyperedges of one node: sums of up to 5,000 terms that may cancel
    assert np.linalg.norm(dw.cpu().numpy() - w_ref) <= 1e-4 * np.linalg.norm(w_ref)


def _time(f):
    import torch
    f()
    best = []
    for _ in range(7):
        t0, t1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        t0.record()
        f()
        t1.record()
        t1.synchronize()
        best.append(t0.elapsed_time(t1))
    return sorted(best)[3]


@pytest.mark.parametrize("nodes,edges,mean,power,d", [(8000, 4000, 10, 4.0, 128), (36000, 25000, 12, 1.0, 256),
                                                      (100000, 60000, 10, 1.0, 16)])
def test_default_tiers_are_not_slower(H, nodes, edges, mean, power, d):
    """Hubs (members drawn by a power), wide rows and narrow ones; a third over is the margin for noise (rows done by
    one wavefront of a workgroup took 1.2 to 2.3 times as long)."""
    import torch
    from synth.hypergraph import Hypergraph
    print("gradient order, time", nodes, d, flush=True)
    rng = np.random.default_rng(nodes)
    sizes = np.minimum(rng.zipf(2.0, edges) + mean // 2, nodes // 8)
    lists = [np.unique((nodes * rng.random(k) ** power).astype(np.int32)) for k in sizes]
    ptr = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int64)
    hg = Hypergraph(nodes, edges, ptr, np.concatenate(lists).astype(np.int32), None)
    hier = H.Hierarchy.build(hg.n_nodes, hg.n_edges, hg.edge_ptr, hg.edge_idx, hg.edge_w, 0)
    z, top = (torch.randn(nodes + edges, d, device="cuda") for _ in range(2))
    took = []
    for options in ({}, PLAIN):
        plan = H.Plan(hier, d, "f32", options=options)
        states = [z] + plan.sweeps(0, z, [True] * 20, 0.5)
        dw, acc = torch.zeros(edges, device="cuda"), torch.zeros(nodes, device="cuda")
        took.append((_time(lambda: plan.sweeps(0, z, [False] * 19 + [True], 0.5)),
                     _time(lambda: plan.sweeps_adjoint(0, top, states, 0.5, dw=dw, node_acc=acc))))
    for what, a, b in zip(("forward", "reverse"), *took):
        assert a <= 4 / 3 * b, f"{what}: {a:.3f} ms by the default tiers, {b:.3f} ms by plain ones"
