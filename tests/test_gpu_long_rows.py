"""Rows on the boundaries of the default degree tiers, which depend on the
size of the level: the lane-group bound (8, 16 or 64 neighbours), the items
that a whole workgroup takes, and the split at 2048 neighbours.  Forward and
reverse sweeps against the oracle, the host-built and the device-built plan
bit for bit, and the static-scratch sweep where its residual partials only
fit with a wavefront per item."""
import numpy as np
import pytest

from tests.cases import assert_close, both_hierarchies

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2103_09660_amd as H
    return H


def _hypergraph(n_nodes, sizes, hubs, seed):
    """Hyperedges of the given sizes, and nodes of the given degrees in singleton hyperedges."""
    from synth.hypergraph import Hypergraph
    rng = np.random.default_rng(seed)
    edges = [np.sort(rng.choice(n_nodes - len(hubs), size=s, replace=False)) for s in sizes]
    for k, degree in enumerate(hubs):
        edges += [np.array([n_nodes - len(hubs) + k])] * degree
    ptr = np.concatenate([[0], np.cumsum([len(e) for e in edges])]).astype(np.int64)
    w = rng.uniform(0.5, 2.0, size=len(edges)).astype(np.float32)
    return Hypergraph(n_nodes, len(edges), ptr, np.concatenate(edges).astype(np.int32), w)


LENGTHS = [1, 4, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 255, 256, 257, 258, 1023, 2047, 2048, 2049, 4097]


@pytest.mark.parametrize("n_nodes", [6000, 40000, 120000])
@pytest.mark.parametrize("d", [8, 64])
def test_default_tiers(oracle_mod, H, n_nodes, d):
    import torch
    hg = _hypergraph(n_nodes, LENGTHS, [n for n in LENGTHS if n > 4], n_nodes + d)
    levels, maps, hier = both_hierarchies(oracle_mod, H, hg, 1)
    host, dev = H.Plan(hier, d, "f32"), H.Plan(hier, d, "f32", build="device")
    rng = np.random.default_rng(d)
    z = rng.standard_normal((levels[0].rows, d)).astype(np.float32)
    g = rng.standard_normal((levels[0].rows, d)).astype(np.float32)
    zd, gd = torch.as_tensor(z).cuda(), torch.as_tensor(g).cuda()
    res = [torch.zeros(1, dtype=torch.float64, device="cuda") for _ in range(2)]
    out = [p.sweep(0, zd, 0.5, resid=r) for p, r in zip((host, dev), res)]
    dw = [torch.zeros(hg.n_edges, device="cuda") for _ in range(2)]
    adj = [p.sweep_adjoint(0, gd, zd, out[0], 0.5, dw=w) for p, w in zip((host, dev), dw)]
    for a, b in (out, res, dw, adj):
        assert torch.equal(a, b)
    ref = oracle_mod.sweep(levels[0], z, 0.5)
    assert_close(out[0].cpu().numpy(), ref, 1e-5, f"sweep of {n_nodes} nodes, d {d}")
    assert abs(res[0].item() - np.linalg.norm(ref - z)) <= 1e-5 * np.linalg.norm(ref - z)
    g_ref, w_ref = oracle_mod.sweep_vjp(levels[0], z, g, 0.5)
    assert_close(adj[0].cpu().numpy(), g_ref, 1e-4, f"reverse sweep of {n_nodes} nodes, d {d}")
    # singleton hyperedges of one node: sums of up to 4,097 terms that may cancel
    assert np.linalg.norm(dw[0].cpu().numpy() - w_ref) <= 1e-4 * np.linalg.norm(w_ref)


def test_static_scratch_with_a_wavefront_per_item(H):
    """30,500 hyperedges of 128 members over 10,000 nodes in chunks of 8: 0.98M
    partial slots of 64 bytes and as many items, whose residual partials pass
    the 64 MiB static array with a workgroup per item and fit with a wavefront
    per item: the sweep is accepted there and equals the workspace sweep."""
    import torch
    from paper_2103_09660_amd.api import Hierarchy, HostLevel
    n_nodes, n_edges, size = 10000, 30500, 128
    idx = np.sort((np.arange(n_edges)[:, None] * 37 + np.arange(size)[None, :] * 78) % n_nodes, axis=1)
    lv = HostLevel(n_nodes, n_edges, np.arange(n_edges + 1, dtype=np.int64) * size, idx.astype(np.int32).ravel(), None)
    z = torch.randn(n_nodes + n_edges, 8, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    for build in ("host", "device"):
        plan = H.Plan(Hierarchy([lv], []), 8, "f32", options={"small_max": 4, "chunk": 8}, build=build)
        ra, rb = (torch.zeros(1, dtype=torch.float64, device="cuda") for _ in range(2))
        assert torch.equal(plan.sweep(0, z, 0.5, resid=ra), plan.sweep_noalloc(0, z, 0.5, resid=rb))
        assert torch.equal(ra, rb)
