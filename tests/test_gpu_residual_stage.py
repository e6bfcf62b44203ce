"""Residuals of sweeps with one, a few thousand and tens of thousands of per-block
partials, around the edges of the reduction's stages: the norm of the change, and
one launch for the reduction up to 8,192 partials."""
import pytest

from tests.graph_nodes import nodes_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blocks,launches", [(1, 2), (2047, 2), (2048, 2), (2049, 2), (5000, 2), (8192, 2), (8193, 3),
                                             (20000, 3)])
def test_residual(blocks, launches):
    """One hyperedge holds two nodes and the other nodes none, so a sweep of d = 8 in FP32 has a block per 128 rows of
    each side (2 lanes a row): `blocks` less one of node rows."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2103_09660_amd as H
    print("residual", blocks, flush=True)
    nodes = max(2, 128 * (blocks - 1))
    dev = torch.device("cuda")
    lv = H.DeviceLevel(nodes, 1, 2, torch.tensor([0, 2], dtype=torch.int32, device=dev),
                       torch.tensor([0, 1], dtype=torch.int32, device=dev))
    plan = H.Plan.from_device([lv], [], 8, "f32")
    z = torch.randn(nodes + 1, 8, device=dev, generator=torch.Generator(dev).manual_seed(blocks))
    z *= 1000.0                                # (only three rows change)
    out, res = torch.empty_like(z), torch.zeros(1, dtype=torch.float64, device=dev)
    plan.sweep(0, z, 0.5, out=out, resid=res)
    want = (out.double() - z.double()).norm().item()
    # FP64 sums of exact squares of at most 24 terms and zeros
    assert abs(res.item() - want) <= 1e-13 * want
    assert nodes_of(lambda: plan.sweep(0, z, 0.5, out=out, resid=res)) == launches
