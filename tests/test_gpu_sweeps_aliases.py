"""Buffers that several sweeps in one call must not share: a kept result with the input or with another kept result,
near or far; a cotangent with a state that a later reverse sweep reads.  What no later sweep reads may be shared."""
import ctypes

import pytest

from tests.cases import random_hypergraph

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def plan():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2103_09660_amd as H
    hg = random_hypergraph(4, 300, 200, 1, 9)
    return H.Plan(H.Hierarchy.build(hg.n_nodes, hg.n_edges, hg.edge_ptr, hg.edge_idx, hg.edge_w, 0), 16, "f32")


def _array(tensors):
    return (ctypes.c_void_p * len(tensors))(*(None if t is None else t.data_ptr() for t in tensors))


def _status(name, *args):
    from paper_2103_09660_amd import _lib as L
    try:
        L.call(name, *args)
    except L.HnvError as e:
        return e.status
    return 0


def test_kept_results(plan):
    import torch
    from paper_2103_09660_amd._lib import HNV_EINVAL
    z, a, b, c = (torch.zeros(plan.rows(0), 16, device="cuda") for _ in range(4))
    s = torch.cuda.current_stream().cuda_stream

    def sweeps(outs):
        return _status("hnv_sweeps", plan._h, 0, z.data_ptr(), _array(outs), len(outs), 0.5, 0, s)

    for outs in ([a, b, a], [a, b, c, a], [a, None, None, a], [a, a], [a, z], [z, a], [None, z], [a, b, c, None, b]):
        assert sweeps(outs) == HNV_EINVAL, len(outs)
    for outs in ([a, b, c], [None, None, a], [a, None, b]):
        assert sweeps(outs) == 0
    torch.cuda.synchronize()


def test_cotangents_and_states(plan):
    import torch
    from paper_2103_09660_amd._lib import HNV_EINVAL
    rows = plan.rows(0)
    n_v, n_e, _ = plan.level_info(0)
    top = torch.randn(rows, 16, device="cuda")
    z = torch.randn(rows, 16, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    dw, acc = torch.zeros(n_e, device="cuda"), torch.zeros(n_v, device="cuda")
    a, b = (torch.empty(rows, 16, device="cuda") for _ in range(2))
    states = [z] + plan.sweeps(0, z, [True] * 3, 0.5)

    def adjoint(outs, grad=True):
        return _status("hnv_sweeps_adjoint", plan._h, 0, top.data_ptr(), _array(outs), _array(states), 3,
                       dw.data_ptr() if grad else None, acc.data_ptr() if grad else None, 0.5, s)

    for outs in ([states[0], a, b], [states[1], a, b], [states[2], a, b], [a, states[0], b], [a, states[1], b]):
        assert adjoint(outs) == HNV_EINVAL
    want = plan.sweeps_adjoint(0, top, states, 0.5, dw=dw, node_acc=acc)
    want_dw, want_acc = dw.clone(), acc.clone()
    # the last state is read by the first reverse sweep only, and no state by none after the last one
    for outs in ([a, b, a], [a, states[3], b], [a, b, states[0]]):
        keep = [t.clone() for t in states]
        dw.zero_(), acc.zero_()
        assert adjoint(outs) == 0
        assert torch.equal(outs[2], want) and torch.equal(dw, want_dw) and torch.equal(acc, want_acc)
        for t, k in zip(states, keep):
            t.copy_(k)
    assert adjoint([states[0], a, b], grad=False) == 0      # (no state is read without a weight gradient)
    assert torch.equal(b, want)
