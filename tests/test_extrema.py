"""Largest and smallest load and utilisation of the links, at the sizes where one workgroup finds them, where several do and
where a thread takes many: ties go to the lowest link.  Against numpy.  (Needs an MI355X.)"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nodes,degree", [
    (2, 1), (33, 2), (1024, 8), (1025, 8),           # nodes: one workgroup for the utilisations, and more
    (8192, 4), (8193, 4), (7000, 5), (4099, 8),      # links: 32768 by one workgroup, and a node more; ragged
    (70000, 4), (70001, 9)])                         # more than four links a thread, more than one node
@pytest.mark.parametrize("ties", [False, True])
def test_extrema_match_numpy(nodes, degree, ties):
    import torch
    import paper_2309_13541_amd as a2a
    print(nodes, degree, flush=True)
    offsets = np.maximum(1, np.round(nodes ** (np.arange(degree) / degree))).astype(np.int64)  # few levels
    col = ((np.arange(nodes)[:, None] + offsets) % nodes).astype(np.int32).reshape(-1)
    topo = a2a.Topology((np.arange(nodes + 1) * degree).astype(np.int32), col)
    rng = np.random.default_rng(nodes + degree)
    load = rng.integers(1, 4, topo.E).astype(np.float64) if ties else rng.random(topo.E) + 0.25
    cap = rng.choice([0.5, 1.0, 2.0], topo.E)
    on_gpu = torch.from_numpy(load).cuda()
    bound, _ = topo.schedule_bound(on_gpu, 1, 0)
    assert bound.max_load == load.max() and bound.min_load == load.min() and bound.argmax_arc == int(load.argmax())
    util = load / cap
    bound, _ = topo.schedule_bound_cap(on_gpu, torch.from_numpy(cap).cuda(), 1, 0)
    assert bound.max_util == util.max() and bound.min_util == util.min() and bound.argmax_arc == int(util.argmax())
    assert bound.total_capacity == cap.sum()  # halves: exact in any order
    assert bound.max_node_capacity == cap.reshape(nodes, degree).sum(axis=1).max()
    topo.close()
