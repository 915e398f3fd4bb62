"""Link loads of a source at a time in LDS, where the queue of its nodes and their path counts stay there and where the queue goes through
memory: at the edges of that and of where the positions of the sort lie, and from sources without links.  (Needs an MI355X.)"""
import numpy as np
import pytest

import a2a_inputs as gen

pytestmark = pytest.mark.gpu


def without_links(csr, every):
    """The same, with no links out of every so many nodes."""
    rp, _ = csr
    return gen.remove_arcs(csr, np.concatenate([np.arange(rp[v], rp[v + 1]) for v in range(0, len(rp) - 1, every)]))


CASES = {
    # positions of the sort behind all that stays, then (one node on) between the words and the queue, which they fill
    "4544 nodes, 12 links": lambda: gen.random_regular(4544, 12, 1),
    "4545 nodes, 12 links": lambda: gen.random_regular(4545, 12, 2),
    "8640 nodes, 9 levels": lambda: gen.imase_itoh(8640, 3),
    "8641 nodes, 9 levels": lambda: gen.imase_itoh(8641, 3),
    # most nodes whose path counts stay in the queue's order, and one more
    "11584 nodes": lambda: gen.random_regular(11584, 5, 7),
    "11585 nodes": lambda: gen.random_regular(11585, 5, 8),
    # most nodes whose queue stays, and one more
    "16256 nodes": lambda: gen.random_regular(16256, 5, 3),
    "16257 nodes": lambda: gen.random_regular(16257, 5, 4),
    "sources without links, path counts in the queue's order": lambda: without_links(gen.random_regular(9000, 8, 5), 7),
    "sources without links, queue in LDS": lambda: without_links(gen.random_regular(12500, 6, 9), 7),
    "sources without links, queue in memory": lambda: without_links(gen.random_regular(17000, 6, 6), 7),
}


@pytest.mark.parametrize("name", CASES)
def test_loads(oracle, name):
    import torch
    import paper_2309_13541_amd as a2a
    csr, cnt = CASES[name](), 1031
    print(name, flush=True)
    topo = a2a.Topology(*csr)
    ws = torch.full((topo.workspace_bytes(cnt, a2a.WS_LOADS),), 0xff, dtype=torch.uint8, device="cuda")
    got = []
    for _ in range(2):
        load = torch.full((topo.E,), -7.0, dtype=torch.float64, device="cuda")
        words = torch.full((2,), -7, dtype=torch.int64, device="cuda")
        topo.profile_enable(len(got))  # the first without
        topo.link_loads(3, cnt, load=load, dist_sum_total=words[:1], flags=words[1:], workspace=ws)
        torch.cuda.synchronize()
        got.append((load, words))
    assert topo.profile_read()["sources"]["launches"] > 0
    topo.profile_enable(0)
    topo.close()
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    o = oracle.run(*csr, 3, cnt, threads=8)
    # sums of up to 1031 x N positive terms in double precision, in two orders
    assert np.allclose(got[0][0].cpu().numpy(), o.load, rtol=1e-11, atol=0)
    assert int(got[0][1][0]) == int(o.dist_sum.sum()) and int(got[0][1][1]) == o.flags
