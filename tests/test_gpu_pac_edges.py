"""Sub-graph extraction at the edges of a thread's eight events and of a workgroup, with ids that are no nodes and arrays on
4-byte boundaries only, against plain numpy."""
import numpy as np
import pytest

from paper_2308_14129_amd import pac

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("n", [1, 7, 8, 9, 2047, 2048, 2049, 300_001])
def test_subgraph_edges(n, offset):
    import torch
    rng = np.random.default_rng(n)
    nodes = max(2, n // 3)
    masks = 1 << rng.integers(0, 4, nodes).astype(np.int64)
    masks[: nodes // 10] = 15  # shared nodes
    ends = rng.integers(-1, nodes + 1, (2, n)).astype(np.int32)  # -1 and `nodes` are no nodes
    group = 0b0101

    def dev(x):
        t = torch.zeros(len(x) + offset, dtype=torch.from_numpy(x).dtype, device="cuda:0")
        t[offset:] = torch.from_numpy(x).cuda()
        return t[offset:]

    eid, local, count = pac.subgraph(dev(ends[0]), dev(ends[1]), torch.from_numpy(masks).cuda(), group)
    shared = np.array([bin(int(m)).count("1") > 1 for m in masks])
    member = shared | ((masks & group) != 0)
    inside = (ends >= 0) & (ends < nodes)
    keep = inside.all(axis=0) & member[np.clip(ends, 0, nodes - 1)].all(axis=0)
    np.testing.assert_array_equal(eid.cpu().numpy(), np.flatnonzero(keep))
    expect = np.where(member, np.cumsum(member) - 1, -1)
    np.testing.assert_array_equal(local.cpu().numpy(), expect)
    assert count == int(member.sum())
