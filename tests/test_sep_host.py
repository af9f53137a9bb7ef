"""The host stage of the partitioner (tig_sep_assign: the sequential edge loop of Alg. 1) against
the oracle, bit for bit, on the oracle's own centralities and hubs.  No GPU needed."""
import json
import os

import numpy as np
import pytest

import tig_synth as S
from oracle import sep_oracle as P

GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "sep_hand_stream.json")


@pytest.fixture(scope="module")
def sep():
    from paper_2308_14129_amd import sep, tig
    if not os.path.exists(tig.LIB_PATH):
        from paper_2308_14129_amd import build
        build.build()
    return sep


def masks(A):
    return np.array([sum(1 << p for p in a) for a in A], dtype=np.uint64)


def test_hand_worked_stream(sep):
    g = json.load(open(GOLDEN))
    is_hub = np.zeros(g["num_nodes"], dtype=np.uint8)
    is_hub[g["hubs"]] = 1
    cfg = sep.make_config(g["num_parts"], 0.0, 0.0, g["lambda"], g["epsilon"])
    part, node_parts, sizes = sep.assign(cfg, g["src"], g["dst"], g["num_nodes"], g["cent"], is_hub)
    assert part.tolist() == g["edge_part"]
    assert node_parts.tolist() == masks(g["A"]).tolist()
    assert sizes.tolist() == g["sizes"]
    parts, shared = sep.node_lists(node_parts, g["num_parts"])
    assert shared.tolist() == g["shared"] and [p.tolist() for p in parts] == g["parts"]


@pytest.mark.parametrize("name,events,num_parts,k,lam", [("c1_tiny", 10000, 4, 0.05, 1.0), ("c1_tiny", 10000, 8, 0.0, 0.3),
                                                         ("c1_tiny", 10000, 3, 0.2, 2.5),
                                                         ("c2_bipartite_medium", 30000, 4, 0.01, 1.0),
                                                         ("c3_bipartite_dense", 30000, 64, 0.05, 1.0)])
def test_assign_matches_oracle(sep, name, events, num_parts, k, lam):
    w = S.WORKLOADS[name].scaled(num_events=events)
    g = S.make_graph(w)
    cent = P.centrality(g.src, g.dst, g.ts, g.num_nodes, beta=1e-5)
    hubs = P.top_k_hubs(cent, k)
    ref_part, A, sizes, _ = P.assign_stream(g.src, g.dst, g.num_nodes, cent, hubs, num_parts, lam, 1e-3)
    is_hub = np.zeros(g.num_nodes, dtype=np.uint8)
    is_hub[hubs] = 1
    part, node_parts, part_edges = sep.assign(sep.make_config(num_parts, 1e-5, k, lam, 1e-3), g.src, g.dst,
                                              g.num_nodes, cent, is_hub)
    assert np.array_equal(part, ref_part)
    assert np.array_equal(node_parts, masks(A))
    assert part_edges.tolist() == sizes
    parts, shared = sep.node_lists(node_parts, num_parts)
    ref_parts, ref_shared = P.node_lists(A, num_parts)
    assert shared.tolist() == ref_shared and [p.tolist() for p in parts] == ref_parts


@pytest.mark.parametrize("num_parts,lam,eps,hubs", [(2, 1.0, 1e-3, 3), (5, 1.0, 1e-3, 40), (64, 0.7, 1.0, 40), (3, 1e-16, 1e-3, 20),
                                                    (4, 60.0, 1e-3, 30), (4, 1.0, 1e-13, 30), (1, 1.0, 1e-3, 5)])
def test_assign_branches_match_oracle(sep, num_parts, lam, eps, hubs):
    # sizes that drift far apart (non-hubs pile up where they reside) and come together again (hubs), balance terms
    # that lose against a replica, beat it, or differ by less than a rounding
    r = np.random.default_rng(num_parts * 100 + hubs)
    n = 60
    src = np.concatenate([np.tile([50, 52], 40), r.integers(0, 12, 1500), r.integers(0, n, 1500)]).astype(np.int32)
    dst = np.concatenate([np.tile([51, 53], 40), r.integers(12, 24, 1500), r.integers(0, n, 1500)]).astype(np.int32)
    dst = np.where(dst == src, (src + 1) % n, dst).astype(np.int32)
    cent = np.bincount(src, minlength=n) + np.bincount(dst, minlength=n) + 0.0
    hub_ids = np.arange(hubs)
    is_hub = np.zeros(n, dtype=np.uint8)
    is_hub[hub_ids] = 1
    ref_part, A, sizes, _ = P.assign_stream(src, dst, n, cent, hub_ids, num_parts, lam, eps)
    part, node_parts, part_edges = sep.assign(sep.make_config(num_parts, 0.0, 0.0, lam, eps), src, dst, n, cent, is_hub)
    assert np.array_equal(part, ref_part) and np.array_equal(node_parts, masks(A)) and part_edges.tolist() == sizes


@pytest.mark.parametrize("num_parts,pile", [(2, 17), (3, 40), (7, 16), (16, 30)])
def test_sizes_that_drift_apart_and_come_together_again(sep, num_parts, pile):
    # blocks of events between two resident non-hubs (one partition grows by `pile`), and of events between hubs, which
    # the balance term sends to the small partitions until all sizes are close again
    r = np.random.default_rng(num_parts)
    hubs = np.arange(30)
    src, dst = [], []
    for k in range(25):
        src += [40 + 2 * (k % 5)] * pile + r.integers(0, 30, num_parts * pile + k).tolist()
        dst += [41 + 2 * (k % 5)] * pile + r.integers(0, 29, num_parts * pile + k).tolist()
    src, dst = np.array(src, dtype=np.int32), np.array(dst, dtype=np.int32)
    dst = np.where(dst == src, 29, dst).astype(np.int32)
    src = np.where(dst == src, 0, src).astype(np.int32)
    n = 60
    cent = np.bincount(src, minlength=n) + np.bincount(dst, minlength=n) + 0.0
    is_hub = (np.arange(n) < 30).astype(np.uint8)
    for lam in (1.0, 8.0):  # (8: a partition that is small enough beats one with both replicas)
        ref_part, A, sizes, _ = P.assign_stream(src, dst, n, cent, hubs, num_parts, lam, 1e-3)
        part, node_parts, part_edges = sep.assign(sep.make_config(num_parts, 0.0, 0.0, lam, 1e-3), src, dst, n, cent, is_hub)
        assert np.array_equal(part, ref_part) and np.array_equal(node_parts, masks(A)) and part_edges.tolist() == sizes


def test_a_stream_without_hubs_costs_no_more_than_one_with(sep):
    # without hubs the sizes are far apart from the start: an edge of such a stream took seven times as long as one of
    # the same stream with hubs while the sets of sizes were rebuilt for each (0.8 times as long without that)
    import time
    r = np.random.default_rng(1)
    n, events = 100_000, 300_000
    cdf = np.cumsum(np.arange(1, n + 1) ** -1.5)
    src, dst = (np.searchsorted(cdf, r.random(events) * cdf[-1]).astype(np.int32) for _ in range(2))
    dst = np.where(dst == src, (src + 1) % n, dst).astype(np.int32)
    cent = np.bincount(src, minlength=n) + np.bincount(dst, minlength=n) + 0.0
    seconds = []
    for hubs in (0, n // 100):
        is_hub = (np.arange(n) < hubs).astype(np.uint8)
        runs = []
        for _ in range(7):
            start = time.perf_counter()
            sep.assign(sep.make_config(16, 0.0, 0.0), src, dst, n, cent, is_hub)
            runs.append(time.perf_counter() - start)
        seconds.append(min(runs))
    assert seconds[0] < 3.0 * seconds[1], seconds


def test_assign_rejects_bad_arguments(sep):
    from paper_2308_14129_amd import tig
    ok = dict(src=[0, 1], dst=[1, 2], num_nodes=3, cent=[1.0, 1.0, 1.0], is_hub=[0, 0, 0])
    for cfg in (sep.make_config(0, 0.1, 0.0), sep.make_config(65, 0.1, 0.0), sep.make_config(2, 0.1, 0.0, lam=0.0),
                sep.make_config(2, 0.1, 0.0, eps=0.0)):
        with pytest.raises(tig.TigError) as ei:
            sep.assign(cfg, **ok)
        assert ei.value.status == tig.TIG_EINVAL
    with pytest.raises(tig.TigError) as ei:
        sep.assign(sep.make_config(2, 0.1, 0.0), [0, 5], [1, 2], 3, [1.0] * 3, [0] * 3)
    assert ei.value.status == tig.TIG_ERANGE


def test_combine_host_call():
    from paper_2308_14129_amd import pac, tig
    from oracle import pac_oracle as E
    order = np.random.default_rng(11).permutation(8)
    assert pac.combine(order, 4) == E.combine(order, 4)
    assert pac.combine(order, 8) == [1 << int(p) for p in order]
    assert pac.combine(order, 1) == [0xFF]
    for bad in (([0, 1, 2], 2), ([0, 0, 1, 2], 2), ([0, 1, 2, 7], 2)):
        with pytest.raises(tig.TigError):
            pac.combine(*bad)
