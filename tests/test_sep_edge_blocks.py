"""The edge loop's blocks: streams that end at and around a block's edge against the oracle, and an id that is no node at any place
of a block (the call is refused)."""
import numpy as np
import pytest

from oracle import sep_oracle as P
from paper_2308_14129_amd import sep, tig


def _stream(n, nodes, seed):
    rng = np.random.default_rng(seed)
    p = np.arange(1, nodes + 1) ** -1.3
    src, dst = (rng.choice(nodes, n, p=p / p.sum()).astype(np.int32) for _ in range(2))
    dst = np.where(dst == src, (src + 1) % nodes, dst).astype(np.int32)
    cent = rng.random(nodes) + 0.1
    return src, dst, cent, (np.arange(nodes) < nodes // 5).astype(np.uint8)


@pytest.mark.parametrize("bad", [0, 1, 63, 64, 65, 127, 128, 199])
@pytest.mark.parametrize("value", [-1, 40])
def test_an_id_that_is_no_node(bad, value):
    src, dst, cent, hub = _stream(200, 40, bad)
    for ends in (src, dst):
        kept = ends[bad]
        ends[bad] = value
        with pytest.raises(tig.TigError) as err:
            sep.assign(sep.make_config(4, 1e-3, 0.2), src, dst, 40, cent, hub)
        assert err.value.status == tig.TIG_ERANGE
        ends[bad] = kept


@pytest.mark.parametrize("n", [0, 1, 63, 64, 65, 128, 129, 5000])
@pytest.mark.parametrize("parts", [1, 2, 8, 64])
def test_blocks_against_one_edge_at_a_time(n, parts):
    src, dst, cent, hub = _stream(n, 300, n)
    part, masks, sizes = sep.assign(sep.make_config(parts, 0.0, 0.0, 1.0, 1e-3), src, dst, 300, cent, hub)
    ref_part, A, ref_sizes, _ = P.assign_stream(src, dst, 300, cent, np.flatnonzero(hub).tolist(), parts, 1.0, 1e-3)
    assert part.tolist() == list(ref_part)
    assert masks.tolist() == [sum(1 << p for p in a) for a in A]
    assert sizes.tolist() == list(ref_sizes)


@pytest.mark.parametrize("n", [23, 24, 25, 26, 49])  # endpoints are requested 24 edges ahead, whatever they are
def test_ends_of_what_is_requested_ahead(n):
    src, dst, cent, hub = _stream(n, 300, n)
    part, masks, _ = sep.assign(sep.make_config(3, 0.0, 0.0, 1.0, 1e-3), src, dst, 300, cent, hub)
    ref_part, A, _, _ = P.assign_stream(src, dst, 300, cent, np.flatnonzero(hub).tolist(), 3, 1.0, 1e-3)
    assert part.tolist() == list(ref_part)
    assert masks.tolist() == [sum(1 << p for p in a) for a in A]
    for bad in (-1, -2**31, 2**31 - 1):
        dst[n - 1] = bad
        with pytest.raises(tig.TigError) as err:
            sep.assign(sep.make_config(3, 0.0, 0.0, 1.0, 1e-3), src, dst, 300, cent, hub)
        assert err.value.status == tig.TIG_ERANGE
