"""The temporal adjacency as the device builds it (csr_build.hip), every array of it against a stable sort on the host: one
and two counting passes, the library sort above 2^22 nodes, the edges of tiles and of a workgroup's run of tiles."""
import numpy as np
import pytest

from paper_2308_14129_amd import tig

pytestmark = pytest.mark.gpu

# nodes, events, exponent of the endpoints' ranks (0: uniform)
SHAPES = [(2, 1, 0.0), (5, 4095, 0.0), (256, 4096, 1.2), (257, 4097, 1.2), (2048, 30_001, 0.0), (2049, 30_001, 1.5), (65_537, 8193, 1.1),
          (300_000, 100_000, 0.0), (4096, 4_300_000, 1.3), (1 << 22, 60_000, 0.0), ((1 << 22) + 1, 60_000, 1.1)]


def _ends(rng, n, count, alpha):
    if alpha == 0.0:
        return rng.integers(0, n, count)
    cdf = np.cumsum(np.arange(1, n + 1, dtype=np.float64) ** -alpha)
    return np.minimum(np.searchsorted(cdf, rng.random(count) * cdf[-1]), n - 1)


def _arrays(ctx, n, e, feat):
    """indptr, entries (neighbour, event, time) and positions out of the persistent workspace (arrays on 256-byte boundaries)."""
    raw = ctx.persistent.cpu().numpy()
    at = 0
    found = []
    for count, dtype in ((e, "<i4"), (e, "<i4"), (e, "<f8"), (e * feat, "<f4"), (n + 1, "<i8"),
                         (2 * e, [("nbr", "<i4"), ("eid", "<i4"), ("ts", "<f8")]), (2 * e, "<i4")):
        size = count * np.dtype(dtype).itemsize
        found.append(raw[at:at + size].view(dtype))
        at = (at + size + 255) // 256 * 256
    return found[4], found[5], found[6]


@pytest.mark.parametrize("n,e,alpha", SHAPES)
def test_adjacency_is_the_stable_sort(n, e, alpha):
    rng = np.random.default_rng(n + e)
    src = _ends(rng, n, e, alpha).astype(np.int32)
    dst = _ends(rng, n, e, alpha).astype(np.int32)
    dst = np.where(dst == src, (src + 1) % n, dst).astype(np.int32)
    ts = np.floor(np.cumsum(rng.exponential(0.3, e)))
    cfg = tig.make_config(4, 4, 1, 4, 5, 1, 8)
    ctx = tig.TigContext(cfg, n, src, dst, ts, np.zeros((e, 1), np.float32), None)
    indptr, entries, pos = _arrays(ctx, n, e, 1)
    ctx.close()
    ends = np.stack([src, dst], axis=1).ravel()
    order = np.argsort(ends, kind="stable")
    np.testing.assert_array_equal(indptr, np.searchsorted(ends[order], np.arange(n + 1)))
    np.testing.assert_array_equal(entries["eid"], order >> 1)
    np.testing.assert_array_equal(entries["nbr"], np.stack([dst, src], axis=1).ravel()[order])
    np.testing.assert_array_equal(entries["ts"], ts[order >> 1])
    where = np.empty(2 * e, np.int64)
    where[order] = np.arange(2 * e)
    np.testing.assert_array_equal(pos, where)


@pytest.mark.parametrize("n", [2000, 5000])  # one pass, two passes
@pytest.mark.parametrize("event", [0, 1, 4095, 4096, 9999])
def test_a_graph_that_is_not_one_is_refused(n, event):
    rng = np.random.default_rng(event)
    src = rng.integers(0, n, 10_000).astype(np.int32)
    dst = ((src + 1 + rng.integers(0, n - 1, 10_000)) % n).astype(np.int32)
    ts = np.arange(10_000, dtype=np.float64)
    cfg = tig.make_config(4, 4, 1, 4, 5, 1, 8)

    def refused(src, dst, ts):
        with pytest.raises(tig.TigError) as err:
            tig.TigContext(cfg, n, src, dst, ts, np.zeros((10_000, 1), np.float32), None)
        return err.value.status

    bad = dst.copy()
    bad[event] = n
    assert refused(src, bad, ts) == tig.TIG_ERANGE
    bad[event] = -1
    assert refused(src, bad, ts) == tig.TIG_ERANGE
    bad[event] = src[event]
    assert refused(src, bad, ts) == tig.TIG_ESELFLOOP
    late = ts.copy()
    late[event] = 20_000.0 if event < 9999 else -1.0
    assert refused(src, dst, late) == tig.TIG_EUNSORTED


# more than 1024 tiles, so that workgroups carry their digits' places from tile to tile, with two and four bins a thread: one pass of 11
# bits, two of 9, 10 and 11; whole runs of tiles, a shorter last run, a last tile of two entries
@pytest.mark.parametrize("n,e,alpha", [(2000, 4_300_000, 1.3), ((1 << 17) + 1, 4_296_000, 1.2), ((1 << 19) + 1, 4_300_000, 1.3),
                                       ((1 << 21) + 1, 4_300_000, 1.1), ((1 << 21) + 1, 4_300_801, 0.0)])
def test_places_carried_from_tile_to_tile(n, e, alpha):
    test_adjacency_is_the_stable_sort(n, e, alpha)


@pytest.mark.parametrize("n,e", [(3_000_001, 60_000_000), (70_000, 60_000_000)])
def test_list_bounds_between_wider_samples(n, e):
    # so many entries that the scratch memory holds the node of every sixteenth only
    import torch
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    src = torch.randint(0, n, (e,), device="cuda:0", generator=gen, dtype=torch.int32)
    dst = torch.randint(0, n // 50, (e,), device="cuda:0", generator=gen, dtype=torch.int32)
    dst = torch.where(dst == src, (src + 1) % n, dst).to(torch.int32)
    ts = torch.arange(e, device="cuda:0", dtype=torch.float64)
    ctx = tig.TigContext(tig.make_config(4, 4, 1, 4, 5, 1, 8), n, src, dst, ts, torch.zeros((e, 1), device="cuda:0"), None)
    at = 0
    for size in (4 * e, 4 * e, 8 * e, 4 * e):
        at = (at + size + 255) // 256 * 256
    indptr = ctx.persistent[at:at + 8 * (n + 1)].view(torch.int64)
    count = torch.bincount(torch.cat([src, dst]).long(), minlength=n)
    assert indptr[0].item() == 0
    assert torch.equal(indptr[1:], torch.cumsum(count, 0))
    ctx.close()
