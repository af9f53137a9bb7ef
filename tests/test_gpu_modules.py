"""Other instances of the general architecture (Sec. II-C: mean aggregator, RNN update, identity /
time-projection embedding; Sec. II-A node features) on the GPU against their oracle, through the C
ABI: tig_init without weights + tig_modules_attach, then ordinary tig_step calls.

Bar: winners and (attention embedding) neighbour tables bit-exact; embeddings, scores and memory
within 1e-4 under the per-tensor gate; last_update bit-exact; rows outside the applied batch
bit-identical."""
import numpy as np
import pytest

import tig_synth as S
from oracle import modules_oracle as G
from oracle import tig_oracle as O
from tests.parity import gate

pytestmark = pytest.mark.gpu

TOL = 1e-4

INSTANCES = {
    "jodie_like": dict(aggregator="last", updater="rnn", embedding="time_projection"),
    "dyrep_like": dict(aggregator="last", updater="rnn", embedding="identity"),
    "mean_gru_identity": dict(aggregator="mean", updater="gru", embedding="identity"),
    "mean_rnn_projection": dict(aggregator="mean", updater="rnn", embedding="time_projection"),
    "mean_gru_attention": dict(aggregator="mean", updater="gru", embedding="attention"),
    "last_rnn_attention": dict(aggregator="last", updater="rnn", embedding="attention"),
    "headline": dict(aggregator="last", updater="gru", embedding="attention"),
}


class Case:
    def __init__(self, w, inst, node_feat, order="update_first", max_batch=None, layers=1):
        import torch
        from paper_2308_14129_amd import tig
        self.w, self.inst = w, inst
        self.g = S.make_graph(w)
        self.W = S.make_module_weights(w, inst["updater"], inst["embedding"])
        self.ix = O.NeighbourIndex(self.g.num_nodes, self.g.src, self.g.dst, self.g.ts)
        self.nf = S.make_node_feat(w, self.g.num_nodes) if node_feat else None
        self.L2 = S.make_layer2_weights(w) if layers == 2 else None
        self.mods = G.Modules(inst["aggregator"], inst["updater"], inst["embedding"], self.nf, layers, self.L2)
        self.deferred = order == "deferred"
        E = w.emb_dim if inst["embedding"] == "attention" else w.mem_dim
        cfg = tig.make_config(w.mem_dim, w.time_dim, w.feat_dim, E, w.num_neighbors, w.num_heads,
                              max_batch or w.batch_size, "fp32", order)
        self.ctx = tig.TigContext(cfg, self.g.num_nodes, self.g.src, self.g.dst, self.g.ts, self.g.edge_feat, None)
        self.ctx.modules_attach(self.W, node_feat=self.nf, layers=layers, layer2=self.L2, **inst)
        self.torch = torch

    def run(self, batches, warm_at=None, with_neg=True, locked=False):
        torch, w, g, ctx = self.torch, self.w, self.g, self.ctx
        attn = self.inst["embedding"] == "attention"
        if warm_at is None:
            st = O.OracleState.zeros(g.num_nodes, w.mem_dim)
            ctx.reset()
        else:
            st = O.OracleState(*S.make_warm_state(w, g, warm_at))
            ctx.state_import(st.mem, st.last_update)
        before = (st.mem.copy(), st.last_update.copy())
        applied = None
        worst = {}
        for first, count in batches:
            print(f"[{w.name} {self.inst}] step first_eid={first} count={count}", flush=True)
            neg = S.make_negatives(w, g, first, count) if with_neg else None
            if locked:
                ctx.state_import(st.mem, st.last_update)
                st.drop_pending()
                before = (st.mem.copy(), st.last_update.copy())
                applied = None
            ref = G.step(st, g.src, g.dst, g.ts, g.edge_feat, self.W, first, count, neg, w.num_neighbors, w.num_heads,
                         self.mods, index=self.ix, deferred=self.deferred)
            out = ctx.alloc_outputs(count, with_neg=with_neg, inspect=True)
            if not attn:
                out.nbr_cnt.fill_(-7)      # must stay untouched
            ctx.step(first, count, torch.from_numpy(neg).to("cuda:0") if with_neg else None, out)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(out.is_winner.cpu().numpy(), ref["is_winner"], err_msg="is_winner")
            if attn:
                for k in ("nbr_cnt", "nbr_node", "nbr_eid", "nbr_ts"):
                    np.testing.assert_array_equal(getattr(out, k).cpu().numpy(), ref[k], err_msg=k)
            else:
                assert int((out.nbr_cnt != -7).sum()) == 0
            res = {"emb": gate(out.emb.cpu().numpy(), ref["emb"], TOL, "emb"),
                   "score_pos": gate(out.score_pos.cpu().numpy(), ref["score_pos"], TOL, "score_pos")}
            if with_neg:
                res["score_neg"] = gate(out.score_neg.cpu().numpy(), ref["score_neg"], TOL, "score_neg")
            mem, lu = ctx.state_export()
            np.testing.assert_array_equal(lu, st.last_update, err_msg="last_update")
            res["mem"] = gate(mem, st.mem, TOL, "mem")
            msg = (first, count) if not self.deferred else applied
            keep = np.ones(g.num_nodes, dtype=bool)
            if msg is not None:
                keep[np.concatenate([g.src[msg[0]:msg[0] + msg[1]], g.dst[msg[0]:msg[0] + msg[1]]])] = False
            assert np.array_equal(mem[keep], before[0][keep]) and np.array_equal(lu[keep], before[1][keep])
            before = (mem, lu)
            applied = (first, count)
            for k, v in res.items():
                worst[k] = max(worst.get(k, 0.0), v)
        print(f"[{w.name} {self.inst}] worst gate ratios: {worst}", flush=True)
        return worst

    def close(self):
        self.ctx.close()


def window(w, frac, steps, batch=None):
    B = batch or w.batch_size
    first = int(w.num_events * frac) // B * B
    return first, list(S.batches(w.num_events, B, first=first, stop=first + steps * B))


@pytest.mark.parametrize("name", list(INSTANCES))
@pytest.mark.parametrize("node_feat", [False, True])
def test_c1_from_reset_and_ragged(name, node_feat):
    """From reset, free running, ragged batch of 136 (tails in every kernel), then a one-event batch
    and a batch without negatives."""
    c = Case(S.WORKLOADS["c1_tiny"], INSTANCES[name], node_feat)
    c.run(list(S.batches(c.w.num_events, 136))[:10])
    c.run([(3000, 1), (3001, 136)], warm_at=3000)
    c.run([(5000, 200), (5200, 200)], warm_at=5000, with_neg=False)
    c.close()


@pytest.mark.parametrize("order", ["update_first", "deferred"])
@pytest.mark.parametrize("name,dims,batch", [("jodie_like", dict(mem_dim=37, time_dim=11, feat_dim=5), 33),
                                             ("mean_rnn_projection", dict(mem_dim=130, time_dim=20, feat_dim=3), 999),
                                             ("last_rnn_attention", dict(mem_dim=33, time_dim=15, emb_dim=50), 137),
                                             ("mean_gru_identity", dict(mem_dim=16, time_dim=4, feat_dim=1), 1)])
def test_steps_that_prepare_each_other(name, dims, batch, order):
    """Without inspection outputs every step's winners (and queries) come from the step before; row widths around
    the tiles' edges, batches that leave tiles ragged, a gap in the stream."""
    c = Case(S.WORKLOADS["c1_tiny"].scaled(**dims), INSTANCES[name], False, order=order, max_batch=batch)
    st = O.OracleState.zeros(c.g.num_nodes, c.w.mem_dim)
    c.ctx.reset()
    for first in [0, batch, 2 * batch, 3 * batch + 50, 4 * batch + 50]:
        neg = S.make_negatives(c.w, c.g, first, batch)
        ref = G.step(st, c.g.src, c.g.dst, c.g.ts, c.g.edge_feat, c.W, first, batch, neg, c.w.num_neighbors, c.w.num_heads,
                     c.mods, index=c.ix, deferred=c.deferred)
        out = c.ctx.alloc_outputs(batch)
        c.ctx.step(first, batch, c.torch.from_numpy(neg).to("cuda:0"), out)
        for k in ("emb", "score_pos", "score_neg"):
            gate(getattr(out, k).cpu().numpy(), ref[k], TOL, k)
    mem, lu = c.ctx.state_export()
    np.testing.assert_array_equal(lu, st.last_update)
    gate(mem, st.mem, TOL, "mem")
    c.close()


@pytest.mark.parametrize("name", ["jodie_like", "mean_gru_attention", "mean_rnn_projection"])
def test_c1_deferred_order(name):
    c = Case(S.WORKLOADS["c1_tiny"], INSTANCES[name], True, order="deferred")
    c.run(list(S.batches(c.w.num_events, 136))[:10])
    c.run([(3000, 100), (3100, 100), (3300, 50)], warm_at=3000)      # a gap; import drops what is kept
    c.close()


@pytest.mark.parametrize("name", ["mean_gru_attention", "jodie_like"])
def test_c1_step_locked_whole_stream_tail(name):
    c = Case(S.WORKLOADS["c1_tiny"], INSTANCES[name], False)
    c.run(list(S.batches(c.w.num_events, 200))[-3:] + [(9990, 10)], warm_at=9400, locked=True)
    c.close()


@pytest.mark.parametrize("name", ["mean_gru_attention", "dyrep_like", "mean_rnn_projection"])
def test_c2_wide_rows_window(name):
    w = S.WORKLOADS["c2_bipartite_medium"]
    c = Case(w, INSTANCES[name], name != "dyrep_like")
    first, bs = window(w, 0.5, 3)
    c.run(bs, warm_at=first)
    c.close()


@pytest.mark.parametrize("name", ["mean_gru_attention", "jodie_like"])
def test_c3_batch_2000_and_above_the_selection_limit(name):
    """K = 20, 2000 events per batch (a hub node collects hundreds of messages for the mean), then a
    5000-event batch (selection in its own launches)."""
    w = S.WORKLOADS["c3_bipartite_dense"]
    c = Case(w, INSTANCES[name], False, max_batch=5000)
    first, bs = window(w, 0.5, 2, 2000)
    c.run(bs, warm_at=first)
    c.run([(first, 5000)], warm_at=first)
    c.close()


@pytest.mark.parametrize("name,node_feat", [("headline", False), ("mean_gru_attention", True), ("last_rnn_attention", False)])
def test_c1_two_layers_from_reset_and_ragged(name, node_feat):
    """Two stacked attention layers (the embedding over the 2-hop neighbourhood): from reset (empty
    and short neighbour tables in both hops), ragged batches, a one-event batch, no negatives."""
    c = Case(S.WORKLOADS["c1_tiny"], INSTANCES[name], node_feat, layers=2)
    c.run(list(S.batches(c.w.num_events, 136))[:6])
    c.run([(3000, 1), (3001, 136)], warm_at=3000)
    c.run([(5000, 200)], warm_at=5000, with_neg=False)
    c.close()


def test_c1_two_layers_deferred_order():
    c = Case(S.WORKLOADS["c1_tiny"], INSTANCES["headline"], True, order="deferred", layers=2)
    c.run([(3000, 100), (3100, 100), (3300, 50)], warm_at=3000)
    c.close()


@pytest.mark.parametrize("order", ["update_first", "deferred"])
@pytest.mark.parametrize("name,dims,batch", [
    ("headline", dict(), 1),                                              # one event: fewer rows than a tile
    ("last_rnn_attention", dict(mem_dim=33, time_dim=15, emb_dim=49, feat_dim=5, num_neighbors=7), 137),
    ("mean_gru_attention", dict(num_heads=1, mem_dim=65, emb_dim=31), 1000),
    ("headline", dict(num_heads=4, num_neighbors=15, emb_dim=64), 999),   # rows of both layers beyond one pass of the grid
    # the second layer's rows do not fit the embedding kernel's tiles: products over all rows instead
    ("headline", dict(num_heads=4, mem_dim=16, time_dim=100, feat_dim=160, emb_dim=252), 50)])
def test_two_layers_that_prepare_each_other(name, dims, batch, order):
    """Without inspection outputs the winners, queries and (but for the mean) staged rows come from the step before;
    a gap in the stream, row widths around the tiles' edges, a step without negatives at the end."""
    c = Case(S.WORKLOADS["c1_tiny"].scaled(**dims), INSTANCES[name], False, order=order, max_batch=batch, layers=2)
    st = O.OracleState.zeros(c.g.num_nodes, c.w.mem_dim)
    c.ctx.reset()
    for n, first in enumerate([0, batch, 2 * batch, 3 * batch + 50, 4 * batch + 50]):
        print(f"two layers {name} {dims} first={first} count={batch}", flush=True)
        neg = S.make_negatives(c.w, c.g, first, batch) if n < 4 else None
        ref = G.step(st, c.g.src, c.g.dst, c.g.ts, c.g.edge_feat, c.W, first, batch, neg, c.w.num_neighbors, c.w.num_heads,
                     c.mods, index=c.ix, deferred=c.deferred)
        out = c.ctx.alloc_outputs(batch, with_neg=n < 4)
        c.ctx.step(first, batch, c.torch.from_numpy(neg).to("cuda:0") if n < 4 else None, out)
        for k in ("emb", "score_pos", "score_neg")[:3 if n < 4 else 2]:
            gate(getattr(out, k).cpu().numpy(), ref[k], TOL, k)
    mem, lu = c.ctx.state_export()
    np.testing.assert_array_equal(lu, st.last_update)
    gate(mem, st.mem, TOL, "mem")
    c.close()


def test_a_new_context_takes_nothing_over_from_one_that_is_gone():
    """The first step of a context is the same bits whatever the context before it ran (contexts take over each other's
    places in the page of hints about recent steps, which size the launches)."""
    def first_step(count):
        c = Case(S.WORKLOADS["c1_tiny"], INSTANCES["headline"], False, max_batch=900, layers=2)
        c.ctx.state_import(*S.make_warm_state(c.w, c.g, 4000))
        out = c.ctx.alloc_outputs(count)
        c.ctx.step(4000, count, c.torch.from_numpy(S.make_negatives(c.w, c.g, 4000, count)).to("cuda:0"), out)
        c.torch.cuda.synchronize()
        c.close()
        return out

    first_step(10)
    behind_small = first_step(900)
    behind_large = first_step(900)
    for k in ("emb", "score_pos", "score_neg"):
        assert getattr(behind_small, k).equal(getattr(behind_large, k)), k


@pytest.mark.parametrize("count", [300, 900, 1300])
def test_bits_of_two_layers_do_not_depend_on_the_step_before(count):
    def play(behind):
        c = Case(S.WORKLOADS["c1_tiny"], INSTANCES["headline"], False, max_batch=1300, layers=2)
        for n in (behind, count):
            c.ctx.state_import(*S.make_warm_state(c.w, c.g, 4000))
            out = c.ctx.alloc_outputs(n)
            c.ctx.step(4000, n, c.torch.from_numpy(S.make_negatives(c.w, c.g, 4000, n)).to("cuda:0"), out)
            c.torch.cuda.synchronize()
        c.close()
        return out

    ref = play(10)
    for behind in (10, 1300):
        out = play(behind)
        for k in ("emb", "score_pos", "score_neg"):
            assert getattr(out, k).equal(getattr(ref, k)), (behind, k)


def test_c2_two_layers_wide_rows_emb_narrower_than_memory():
    """E = 100 != M = 172: the second layer's rows have a width of their own."""
    w = S.WORKLOADS["c2_bipartite_medium"]
    c = Case(w, INSTANCES["headline"], True, layers=2)
    first, bs = window(w, 0.5, 2)
    c.run(bs, warm_at=first)
    c.close()


def test_c3_two_layers_twenty_neighbours():
    w = S.WORKLOADS["c3_bipartite_dense"]
    c = Case(w, INSTANCES["mean_gru_attention"], False, layers=2)
    first, bs = window(w, 0.5, 1)
    c.run(bs, warm_at=first)
    c.close()


@pytest.mark.parametrize("layers", [1, 2])
def test_c1_four_heads_with_node_features(layers):
    """Four attention heads (the kernels keep per-head rows in registers: another instantiation) over
    K = 12 neighbours, node features on, one and two layers."""
    w = S.WORKLOADS["c1_tiny"].scaled(num_heads=4, num_neighbors=12)
    c = Case(w, INSTANCES["headline"], True, layers=layers)
    c.run(list(S.batches(w.num_events, 136))[:4])
    c.run([(5000, 200), (5200, 77)], warm_at=5000)
    c.close()


def test_two_layers_need_the_attention_embedding_and_their_weights():
    import ctypes
    from paper_2308_14129_amd import tig
    w = S.WORKLOADS["c1_tiny"]
    cfg = tig.make_config(w.mem_dim, w.time_dim, w.feat_dim, w.mem_dim, w.num_neighbors, w.num_heads, 200)
    lib = tig.load_library()
    n = ctypes.c_size_t(0)
    for emb, l2 in ((1, True), (0, False)):
        L2 = S.make_layer2_weights(w)
        lw = tig.tig_layer_weights(ctypes.sizeof(tig.tig_layer_weights), 0, *[L2[k].ctypes.data for k in tig.LAYER_WEIGHT_NAMES])
        m = tig.tig_modules(ctypes.sizeof(tig.tig_modules), 0, 0, emb, None, None, 2, 0, ctypes.pointer(lw) if l2 else None)
        assert lib.tig_modules_workspace_bytes(ctypes.byref(cfg), ctypes.byref(m), 1000, ctypes.byref(n)) == tig.TIG_EINVAL


def test_headline_selection_matches_the_fused_step():
    """The module path with (last, GRU, attention, no node features) and the fused kernels of the
    headline instance compute the same step: both within the gate of the same oracle."""
    import torch
    from paper_2308_14129_amd import tig
    w = S.WORKLOADS["c1_tiny"]
    c = Case(w, INSTANCES["headline"], False)
    cfg = tig.make_config(w.mem_dim, w.time_dim, w.feat_dim, w.emb_dim, w.num_neighbors, w.num_heads, w.batch_size)
    fused = tig.TigContext(cfg, c.g.num_nodes, c.g.src, c.g.dst, c.g.ts, c.g.edge_feat, c.W)
    warm = S.make_warm_state(w, c.g, 4000)
    neg = torch.from_numpy(S.make_negatives(w, c.g, 4000, 200)).to("cuda:0")
    outs = []
    for ctx in (c.ctx, fused):
        ctx.state_import(*warm)
        o = ctx.alloc_outputs(200)
        ctx.step(4000, 200, neg, o)
        torch.cuda.synchronize()
        outs.append(o)
    gate(outs[0].emb.cpu().numpy(), outs[1].emb.cpu().numpy(), 2e-4, "emb (module path vs fused path)")
    gate(outs[0].score_pos.cpu().numpy(), outs[1].score_pos.cpu().numpy(), 2e-4, "score_pos")
    fused.close()
    c.close()


def test_context_without_weights_refuses_steps_and_static_and_training():
    import ctypes
    import torch
    from paper_2308_14129_amd import tig
    w = S.WORKLOADS["c1_tiny"]
    g = S.make_graph(w)
    cfg = tig.make_config(w.mem_dim, w.time_dim, w.feat_dim, w.mem_dim, w.num_neighbors, w.num_heads, 200)
    ctx = tig.TigContext(cfg, g.num_nodes, g.src, g.dst, g.ts, g.edge_feat, None)
    out = ctx.alloc_outputs(200)
    neg = torch.from_numpy(S.make_negatives(w, g, 0, 200)).to("cuda:0")
    with pytest.raises(tig.TigError) as ei:
        ctx.step(0, 200, neg, out)
    assert ei.value.status == tig.TIG_EINVAL
    W = S.make_module_weights(w, "rnn", "identity")
    ctx.modules_attach(W, updater="rnn", embedding="identity")
    ctx.step(0, 200, neg, out)
    with pytest.raises(tig.TigError) as ei:
        ctx.step(200, 200, neg, out, static=True)
    assert ei.value.status == tig.TIG_EINVAL
    torch.cuda.synchronize()
    # emb_dim != mem_dim with a non-attention embedding is refused
    cfg2 = tig.make_config(w.mem_dim, w.time_dim, w.feat_dim, w.mem_dim + 4, w.num_neighbors, w.num_heads, 200)
    m = tig.tig_modules(ctypes.sizeof(tig.tig_modules), 0, 1, 1, None, None, 1, 0, None)
    n = ctypes.c_size_t(0)
    assert ctx.lib.tig_modules_workspace_bytes(ctypes.byref(cfg2), ctypes.byref(m), g.num_nodes, ctypes.byref(n)) == tig.TIG_EINVAL
    ctx.close()


# Median over the steps below of the embeddings' and the scores' relative errors (2-norm).  Measured here: in direct form,
# item by item, 2.9e-7 and 6.0e-7; by the layers' kernel with the softmax's hardware exponential and the merge layer's
# sums in one chain 3.8e-7 and 6.1e-7; with expf and sums in parts 2.6e-7 and 4.7e-7.
TWO_LAYER_EMB, TWO_LAYER_SCORE = 2.9e-7, 5.5e-7


def test_two_layers_errors_against_64_bits():
    emb, score = [], []
    for mem, time, feat, width, heads, K in ((100, 100, 8, 100, 2, 10), (172, 100, 30, 100, 2, 10), (61, 39, 20, 53, 1, 7),
                                             (120, 60, 90, 128, 4, 13), (33, 95, 64, 41, 2, 15), (150, 18, 5, 70, 2, 9)):
        c = Case(S.WORKLOADS["c1_tiny"].scaled(mem_dim=mem, time_dim=time, feat_dim=feat, emb_dim=width, num_heads=heads,
                                               num_neighbors=K), INSTANCES["headline"], False, max_batch=100, layers=2)
        st = O.OracleState(*S.make_warm_state(c.w, c.g, 4000))
        for first in (4000, 4100, 4200):
            c.ctx.state_import(st.mem, st.last_update)
            neg = S.make_negatives(c.w, c.g, first, 100)
            ref = G.step(st, c.g.src, c.g.dst, c.g.ts, c.g.edge_feat, c.W, first, 100, neg, c.w.num_neighbors, c.w.num_heads,
                         c.mods, index=c.ix, deferred=False)
            out = c.ctx.alloc_outputs(100)
            c.ctx.step(first, 100, c.torch.from_numpy(neg).to("cuda:0"), out)
            emb.append(np.linalg.norm(out.emb.cpu().numpy() - ref["emb"]) / np.linalg.norm(ref["emb"]))
            score.append(np.linalg.norm(out.score_pos.cpu().numpy() - ref["score_pos"]) / np.linalg.norm(ref["score_pos"]))
        c.close()
    print(f"medians: embeddings {np.median(emb):.3g}, scores {np.median(score):.3g}", flush=True)
    assert np.median(emb) < TWO_LAYER_EMB and np.median(score) < TWO_LAYER_SCORE, (emb, score)


# a mean message's columns are gathered as two halves beside the state row: the fewest columns, an odd number of them, halves and
# state rows on either side of what one round of a wavefront's loads takes (192 columns)
@pytest.mark.parametrize("name,dims", [("mean_rnn_projection", dict(mem_dim=2, time_dim=2, feat_dim=1)),
                                       ("mean_gru_identity", dict(mem_dim=200, time_dim=8, feat_dim=3)),
                                       ("mean_gru_attention", dict(mem_dim=150, time_dim=150, feat_dim=151)),
                                       ("mean_rnn_projection", dict(mem_dim=192, time_dim=100, feat_dim=92))])
def test_mean_messages_in_two_halves(name, dims):
    c = Case(S.WORKLOADS["c1_tiny"].scaled(**dims), INSTANCES[name], False)
    c.run([(3000, 150), (3150, 150)], warm_at=3000)
    c.close()
