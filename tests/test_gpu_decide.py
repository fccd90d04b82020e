"""sage_decide: a whole decision (ingest, predict, index, rank) in one call gives
the separate calls' bits, for every form of the queries and the store that it
takes; forms that it does not take go through the separate calls."""
import numpy as np
import pytest
import torch

from paper_2603_07917_amd import sage, workloads

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def same(a, b):
    torch.cuda.synchronize()
    return all(x.dtype == y.dtype and torch.equal(x.view(torch.uint8), y.view(torch.uint8)) for x, y in zip(a, b))


def separate(store, queries, plen):
    pred = store.predict(queries)
    g = sage.index(pred[3], plen, store.bin_repr)
    return (*pred, g, sage.rank(g))


@pytest.mark.parametrize("Q,N,k", [(1, 900, 8), (9, 50000, 64), (33, 3000, 100), (300, 40000, 64), (9000, 2000, 16)])
@pytest.mark.parametrize("layout", ["rows", "panels"])
def test_decide_equals_the_separate_calls(Q, N, k, layout):
    w = workloads.small_predict(Q=Q, N=N, d=96, k=k, B=64, seed=Q + N, clusters=6)
    store = sage.Store(dev(w.hist_emb), dev(w.hist_len), dev(w.bin_edges), dev(w.bin_repr), k, layout=layout)
    qf, plen = dev(w.queries), dev(w.prompt_len)
    want = separate(store, qf, plen)
    wide = torch.zeros((Q, 128), device="cuda")
    wide[:, :96] = qf
    forms = [qf, sage.ingest_bf16(qf), sage.ingest_bf16(qf, "panels"), wide[:, :96]]      # the last: not contiguous
    for q in forms:
        assert same(store.decide(q, plen), want)
    out = [torch.full_like(t, 7) for t in want]
    got = store.decide(qf, plen, out=out)
    assert all(a is b for a, b in zip(got, out)) and same(out, want)
    # a store in the other layout than the one declared: the separate calls
    other = sage.Store(sage.ingest_bf16(dev(w.hist_emb), "panels" if layout == "rows" else "rows"), dev(w.hist_len),
                       dev(w.bin_edges), dev(w.bin_repr), k, layout=layout)
    assert same(other.decide(qf, plen), want)


def test_decide_keeps_errors_and_overrides():
    w = workloads.small_predict(Q=4, N=500, d=64, k=8, B=16, seed=2, clusters=3)
    store = sage.Store(dev(w.hist_emb), dev(w.hist_len), dev(w.bin_edges), dev(w.bin_repr), 8)
    qf, plen = dev(w.queries), dev(w.prompt_len)
    for q, p in ((qf, plen[:3]), (qf.cpu(), plen), (qf, plen.long()), (qf[:, :32], plen), (qf.double(), plen)):
        with pytest.raises(sage.SageError):
            store.decide(q, p)
    full = store.decide(qf, plen)
    for i, t in ((3, full[3].double()), (3, full[3].repeat(2, 1)), (3, torch.zeros((16, 4), device="cuda").t()),
                 (3, full[3].int()), (4, full[4].double()), (4, full[4].reshape(2, 2))):
        out = [torch.zeros_like(x) for x in full]
        out[i] = t                                             # of the size written or larger
        with pytest.raises(sage.SageError):
            store.decide(qf, plen, out=out)
    for left_out in ((4, 5), (5,)):                            # allocated by the index and the rank
        out = [None if i in left_out else torch.zeros_like(x) for i, x in enumerate(full)]
        assert same(store.decide(qf, plen, out=out), full)
    with pytest.raises(sage.SageError):
        store.decide(qf, plen, out=[None, *full[1:]])
    ring = sage.RingStore(100, 64, dev(w.bin_edges), dev(w.bin_repr), 8)
    with pytest.raises(sage.SageError, match="empty"):
        ring.decide(qf, plen)
    ring.insert(dev(w.hist_emb[:300]), dev(w.hist_len[:300]))
    assert same(ring.decide(qf, plen), separate(ring, qf, plen))

    class Mine(sage.Store):
        def predict(self, queries, out=None):
            self.called = True
            return super().predict(queries, out=out)

    mine = Mine(dev(w.hist_emb), dev(w.hist_len), dev(w.bin_edges), dev(w.bin_repr), 8)
    assert same(mine.decide(qf, plen), store.decide(qf, plen)) and mine.called
    empty = store.decide(qf[:0], plen[:0])
    assert [t.shape[0] for t in empty] == [0] * 6


@pytest.mark.parametrize("Q,N,k,path", [(40, 50000, 32, "filtered"), (4, 60000, 16, "stream")])
@pytest.mark.parametrize("f32", [True, False])
def test_stats_of_a_decision(Q, N, k, path, f32):
    """predict_stats on the store's workspace after decide: what the same search
    reports after predict (the candidates depend on the inputs only), with every
    query flagged and with none."""
    w = workloads.small_predict(Q=Q, N=N, d=64, k=k, B=32, seed=Q + N, clusters=6)
    store = sage.Store(dev(w.hist_emb), dev(w.hist_len), dev(w.bin_edges), dev(w.bin_repr), k)
    queries, plen = dev(w.queries), dev(w.prompt_len)
    if not f32:
        queries = sage.ingest_bf16(queries, "panels")
    stats = lambda: sage.predict_stats(store._ws, Q, N, 64, k, 32)
    try:
        for floor, flagged in ((-np.inf, 0), (2.0, Q)):
            sage.debug_theta_floor(floor)
            store.predict(queries)
            want = stats()
            assert want["path"] == path and want["flagged"] == flagged
            store._ws.fill_(0x5A)
            store.decide(queries, plen)
            assert stats() == want
    finally:
        sage.debug_theta_floor(-np.inf)
