"""The filtered neighbour search (Sec. 3.1: brute-force similarity and top-k)
at the edges of its tiles, chunk counts and candidate segments, against the
oracle. Bounds as in tests/parity.py: similarities within the fp32
accumulation error, neighbour sets exact outside the band around the k-th
score, counts exact and masses within the bound that follows."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_07917_amd import sage, workloads
from tests import parity

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def check(w, k, layout, workspace=None):
    qb, hb = sage.ingest_bf16(dev(w.queries), layout), sage.ingest_bf16(dev(w.hist_emb), layout)
    out = [host(t) for t in sage.predict(qb, hb, dev(w.hist_len), k, 0.8, dev(w.bin_edges), workspace=workspace)]
    S = oracle.similarity(oracle.round_to_bf16(w.queries), oracle.round_to_bf16(w.hist_emb))
    parity.check_predict(*out, S, w.hist_len, w.bin_edges, 0.8, k)
    return out


@pytest.mark.parametrize("Q,N,d,k,layout", [
    (17, 32769, 32, 64, "rows"),        # 128-query tile, one row past the stores whose scores are all written
    (64, 33024, 64, 16, "panels"),      # 129 whole steps, each a chunk with a small segment
    (65, 140000, 96, 64, "panels"),     # more chunks than 512: two steps each
    (128, 40000, 384, 50, "rows"),      # the whole 128-query tile
    (129, 40001, 64, 64, "panels"),     # one query into the 256-query tile
    (257, 33333, 96, 32, "panels"),     # two tiles, four waves per query in the select
    (2049, 9000, 32, 64, "rows"),       # nine tiles, at most 64 chunks, one wave per query
    (321, 16384, 64, 128, "panels"),    # k > 64: the smallest store with a pre-pass at k = 128
    (300, 40000, 96, 65, "rows"),       # two list registers per lane, four waves per query
    (129, 65537, 32, 256, "panels"),    # four list registers, sixteen waves
    (2100, 33000, 32, 200, "rows"),     # ... and one wave per query
    (2100, 33000, 32, 128, "panels"),   # two list registers and one wave per query
])
def test_filtered_search_edges(Q, N, d, k, layout):
    print(f"case Q={Q} N={N} d={d} k={k} {layout}", flush=True)
    w = workloads.small_predict(Q=Q, N=N, d=d, k=k, B=64, seed=Q + N + k, clusters=12)
    ws = torch.empty(sage.predict_workspace_bytes(Q, N, d, k, 64), dtype=torch.uint8, device="cuda")
    check(w, k, layout, ws)
    stats = sage.predict_stats(ws, Q, N, d, k, 64)
    assert stats["path"] == "filtered" and stats["flagged"] == 0


@pytest.mark.parametrize("Q,k", [(300, 100), (40, 256)])
def test_long_lists_on_the_exact_fallback(Q, k):
    """theta0 raised from the host until about half, then all, of the queries
    have fewer than k candidates: the exact lists of 128 and 256 keys answer
    them with the unforced run's bits (both compute the same fp32 scores)."""
    w = workloads.small_predict(Q=Q, N=50000, d=96, k=k, B=64, seed=77 + k, clusters=6)
    base = check(w, k, "panels")
    try:
        for floor in (float(np.median(base[1][:, k - 1])), 2.0):
            sage.debug_theta_floor(floor)
            for a, b in zip(base, check(w, k, "panels")):
                assert np.array_equal(a.view(np.uint8), b.view(np.uint8)), f"floor {floor}"
    finally:
        sage.debug_theta_floor(-np.inf)


@pytest.mark.parametrize("Q", [40, 200])
def test_full_segments_spill(Q):
    """200 rows of one 256-row step (its whole chunk here) lie around the first
    queries' cluster, more than a segment of 32 keys holds: the keys past it go
    to the spill arrays, and no query to the exact path."""
    N, d, k, B = 139 * 256, 64, 16, 32
    print(f"case Q={Q}", flush=True)
    w = workloads.small_predict(Q=Q, N=N, d=d, k=k, B=B, seed=31 + Q, clusters=12)
    rng = np.random.default_rng(4)
    x = w.queries[0] + 0.02 * rng.standard_normal((200, d)).astype(np.float32)
    w.hist_emb[300:500] = x / np.linalg.norm(x, axis=1, keepdims=True)
    ws = torch.empty(sage.predict_workspace_bytes(Q, N, d, k, B), dtype=torch.uint8, device="cuda")
    ids = check(w, k, "panels", ws)[0]
    stats = sage.predict_stats(ws, Q, N, d, k, B)
    assert stats["path"] == "filtered" and stats["segment_capacity"] == 32 and stats["flagged"] == 0
    assert np.all((ids[0] >= 300) & (ids[0] < 500))


@pytest.mark.parametrize("Q,N,d,k,layout", [
    (1, 1, 32, 1, "rows"),              # one score
    (3, 31, 64, 64, "panels"),          # fewer rows than neighbours: padded
    (32, 1023, 96, 16, "rows"),         # a whole query tile; less than one score per thread
    (33, 1025, 416, 64, "panels"),      # one query and one row past; 13 panels: two rounds of loads
    (5, 10000, 768, 128, "rows"),       # two list registers, every fourth thread a group
    (160, 32768, 32, 129, "panels"),    # the largest store; a group per thread; as many scores as allowed
    (7, 20011, 64, 256, "rows"),
    (97, 20011, 224, 50, "panels"),     # two history tiles per wave, the last one ragged
])
def test_dense_search_edges(Q, N, d, k, layout):
    """Stores small enough that every score is written out."""
    print(f"case Q={Q} N={N} d={d} k={k} {layout}", flush=True)
    w = workloads.small_predict(Q=Q, N=N, d=d, k=k, B=64, seed=Q + N + k, clusters=4)
    ws = torch.empty(sage.predict_workspace_bytes(Q, N, d, k, 64), dtype=torch.uint8, device="cuda")
    check(w, k, layout, ws)
    assert sage.predict_stats(ws, Q, N, d, k, 64)["path"] == "dense"


@pytest.mark.parametrize("Q,N,d,k,path", [
    (256, 300, 64, 32, "dense"), (1024, 2000, 64, 32, "dense"), (1025, 300, 64, 32, "filtered"),
    (1024, 300, 64, 32, "filtered"),    # few rows: a workgroup of 16 waves per query is too many
    (1024, 300, 64, 65, "dense"), (1025, 2500, 64, 100, "lists"),
    (1024, 100, 64, 256, "lists"), (600, 20, 64, 129, "lists"), (300, 100, 64, 256, "dense"), (1024, 100, 64, 128, "dense"),
    (3000, 40, 64, 64, "filtered"),
    # no pre-pass: every row of a chunk is a candidate
    (1025, 8191, 32, 64, "filtered"),   # the largest such store, its last step and quad cut
    (1300, 255, 64, 8, "filtered"),
    (16000, 514, 32, 64, "filtered"),   # chunks of two steps and of two rows
    (100, 1027, 8224, 64, "filtered"),  # the 128-query tile
])
def test_batches_past_the_dense_search(Q, N, d, k, path):
    print(f"case Q={Q} N={N} d={d} k={k}", flush=True)
    w = workloads.small_predict(Q=Q, N=N, d=d, k=k, B=64, seed=Q + N + k, clusters=4)
    ws = torch.empty(sage.predict_workspace_bytes(Q, N, d, k, 64), dtype=torch.uint8, device="cuda")
    check(w, k, "panels", ws)
    assert sage.predict_stats(ws, Q, N, d, k, 64)["path"] == path


@pytest.mark.parametrize("Q,N,d,k", [(512, 10000, 768, 64), (1024, 2500, 384, 32), (300, 6000, 4096, 50)])
def test_search_chosen_by_layout(Q, N, d, k):
    """Sizes at which panels are searched by writing every score out and rows are
    filtered: one workspace serves both in turn, predict_stats tells which ran,
    and the bits are the same; one operand in rows counts as rows."""
    B = 64
    print(f"case Q={Q} N={N} d={d} k={k}", flush=True)
    w = workloads.small_predict(Q=Q, N=N, d=d, k=k, B=B, seed=Q + N + k, clusters=8)
    ws = torch.empty(sage.predict_workspace_bytes(Q, N, d, k, B), dtype=torch.uint8, device="cuda")
    hist_len, edges = dev(w.hist_len), dev(w.bin_edges)
    emb = {lay: (sage.ingest_bf16(dev(w.queries), lay), sage.ingest_bf16(dev(w.hist_emb), lay))
           for lay in ("rows", "panels")}
    outs = []
    for ql, hl, path in (("panels", "panels", "dense"), ("rows", "rows", "filtered"), ("panels", "panels", "dense"),
                         ("rows", "panels", "filtered"), ("panels", "rows", "filtered")):
        out = sage.predict(emb[ql][0], emb[hl][1], hist_len, k, 0.8, edges, workspace=ws)
        stats = sage.predict_stats(ws, Q, N, d, k, B)
        assert stats["path"] == path and stats["flagged"] == 0, (ql, hl)
        outs.append([host(t) for t in out])
        if Q * 8192 * 8 < 60 << 20 and N < 9000:      # both fit the static scratch: either way without a workspace
            again = [torch.full_like(t, 7) for t in out]
            assert sage.load_library().sage_predict_noalloc(
                emb[ql][0].data_ptr(), sage.LAYOUTS[ql], Q, emb[hl][1].data_ptr(), sage.LAYOUTS[hl], hist_len.data_ptr(),
                N, d, k, 0.8, edges.data_ptr(), B, *[t.data_ptr() for t in again], sage._stream()) == 0
            outs.append([host(t) for t in again])
    for other in outs[1:]:
        for a, b in zip(outs[0], other):
            assert np.array_equal(a.view(np.uint8), b.view(np.uint8))
    S = oracle.similarity(oracle.round_to_bf16(w.queries), oracle.round_to_bf16(w.hist_emb))
    parity.check_predict(*outs[0], S, w.hist_len, w.bin_edges, 0.8, k)


@pytest.mark.parametrize("Q,k,path,cap", [
    (12, 8, "stream", 4096),        # the stream search's array
    (12, 128, "stream", 0),
    (100, 64, "filtered", 0),       # more than 64 chunks: segments and the spill array
    (300, 100, "filtered", 0),      # k > 64: the same
    (300, 256, "filtered", 0),
    (2200, 32, "filtered", 0),      # segments without a spill array, one wave per query in the select
    (2200, 128, "filtered", 0),     # with one, two list registers
    (2200, 200, "filtered", 0),     # four
])
@pytest.mark.parametrize("layout", ["panels", "rows"])
def test_overflowing_candidates_take_the_exact_path(Q, k, path, cap, layout):
    """Half of the store repeats one row: a query equal to it has more candidates
    than any array holds, and is answered by the exact path (the lowest ids of
    the copies, in order); the others are not disturbed. Every seventh query is
    one, so that tiles hold both."""
    N, d, B = 60000, 64, 16
    print(f"case Q={Q} k={k} {layout}", flush=True)
    w = workloads.small_predict(Q=Q, N=N, d=d, k=k, B=B, seed=21 + Q + k, clusters=12)
    w.hist_emb[: N // 2] = w.hist_emb[N // 2]
    w.queries[::7] = w.hist_emb[N // 2]
    qb, hb = sage.ingest_bf16(dev(w.queries), layout), sage.ingest_bf16(dev(w.hist_emb), layout)
    ws = torch.empty(sage.predict_workspace_bytes(Q, N, d, k, B), dtype=torch.uint8, device="cuda")
    for _ in range(2):                               # the second call with the first one's counters and flags
        out = [host(t) for t in sage.predict(qb, hb, dev(w.hist_len), k, 0.8, dev(w.bin_edges), workspace=ws)]
        stats = sage.predict_stats(ws, Q, N, d, k, B)
        assert stats["path"] == path and len(w.queries[::7]) <= stats["flagged"] < Q
        assert cap == 0 or stats["segment_capacity"] == cap
        assert np.array_equal(out[0][::7], np.tile(np.arange(k), (len(w.queries[::7]), 1)))
    rows = np.unique(np.concatenate([np.arange(0, Q, max(1, Q // 60)), [Q - 1]]))
    S = oracle.similarity(oracle.round_to_bf16(w.queries[rows]), oracle.round_to_bf16(w.hist_emb))
    parity.check_predict(*[t[rows] for t in out], S, w.hist_len, w.bin_edges, 0.8, k)


@pytest.mark.parametrize("Q,N,k", [(2047, 100000, 128), (2048, 100000, 128), (1001, 100003, 128), (481, 60001, 256),
                                   (963, 50000, 100), (327, 500000, 256)])
def test_long_lists_of_any_batch_are_filtered(Q, N, k):
    """k > 64 with a workspace of its own takes the filtered search, whether or
    not the exact lists would fit the scratch of sage_predict_noalloc; that call
    takes them where only they fit (all but the fourth: lists of 128 and, the
    last, 256 keys, with the threshold of their own sample), and gives the same
    bits."""
    d, B = 32, 16
    print(f"case Q={Q} N={N} k={k}", flush=True)
    w = workloads.small_predict(Q=Q, N=N, d=d, k=k, B=B, seed=Q + N + k, clusters=12)
    qb, hb = sage.ingest_bf16(dev(w.queries), "panels"), sage.ingest_bf16(dev(w.hist_emb), "panels")
    hist_len, edges = dev(w.hist_len), dev(w.bin_edges)
    need = sage.predict_workspace_bytes(Q, N, d, k, B)
    assert (need > 64 << 20) == (Q != 481)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    out = sage.predict(qb, hb, hist_len, k, 0.8, edges, workspace=ws)
    stats = sage.predict_stats(ws, Q, N, d, k, B)
    assert stats["path"] == "filtered" and stats["flagged"] == 0
    rows = np.unique(np.linspace(0, Q - 1, 64).astype(int))
    S = oracle.similarity(oracle.round_to_bf16(w.queries[rows]), oracle.round_to_bf16(w.hist_emb))
    parity.check_predict(*[host(t)[rows] for t in out], S, w.hist_len, w.bin_edges, 0.8, k)
    again = [torch.full_like(t, 7) for t in out]
    assert sage.load_library().sage_predict_noalloc(
        qb.data_ptr(), 1, Q, hb.data_ptr(), 1, hist_len.data_ptr(), N, d, k, 0.8, edges.data_ptr(), B,
        *[t.data_ptr() for t in again], sage._stream()) == 0
    for a, b in zip(out, again):
        assert np.array_equal(host(a).view(np.uint8), host(b).view(np.uint8))


@pytest.mark.parametrize("k", [16, 100, 256])
def test_dense_search_many_equal_scores(k):
    """6,000 copies of one row: more keys reach the bound than the select
    gathers, so every wave folds its keys; the lowest ids come first."""
    w = workloads.small_predict(Q=9, N=12000, d=64, k=k, B=16, seed=21, clusters=4)
    w.hist_emb[:6000] = w.hist_emb[6000]
    w.queries[:4] = w.hist_emb[6000]
    ids = check(w, k, "rows")[0]
    assert list(ids[0]) == list(range(k))
