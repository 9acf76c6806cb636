"""Kernels at the sizes where their work splits change: list lengths around
the classes and chunks of the adjustments, tile and remainder edges of the
others, each against the oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from gpu_common import L, api, gpu_graph, gpu_vectors, host, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("deg", [64, 65, 128, 129, 512, 513, 2048, 2049, 4097])
def test_adjust_path_list_length_classes(deg):
    """Hubs whose lists end just at and past the node classes (128, 512) and
    the target chunks (2048) of the path adjustment, among ordinary nodes,
    with ties, repeated neighbours and self edges; bit-exact."""
    say("adjust_path list length", deg)
    A, Lb = api(), L()
    g = np.random.default_rng(deg)
    n = 700
    offs, nbs, lns = [0], [], []
    for v in range(n):
        m = deg if v in (0, 5, 351, n - 1) else deg - 1 if v == 350 else int(g.integers(0, 40))
        nb = g.integers(0, n, size=m)
        ln = g.integers(1, 200, size=m)
        o = np.lexsort((nb, ln))
        nbs.append(nb[o]); lns.append(ln[o]); offs.append(offs[-1] + m)
    off = np.array(offs, dtype=np.int64)
    nb = np.concatenate(nbs).astype(np.int32)
    ln = np.concatenate(lns).astype(np.int32)
    po, pn, pl = orc.adjust_path(off, nb, ln)
    for dt, lens in ((Lb.U8, ln), (Lb.F32, ln.astype(np.float32) * 0.25)):
        gg = A.adjust_path(gpu_graph(off, nb, lens, int_len=dt == Lb.U8), dt, Lb.L2SQ)
        assert np.array_equal(host(gg.offsets), po)
        assert np.array_equal(host(gg.nbrs), pn)
        assert np.array_equal(host(gg.lens), pl * (1 if dt == Lb.U8 else 0.25))


def knn_like_table(n, k, seed, hubs=0, pad=False):
    """Rows of k distinct ids (the first `hubs` rows' ids near the head of
    every row), (distance, id)-sorted with many ties; some rows padded."""
    g = np.random.default_rng(seed)
    ids = np.empty((n, k), dtype=np.int32)
    d = np.empty((n, k), dtype=np.int32)
    for v in range(n):
        r = g.permutation(n)[:k + hubs + 1]
        if hubs:
            r = np.concatenate([g.permutation(hubs), r[r >= hubs]])
        r = r[r != v][:k]
        ln = np.sort(g.integers(1, 3 * k, size=k))
        o = np.lexsort((r, ln))
        ids[v], d[v] = r[o], ln[o]
        if pad and v % 7 == 0:
            m = int(g.integers(0, k))
            ids[v, m:], d[v, m:] = -1, np.iinfo(np.int32).max
    return ids, d


@pytest.mark.parametrize("n,k,eo,ei,hubs,pad", [
    (300, 70, 64, 65, 0, False), (300, 150, 129, 150, 0, True), (500, 40, 0, 40, 3, False),
    (500, 40, 40, 0, 0, True), (300, 9, 3, 7, 2, True), (4300, 5, 2, 5, 2, False)])
def test_degree_adjustments_list_lengths(n, k, eo, ei, hubs, pad):
    """Algorithms 2 and 3 on tables whose rows need one, two and three 64-lane
    steps, with padded rows and hubs of up to n incoming edges (lists of one
    wave, of a block in LDS, and longer); bit-exact."""
    say("degree adjustments", n, k, eo, ei)
    A, Lb = api(), L()
    ids, d = knn_like_table(n, k, n + k, hubs, pad)
    for mine, ref in ((A.adjust_degree, orc.adjust_degree),
                      (A.adjust_degree_constrained, orc.adjust_degree_constrained)):
        off, nb, ln = ref(ids, d.astype(np.float64), eo, ei)
        got = mine(to_dev(ids), to_dev(d), Lb.U8, Lb.L2SQ, eo, ei)
        assert np.array_equal(host(got.offsets), off)
        assert np.array_equal(host(got.nbrs), nb)
        assert np.array_equal(host(got.lens), ln.astype(np.int32))


def test_edge_insertion_keeps_equal_edges():
    """Edges of equal length and target each keep a place in the list."""
    say("graph_add_edges repeats")
    A, Lb = api(), L()
    g = np.random.default_rng(5)
    n, m = 40, 3000
    src = g.integers(0, n, size=m).astype(np.int32)
    src[:700] = 3
    dst = g.integers(0, 6, size=m).astype(np.int32)
    ln = g.integers(1, 5, size=m).astype(np.int32)
    e = np.zeros(n + 1, dtype=np.int64)
    out = A.graph_add_edges(gpu_graph(e, np.zeros(0, np.int32), np.zeros(0, np.int32)), to_dev(src),
                            to_dev(dst), to_dev(ln), Lb.U8, Lb.L2SQ)
    o = np.lexsort((dst, ln, src))
    assert np.array_equal(host(out.nbrs), dst[o])
    assert np.array_equal(host(out.lens), ln[o])


@pytest.mark.parametrize("dim,pitch,inrow", [(1, None, True), (3, None, False), (100, 128, True), (127, None, True),
                                             (128, 160, False), (129, None, True), (260, None, False),
                                             (37, 37, False), (38, 42, False)])
def test_encode_row_shapes(dim, pitch, inrow):
    """Rows of every step of the four-element encoder (below, at and past 128
    components, ragged ends, wide padding) and of pitches that only the general
    form takes; byte for byte."""
    A, Lb = api(), L()
    g = np.random.default_rng(dim)
    x = (g.standard_normal((71, dim)) * 10.0 ** g.integers(-6, 4, size=(71, 1))).astype(np.float32)
    x[3] = 0.0
    for dt, odt, esz in ((Lb.F16, orc.F16, 2), (Lb.BF16, orc.BF16, 2), (Lb.FP8_E4M3, orc.FP8, 1)):
        if pitch is not None and pitch < dim * esz:
            continue
        if pitch is not None and pitch % 16 and dt == Lb.FP8_E4M3 and inrow:
            continue
        say("encode", dim, pitch, dt)
        row_in = inrow and dt == Lb.FP8_E4M3
        v = A.encode(to_dev(x), dt, Lb.L2SQ, pitch=pitch, scale_in_row=row_in)
        codes = host(v.data)
        ref, rs = orc.encode_rows(x, odt, pitch=v.pitch)
        if row_in:
            assert np.array_equal(codes[:, -4:].copy().view(np.float32)[:, 0], rs)
            codes, ref = codes[:, :-4], ref[:, :-4]
        elif rs is not None:
            assert np.array_equal(host(v.scale), rs)
        assert np.array_equal(codes, ref)


def test_encode_fp8_every_rounding_case():
    """Every e4m3 value, every midpoint of two of them and their f32
    neighbours (scale 1: the row's largest element is 448), and NaN."""
    say("encode fp8 grid")
    A, Lb = api(), L()
    vals = sorted({orc.decode(orc.FP8, c) for c in range(0x7f)})
    mid = [(a + b) / 2 for a, b in zip(vals, vals[1:])]
    v = np.array(vals + mid, dtype=np.float32)
    v = np.concatenate([v, np.nextafter(v, np.float32(1e9)), np.nextafter(v, np.float32(-1e9))])
    v = v[np.abs(v) <= 448]
    v = np.concatenate([v, -v])
    rows = np.zeros((-(-len(v) // 99), 100), dtype=np.float32)
    rows[:, 0] = 448
    rows.reshape(-1)[np.flatnonzero(np.arange(rows.size) % 100 > 0)[:len(v)]] = v
    out = A.encode(to_dev(rows), Lb.FP8_E4M3, Lb.L2SQ)
    ref, rs = orc.encode_rows(rows, orc.FP8, pitch=out.pitch)
    assert np.array_equal(host(out.scale), rs)
    assert np.array_equal(host(out.data), ref)
    nan = np.array([[448, np.nan, -1.0, 2.0, 0.5, -np.nan, 1e-9, -448.0]], dtype=np.float32)
    nan[0, 5] = np.copysign(np.float32(np.nan), np.float32(-1))
    got = host(A.encode(to_dev(nan), Lb.FP8_E4M3, Lb.L2SQ).data)[0]
    assert got[:8].tolist() == [0x7e, 0x7f, 0xb8, 0x40, 0x30, 0xff, 0x00, 0xfe]


@pytest.mark.parametrize("nq,pool,dim,metric", [(1, 1, 3, orc.L2SQ), (3, 15, 64, orc.COS), (5, 65, 65, orc.L2SQ),
                                                (300, 128, 37, orc.COS), (2, 1000, 130, orc.L2SQ),
                                                (9000, 20, 100, orc.COS)])
def test_rerank_row_splits(nq, pool, dim, metric):
    """The rerank over lane-group remainders of the pool, components past 64
    and 128, and one to four waves per query.  f64: 1e-12 of the oracle; f32:
    a sum of at most dim terms, (dim / 64 + 8) roundings of 2^-24 each on
    terms whose magnitudes sum to at most |x|^2 + |q|^2 + |d|."""
    say("rerank", nq, pool, dim)
    A = api()
    g = np.random.default_rng(pool)
    x = g.standard_normal((1200, dim)).astype(np.float32)
    q = g.standard_normal((nq, dim)).astype(np.float32)
    if metric == orc.COS:
        x /= np.linalg.norm(x, axis=1, keepdims=True)
        q /= np.linalg.norm(q, axis=1, keepdims=True)
    ids = np.argsort(g.random((nq, 1200)), axis=1)[:, :pool].astype(np.int32)
    ids[:, pool // 2] = -1
    k = min(10, pool)
    bv, qv = orc.Vectors.from_array(x, metric), orc.Vectors.from_array(q, metric)
    rid, rd = orc.rerank(qv, bv, ids, k)
    gid, gd = A.rerank(gpu_vectors(q, metric), gpu_vectors(x, metric), to_dev(ids), k, use_f64=True)
    fin = np.isfinite(rd)
    assert np.array_equal(host(gid), rid)
    assert np.array_equal(np.isfinite(host(gd)), fin)
    assert np.allclose(host(gd)[fin], rd[fin], rtol=1e-12, atol=1e-12)
    _, gd = A.rerank(gpu_vectors(q, metric), gpu_vectors(x, metric), to_dev(ids), k)
    size = 2.0 * (1.0 if metric == orc.COS else rd[fin].max(initial=0.0))
    assert np.abs(host(gd)[fin] - rd[fin]).max(initial=0.0) <= (dim / 64 + 8) * 2.0 ** -24 * size
    if metric == orc.L2SQ and dim == 65:   # stored types other than f32
        for dt, odt in ((L().F16, orc.F16), (L().FP8_E4M3, orc.FP8)):
            lp = A.encode(to_dev(x), dt, L().L2SQ)
            codes, rs = orc.encode_rows(x, odt, pitch=lp.pitch)
            dec = np.array([orc.decode(odt, c) for c in range(256 if odt == orc.FP8 else 65536)])
            xd = dec[codes.view(np.uint16 if odt == orc.F16 else np.uint8)[:, :dim].astype(np.int64)]
            if rs is not None:
                xd = xd * rs[:, None].astype(np.float64)
            d = np.where(ids >= 0, ((xd[ids] - q[:, None, :].astype(np.float64)) ** 2).sum(2), np.inf)
            got = host(A.rerank(gpu_vectors(q, metric), lp, to_dev(ids), k, use_f64=True)[1])
            assert np.allclose(got, np.sort(d, axis=1)[:, :k], rtol=1e-12)


@pytest.mark.parametrize("B,F,H,T", [(1, 14, 64, 16), (5, 1, 1, 1), (63, 33, 33, 3), (1026, 32, 64, 16), (300, 70, 17, 5)])
def test_mlp_sizes(B, F, H, T):
    """Sample-group remainders, one to full widths, and inputs past the
    staged width; every result is an f32 sum of at most F + H + B terms in a
    fixed order: 1e-5 of its norm."""
    say("mlp", B, F, H, T)
    A = api()
    g = np.random.default_rng(B)
    X, Y, W = (g.standard_normal(s).astype(np.float32) for s in ((B, F), (B, T), (B, T)))
    W = np.abs(W)
    W1, b1, W2, b2 = ((g.standard_normal(s) * 0.3).astype(np.float32) for s in ((H, F), (H,), (T, H), (T,)))
    ref_h, ref_y = orc.mlp_forward(X, W1, b1, W2, b2)
    ref_loss, ref_g = orc.mlp_loss_grad(X, Y, W1, b1, W2, b2, W)
    dev_w = [to_dev(a) for a in (W1, b1, W2, b2)]
    y, hid = A.mlp_forward(to_dev(X), *dev_w, want_hidden=True)
    loss, grads = A.mlp_backward(to_dev(X), to_dev(Y), *dev_w, w=to_dev(W))
    for got, ref in zip([y, hid, loss, *grads], [ref_y, ref_h, np.array([ref_loss]), *ref_g]):
        assert np.linalg.norm(host(got) - ref) <= 1e-5 * np.linalg.norm(ref) + 1e-7


@pytest.mark.parametrize("kind,nq,nb,dim,k,form", [
    ("u8", 1, 1024, 128, 8, "cand"), ("u8", 16, 1023, 64, 10, ""), ("u8", 17, 1025, 65, 1, ""),
    ("u8", 64, 5000, 300, 40, "cand"), ("u8", 65, 4097, 17, 100, ""), ("u8", 1500, 1500, 40, 20, "self"),
    ("u8", 2049, 2049, 128, 100, "self"), ("u8", 129, 3000, 128, 256, ""), ("u8tie", 200, 6000, 4, 50, ""),
    ("u8tie", 1300, 1300, 3, 9, "self"), ("f32l2", 3, 70000, 96, 20, ""), ("f32l2", 130, 20000, 33, 100, "cand"),
    ("f32l2", 1100, 1100, 128, 10, "self"), ("f32l2", 20, 3000, 200, 5, ""), ("f32cos", 64, 2000, 100, 8, "cand"),
    ("f32cos", 300, 9000, 112, 74, ""), ("f32cos", 10, 1200, 256, 3, ""), ("f32tie", 90, 8000, 5, 30, ""),
    ("f32tie", 1040, 1040, 6, 12, "self")])
def test_topk_bound_and_filter(kind, nq, nb, dim, k, form):
    """Top-k by a bound and a filter at the edges of its layouts: 1 / 16 / 17 / 64
    / 65 / 128 / 129 query rows, base rows around 1024 and ragged tiles, one to
    all k-steps, k from 1 to 256, candidate lists, self exclusion, and rows of so
    few distinct distances that every candidate buffer overflows.  f32 rows hold
    small integers, whose distances are exact in f32: ids and distances equal
    the oracle's."""
    say("topk bound", kind, nq, nb, dim, k, form)
    A = api()
    g = np.random.default_rng(nb + k)
    n = nb + 500 if form == "cand" else nb
    metric = orc.COS if kind == "f32cos" else orc.L2SQ
    hi = 3 if kind.endswith("tie") else 200 if kind == "u8" else 9
    dt = np.uint8 if kind.startswith("u8") else np.float32
    x = g.integers(0, hi, size=(n, dim)).astype(dt)
    q = x if form == "self" else g.integers(0, hi, size=(nq, dim)).astype(dt)
    cand = g.permutation(n)[:nb].astype(np.int32) if form == "cand" else None
    bv, qv = orc.Vectors.from_array(x, metric), orc.Vectors.from_array(q, metric)
    B = gpu_vectors(x, metric)
    if form == "self":
        rid, rd = orc.knn_graph(bv, k)
        ids, d = A.build_knn(B, k)
    else:
        rid, rd = orc.topk(qv, bv, k, cand=cand)
        ids, d = A.topk(gpu_vectors(q, metric), B, k, cand=None if cand is None else to_dev(cand))
    assert np.array_equal(host(ids), rid)
    assert np.array_equal(host(d).astype(np.float64), rd)


@pytest.mark.parametrize("kind,n,dim,k", [("f32l2", 33000, 1, 5), ("f32l2", 33001, 33, 20), ("f32cos", 32800, 96, 256),
                                          ("f32l2", 40000, 128, 100), ("f32tie", 33000, 4, 20),
                                          ("u8", 65600, 64, 100), ("u8", 66000, 17, 10), ("u8tie", 65536, 3, 12)])
def test_topk_wide_bound_and_filter(kind, n, dim, k):
    """The wide two-pass kNN over its k-steps (one to four of 32 f16 components,
    one and two of 64 bytes), more than one chunk of query rows with a ragged
    last block, k up to 256, and rows whose few distinct distances overflow
    every candidate buffer; integer rows, whose f32 distances are exact, so the
    sampled rows equal the oracle's."""
    say("wide bound", kind, n, dim, k)
    A = api()
    g = np.random.default_rng(n + dim)
    metric = orc.COS if kind == "f32cos" else orc.L2SQ
    hi = 2 if kind.endswith("tie") else 250 if kind == "u8" else 16
    x = g.integers(0, hi, size=(n, dim)).astype(np.uint8 if kind.startswith("u8") else np.float32)
    if kind == "f32l2":
        x[:, 0] += np.arange(n) % 1009   # (one component alone has few distinct values)
    bv = orc.Vectors.from_array(x, metric)
    rows = np.unique(np.concatenate([np.arange(70), np.arange(n - 70, n), [255, 256, 16639, 16640, 32767],
                                     g.choice(n, 60, replace=False)])).astype(np.int32)
    rid, rd = orc.knn_graph(bv, k, rows=rows)
    ids, d = A.build_knn(gpu_vectors(x, metric), k)
    assert np.array_equal(host(ids)[rows], rid)
    assert np.array_equal(host(d)[rows].astype(np.float64), rd)


def _random_lists(n, degs, seed):
    """Lists of the given lengths in turn; ids at random, so that some repeat."""
    g = np.random.default_rng(seed)
    off = np.zeros(n + 1, np.int64)
    off[1:] = np.cumsum(np.resize(degs, n))
    return off, g.integers(0, n, off[-1]).astype(np.int32)


@pytest.mark.parametrize("kind,dim", [("u8", 16), ("u8", 128), ("f32", 17), ("f32", 100), ("f32", 128)])
@pytest.mark.parametrize("shape", [None, dict(visited_log2=-1, s_capacity=64)])
def test_search_batch_and_list_sizes(kind, dim, shape):
    """List lengths around the 64-edge chunks and the two of a pass, batches of
    every number of row passes, merges of few and of many keys.  The components
    are whole numbers, so that float distances are exact in any order: ids,
    distances and counts equal the oracle's."""
    n, nq = 2500, 6
    g = np.random.default_rng(dim)
    hi = 256 if kind == "u8" else 40
    x, q = (g.integers(0, hi, (m, dim)).astype(np.uint8 if kind == "u8" else np.float32) for m in (n, nq))
    off, nb = _random_lists(n, [0, 1, 3, 63, 64, 65, 127, 128, 129, 191, 257, 20, 33], 5)
    seeds = g.integers(0, n, (nq, 8)).astype(np.int32)
    seeds[:, 5] = seeds[:, 2]
    bv, qv = orc.Vectors.from_array(x, orc.L2SQ), orc.Vectors.from_array(q, orc.L2SQ)
    A = api()
    cfg = A.launch_config(**shape) if shape else None
    B, Q, G = gpu_vectors(x, orc.L2SQ), gpu_vectors(q, orc.L2SQ), gpu_graph(off, nb)
    for k, eps, ep in ((1, 0.0, orc.INF_EP), (4, 0.05, 65), (64, 0.1, orc.INF_EP), (100, 0.02, 130)):
        say("search sizes", kind, dim, shape, k, eps, ep)
        ref = orc.search(bv, off, nb, qv, seeds, k, eps, ep)
        r = A.search(B, G, Q, to_dev(seeds), k=k, eps=eps, ep=ep, launch=cfg)
        assert np.array_equal(host(r.ids), ref["ids"])
        d = host(r.dists).astype(np.float64)
        if kind == "u8":
            d[d == 2 ** 31 - 1] = np.inf
        assert np.array_equal(d, ref["dists"])
        assert np.array_equal(host(r.dc), ref["dc"])
        assert np.array_equal(host(r.hops), ref["hops"])


@pytest.mark.parametrize("nq", [1, 5, 1024, 1025])
def test_search_small_batch_window(nq):
    """The launch of a batch that leaves the chip idle (window of 2^18 ids, a
    block a wave) against the general one and the off-chip bitset."""
    n, dim = 140_000, 16
    g = np.random.default_rng(9)
    x, q = (g.integers(0, 256, (m, dim)).astype(np.uint8) for m in (n, nq))
    off, nb = _random_lists(n, [12, 70, 24], 6)
    A = api()
    B, Q, G = gpu_vectors(x, orc.L2SQ), gpu_vectors(q, orc.L2SQ), gpu_graph(off, nb)
    seeds = to_dev(g.integers(0, n, (nq, 8)).astype(np.int32))
    say("search window", nq)
    out = [A.search(B, G, Q, seeds, k=10, eps=0.1, ep=orc.INF_EP, launch=c)
           for c in (None, A.launch_config(visited_log2=11, waves_per_block=4),
                     A.launch_config(visited_log2=-1))]
    for r in out[1:]:
        for name in ("ids", "dists", "dc", "hops", "scanned"):
            assert np.array_equal(host(getattr(r, name)), host(getattr(out[0], name))), name


@pytest.mark.parametrize("nq", [5, 901, 1023])
def test_search_small_batch_scratch(nq):
    """Batches whose own launch is a block a wave: the static scratch (fewer
    slots than queries) and the autotuner on the default workspace take them as
    they take larger ones."""
    n, dim = 12_000, 32
    g = np.random.default_rng(nq)
    x, q = (g.integers(0, 256, (m, dim)).astype(np.uint8) for m in (n, nq))
    off, nb = _random_lists(n, [12, 70, 24], 6)
    A = api()
    B, Q, G = gpu_vectors(x, orc.L2SQ), gpu_vectors(q, orc.L2SQ), gpu_graph(off, nb)
    seeds = to_dev(g.integers(0, n, (nq, 8)).astype(np.int32))
    say("search scratch", nq)
    kw = dict(k=10, eps=0.05, ep=40)
    ref = A.search(B, G, Q, seeds, **kw)
    ids, dc = host(ref.ids), host(ref.dc)
    got = A.search(B, G, Q, seeds, static_scratch=True, **kw)
    assert np.array_equal(host(got.ids), ids) and np.array_equal(host(got.dc), dc)
    r = A.SearchRequest(B, G, Q, seeds, **kw)
    ws = r.ws.numel()
    best = r.autotune()
    # the largest shape the tuner tries has the default one's slots
    assert best.waves_per_block in (2, 4) and r.ws_bytes <= ws
    r.run()
    assert np.array_equal(host(r.ids), ids) and np.array_equal(host(r.dc), dc)
