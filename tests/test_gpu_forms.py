"""Shapes beside the usual ones of the training, encoding, rerank and list-sorting
kernels, at the edges of the rules that split their work."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from gpu_common import L, api, gpu_graph, gpu_vectors, host, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,F,H,T", [(2047, 14, 16, 2), (2048, 14, 16, 2), (4099, 1, 1, 1), (6001, 33, 33, 3),
                                     (2050, 14, 64, 16), (5000, 110, 40, 16), (3000, 250, 64, 16), (2300, 60, 20, 9)])
def test_mlp_large_batches(B, F, H, T):
    """Gradient sums of batches whose units are split over blocks (1 to 16
    partial sums beside each other in a wave); every result is an f32 sum in 256
    partial sums and a tree, of terms of both signs: 1e-5 of its norm."""
    say("mlp large", B, F, H, T)
    A = api()
    g = np.random.default_rng(B)
    X, Y, W = (g.standard_normal(s).astype(np.float32) for s in ((B, F), (B, T), (B, T)))
    W = np.abs(W)
    W1, b1, W2, b2 = ((g.standard_normal(s) * 0.3).astype(np.float32) for s in ((H, F), (H,), (T, H), (T,)))
    ref_loss, ref_g = orc.mlp_loss_grad(X, Y, W1, b1, W2, b2, W)
    loss, grads = A.mlp_backward(to_dev(X), to_dev(Y), *(to_dev(a) for a in (W1, b1, W2, b2)), w=to_dev(W))
    for got, ref in zip([loss, *grads], [np.array([ref_loss]), *ref_g]):
        assert np.linalg.norm(host(got) - ref) <= 1e-5 * np.linalg.norm(ref) + 1e-7


@pytest.mark.parametrize("n", [1, 3, 130])
@pytest.mark.parametrize("dim,pitch", [(128, None), (129, None), (132, None), (252, 384), (256, None), (257, None),
                                       (300, 512), (515, None), (960, None)])
def test_encode_wide_rows(n, dim, pitch):
    """Rows of one and of several steps of a wave, ragged ends and wide padding,
    the scale beside the rows and in them, byte for byte."""
    A, Lb = api(), L()
    g = np.random.default_rng(dim + n)
    x = (g.standard_normal((n, dim)) * 10.0 ** g.integers(-6, 4, size=(n, 1))).astype(np.float32)
    for dt, odt, esz, inrow in ((Lb.F32, orc.F32, 4, False), (Lb.F16, orc.F16, 2, False), (Lb.BF16, orc.BF16, 2, False),
                                (Lb.FP8_E4M3, orc.FP8, 1, False), (Lb.FP8_E4M3, orc.FP8, 1, True)):
        if pitch is not None and pitch < dim * esz + 16:
            continue
        say("encode wide", n, dim, pitch, dt, inrow)
        v = A.encode(to_dev(x), dt, Lb.L2SQ, pitch=pitch, scale_in_row=inrow)
        codes = host(v.data)
        ref, rs = orc.encode_rows(x, odt, pitch=v.pitch)
        codes = codes.view(np.uint8).reshape(n, -1)
        ref = ref.view(np.uint8).reshape(n, -1)
        if inrow:
            assert np.array_equal(codes[:, -4:].copy().view(np.float32)[:, 0], rs)
            codes, ref = codes[:, :-4], ref[:, :-4]
        elif rs is not None:
            assert np.array_equal(host(v.scale), rs)
        assert np.array_equal(codes, ref)


@pytest.mark.parametrize("pool", [1, 3, 4, 5])
@pytest.mark.parametrize("nq,dim,metric", [(1, 8, orc.L2SQ), (700, 65, orc.COS), (40_000, 5, orc.L2SQ)])
def test_rerank_small_pools(nq, pool, dim, metric):
    """Pools that the four lane groups of a wave hold at once, and one row more;
    whole numbers, so that f32 and f64 sums are exact; some places empty."""
    say("rerank small pool", nq, pool, dim)
    A = api()
    g = np.random.default_rng(pool + nq)
    x, q = (g.integers(-7, 8, (n, dim)).astype(np.float32) for n in (500, nq))
    ids = np.argsort(g.random((nq, 500)), axis=1)[:, :pool].astype(np.int32)
    ids[::3, pool // 2] = -1
    k = min(3, pool)
    rid, rd = orc.rerank(orc.Vectors.from_array(q, metric), orc.Vectors.from_array(x, metric), ids, k)
    for f64 in (False, True):
        gid, gd = A.rerank(gpu_vectors(q, metric), gpu_vectors(x, metric), to_dev(ids), k, use_f64=f64)
        assert np.array_equal(host(gid), rid)
        assert np.array_equal(host(gd).astype(np.float64), rd)


@pytest.mark.parametrize("n", [1, 2, 1023, 1024, 1025, 1500])
def test_list_sorts_around_the_queue(n):
    """Degree adjustments and edge insertion with as many lists as are sorted
    without a queue, and one more: hubs of all lengths among short lists, empty
    ones too; bit-exact."""
    say("list sorts", n)
    A, Lb = api(), L()
    g = np.random.default_rng(n)
    k = min(7, max(n - 1, 1))
    ids = np.empty((n, k), dtype=np.int32)
    d = np.empty((n, k), dtype=np.int32)
    for v in range(n):
        r = np.concatenate([g.permutation(min(n, 3)), 3 + g.permutation(max(n - 3, 0))])
        r = r[r != v][:k]
        o = np.lexsort((r, ln := np.sort(g.integers(1, 9, size=len(r)))))
        ids[v], d[v] = -1, np.iinfo(np.int32).max
        ids[v, :len(r)], d[v, :len(r)] = r[o], ln[o]
    for eo, ei in ((k, k), (0, 2), (2, 0), (3, 5)):
        for mine, ref in ((A.adjust_degree, orc.adjust_degree), (A.adjust_degree_constrained, orc.adjust_degree_constrained)):
            off, nb, ln = ref(ids, d.astype(np.float64), eo, ei)
            got = mine(to_dev(ids), to_dev(d), Lb.U8, Lb.L2SQ, eo, ei)
            assert np.array_equal(host(got.offsets), off)
            assert np.array_equal(host(got.nbrs), nb)
            assert np.array_equal(host(got.lens), ln.astype(np.int32))
    m = 5000
    src = np.where(g.random(m) < 0.3, 0, g.integers(0, n, size=m)).astype(np.int32)
    dst, ln = g.integers(0, n, size=m).astype(np.int32), g.integers(1, 50, size=m).astype(np.int32)
    e = np.zeros(n + 1, dtype=np.int64)
    out = A.graph_add_edges(gpu_graph(e, np.zeros(0, np.int32), np.zeros(0, np.int32)), to_dev(src), to_dev(dst),
                            to_dev(ln), Lb.U8, Lb.L2SQ)
    o = np.lexsort((dst, ln, src))
    assert np.array_equal(host(out.nbrs), dst[o])
    assert np.array_equal(host(out.lens), ln[o])


@pytest.mark.parametrize("n", [2, 40, 3999, 4001])
@pytest.mark.parametrize("k,eo,ei", [(1, 1, 1), (5, 5, 5), (5, 0, 5), (5, 4, 0), (30, 3, 5), (30, 5, 1), (30, 6, 5)])
def test_degree_adjustment_short_rows(n, k, eo, ei):
    """Algorithm 2 with few edges a row, over the rule that a lane takes a row,
    below and above its number of nodes; rows with padding and hubs; bit-exact."""
    say("degree short rows", n, k, eo, ei)
    A, Lb = api(), L()
    g = np.random.default_rng(n + k)
    k = min(k, n - 1)
    ids = np.full((n, k), -1, dtype=np.int32)
    d = np.full((n, k), np.iinfo(np.int32).max, dtype=np.int32)
    for v in range(n):
        r = np.concatenate([g.permutation(2), 2 + g.permutation(min(n - 2, 60))]) if v % 3 else (v + 1 + g.permutation(min(n - 1, 40))) % n
        r = r[r != v][:k if v % 5 else int(g.integers(0, k + 1))]
        ln = np.sort(g.integers(1, 9, size=len(r)))
        o = np.lexsort((r, ln))
        ids[v, :len(r)], d[v, :len(r)] = r[o], ln[o]
    off, nb, ln = orc.adjust_degree(ids, d.astype(np.float64), eo, ei)
    for dt, dd in ((Lb.U8, d), (Lb.F32, np.where(ids >= 0, d * 0.5, np.inf).astype(np.float32))):
        got = A.adjust_degree(to_dev(ids), to_dev(dd), dt, Lb.L2SQ, eo, ei)
        assert np.array_equal(host(got.offsets), off)
        assert np.array_equal(host(got.nbrs), nb)
        assert np.array_equal(host(got.lens).astype(np.float64), ln if dt == Lb.U8 else ln * 0.5)
