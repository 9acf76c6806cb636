"""Top-k over the forms of its arguments that change its path: far u8 rows,
candidate lists with self exclusion and with repeats, and rows of one buffer at
two pitches; ids and distances against the oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from gpu_common import L, api, gpu_vectors, host, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,nq", [(259, 3), (259, 60), (300, 200), (512, 16), (512, 130), (512, 0)])
def test_topk_u8_distances_past_24_bits(dim, nq):
    """u8 rows whose squared distances exceed 2^24 (from 259 components on; at
    512 up to 33,292,800), in each of the three block shapes; nq = 0: a kNN
    table of two far groups, the smaller of fewer than k rows."""
    say("topk far u8", dim, nq)
    A = api()
    g = np.random.default_rng(dim + nq)
    nb, k = 1100, 40
    x = (g.random((nb, dim)) < 0.25).astype(np.uint8)
    far = 255 - (g.random((max(nq, 25), dim)) < 0.02 * (dim > 259)).astype(np.uint8)
    if nq:
        rid, rd = orc.topk(orc.Vectors.from_array(far, orc.L2SQ), orc.Vectors.from_array(x, orc.L2SQ), k)
        ids, d = A.topk(gpu_vectors(far, orc.L2SQ), gpu_vectors(x, orc.L2SQ), k)
        assert rd.min() > 2 ** 24
    else:
        x[::44] = far[:25]
        rid, rd = orc.knn_graph(orc.Vectors.from_array(x, orc.L2SQ), k)
        ids, d = A.build_knn(gpu_vectors(x, orc.L2SQ), k)
        assert (rd[::44, 24:] > 2 ** 24).all()
    assert np.array_equal(host(ids), rid)
    assert np.array_equal(host(d).astype(np.float64), rd)


@pytest.mark.parametrize("kind,n,nq,nc,k", [
    ("u8", 5000, 12, 1500, 8), ("u8", 5000, 60, 1024, 20), ("u8", 1700, 1700, 1600, 8), ("u8", 65536, 65536, 1100, 8),
    ("u8", 900, 900, 500, 8), ("f32l2", 5000, 12, 1500, 8), ("f32cos", 1700, 1700, 1600, 20),
    ("f32l2", 32768, 32768, 1100, 8), ("f32cos", 32768, 32768, 1500, 20)])
@pytest.mark.parametrize("repeat", [False, True])
def test_topk_candidates_without_self(kind, n, nq, nc, k, repeat):
    """A candidate list (in no order) with self exclusion: the base id that
    equals the query's row is left out, wherever it stands in the list.  With
    `repeat` the list also holds some rows' own ids many times over: all copies
    are left out there and kept elsewhere.  Narrow and wide forms, with f32
    rows of small whole numbers, whose distances are exact."""
    say("topk candidates without self", kind, n, nq, nc, repeat)
    A = api()
    g = np.random.default_rng(n + nq + nc)
    metric = orc.COS if kind == "f32cos" else orc.L2SQ
    dim = 24
    x = g.integers(0, 250 if kind == "u8" else 14, (n, dim)).astype(np.uint8 if kind == "u8" else np.float32)
    cand = g.permutation(n)[:nc].astype(np.int32)
    own = [1, nq // 2, nq - 1]
    cand[g.permutation(nc)[:3]] = own
    if repeat:
        at = g.permutation(nc)[:90]
        cand[at] = np.repeat(own, 30)
    rows = np.unique(np.concatenate([own, g.choice(nq, min(nq, 150), replace=False),
                                     [c for c in cand if c < nq][:60], np.arange(min(nq, 20))]))
    bv = orc.Vectors.from_array(x, metric)
    rid, rd = orc.topk(bv, bv, k, q_rows=rows, cand=cand, exclude_self=True)
    ids, d = A.topk(gpu_vectors(x[:nq], metric), gpu_vectors(x, metric), k, cand=to_dev(cand), exclude_self=True)
    assert np.array_equal(host(ids)[rows], rid)
    assert np.array_equal(host(d)[rows].astype(np.float64), rd)


@pytest.mark.parametrize("dtype", [torch.uint8, torch.float32])
def test_topk_one_buffer_two_pitches(dtype):
    """Queries and base over one buffer, the same number of rows, the base's
    twice as far apart: the queries are the buffer's first rows, not the base's."""
    say("topk two pitches", dtype)
    A, Lb = api(), L()
    n, k, dim = 65536, 8, 16 if dtype == torch.uint8 else 4
    g = np.random.default_rng(4)
    buf = g.integers(0, 250 if dtype == torch.uint8 else 30, (2 * n, dim)).astype(
        np.uint8 if dtype == torch.uint8 else np.float32)
    t = to_dev(buf)
    Q = A.Vectors(t[:n], Lb.U8 if dtype == torch.uint8 else Lb.F32, Lb.L2SQ, dim)
    B = A.Vectors(t.view(n, 2 * dim), Q.dtype, Lb.L2SQ, dim)
    rows = np.unique(np.concatenate([np.arange(40), g.choice(n, 60, replace=False), [n - 1]]))
    rid, rd = orc.topk(orc.Vectors.from_array(buf[:n], orc.L2SQ),
                       orc.Vectors.from_array(np.ascontiguousarray(buf[::2]), orc.L2SQ), k, q_rows=rows)
    ids, d = A.topk(Q, B, k)
    assert np.array_equal(host(ids)[rows], rid)
    assert np.array_equal(host(d)[rows].astype(np.float64), rd)


def test_topk_rows_past_the_screen_scale():
    """f32 rows whose components overflow f16, beside one row whose squared
    length overflows f32, so that no power of two brings all into f16's range:
    the other rows' neighbours are those of the f32 distances (odd multiples of
    2^17, whose squared differences sum exactly)."""
    say("topk past the screen's scale")
    A = api()
    g = np.random.default_rng(3)
    n, dim, k = 33000, 9, 8
    x = ((2 * g.integers(-4, 4, (n, dim)) + 1) * 2.0 ** 17).astype(np.float32)
    x[n // 2] = 1e20
    rows = np.setdiff1d(np.unique(np.concatenate([np.arange(40), g.choice(n, 80, replace=False)])), [n // 2])
    rid, rd = orc.knn_graph(orc.Vectors.from_array(x, orc.L2SQ), k, rows=rows)
    ids, d = A.build_knn(gpu_vectors(x, orc.L2SQ), k)
    assert np.array_equal(host(d)[rows].astype(np.float64), rd)
    assert np.array_equal(host(ids)[rows], rid)


@pytest.mark.parametrize("kind,nq", [("u8", 66000), ("f32l2", 65537)])
def test_topk_query_chunks(kind, nq):
    """More query rows of over 128 components than one pass holds candidates
    for: rows around the cut, with a candidate list and self exclusion, some of
    them redone (all components equal, so tied with many)."""
    say("topk query chunks", kind, nq)
    A = api()
    g = np.random.default_rng(nq)
    dim, k = 130, 8
    x = g.integers(0, 250 if kind == "u8" else 5, (nq, dim)).astype(np.uint8 if kind == "u8" else np.float32)
    x[g.permutation(nq)[:nq // 2]] = 2
    cand = g.permutation(nq)[:1500].astype(np.int32)
    cut = -(-(nq // 2) // 128) * 128
    rows = np.unique(np.concatenate([np.arange(20), np.arange(cut - 140, cut + 140), [nq - 1], cand[:60]]))
    bv = orc.Vectors.from_array(x, orc.L2SQ)
    rid, rd = orc.topk(bv, bv, k, q_rows=rows, cand=cand, exclude_self=True)
    V = gpu_vectors(x, orc.L2SQ)
    ids, d = A.topk(V, V, k, cand=to_dev(cand), exclude_self=True)
    assert np.array_equal(host(ids)[rows], rid)
    assert np.array_equal(host(d)[rows].astype(np.float64), rd)


@pytest.mark.parametrize("kind,n,dim,k,equal", [
    ("u8", 1500, 20, 8, 1.0), ("u8", 6000, 300, 100, 0.4), ("f32l2", 20000, 33, 8, 0.5), ("f32cos", 1100, 12, 20, 1.0),
    ("u8", 65536, 16, 20, 0.1), ("u8", 65600, 100, 100, 1.0), ("f32l2", 32768, 40, 30, 0.2), ("f32cos", 33000, 8, 10, 1.0)])
def test_topk_many_equal_rows(kind, n, dim, k, equal):
    """Rows of which a share are equal, so that their queries' bounds are tied
    with far more rows than the candidate buffers hold: those are foreseen and
    left to the list kernel, the others are not; whole numbers, so exact."""
    say("topk equal rows", kind, n, dim, k, equal)
    A = api()
    g = np.random.default_rng(n + dim)
    metric = orc.COS if kind == "f32cos" else orc.L2SQ
    x = g.integers(0, 250 if kind == "u8" else 16, (n, dim)).astype(np.uint8 if kind == "u8" else np.float32)
    same = g.random(n) < equal
    x[same] = x[0]
    rows = np.unique(np.concatenate([np.arange(60), np.arange(n - 60, n), g.choice(n, 80, replace=False)]))
    rid, rd = orc.knn_graph(orc.Vectors.from_array(x, metric), k, rows=rows)
    ids, d = A.build_knn(gpu_vectors(x, metric), k)
    assert np.array_equal(host(ids)[rows], rid)
    assert np.array_equal(host(d)[rows].astype(np.float64), rd)


@pytest.mark.parametrize("kind,nb,dim,k,cands", [("u8", 5000, 300, 256, False), ("u8", 5001, 150, 256, True),
                                                 ("f32l2", 5000, 200, 132, False), ("f32l2", 5003, 131, 132, True),
                                                 ("f32cos", 5000, 140, 132, False)])
def test_topk_list_kernel_long_sweeps(kind, nb, dim, k, cands):
    """Shapes that the list kernel takes by itself (k too large for a sample of
    so few base rows) and sweeps in one part, long enough for base norms from a
    launch of their own; a ragged last tile, candidate lists; whole numbers, so
    exact."""
    say("topk long sweeps", kind, nb, dim, k, cands)
    A = api()
    g = np.random.default_rng(nb + dim)
    metric = orc.COS if kind == "f32cos" else orc.L2SQ
    nq = 33000
    x, q = (g.integers(0, 250 if kind == "u8" else 16, (n, dim)).astype(np.uint8 if kind == "u8" else np.float32)
            for n in (nb + 700 * cands, nq))
    cand = g.permutation(nb + 700)[:nb].astype(np.int32) if cands else None
    rows = np.unique(np.concatenate([np.arange(40), np.arange(nq - 40, nq), g.choice(nq, 60, replace=False)]))
    rid, rd = orc.topk(orc.Vectors.from_array(q, metric), orc.Vectors.from_array(x, metric), k, q_rows=rows,
                       cand=cand, exclude_self=cands)
    ids, d = A.topk(gpu_vectors(q, metric), gpu_vectors(x, metric), k, cand=to_dev(cand) if cands else None,
                    exclude_self=cands)
    assert np.array_equal(host(ids)[rows], rid)
    assert np.array_equal(host(d)[rows].astype(np.float64), rd)
