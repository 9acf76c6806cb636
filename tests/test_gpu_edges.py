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
