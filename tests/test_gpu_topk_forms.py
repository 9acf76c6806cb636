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
