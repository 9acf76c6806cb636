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
