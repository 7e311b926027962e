"""The block-tiled weight gradient against the per-site gather kernel (which the
other network tests hold against the oracle).  Activations agree bit for bit, so
the gradients differ by the order of their FP32 sums only: with n additions of
random sign the rounding is about 2^-24 sqrt(n / 2) of the result, 1e-6 for the
256 additions of a partial sum; ten times that is allowed.  Lattices of one
block, of blocks that are their own neighbours, with C* crossings, and of 87
blocks, where a workgroup's run of blocks passes from one d0 to the next."""
import os

import numpy as np
import pytest

import synthgen as sg
from tests.gpu_common import make_pair

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
qxd = pytest.importorskip("paper_1908_11673_amd")


@pytest.mark.parametrize("L,cstar,n", [((4, 4, 4, 8), 0, 1), ((4, 2, 4, 8), 1, 2), ((8, 4, 8, 8), 2, 1),
                                       ((8, 4, 4, 16), 3, 66), ((116, 4, 4, 24), 0, 1)])
def test_block_and_gather_gradients_agree(L, cstar, n):
    o, lat, _ = make_pair(L, cstar, sg.FLAVOURS["d"], seed=31)
    rng = np.random.default_rng(3)
    w = np.concatenate([rng.standard_normal(81 * a * b) * np.sqrt(2.0 / (81 * a))
                        for a, b in ((24, 32), (32, 32), (32, 24))]).astype(np.float32)
    g = torch.Generator(device="cuda").manual_seed(7)
    r, e = (torch.randn(n, 12 * lat.Ve, dtype=torch.complex64, device="cuda", generator=g) for _ in range(2))
    got = {}
    for gather in ("0", "1"):
        old = os.environ.get("QXD_NN_GATHER")
        os.environ["QXD_NN_GATHER"] = gather
        try:
            net = qxd.qxd_nn_create(lat.h)
        finally:
            if old is None:
                del os.environ["QXD_NN_GATHER"]
            else:
                os.environ["QXD_NN_GATHER"] = old
        qxd.qxd_nn_set_weights(net, w)
        got[gather] = qxd.qxd_nn_loss_grad(lat.h, net, r, e, n, 0)
        again = qxd.qxd_nn_loss_grad(lat.h, net, r, e, n, 0)
        assert again[0] == got[gather][0] and np.array_equal(again[1], got[gather][1])
        qxd.qxd_nn_destroy(net)
    assert got["0"][0] == got["1"][0]
    at = 0
    for a, b in ((24, 32), (32, 32), (32, 24)):
        u, v = (got[k][1][at:at + 81 * a * b].astype(np.float64) for k in "01")
        assert np.linalg.norm(u - v) <= 1e-5 * np.linalg.norm(v)
        at += 81 * a * b
    lat.close()
