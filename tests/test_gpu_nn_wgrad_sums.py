"""The length of the FP32 sums of the weight gradient, 2048 terms in both kernels
(products with sites where the input or the gradient vanishes not counted).  The
activations and the gradients at every layer's output are small whole numbers
(times a power of two), so that a sum of 2048 terms stays below 2^24 and is exact
in FP32, one of 3072 or more does not and is not; the partial sums meet in FP64.
The block kernel, with a run of eight blocks (512 sites each) for each
workgroup, and the per-site one then return the same bits.

Layers 1 and 3 move the field one site along x3 besides leaving it in place, so
that from an even half field both parities are filled; layer 2 is the identity.
|r| is 2^17 to 1e-4 and e solves f d = q for the gradient f d at the output (f
depends on |e|), both closely enough that the rounding to bfloat16 gives the
whole numbers."""
import os

import numpy as np
import pytest

import synthgen as sg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
qxd = pytest.importorskip("paper_1908_11673_amd")

L = (80, 16, 16, 16)  # 640 blocks
HERE, NEXT = 40, 41   # taps (0, 0, 0, 0) and (0, 0, 0, 1)


def network(lat, w, gather):
    old = os.environ.get("QXD_NN_GATHER")
    os.environ["QXD_NN_GATHER"] = "1" if gather else "0"
    try:
        net = qxd.qxd_nn_create(lat.h)
    finally:
        if old is None:
            del os.environ["QXD_NN_GATHER"]
        else:
            os.environ["QXD_NN_GATHER"] = old
    qxd.qxd_nn_set_weights(net, w)
    return net


def test_partial_sums_are_exact_over_2048_sites():
    vp = int(np.prod(L))
    lat = qxd.Lattice(L, 0)
    lat.setup(sg.gauge_su3(3, 0.2, vp), sg.gauge_u1(3, 0.3, vp), sg.FLAVOURS["d"])
    w = [np.zeros((81, co, ci), np.float32) for ci, co in ((24, 32), (32, 32), (32, 24))]
    for k, taps in enumerate(((HERE, NEXT), (HERE,), (HERE, NEXT))):
        for t in taps:
            np.fill_diagonal(w[k][t], 1.0)
    w = np.concatenate([x.reshape(-1) for x in w])

    rng = np.random.default_rng(4)
    m = 24 * lat.Ve
    n = rng.integers(56, 77, m).astype(np.float64)  # mean 66
    want = 4.0 ** 17 - np.sum(n * n)
    n[rng.random(m) < -want / np.sum(2 * n - 1)] -= 1  # now |n| = 2^17
    norm = np.sqrt(np.sum(n * n))
    assert abs(norm / 2 ** 17 - 1) < 1e-4
    q = rng.integers(105, 126, m).astype(np.float64)  # mean 115: 66 * 115 * 2048 < 2^24 < 66 * 115 * 3072
    qs = q * 2.0 ** -18
    dev = lambda a: torch.from_numpy(a.astype(np.float32)).cuda().view(torch.complex64)  # noqa: E731
    r = dev(n)

    grads = []
    for gather in (False, True):
        net = network(lat, w, gather)
        out = lat.field(qxd.F32)
        qxd.qxd_nn_apply(lat.h, net, out, r)
        y = torch.view_as_real(out).cpu().double().numpy().reshape(-1) / norm
        # f = 2 |r|^2 / |e|^2 with e / |r| = y - qs / f
        Y, C, Q = np.sum(y * y), np.sum(y * qs), np.sum(qs * qs)
        f = ((C + 1) + np.sqrt((C + 1) ** 2 - Y * Q)) / Y
        e = dev(norm * (y - qs / f))
        grads.append(np.asarray(qxd.qxd_nn_loss_grad(lat.h, net, r, e, 1, 0)[1]))
        qxd.qxd_nn_destroy(net)
    # the gradient of layer 2's own tap is a sum over every site
    at = 81 * 32 * 24 + HERE * 32 * 32
    assert abs(grads[0][at] / (66 * 115 * lat.V * 2.0 ** -35) - 1) < 0.02
    assert np.array_equal(grads[0], grads[1])
    lat.close()
