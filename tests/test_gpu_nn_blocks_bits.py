"""The block convolution gives the bits of the per-site one, on lattices that its
blocks divide and on those where the last blocks lie back over their neighbours:
application, both losses (their forward passes and, through the gradients, the
masked data gradients).  Both contract a tap's 32 channels in one matrix-core
instruction and take the taps in the same order, so nothing may differ.  The
weight gradients sum the sites in another order: with the 128 additions of a
partial sum of random sign the rounding is about 2^-24 sqrt(128 / 2) = 5e-7 of
the result; ten times that is allowed, layer by layer."""
import numpy as np
import pytest

import synthgen as sg
from tests.test_gpu_nn_blocks import GEOMS, network

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
qxd = pytest.importorskip("paper_1908_11673_amd")

SHAPES = ((24, 32), (32, 32), (32, 24))


@pytest.mark.parametrize("L,cstar", GEOMS)
def test_block_and_gather_kernels_agree_to_the_bit(L, cstar):
    vp = int(np.prod(L))
    lat = qxd.Lattice(L, cstar)
    lat.setup(sg.gauge_su3(35, 0.2, vp), sg.gauge_u1(35, 0.3, vp), sg.FLAVOURS["d"])
    rng = np.random.default_rng(12)
    w = np.concatenate([rng.standard_normal(81 * ci * co) * np.sqrt(2.0 / (81 * ci))
                        for ci, co in SHAPES]).astype(np.float32)
    gen = torch.Generator(device="cuda").manual_seed(13)
    r, e = torch.randn(2, 12 * lat.Ve, dtype=torch.complex64, device="cuda", generator=gen)
    outs, losses, grads = [], [], []
    for gather in (False, True):
        net = network(lat, gather)
        qxd.qxd_nn_set_weights(net, w)
        qxd.qxd_nn_set_skip(net, 0.1)
        out = lat.field(qxd.F32)
        qxd.qxd_nn_apply(lat.h, net, out, r)
        outs.append(out)
        got = [qxd.qxd_nn_loss_grad(lat.h, net, r, e, 1, kind) for kind in (0, 1)]
        losses.append([x[0] for x in got])
        grads.append([np.asarray(x[1], dtype=np.float64) for x in got])
        qxd.qxd_nn_destroy(net)
    assert torch.equal(outs[0], outs[1])
    assert losses[0] == losses[1]
    cuts = np.cumsum([81 * ci * co for ci, co in SHAPES])[:-1]
    for a, b in zip(*grads):
        for u, v in zip(np.split(a, cuts), np.split(b, cuts)):
            assert np.linalg.norm(u - v) <= 5e-6 * np.linalg.norm(v)
    lat.close()


def test_application_in_place_is_refused():
    """Where blocks lie over one another a site's input is read by two of them,
    so output and input have to be distinct fields."""
    lat = qxd.Lattice((6, 4, 4, 8), 0)
    net = qxd.qxd_nn_create(lat.h)
    f = lat.field(qxd.F32)
    with pytest.raises(qxd.QxdError) as e:
        qxd.qxd_nn_apply(lat.h, net, f, f)
    assert e.value.code == 1
    qxd.qxd_nn_destroy(net)
    lat.close()
