"""The block convolution against the per-site one where its walk over the blocks
can go wrong: a single block (fewer workgroups than XCDs, every halo wrapping
onto the block itself), a number of blocks that eight does not divide, C* shifts
at block borders, two blocks for each workgroup, whose halo table and
weights are those of the next, and extents that the block's do not divide, along
one direction and along all; forward, and the loss gradient, whose data
gradients run the masked forms."""
import os

import numpy as np
import pytest

import synthgen as sg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
qxd = pytest.importorskip("paper_1908_11673_amd")

GEOMS = [((4, 4, 4, 8), 0), ((12, 4, 8, 24), 0), ((8, 6, 8, 16), 2), ((20, 4, 12, 8), 3), ((32, 16, 16, 16), 3),
         ((4, 4, 4, 10), 0), ((6, 4, 4, 8), 1), ((4, 6, 6, 10), 1), ((6, 6, 6, 10), 3), ((10, 6, 14, 26), 2), ((22, 14, 18, 18), 3)]


def network(lat, gather):
    old = os.environ.get("QXD_NN_GATHER")
    os.environ["QXD_NN_GATHER"] = "1" if gather else "0"
    try:
        return qxd.qxd_nn_create(lat.h)
    finally:
        if old is None:
            del os.environ["QXD_NN_GATHER"]
        else:
            os.environ["QXD_NN_GATHER"] = old


@pytest.mark.parametrize("L,cstar", GEOMS)
def test_block_convolution_on_edge_lattices(L, cstar):
    fl = sg.FLAVOURS["d"]
    vp = int(np.prod(L))
    lat = qxd.Lattice(L, cstar)
    lat.setup(sg.gauge_su3(33, 0.2, vp), sg.gauge_u1(33, 0.3, vp), fl)
    rng = np.random.default_rng(8)
    w = np.concatenate([rng.standard_normal(81 * ci * co) * np.sqrt(2.0 / (81 * ci))
                        for ci, co in ((24, 32), (32, 32), (32, 24))]).astype(np.float32)
    gen = torch.Generator(device="cuda").manual_seed(9)
    r, e = torch.randn(2, 12 * lat.Ve, dtype=torch.complex64, device="cuda", generator=gen)
    outs, grads = [], []
    for gather in (False, True):
        net = network(lat, gather)
        qxd.qxd_nn_set_weights(net, w)
        qxd.qxd_nn_set_skip(net, 0.1)
        out = lat.field(qxd.F32)
        qxd.qxd_nn_apply(lat.h, net, out, r)
        outs.append(out.cpu().to(torch.complex128))
        grads.append(np.asarray(qxd.qxd_nn_loss_grad(lat.h, net, r, e, 1, 0)[1], dtype=np.float64))
        qxd.qxd_nn_destroy(net)
    # sums in another order turn single bfloat16 roundings (2^-8) of two layers of
    # activations, and of two more on the way back
    assert torch.linalg.norm(outs[0] - outs[1]) < 5e-3 * torch.linalg.norm(outs[1])
    assert np.linalg.norm(grads[0] - grads[1]) < 1e-2 * np.linalg.norm(grads[1])
    lat.close()
