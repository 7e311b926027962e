"""GPU set-up kernels (gauge copy, links, clover blocks and their inverses) on
lattices whose physical volume leaves partial workgroups, with and without the
mirror half, from host and from device arrays."""
import numpy as np
import pytest

import oracle
import synthgen as sg
from tests.gpu_common import even_only, rel_err, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
qxd = pytest.importorskip("paper_1908_11673_amd")

# a small diagonal and a large SW term: the eliminations of many blocks swap rows
STRONG = dict(qhat=3, invqel=6.0, kappa=0.5, su3csw=6.0, u1csw=1.5)


@pytest.mark.parametrize("L,cstar", [((2, 2, 2, 2), 0), ((2, 2, 2, 2), 3), ((6, 2, 10, 4), 1), ((10, 6, 2, 6), 2),
                                     ((4, 6, 6, 10), 3), ((6, 6, 4, 4), 0)])
@pytest.mark.parametrize("on_device", [False, True])
def test_setup_against_the_oracle(L, cstar, on_device):
    o = oracle.Oracle(L, cstar)
    U, A = sg.gauge_su3(31, 0.5, o.Vphys), sg.gauge_u1(31, 0.7, o.Vphys)
    o.set_gauge_physical(U, A)
    o.set_flavour(**STRONG)
    lat = qxd.Lattice(L, cstar)
    lat.setup(to_dev(U) if on_device else U, to_dev(A) if on_device else A, STRONG)
    psi = sg.spinor(32, o.V)
    out = lat.field(qxd.F64, full=True)
    qxd.qxd_dw_apply(lat.h, qxd.F64, out, lat.pack(to_dev(psi)))
    assert rel_err(lat.unpack(out).cpu().numpy(), o.dirac(psi)) < 1e-13
    # both sides invert the odd blocks: elimination with pivoting is off by a
    # modest multiple of eps times the condition number (order 6, growth < 2^5)
    cond = max(np.linalg.cond(o.site_block(s)) for s in np.nonzero(o.parity() == 1)[0])
    pe = even_only(o, psi)
    out.zero_()
    qxd.qxd_dw_eo_schur(lat.h, qxd.F64, 0, out[:12 * lat.Ve], lat.pack(to_dev(pe))[:12 * lat.Ve])
    assert rel_err(lat.unpack(out).cpu().numpy(), o.schur(pe)) < 200 * np.finfo(float).eps * cond
    lat.close()


@pytest.mark.parametrize("L,cstar", [((2, 2, 2, 2), 1), ((6, 6, 2, 10), 3)])
def test_lower_precision_copies_round_the_links(L, cstar):
    """D in FP32 and with bf16 storage on a source whose entries both types hold
    exactly: within the rounding of the operator (2^-24 and 2^-9 per entry, of
    some hundred terms of either sign)."""
    o = oracle.Oracle(L, cstar)
    U, A = sg.gauge_su3(33, 0.3, o.Vphys), sg.gauge_u1(33, 0.3, o.Vphys)
    o.set_gauge_physical(U, A)
    fl = sg.FLAVOURS["u"]
    o.set_flavour(**fl)
    lat = qxd.Lattice(L, cstar)
    lat.setup(U, A, fl)
    psi = np.round(4 * sg.spinor(34, o.V).view(np.float64)).view(np.complex128) / 4
    want = o.dirac(psi)
    for prec, tol in ((qxd.F32, 1e-6), (qxd.BF16, 2e-2)):
        out = lat.field(prec, full=True)
        qxd.qxd_dw_apply(lat.h, prec, out, lat.pack(to_dev(psi), prec))
        assert rel_err(lat.unpack(out, prec).cpu().numpy(), want) < tol
    lat.close()
