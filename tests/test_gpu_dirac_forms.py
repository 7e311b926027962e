"""The forms of the operator kernels against one another, to the bit.

Four waves for 64 sites, one wave for 64 and 256 work-items are chosen by the half
volume.  A lattice repeated n times along x0, links and fields alike, gives on
each copy what the single one gives, so a small lattice (four waves) and its
repetitions (the other two) compare the forms.  With an antiperiodic time
direction the copies alternate in sign (n odd)."""
import numpy as np
import pytest

import synthgen as sg
from tests.gpu_common import to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
qxd = pytest.importorskip("paper_1908_11673_amd")

FL = sg.FLAVOURS["u"]
PRECS = [qxd.F64, qxd.F32, qxd.BF16]


def lattice(L, cstar, tanti, U, A, flavour=FL):
    lat = qxd.Lattice(L, cstar, tanti)
    lat.setup(U, A, flavour)
    return lat


def applied(lat, prec, psi):
    """D_hat, its adjoint (even sites) and D of psi, as (V, 12) arrays."""
    x = lat.pack(psi, prec)
    n = x.numel() // 2
    res = []
    for dag in (0, 1):
        out = torch.zeros_like(x)
        qxd.qxd_dw_eo_schur(lat.h, prec, dag, out[:n], x[:n])
        res.append(lat.unpack(out, prec))
    out = torch.zeros_like(x)
    qxd.qxd_dw_apply(lat.h, prec, out, x)
    res.append(lat.unpack(out, prec))
    return [r.reshape(lat.V, 12) for r in res]


# even sites 8,192 and 5,040 (no multiple of a wave); their repetitions lie in
# the ranges of one wave for 64 sites (65,536, 2^18] and of 256 work-items
@pytest.mark.parametrize("L,cstar,tanti,copies", [((8, 8, 16, 16), 0, False, (9, 33)),
                                                  ((6, 6, 10, 14), 3, True, (15, 55))])
@pytest.mark.parametrize("prec", PRECS, ids=["f64", "f32", "bf16"])
def test_every_form_gives_the_same_bits(L, cstar, tanti, copies, prec):
    vp = int(np.prod(L))
    U, A = sg.gauge_su3(61, 0.3, vp), sg.gauge_u1(61, 0.4, vp)
    one = lattice(L, cstar, tanti, U, A)
    psi = to_dev(sg.spinor(62, one.V))
    assert one.Ve <= 32768
    want = applied(one, prec, psi)
    for n in copies:
        sign = torch.tensor([-1.0 if tanti and k & 1 else 1.0 for k in range(n)], dtype=torch.float64, device="cuda")
        big = lattice((n * L[0],) + L[1:], cstar, tanti, np.concatenate([U] * n, axis=1), np.concatenate([A] * n, axis=1))
        assert big.Ve > 65536 and (big.Ve > 1 << 18) == (n == copies[-1])
        field = torch.cat([s * psi for s in sign])
        for got, ref in zip(applied(big, prec, field), want):
            got = got.reshape(n, one.V, 12)
            for k in range(n):
                assert torch.equal(sign[k] * got[k], ref), (n, k)
        big.close()
    one.close()
