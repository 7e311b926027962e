"""The chunked order of time slices, forced through QXD_SCHUR_SLICES, against two
plain launches, on lattices of the two kernel forms that large lattices use: the
operators, and a CG solve, whose norms come from the partial sums of the second
pass.  (The small lattice of the test in test_gpu_dirac.py takes the form with
four waves for 64 sites; the library itself takes chunks where t_o and psi_e
exceed 256 MB.)"""
import os

import numpy as np
import pytest

import synthgen as sg
from tests.gpu_common import to_dev
from tests.test_gpu_dirac_forms import FL, PRECS, applied, lattice

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
qxd = pytest.importorskip("paper_1908_11673_amd")

HEAVY = dict(FL, kappa=0.11)  # a solve of some tens of iterations


def with_slices(slices, make):
    old = os.environ.get("QXD_SCHUR_SLICES")
    os.environ["QXD_SCHUR_SLICES"] = str(slices)
    try:
        return make()
    finally:
        if old is None:
            del os.environ["QXD_SCHUR_SLICES"]
        else:
            os.environ["QXD_SCHUR_SLICES"] = old


# even sites 73,728 (one wave for 64 sites) and 327,680 (256 work-items); chunks
# of two slices have no second pass after the first
@pytest.mark.parametrize("L,cstar,slices", [((36, 16, 16, 16), 0, (2, 9)), ((40, 16, 16, 32), 1, (2, 8, 20))])
def test_chunked_order_gives_the_bits_of_two_launches(L, cstar, slices):
    vp = int(np.prod(L))
    U, A = sg.gauge_su3(63, 0.3, vp), sg.gauge_u1(63, 0.4, vp)
    runs = []
    for s in (0,) + slices:
        lat = with_slices(s, lambda: lattice(L, cstar, False, U, A, HEAVY))
        assert lat.Ve > 65536 and (lat.Ve > 1 << 18) == (cstar == 1)
        psi = to_dev(sg.spinor(64, lat.V))
        outs = []
        for prec in PRECS:
            outs += applied(lat, prec, psi)[:2]
        x = lat.field(qxd.F64, full=True)
        st = qxd.qxd_solve_cg(lat.h, qxd.solver_params(res=1e-8, inner_prec=qxd.F64), x, lat.pack(psi))
        runs.append((outs + [x], st["inner_it"]))
        lat.close()
    for outs, its in runs[1:]:
        assert its == runs[0][1]
        for got, ref in zip(outs, runs[0][0]):
            assert torch.equal(got, ref)
