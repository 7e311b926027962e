"""CG and multi-shift CG whatever the interval of the host's convergence checks:
the iteration does not depend on it, so a solve stops at the first multiple of
the interval at which it has converged, and an iteration limit between two checks ends
it there.  On 384 even sites (sums left as partials) and on 147,456 (2304
partials: summed by a kernel)."""
import numpy as np
import pytest

import synthgen as sg

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
qxd = pytest.importorskip("paper_1908_11673_amd")

FL = dict(sg.FLAVOURS["d"], kappa=0.12)


@pytest.fixture(scope="module", params=[((8, 4, 4, 6), 0), ((16, 12, 16, 48), 3)], ids=["384", "147456"])
def lat(request):
    L, cstar = request.param
    vp = int(np.prod(L))
    lat = qxd.Lattice(L, cstar)
    lat.setup(sg.gauge_su3(51, 0.2, vp), sg.gauge_u1(51, 0.3, vp), FL)
    yield lat
    lat.close()


def source(lat):
    gen = torch.Generator(device="cuda").manual_seed(6)
    return torch.randn(24 * lat.Ve, dtype=torch.complex128, device="cuda", generator=gen)


def test_cg_by_check_interval(lat):
    b, its = source(lat), {}
    for check in (1, 3, 50):
        x = lat.field(qxd.F64, full=True)
        st = qxd.qxd_solve_cg(lat.h, qxd.solver_params(res=1e-9, inner_prec=qxd.F64, check_every=check), x, b)
        assert st["status"] == 0 and st["true_residual"] <= 1e-9
        its[check] = st["inner_it"]
    assert its[3] == -(-its[1] // 3) * 3 and its[50] == -(-its[1] // 50) * 50
    x = lat.field(qxd.F64, full=True)
    st = qxd.qxd_solve_cg(lat.h, qxd.solver_params(nmx=5, res=1e-9, inner_prec=qxd.F64, check_every=4), x, b,
                          check=False)
    assert st["status"] != 0 and st["inner_it"] == 5
    x = lat.field(qxd.F64, full=True)
    st = qxd.qxd_solve_cg(lat.h, qxd.solver_params(res=1e-9, inner_prec=qxd.F32, check_every=7), x, b)
    assert st["status"] == 0 and st["true_residual"] <= 1e-9


def test_mscg_by_check_interval(lat):
    b, its, sols = source(lat)[:12 * lat.Ve].clone(), {}, {}
    shifts = [0.01, 0.3]
    for check in (1, 3, 50):
        xs = [lat.field(qxd.F64) for _ in shifts]
        st = qxd.qxd_solve_mscg(lat.h, qxd.solver_params(res=1e-9, check_every=check), shifts, xs, b)
        its[check], sols[check] = st["inner_it"], xs
    assert its[3] == -(-its[1] // 3) * 3 and its[50] == -(-its[1] // 50) * 50
    for check in (3, 50):  # a converged shift is not updated any more
        assert all(torch.equal(p, q) for p, q in zip(sols[1], sols[check]))
    xs = [lat.field(qxd.F64) for _ in shifts]
    st = qxd.qxd_solve_mscg(lat.h, qxd.solver_params(nmx=5, res=1e-9, check_every=4), shifts, xs, b, check=False)
    assert st["status"] != 0 and st["inner_it"] == 5
