"""The operator on either side of the half volumes at which its kernels change
(four waves for 64 sites up to 32,768 even sites, 65,536 with bf16 storage; then
one wave for 64; 256 work-items beyond 2^18), each on a ragged volume too:
against the oracle on sampled sites, D_hat, its adjoint and D, and the norms that
the solvers take from the second pass."""
import numpy as np
import pytest

import oracle
import synthgen as sg
from tests.gpu_common import to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
qxd = pytest.importorskip("paper_1908_11673_amd")

FL = sg.FLAVOURS["u"]
# even sites: 96, 32,760, 32,768, 33,000, 65,536, 65,664, 262,144, 264,384
GEOMS = [((2, 2, 4, 6), 1, False), ((26, 6, 14, 30), 0, True), ((16, 16, 16, 16), 0, False),
         ((22, 10, 10, 30), 0, False), ((32, 8, 16, 16), 2, True), ((38, 12, 12, 12), 3, False),
         ((64, 16, 16, 16), 3, False), ((34, 18, 18, 24), 1, False)]


@pytest.mark.parametrize("L,cstar,tanti", GEOMS)
def test_operator_at_the_kernel_boundaries(L, cstar, tanti):
    o = oracle.Oracle(L, cstar, tanti)
    U, A = sg.gauge_su3(41, 0.3, o.Vphys), sg.gauge_u1(41, 0.4, o.Vphys)
    o.set_gauge_physical(U, A)
    o.set_flavour(**FL, cache=False, blocks=False)
    lat = qxd.Lattice(L, cstar, tanti)
    lat.setup(U, A, FL)
    par = o.parity()
    rng = np.random.default_rng(5)
    even, odd = np.nonzero(par == 0)[0], np.nonzero(par == 1)[0]
    pick = lambda a: np.unique(np.concatenate([a[:4], a[-4:], rng.choice(a, size=min(24, len(a)), replace=False)]))  # noqa: E731
    se, so = pick(even), pick(odd)
    full = sg.spinor(42, o.V)
    psi = full.copy()
    psi[par == 1] = 0
    # FP64 rounding; FP32 2^-24 and bf16 2^-9 per stored entry, of some hundred terms
    for prec, tol in ((qxd.F64, 1e-13), (qxd.F32, 2e-6), (qxd.BF16, 3e-2)):
        x = lat.pack(to_dev(psi), prec)
        n = x.numel() // 2
        for dag in (False, True):
            out = torch.zeros_like(x)
            qxd.qxd_dw_eo_schur(lat.h, prec, dag, out[:n], x[:n])
            got = lat.unpack(out, prec).cpu().numpy()[se]
            want = o.schur_sites(psi, se, dagger=dag)
            assert np.abs(got - want).max() <= tol * np.abs(want).max(), (prec, dag)
        y = lat.pack(to_dev(full), prec)
        out = torch.zeros_like(y)
        qxd.qxd_dw_apply(lat.h, prec, out, y)
        got = lat.unpack(out, prec).cpu().numpy()
        for s in (se, so):
            want = o.dirac_sites(full, s)
            assert np.abs(got[s] - want).max() <= tol * np.abs(want).max(), prec
    # one CG iteration's step lengths are ratios of the norms of the second pass
    b = lat.pack(to_dev(full))
    sol = lat.field(qxd.F64, full=True)
    st = qxd.qxd_solve_cg(lat.h, qxd.solver_params(res=1e-10, inner_prec=qxd.F64), sol, b)
    xs = lat.unpack(sol).cpu().numpy()
    r = full[se] - o.dirac_sites(xs, se)
    assert np.linalg.norm(r) <= 1e-8 * np.linalg.norm(full[se]) and st["true_residual"] <= 1e-10
    lat.close()
