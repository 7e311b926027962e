"""The cycles and the coarse solve at the ends of their ranges, against the FP64
oracle: SAP on fields of both parities from one cycle (first and last at once)
to four, where the solution is summed in the output, with an antiperiodic time
direction; and the two-level preconditioner for subspaces of 1 to 24 vectors
(partial groups of rows, more than half a wavefront) and 1 to 32 coarse steps."""
import numpy as np
import pytest

import synthgen as sg
from oracle import dfl as odfl
from oracle import sap as osap
from tests.gpu_common import from_half32, half32, make_pair, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
qxd = pytest.importorskip("paper_1908_11673_amd")


@pytest.fixture(scope="module")
def pair():
    o, lat, _ = make_pair((8, 8, 8, 8), 3, sg.FLAVOURS["u"], sigma=0.2, su1=0.3, seed=43, tanti=True)
    yield o, lat, osap.site_blocks(o)
    lat.close()


@pytest.mark.parametrize("eo", [1, 0], ids=["eo", "plain"])
@pytest.mark.parametrize("ncy,nmr", [(1, 1), (1, 6), (3, 1), (4, 4)])
def test_sap_cycles_on_full_fields(pair, ncy, nmr, eo):
    o, lat, blocks = pair
    eta = sg.spinor(64, o.V)
    out = lat.field(qxd.F32, full=True)
    out.fill_(float("nan"))  # nothing of the output's old content is used
    qxd.qxd_sap_apply_full(lat.h, ncy, nmr, eo, out, lat.pack(to_dev(eta), qxd.F32))
    got = lat.unpack(out, qxd.F32).cpu().numpy()
    want = osap.sap(o, eta, ncy, nmr, bool(eo), blocks)
    # 16 FP32 unit roundoffs: some 30 operator sums, each rounded to about one
    assert np.linalg.norm(got - want) <= 1e-6 * np.linalg.norm(want)


@pytest.mark.parametrize("ns,nc", [(1, 32), (3, 1), (9, 2), (20, 5), (24, 32)])
def test_coarse_solve_by_subspace_size(pair, ns, nc):
    o, lat, _ = pair
    v0 = [sg.spinor(300 + k, o.V) for k in range(ns)]
    vs = odfl.subspace_vectors(o, v0, 1, 1, 2)
    sites, basis = odfl.block_basis(o, vs)
    A = odfl.little_operator(o, sites, basis)
    d = qxd.qxd_dfl_create(lat.h, ns)
    v = torch.cat([lat.pack(to_dev(x), qxd.F32) for x in v0])
    qxd.qxd_dfl_generate(lat.h, d, v, 1, 1, 2)
    r = sg.spinor(32, o.V)
    r[o.parity() == 1] = 0
    out = lat.field(qxd.F32)
    qxd.qxd_dfl_apply(lat.h, d, nc, 1, 2, 0, out, half32(lat, r))
    got = from_half32(lat, out)
    want = odfl.precondition_even(o, sites, basis, A, r, nc, 1, 2, False, None)
    qxd.qxd_dfl_destroy(d)
    # FP32 rounding 6e-8 times the condition number of the little operator, some tens
    assert np.linalg.norm(got - want) <= 1e-5 * np.linalg.norm(want)
