"""The rounding error of a SAP application against the FP64 oracle on the same
FP32 source.  With each block's residual formed from the iterate, earlier
rounding is corrected and two sources are left, the last residual and the
solution, about one FP32 unit roundoff (2^-24) each: 1.0 to 1.3e-7 were measured
on larger lattices, whatever the cycles.  Rounding that a residual carries over
from visit to visit adds up instead (1.4 to 1.7e-7)."""
import numpy as np
import pytest

import synthgen as sg
from oracle import sap as osap
from tests.gpu_common import even_only, from_half32, half32, make_pair

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
qxd = pytest.importorskip("paper_1908_11673_amd")


@pytest.fixture(scope="module")
def pair():
    o, lat, _ = make_pair((8, 8, 8, 8), 3, sg.FLAVOURS["d"], sigma=0.2, su1=0.3, seed=51)
    yield o, lat, osap.site_blocks(o)
    lat.close()


@pytest.mark.parametrize("eo", [1, 0], ids=["eo", "plain"])
@pytest.mark.parametrize("ncy,nmr", [(2, 8), (5, 5)])
def test_rounding_does_not_add_up_over_the_visits(pair, ncy, nmr, eo):
    o, lat, blocks = pair
    src = half32(lat, even_only(o, sg.spinor(52, o.V)))
    out = lat.field(qxd.F32)
    qxd.qxd_sap_apply(lat.h, ncy, nmr, eo, out, src)
    got = from_half32(lat, out)
    want = even_only(o, osap.sap(o, from_half32(lat, src), ncy, nmr, bool(eo), blocks))
    assert np.linalg.norm(got - want) <= 1.3e-7 * np.linalg.norm(want)
