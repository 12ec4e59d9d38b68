"""The bucket tables' scatter forms (csrc/tables.hip) against the fp64 oracle: one, two and four
keys per step at each slice width, several passes of hashes, the general form (odd or
few hashes), a few heads (narrower slices) and many, at the ends of the 64-key
chunks and of the eight waves' turns.  Bars as in parity.py."""
import numpy as np
import pytest

import oracle
import workloads
from parity import TOL, check_all
from workloads import make_inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2111_09714_amd as Y  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    Y.lib()


# (m, tau): 8-dim slices with one (16), two (8) and four (4) keys per step; 4-dim with one (32) and
# four (8 at tau 10); 2-dim with one (64), two (32 at tau 9) and four (16 at tau 10), the last also
# in passes of hashes (48); a hash count below the power of two; and the general form
FORMS = [(16, 7), (14, 6), (8, 8), (6, 6), (4, 8), (32, 6), (24, 8), (8, 10), (64, 7), (32, 9), (16, 10), (48, 10),
         (2, 8), (15, 7), (8, 12)]


@pytest.mark.parametrize("m,tau", FORMS)
@pytest.mark.parametrize("bh,nq,nk,dtype", [
    (1, 65, 1, "f32"), (2, 63, 513, "bf16"), (3, 1, 577, "f32"), (20, 130, 1089, "f32"), (65, 64, 64, "bf16"),
    (2, 1025, 700, "bf16"),
])
def test_table_forms(bh, nq, nk, dtype, m, tau):
    w = workloads.Workload("tables", 1, bh, nq, 64, tau, m, dtype, "gauss", 31 + nq + 3 * nk + m + 100 * tau)
    inp = make_inputs(w, n=nq, n_k=nk)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    q, k, v = (torch.from_numpy(np.ascontiguousarray(inp[s], np.float32)).to("cuda", dt) for s in ("q", "k", "v"))
    qc, kc = Y.hash_qk(q, k, torch.from_numpy(inp["R"]).cuda(), m, tau)

    Y.yoso_timing_enable(64)
    Y.yoso_timing_reset()
    try:
        y = Y.forward(qc, kc, v, m, tau, n_q=nq)
        torch.cuda.synchronize()
        assert Y.yoso_timing_query("table_kernel")[1] == 1
    finally:
        Y.yoso_timing_enable(0)
    host = lambda c: np.ascontiguousarray(c.cpu().numpy().view(np.uint16).transpose(0, 2, 1))
    ref = oracle.forward(host(qc), host(kc), inp["v"], m, tau)
    check_all(f"tables {bh} {nq} {nk} {m} {tau} {dtype}", [("y", y.float().cpu().numpy().astype(np.float64), ref)],
              TOL[dtype])
