"""The pair passes and the bucket form of the backward (csrc/pairs.hip) against the fp64 oracle,
at sizes that the dense tiles would take by their number of pairs alone: codes with more than 32
hashes of more than 8 bits have no bit planes, and a side of fewer than 64 rows against more
than 1024 stays with the pairs.  The library's kernel timer says that these kernels ran.
Bars as in parity.py."""
import numpy as np
import pytest

import oracle
import workloads
from parity import TOL, check_all
from test_parity_gpu import large_bucket_share
from workloads import make_inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2111_09714_amd as Y  # noqa: E402

KERNELS = ("tile_kernel", "tile_star_kernel", "dense_kernel", "pass_kernel", "pass_star_kernel", "bucket_kernel")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    Y.lib()


def to_dev(a, dtype):
    t = torch.from_numpy(np.ascontiguousarray(a, np.float32))
    return t.to(device="cuda", dtype=torch.bfloat16 if dtype == "bf16" else torch.float32).contiguous()


def codes_np(t):
    return np.ascontiguousarray(t.cpu().numpy().view(np.uint16).transpose(0, 2, 1))


def host(t):
    return t.float().cpu().numpy().astype(np.float64)


def case(bh, nq, nk, m, tau, dtype, dist="gauss", change=None, star=False):
    """Runs the backward (*YOSO if `star`), checks dQ and dK (and dV), returns the launches and the codes."""
    inp = make_inputs(workloads.Workload("pairs", 1, bh, nq, 64, tau, m, dtype, dist, 31 + nq + 2 * nk + m), n=nq, n_k=nk)
    if change is not None:
        change(inp)
    q, k, v, dy = (to_dev(inp[s], dtype) for s in ("q", "k", "v", "dy"))
    qc, kc = Y.hash_qk(q, k, torch.from_numpy(inp["R"]).cuda(), m, tau)
    torch.cuda.synchronize()
    Y.yoso_timing_enable(256)
    Y.yoso_timing_reset()
    try:
        got = (Y.backward_star if star else Y.backward)(qc, kc, q, k, v, dy, m, tau)
        torch.cuda.synchronize()
        ran = {n: Y.yoso_timing_query(n)[1] for n in KERNELS}
    finally:
        Y.yoso_timing_enable(0)
    c = (codes_np(qc), codes_np(kc))
    ref = (oracle.backward_star if star else oracle.backward)(*c, host(q), host(k), host(v), host(dy), m, tau)
    check_all(f"pairs {bh}x{nq}x{nk} m{m} tau{tau} {dtype} {dist}{' star' if star else ''}",
              [(n, host(g), r) for n, g, r in zip(("dq", "dk", "dv"), got, ref)], TOL[dtype])
    return ran, c


def clusters(inp):
    """16 clusters, their rows about 0.16 rad from the centre: the rows of a cluster (some 65 on either
    side) mostly share their bucket of 9 to 12 bits."""
    g = np.random.default_rng(97)
    centres = g.standard_normal((16, 64))
    for s in ("q", "k"):
        x = centres[g.integers(0, 16, inp[s].shape[:2])]
        x = x / np.linalg.norm(x, axis=-1, keepdims=True) + 0.02 * g.standard_normal(x.shape)
        inp[s] = x / np.linalg.norm(x, axis=-1, keepdims=True)


def clusters_of_unlike_rows(inp):
    clusters(inp)
    g = np.random.default_rng(98)
    inp["dy"] = inp["dy"] * 10.0 ** g.uniform(-4, 0, size=inp["dy"].shape[:2] + (1,))
    inp["v"] = inp["v"] * 10.0 ** g.uniform(-3, 1, size=inp["v"].shape[:2] + (1,))


@pytest.mark.parametrize("bh,nq,nk,m,tau,dtype", [
    (1, 1025, 1100, 40, 9, "f32"),     # a row past the short sequences; ragged last tiles
    (2, 1100, 1030, 56, 9, "bf16"),
    (1, 1300, 1070, 33, 12, "f32"),    # (sides on which rows have several partners: a row of one
                                       # partner is G times a vector, exact only to G's cancellation)
    (2, 5, 1200, 32, 8, "f32"),        # a few rows on a side
    (1, 1025, 1, 8, 3, "bf16"),
])
def test_pair_passes(bh, nq, nk, m, tau, dtype):
    ran, _ = case(bh, nq, nk, m, tau, dtype)
    assert ran["pass_kernel"] > 0 and ran["tile_kernel"] + ran["dense_kernel"] == 0, ran


@pytest.mark.parametrize("bh,nq,nk,m,tau,dtype,change", [
    (2, 1200, 1400, 40, 9, "f32", clusters),
    (2, 1200, 1400, 40, 9, "f32", clusters_of_unlike_rows),  # dY over 10^4, V over 10^4 within a bucket
    (1, 1025, 1031, 36, 10, "bf16", clusters),               # short and ragged
    (3, 1111, 1050, 42, 12, "f32", clusters),
])
def test_bucket_form(bh, nq, nk, m, tau, dtype, change):
    """Clustered rows: the rows of a large bucket take one 64 x 64 matrix."""
    ran, c = case(bh, nq, nk, m, tau, dtype, change=change)
    assert ran["bucket_kernel"] > 0 and ran["tile_kernel"] + ran["dense_kernel"] == 0, ran
    assert large_bucket_share(*c, tau) > 0.05


def test_one_bucket():
    """Every row in one bucket of every hash: one matrix of all rows.  (Positive V and dY: rows of dQ are
    the scalar product dY_i . sum V times one vector, and that must not cancel.)"""
    def one(inp):
        inp["v"], inp["dy"] = np.abs(inp["v"]), np.abs(inp["dy"])
        inp["q"][:] = inp["q"][:1, :1]
        inp["k"][:] = inp["q"][:1, :1]

    ran, c = case(1, 1100, 1300, 33, 9, "f32", change=one)
    assert ran["bucket_kernel"] > 0 and ran["tile_kernel"] == 0, ran
    assert large_bucket_share(*c, 9) == 1.0


@pytest.mark.parametrize("bh,nq,nk,m,tau,dtype", [
    (1, 300, 257, 40, 9, "bf16"),      # no plane layout
    (2, 129, 400, 33, 12, "bf16"),
    (1, 2100, 1030, 40, 9, "f32"),
])
def test_star_pair_passes(bh, nq, nk, m, tau, dtype):
    ran, _ = case(bh, nq, nk, m, tau, dtype, "mixture", star=True)
    assert ran["pass_star_kernel"] > 0 and ran["tile_star_kernel"] == 0, ran
