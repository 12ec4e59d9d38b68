"""Parity of *YOSO's backward (yoso_backward_star, the sampled estimate of the true
gradient of eq. gradient-q) with the fp64 oracle on the GPU's own codes.

Bars as for the other backward (tests/parity.py): per head Frobenius ratio and the
element-wise |gpu - ref| / (|ref| + rms(ref row)), <= 1e-4 for fp32 storage,
<= 2e-2 for bf16."""
import numpy as np
import pytest

import oracle
import workloads
from parity import TOL, check_all, log
from workloads import WORKLOADS, make_inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2111_09714_amd as Y  # noqa: E402


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


def run(inp, m, tau, dtype, heads=None):
    q, k, v, dy = (to_dev(inp[s], dtype) for s in ("q", "k", "v", "dy"))
    R = torch.from_numpy(inp["R"]).cuda()
    qc, kc = Y.hash_qk(q, k, R, m, tau)
    dq, dk, dv = Y.backward_star(qc, kc, q, k, v, dy, m, tau)
    torch.cuda.synchronize()
    sl = slice(None) if heads is None else heads
    # the oracle sees the values the GPU read (bf16-rounded for bf16 storage)
    ref = oracle.backward_star(codes_np(qc)[sl], codes_np(kc)[sl], host(q)[sl], host(k)[sl], host(v)[sl],
                               host(dy)[sl], m, tau)
    return [(name, host(g)[sl], r) for name, g, r in zip(("dq", "dk", "dv"), (dq, dk, dv), ref)]


@pytest.mark.parametrize("bh,nq,nk,m,tau,dtype", [
    (1, 512, 512, 32, 8, "f32"),
    (2, 300, 257, 16, 8, "f32"),
    (1, 100, 77, 4, 1, "f32"),      # every pair counts once per hash (the estimator is exact)
    (1, 200, 150, 8, 12, "f32"),
    (2, 300, 300, 8, 9, "bf16"),
    (3, 65, 130, 1, 3, "f32"),
    (1, 17, 33, 5, 2, "bf16"),
])
def test_star_small(bh, nq, nk, m, tau, dtype):
    name = f"star bh{bh} nq{nq} nk{nk} m{m} tau{tau} {dtype}"
    log(f"[{name}] start")
    w = workloads.Workload(name, 1, bh, nq, 64, tau, m, dtype, "gauss", 9000 + nq + nk + m + tau)
    check_all(name, run(make_inputs(w, n=nq, n_k=nk), m, tau, dtype), TOL[dtype])


@pytest.mark.parametrize("name", ["single_head_n512", "bert_base_n512", "lra_n4096"])
def test_star_workload_full_size(name):
    """All heads on the GPU; the oracle recomputes the first and the last head."""
    w = WORKLOADS[name]
    log(f"[star {name}] start: bh={w.bh} n={w.n} m={w.m} tau={w.tau}")
    heads = np.array(sorted({0, w.bh - 1}))
    check_all(f"star {name}", run(make_inputs(w), w.m, w.tau, w.dtype, heads=heads), TOL[w.dtype])


@pytest.mark.parametrize("n,nk,m,tau,dist,what,scale", [
    (700, 650, 32, 8, "gauss", "dy", 1e3),
    (700, 650, 32, 8, "gauss", "dy", 1e4),
    (700, 650, 32, 8, "gauss", "v", 1e4),
    (300, 1100, 20, 12, "gauss", "dy", 1e4),    # twelve plane words
    (600, 500, 64, 8, "gauss", "v", 1e4),       # two words per plane
    (700, 650, 32, 8, "mixture", "dy", 1e4),    # hundreds of hashes and bits in one weight
])
def test_star_one_large_row(n, nk, m, tau, dist, what, scale):
    """One row of dY (or V) far above the others: the rows of dK (or dQ) that it does not reach
    consist of weights that far below the largest of their head, and keep the fp32 bar."""
    name = f"star large {what} {scale:g} {n}x{nk} m{m} tau{tau} {dist}"
    log(f"[{name}] start")
    w = workloads.Workload(name, 1, 2, n, 64, tau, m, "f32", dist, 31000 + n + m)
    inp = make_inputs(w, n=n, n_k=nk)
    inp[what][:, inp[what].shape[1] // 2] *= scale
    check_all(name, run(inp, m, tau, "f32"), TOL["f32"])


def test_star_golden_worked_example(golden):
    g = golden["star_backward"]
    m, tau = g["m"], g["tau"]
    pad = lambda a: np.pad(np.array(a, np.float32), ((0, 0), (0, 62)))[None]
    q, k, v, dy = (to_dev(pad(g[s]), "f32") for s in ("q", "k", "v", "dy"))
    qc = torch.from_numpy(np.ascontiguousarray(np.array(g["qc"], np.int16).T)[None]).cuda()
    kc = torch.from_numpy(np.ascontiguousarray(np.array(g["kc"], np.int16).T)[None]).cuda()
    dq, dk, dv = Y.backward_star(qc, kc, q, k, v, dy, m, tau)
    torch.cuda.synchronize()
    for t, key in ((dq, "dq_times_pi"), (dk, "dk_times_pi"), (dv, "dv")):
        got = t.cpu().numpy()[0]
        scale = np.pi if key.endswith("_pi") else 1.0
        np.testing.assert_allclose(got[:, :2] * scale, np.array(g[key]), rtol=1e-5, atol=1e-5, err_msg=key)
        assert not got[:, 2:].any()


def test_star_empty():
    m, tau = 4, 3
    R = torch.randn(64, m * tau, device="cuda")
    for bh, nq, nk in [(0, 5, 5), (2, 0, 6), (2, 6, 0)]:
        q = torch.nn.functional.normalize(torch.randn(bh, nq, 64, device="cuda"), dim=-1)
        k = torch.nn.functional.normalize(torch.randn(bh, nk, 64, device="cuda"), dim=-1)
        v = torch.randn(bh, nk, 64, device="cuda")
        dy = torch.randn(bh, nq, 64, device="cuda")
        qc, kc = Y.hash_qk(q, k, R, m, tau)
        dq, dk, dv = Y.backward_star(qc, kc, q, k, v, dy, m, tau)
        torch.cuda.synchronize()
        for t in (dq, dk, dv):
            assert t.numel() == 0 or float(t.abs().max()) == 0.0
