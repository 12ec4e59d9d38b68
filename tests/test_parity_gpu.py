"""Parity of the HIP path (through the C ABI) with the fp64 CPU oracle.

Bars:
  * hash codes bit-exact wherever the oracle's smallest |projection| of the hash
    exceeds 1e-4; the excluded fraction is reported;
  * forward/backward evaluated on the GPU's own codes (so a legitimate flip of a
    near-zero bit cannot fail output parity): per head ||gpu - ref||_F / ||ref||_F
    and, element by element, |gpu - ref| / (|ref| + rms(ref row)), both <= 1e-4
    for fp32 storage and <= 2e-2 for bf16 (tests/parity.py).
"""
import math

import numpy as np
import pytest

import oracle
import workloads
import parity
from parity import TOL, check_all, log
from workloads import WORKLOADS, make_inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2111_09714_amd as Y  # noqa: E402

MARGIN = 1e-4


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    Y.lib()  # fails loudly if the HIP library is missing


def to_dev(a, dtype):
    t = torch.from_numpy(np.ascontiguousarray(a, np.float32))
    return t.to(device="cuda", dtype=torch.bfloat16 if dtype == "bf16" else torch.float32).contiguous()


def codes_np(t):
    """GPU codes [bh, n, m] as the oracle's [bh, m, n] layout."""
    return np.ascontiguousarray(t.cpu().numpy().view(np.uint16).transpose(0, 2, 1))


def run_gpu(inp, m, tau, dtype):
    q, k, v, dy = (to_dev(inp[s], dtype) for s in ("q", "k", "v", "dy"))
    R = torch.from_numpy(inp["R"]).cuda()
    qc, kc = Y.hash_qk(q, k, R, m, tau)
    y = Y.forward(qc, kc, v, m, tau, n_q=q.shape[1])
    dq, dk, dv = Y.backward(qc, kc, q, k, v, dy, m, tau)
    torch.cuda.synchronize()
    f = lambda t: t.float().cpu().numpy().astype(np.float64)
    return dict(qc=codes_np(qc), kc=codes_np(kc), y=f(y), dq=f(dq), dk=f(dk), dv=f(dv))


def check_codes(name, x, R, m, tau, gpu_codes):
    ref, margin = oracle.hash_codes(x, R, m, tau, with_margin=True)
    sure = margin > MARGIN
    mism = (ref != gpu_codes) & sure
    excluded = 1.0 - sure.mean() if sure.size else 0.0
    log(f"[{name}] codes: {sure.size} checked, excluded fraction {excluded:.2e}, mismatches {int(mism.sum())}")
    assert not mism.any()
    return excluded


def check_outputs(name, inp, g, m, tau, dtype, heads=None):
    sl = slice(None) if heads is None else heads
    q, k, v, dy = (inp[s][sl] for s in ("q", "k", "v", "dy"))
    qc, kc = g["qc"][sl], g["kc"][sl]
    y = oracle.forward(qc, kc, v, m, tau)
    dq, dk, dv = oracle.backward(qc, kc, q, k, v, dy, m, tau)
    check_all(name, [(key, g[key][sl], ref) for key, ref in (("y", y), ("dq", dq), ("dk", dk), ("dv", dv))],
              TOL[dtype])


SMALL = [
    # (bh, n_q, n_k, m, tau, dtype)
    (1, 512, 512, 32, 8, "f32"),
    (3, 77, 77, 5, 3, "f32"),
    (2, 1000, 640, 16, 8, "f32"),
    (2, 300, 300, 32, 9, "bf16"),
    (1, 129, 257, 64, 8, "f32"),
    (2, 65, 65, 1, 1, "f32"),
    (1, 100, 100, 42, 12, "f32"),
    (1, 200, 150, 32, 12, "bf16"),
    (2, 1, 1, 8, 4, "f32"),
    (1, 17, 33, 7, 2, "bf16"),
    # many heads of short sequences: the dense forms of the forward and the backward
    (40, 300, 257, 32, 8, "f32"),
    (32, 129, 1000, 33, 12, "bf16"),
    # above 1024 rows on a side the rule weighs the dense tiles against the pair passes (which form
    # serves these is the library's choice; test_pairs_gpu.py holds the pairs' own cases)
    (1, 1025, 1100, 7, 5, "f32"),
    (2, 1500, 1030, 16, 8, "bf16"),
    # the most hashes (m = 64): eight gather lanes per query in the tables, two plane words per
    # bit in the dense tiles
    (1, 1100, 1500, 64, 8, "f32"),
    (1, 2000, 1100, 64, 7, "bf16"),
]


@pytest.mark.parametrize("bh,nq,nk,m,tau,dtype", SMALL)
def test_small_shapes(bh, nq, nk, m, tau, dtype):
    run_case(bh, nq, nk, m, tau, dtype)


FORWARD_FORMS = [
    # (bh, n_q, n_k, m, tau, dtype, kernel): many heads of short sequences take the
    # dense forward (ragged tiles, one and two words of hashes, tau 1 to 12); few
    # heads, or n_q n_k past the rule's bound, take the bucket tables
    (512, 37, 50, 5, 3, "f32", "dense_fwd_kernel"),
    (160, 200, 333, 32, 8, "f32", "dense_fwd_kernel"),
    (96, 400, 1024, 64, 6, "f32", "dense_fwd_kernel"),
    (128, 300, 1000, 33, 12, "bf16", "dense_fwd_kernel"),
    (256, 129, 65, 17, 9, "bf16", "dense_fwd_kernel"),
    (520, 1, 1, 1, 1, "f32", "dense_fwd_kernel"),
    (8, 512, 512, 32, 8, "f32", "table_kernel"),
    (64, 1024, 1000, 32, 8, "f32", "table_kernel"),
]


@pytest.mark.parametrize("bh,nq,nk,m,tau,dtype,kernel", FORWARD_FORMS)
def test_forward_forms(bh, nq, nk, m, tau, dtype, kernel):
    """The forward's two forms (dense counts C V, or bucket tables) against the
    oracle on every head; the library's kernel timer confirms which form ran."""
    name = f"fwd_bh{bh}_nq{nq}_nk{nk}_m{m}_tau{tau}_{dtype}"
    log(f"[{name}] start")
    w = workloads.Workload(name, 1, bh, nq, 64, tau, m, dtype, "gauss", 4321 + nq + 7 * nk + m + tau)
    inp = make_inputs(w, n=nq, n_k=nk)
    q, k, v = (to_dev(inp[s], dtype) for s in ("q", "k", "v"))
    R = torch.from_numpy(inp["R"]).cuda()
    qc, kc = Y.hash_qk(q, k, R, m, tau)
    torch.cuda.synchronize()
    Y.yoso_timing_enable(64)
    Y.yoso_timing_reset()
    try:
        y = Y.forward(qc, kc, v, m, tau, n_q=nq)
        torch.cuda.synchronize()
        launches = {kn: Y.yoso_timing_query(kn)[1] for kn in ("dense_fwd_kernel", "table_kernel")}
    finally:
        Y.yoso_timing_enable(0)
    assert launches[kernel] >= 1 and sum(launches.values()) == launches[kernel], launches
    ref = oracle.forward(codes_np(qc), codes_np(kc), inp["v"], m, tau)
    check_all(name, [("y", y.float().cpu().numpy().astype(np.float64), ref)], TOL[dtype])


def test_dense_forward_without_keys():
    """Many heads with no keys at all: the dense forward runs (enough workgroups) and
    every query reads empty buckets, so Y is exactly zero; one key per head gives
    Y_i = (C_i0 / m) V_0 with C_i0 counted from the codes."""
    bh, nq, m, tau = 600, 10, 4, 3
    g = torch.Generator().manual_seed(5)
    q = torch.nn.functional.normalize(torch.randn(bh, nq, 64, generator=g), dim=-1).cuda()
    R = torch.randn(64, m * tau, generator=g).cuda()
    for nk in (0, 1):
        k = torch.nn.functional.normalize(torch.randn(bh, nk, 64, generator=g), dim=-1).cuda()
        v = torch.randn(bh, nk, 64, generator=g).cuda()
        qc, kc = Y.hash_qk(q, k, R, m, tau)
        torch.cuda.synchronize()
        Y.yoso_timing_enable(64)
        Y.yoso_timing_reset()
        try:
            y = Y.forward(qc, kc, v, m, tau, n_q=nq)
            torch.cuda.synchronize()
            dense = Y.yoso_timing_query("dense_fwd_kernel")[1]
        finally:
            Y.yoso_timing_enable(0)
        assert dense == 1
        if nk == 0:
            assert float(y.abs().max()) == 0.0
        else:
            c = (qc.long() == kc.long()).sum(-1, keepdim=True).float()  # [bh, nq, 1]
            ref = c / m * v[:, :1, :]
            assert torch.allclose(y, ref, rtol=1e-6, atol=1e-6)


@pytest.mark.parametrize("bh,nq,nk,m,tau,dtype", [(1, 65536, 65536, 3, 10, "f32"), (1, 65535, 65536, 2, 12, "bf16")])
def test_maximum_length(bh, nq, nk, m, tau, dtype):
    """Sequences at the library's limit of 65536 rows (the most that the 16-bit row
    field of a sorted entry addresses): the bucket sort takes its global-memory path,
    and in the second case the last row tile is ragged.  Every row is checked.  With
    fp32 outputs the tables' fixed-point scale comes from the largest bucket count
    (about 64 rows here) rather than the sum of |v| over all 65536 rows, whose
    rounding step would put Y and dV near 1e-4: both must stay below 1e-5."""
    run_case(bh, nq, nk, m, tau, dtype)
    if dtype == "f32":
        name = f"bh{bh}_nq{nq}_nk{nk}_m{m}_tau{tau}_{dtype}"
        got = {k: e for tag, k, f, e, tol in parity.RECORD if tag == name and k in ("y", "dv")}
        assert len(got) == 2 and max(got.values()) < 1e-5, got


@pytest.mark.parametrize("bh,nq,nk,m,tau", [(1, 8193, 8200, 16, 9), (2, 9000, 8209, 7, 8)])
def test_count_bound_lengths(bh, nq, nk, m, tau):
    """Just past 8192 source rows (fp32) the tables' fixed-point scale also bounds the
    bucket sums by the largest bucket count: with m = 16 the counts read a row's
    codes 16 bytes at a time, with m = 7 one code at a time.  Ragged lengths on both
    sides; every row checked, and Y, dV at the count bound's precision (1e-5)."""
    run_case(bh, nq, nk, m, tau, "f32")
    name = f"bh{bh}_nq{nq}_nk{nk}_m{m}_tau{tau}_f32"
    got = {k: e for tag, k, f, e, tol in parity.RECORD if tag == name and k in ("y", "dv")}
    assert len(got) == 2 and max(got.values()) < 1e-5, got


@pytest.mark.parametrize("bh,nq,nk,m,tau,dtype", [(1, 1, 65536, 4, 10, "f32"), (2, 65536, 3, 5, 10, "f32"),
                                                   (1, 3, 40000, 6, 9, "bf16")])
def test_extreme_aspect(bh, nq, nk, m, tau, dtype):
    """A handful of queries against the longest key sequence, and the reverse: one
    side's pair pass has a single ragged row tile whose partners span a long sorted
    range, the other side's rows have at most a few partners each; the tables sum
    65536 source rows into a few destinations (and a few into many)."""
    run_case(bh, nq, nk, m, tau, dtype)


def run_case(bh, nq, nk, m, tau, dtype, dist="gauss"):
    name = f"bh{bh}_nq{nq}_nk{nk}_m{m}_tau{tau}_{dtype}" + ("" if dist == "gauss" else f"_{dist}")
    log(f"[{name}] start")
    w = workloads.Workload(name, 1, bh, nq, 64, tau, m, dtype, dist, 1234 + nq + 7 * nk + m + tau)
    inp = make_inputs(w, n=nq, n_k=nk)
    g = run_gpu(inp, m, tau, dtype)
    check_codes(name + "/q", inp["q"], inp["R"], m, tau, g["qc"])
    check_codes(name + "/k", inp["k"], inp["R"], m, tau, g["kc"])
    check_outputs(name, inp, g, m, tau, dtype)
    return g


def large_bucket_share(qc, kc, tau, t=None):
    """Fraction of the (row, hash) pairs of both sides that sit in buckets with
    b_q b_k > t (b_q + b_k): with the library's own threshold (the default), the
    buckets whose dQ, dK rows the backward computes in the bucket-table form."""
    if t is None:
        t = Y.yoso_backward_table_threshold()
    nb = 1 << tau
    rows = big = 0
    for b in range(qc.shape[0]):
        for h in range(qc.shape[1]):
            bq = np.bincount(qc[b, h], minlength=nb).astype(np.int64)
            bk = np.bincount(kc[b, h], minlength=nb).astype(np.int64)
            sel = bq * bk > t * (bq + bk)
            big += int((bq + bk)[sel].sum())
            rows += int((bq + bk).sum())
    return big / max(rows, 1)


TABLE_FORM = [
    # (bh, n_q, n_k, m, tau, dtype, dist): buckets of hundreds of rows on both sides.  (The dense tiles
    # serve all but the last; test_pairs_gpu.py holds the bucket form at such lengths.)
    (2, 1500, 1100, 4, 4, "f32", "gauss"),     # 16 buckets, every one large
    (1, 2000, 1300, 6, 6, "f32", "mixture"),   # large and small buckets side by side in one row tile
    (2, 1100, 3000, 3, 3, "bf16", "mixture"),
    (1, 1025, 1030, 2, 1, "f32", "gauss"),     # two buckets; ragged last tiles and partner groups
    (1, 16000, 15999, 2, 12, "f32", "mixture"),  # a few large buckets among thousands of tiny ones
]


@pytest.mark.parametrize("bh,nq,nk,m,tau,dtype,dist", TABLE_FORM)
def test_bucket_table_form(bh, nq, nk, m, tau, dtype, dist):
    """Large buckets: where the pair passes serve the call, their dQ, dK rows come from one
    64 x 64 matrix per bucket (the table form) while the other buckets keep the passes; every row
    is checked against the oracle's pairwise sums."""
    g = run_case(bh, nq, nk, m, tau, dtype, dist)
    share = large_bucket_share(g["qc"], g["kc"], tau)
    log(f"[table form {bh}x{nq}x{nk} tau {tau} {dist}] rows in large buckets: {share:.3f}")
    assert share > 0.05


@pytest.mark.parametrize("name", list(WORKLOADS))
def test_workload_full_size(name):
    """Every head runs on the GPU exactly as the bench launches it; the oracle
    recomputes the first and the last head (heads are independent, so this is
    exact)."""
    w = WORKLOADS[name]
    log(f"[{name}] start: bh={w.bh} n={w.n} m={w.m} tau={w.tau} {w.dtype}")
    inp = make_inputs(w)
    g = run_gpu(inp, w.m, w.tau, w.dtype)
    heads = [0, w.bh - 1]
    sl = np.array(sorted(set(heads)))
    check_codes(name + "/q", inp["q"][sl], inp["R"], w.m, w.tau, g["qc"][sl])
    check_codes(name + "/k", inp["k"][sl], inp["R"], w.m, w.tau, g["kc"][sl])
    check_outputs(name, inp, g, w.m, w.tau, w.dtype, heads=sl)


@pytest.mark.parametrize("what,scale", [("dy", 1e-6), ("dy", 1e3), ("v", 1e-5), ("rows", None)])
def test_backward_far_from_unit_scale(what, scale):
    """Upstream gradients (and values) far from unit size: typical training
    gradients are small, and the fp16 (hi, lo) split would lose them without the
    per-head power-of-two scaling; "rows" gives every row of dY and V its own scale
    (10^-4 .. 1 and 10^-3 .. 10), which the per-row factor on S covers."""
    bh, n, m, tau = 2, 700, 16, 8
    name = f"scaled {what} {scale}"
    log(f"[{name}] start")
    w = workloads.Workload(name, 1, bh, n, 64, tau, m, "f32", "gauss", 4321)
    inp = make_inputs(w)
    if what == "rows":
        g = np.random.default_rng(99)
        inp["dy"] = inp["dy"] * 10.0 ** g.uniform(-4, 0, size=(bh, n, 1))
        inp["v"] = inp["v"] * 10.0 ** g.uniform(-3, 1, size=(bh, n, 1))
    else:
        inp[what] = inp[what] * scale
    # the oracle sees the fp32 values the GPU reads
    for key in ("dy", "v"):
        inp[key] = inp[key].astype(np.float32).astype(np.float64)
    g = run_gpu(inp, m, tau, "f32")
    y = oracle.forward(g["qc"], g["kc"], inp["v"], m, tau)
    dq, dk, dv = oracle.backward(g["qc"], g["kc"], inp["q"], inp["k"], inp["v"], inp["dy"], m, tau)
    check_all(name, [(key, g[key], ref) for key, ref in (("y", y), ("dq", dq), ("dk", dk), ("dv", dv))], TOL["f32"])


@pytest.mark.parametrize("what,scale", [("dy", 1e-6), ("v", 1e3), ("rows", None)])
def test_bucket_table_form_far_from_unit_scale(what, scale):
    """Small and large gradients and rows of very different size (10^-4 .. 1 in dY, 10^-3 .. 10
    in V) in buckets of a few hundred rows.  (The dense tiles serve this length; test_pairs_gpu.py holds the
    per-bucket power-of-two scaling of M = sum a' b^T.)"""
    bh, nq, nk, m, tau = 2, 1200, 1400, 6, 4
    name = f"table form scaled {what} {scale}"
    log(f"[{name}] start")
    w = workloads.Workload(name, 1, bh, nq, 64, tau, m, "f32", "mixture", 8642)
    inp = make_inputs(w, n=nq, n_k=nk)
    if what == "rows":
        g = np.random.default_rng(98)
        inp["dy"] = inp["dy"] * 10.0 ** g.uniform(-4, 0, size=(bh, nq, 1))
        inp["v"] = inp["v"] * 10.0 ** g.uniform(-3, 1, size=(bh, nk, 1))
    else:
        inp[what] = inp[what] * scale
    for key in ("dy", "v"):
        inp[key] = inp[key].astype(np.float32).astype(np.float64)
    g = run_gpu(inp, m, tau, "f32")
    assert large_bucket_share(g["qc"], g["kc"], tau) > 0.05
    dq, dk, _ = oracle.backward(g["qc"], g["kc"], inp["q"], inp["k"], inp["v"], inp["dy"], m, tau)
    check_all(name, [(key, g[key], ref) for key, ref in (("dq", dq), ("dk", dk))], TOL["f32"])


def test_tables_resolve_every_feature_dim():
    """Feature dims of very different scales (10^-3 .. 10^3 within every table slice):
    each dim has its own fixed-point scale, so each column of Y and dV meets the bar
    on its own, not only the rows dominated by the largest dims."""
    bh, n, m, tau = 1, 16384, 8, 8
    w = workloads.Workload("anisotropic", 1, bh, n, 64, tau, m, "f32", "gauss", 777)
    inp = make_inputs(w)
    g = np.random.default_rng(5)
    for key in ("v", "dy"):
        scales = 10.0 ** g.permutation(np.linspace(-3, 3, 64))
        inp[key] = (inp[key] * scales).astype(np.float32).astype(np.float64)
    out = run_gpu(inp, m, tau, "f32")
    y = oracle.forward(out["qc"], out["kc"], inp["v"], m, tau)
    _, _, dv = oracle.backward(out["qc"], out["kc"], inp["q"], inp["k"], inp["v"], inp["dy"], m, tau)
    for key, ref in (("y", y), ("dv", dv)):
        got = out[key][0]
        col = np.linalg.norm(got - ref[0], axis=0) / np.linalg.norm(ref[0], axis=0)
        log(f"[anisotropic] {key}: worst column rel err {col.max():.2e} (dim {int(col.argmax())})")
        assert col.max() <= TOL["f32"], (key, col.max())


def test_empty_and_degenerate():
    # bh = 0, n_q = 0, n_k = 0: valid calls; empty key set gives zero outputs
    m, tau = 4, 3
    R = torch.randn(64, m * tau, device="cuda")
    for bh, nq, nk in [(0, 5, 5), (2, 0, 6), (2, 6, 0)]:
        q = torch.nn.functional.normalize(torch.randn(bh, nq, 64, device="cuda"), dim=-1)
        k = torch.nn.functional.normalize(torch.randn(bh, nk, 64, device="cuda"), dim=-1)
        v = torch.randn(bh, nk, 64, device="cuda")
        dy = torch.randn(bh, nq, 64, device="cuda")
        qc, kc = Y.hash_qk(q, k, R, m, tau)
        y = Y.forward(qc, kc, v, m, tau, n_q=nq)
        dq, dk, dv = Y.backward(qc, kc, q, k, v, dy, m, tau)
        torch.cuda.synchronize()
        for t in (y, dq, dk, dv):
            assert t.numel() == 0 or float(t.abs().max()) == 0.0


def test_golden_worked_example(golden):
    """The hand-worked example (d = 2 padded to 64 with zeros) through the GPU path."""
    g = golden["forward_backward"]
    m, tau = g["m"], g["tau"]
    pad = lambda a: np.pad(np.array(a, np.float32), ((0, 0), (0, 62)))[None]
    q, k, v, dy = (to_dev(pad(g[s]), "f32") for s in ("q", "k", "v", "dy"))
    qc = torch.from_numpy(np.ascontiguousarray(np.array(g["qc"], np.int16).T)[None]).cuda()
    kc = torch.from_numpy(np.ascontiguousarray(np.array(g["kc"], np.int16).T)[None]).cuda()
    y = Y.forward(qc, kc, v, m, tau, n_q=2)
    dq, dk, dv = Y.backward(qc, kc, q, k, v, dy, m, tau)
    torch.cuda.synchronize()
    for t, key in ((y, "y"), (dq, "dq"), (dk, "dk"), (dv, "dv")):
        got = t.cpu().numpy()[0]
        ref = np.array(g[key])
        np.testing.assert_allclose(got[:, :2], ref, rtol=1e-5, atol=1e-5, err_msg=key)
        assert not got[:, 2:].any()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_hash_rows_of_any_magnitude(dtype):
    """Rows scaled by powers of ten from 1e-30 to 1e30 (each row its own): the hash
    scales every row by a power of two before its fp16 split, so its codes equal the
    oracle's wherever every projection of the hash exceeds 1e-4 |x| |R[:, c]|."""
    g = np.random.default_rng(11)
    bh, n, m, tau = 2, 300, 8, 9
    x = g.standard_normal((bh, n, 64)) * 10.0 ** g.uniform(-30, 30, size=(bh, n, 1))
    x = x.astype(np.float32)
    if dtype == "bf16":
        x = workloads.bf16_round(x)
    R = g.standard_normal((64, m * tau)).astype(np.float32)
    codes = torch.empty((bh, n, m), dtype=torch.int16, device="cuda")
    Y.yoso_hash(to_dev(x, dtype), torch.from_numpy(R).cuda(), m, tau, codes)
    got = codes_np(codes)  # [bh, m, n]
    ref = oracle.hash_codes(x.astype(np.float64), R, m, tau)
    proj = np.einsum("bnd,dc->bnc", x.astype(np.float64), R.astype(np.float64))
    rel = np.abs(proj) / (np.linalg.norm(x.astype(np.float64), axis=-1, keepdims=True) *
                          np.linalg.norm(R.astype(np.float64), axis=0))
    sure = rel.reshape(bh, n, m, tau).min(-1).transpose(0, 2, 1) > 1e-4  # [bh, m, n]
    mism = (got != ref) & sure
    log(f"[hash any magnitude {dtype}] {sure.size} codes, excluded {1 - sure.mean():.2e}, mismatches {int(mism.sum())}")
    assert sure.mean() > 0.95
    assert not mism.any()


def test_golden_hash_example(golden):
    g = golden["hash"]
    m, tau = g["m"], g["tau"]
    x = np.pad(np.array(g["x"], np.float32), ((0, 0), (0, 61)))[None]
    R = np.pad(np.array(g["R"], np.float32), ((0, 61), (0, 0)))
    codes = torch.empty((1, x.shape[1], m), dtype=torch.int16, device="cuda")
    Y.yoso_hash(to_dev(x, "f32"), torch.from_numpy(R).cuda(), m, tau, codes)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(codes_np(codes)[0], np.array(g["codes"]))


def test_repeatable_and_side_stream():
    w = WORKLOADS["single_head_n512"]
    inp = make_inputs(w)
    a = run_gpu(inp, w.m, w.tau, w.dtype)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        b = run_gpu(inp, w.m, w.tau, w.dtype)
    np.testing.assert_array_equal(a["qc"], b["qc"])
    np.testing.assert_array_equal(a["kc"], b["kc"])
    # every accumulation order is fixed (integer tables; stable bucket order; partial
    # rows summed in hash order), so a repeat is bitwise identical
    for key in ("y", "dq", "dk", "dv"):
        np.testing.assert_array_equal(b[key], a[key], err_msg=key)


def one_bucket_inputs(n):
    """Every row of Q and K is the same unit vector u, so every hash puts every key
    in one bucket; V and dY are constant rows of dyadic values, so every sum is exact."""
    u = torch.zeros(64, device="cuda")
    u[0] = 1.0
    x = u.expand(1, n, 64).contiguous()
    v = torch.cat([torch.full((1, n, 32), 1.0), torch.full((1, n, 32), -0.75)], dim=-1).cuda()
    dy = torch.cat([torch.full((1, n, 32), 0.5), torch.full((1, n, 32), 0.25)], dim=-1).cuda()
    return u, x, v, dy


def test_all_keys_in_one_bucket_forward_at_the_length_limit():
    """The worst case of the tables' fixed-point bound: all 65536 keys in one bucket,
    all values of a dim of one sign.  Y is exact (every query reads the sum of V)."""
    n, m, tau = 65536, 2, 8
    _, x, v, _ = one_bucket_inputs(n)
    R = torch.randn(64, m * tau, device="cuda", generator=torch.Generator("cuda").manual_seed(5))
    qc, kc = Y.hash_qk(x, x, R, m, tau)
    y = Y.forward(qc, kc, v, m, tau)
    torch.cuda.synchronize()
    assert bool((qc == qc[0, 0]).all()) and bool((kc == qc[0, 0]).all())
    expect = v[0].sum(dim=0)                      # [65536]*32 + [-49152]*32, exact
    log(f"[one bucket, n={n}] Y row 0 {y[0, 0, :2].tolist()} ... expected {expect[:2].tolist()}")
    assert torch.equal(y[0], expect.expand(n, 64))


def test_all_keys_in_one_bucket_backward_closed_form():
    """Every pair collides in every hash: dV_j = sum_i dY_i, dQ_i = (tau/2)(dY_i . sum V) u
    and dK_j = (tau/2)(V_j . sum dY) u (eq. pseudo-gradient-q with B = 1)."""
    n, m, tau = 4096, 2, 8
    u, x, v, dy = one_bucket_inputs(n)
    R = torch.randn(64, m * tau, device="cuda", generator=torch.Generator("cuda").manual_seed(6))
    qc, kc = Y.hash_qk(x, x, R, m, tau)
    dq, dk, dv = Y.backward(qc, kc, x, x, v, dy, m, tau)
    torch.cuda.synchronize()
    sv, sdy = v[0].double().sum(0), dy[0].double().sum(0)
    dq_ref = (tau / 2) * (dy[0].double() @ sv)[:, None] * u.double()[None, :]
    dk_ref = (tau / 2) * (v[0].double() @ sdy)[:, None] * u.double()[None, :]
    assert torch.equal(dv[0].double(), sdy.expand(n, 64))
    check_all(f"one bucket, n={n}", [(name, got.double().cpu().numpy()[None], ref.cpu().numpy()[None])
                                     for name, got, ref in (("dq", dq[0], dq_ref), ("dk", dk[0], dk_ref))],
              TOL["f32"])
