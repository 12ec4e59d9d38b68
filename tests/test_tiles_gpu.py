"""The dense tiles (csrc/dense.hip) against the fp64 oracle, at the sizes where they can
go wrong: edges of the 32-row blocks, of the 32- and 64-row tiles and of the 128- and
256-row workgroups, one to 64 hashes, one to twelve bits (the three plane layouts),
streamed rows split among workgroups, and the shapes beside them that keep the pair and
table forms.  The library's kernel timer says which form ran.  Bars as in parity.py."""
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


def to_dev(a, dtype):
    t = torch.from_numpy(np.ascontiguousarray(a, np.float32))
    return t.to(device="cuda", dtype=torch.bfloat16 if dtype == "bf16" else torch.float32).contiguous()


def codes_np(t):
    return np.ascontiguousarray(t.cpu().numpy().view(np.uint16).transpose(0, 2, 1))


def host(t):
    return t.float().cpu().numpy().astype(np.float64)


def inputs(bh, nq, nk, m, tau, dtype, dist="gauss"):
    w = workloads.Workload("tiles", 1, bh, nq, 64, tau, m, dtype, dist, 977 + nq + 3 * nk + m + 100 * tau)
    inp = make_inputs(w, n=nq, n_k=nk)
    q, k, v, dy = (to_dev(inp[s], dtype) for s in ("q", "k", "v", "dy"))
    R = torch.from_numpy(inp["R"]).cuda()
    return Y.hash_qk(q, k, R, m, tau), (q, k, v, dy)


def timed(names, call):
    torch.cuda.synchronize()
    Y.yoso_timing_enable(64)
    Y.yoso_timing_reset()
    try:
        out = call()
        torch.cuda.synchronize()
        return out, {n: Y.yoso_timing_query(n)[1] for n in names}
    finally:
        Y.yoso_timing_enable(0)


FORMS = ("tile_kernel", "dense_kernel", "pass_kernel", "dense_sum_kernel")

BACKWARD = [
    # (bh, n_q, n_k, m, tau, dtype, form, split): heads 0 and bh - 1 are compared
    (2100, 17, 33, 5, 2, "f32", "tile_kernel", False),      # one partial block; 8 waves
    (520, 33, 31, 32, 8, "bf16", "tile_kernel", False),
    (512, 200, 200, 32, 8, "f32", "tile_kernel", False),    # 8 waves, ragged tile and rows
    (512, 129, 257, 31, 7, "bf16", "tile_kernel", False),
    (260, 65, 255, 8, 8, "f32", "tile_kernel", False),      # 4 waves
    (9, 64, 5000, 32, 8, "f32", "tile_kernel", True),       # the fewest rows beside a long side
    (9, 5000, 65, 7, 5, "bf16", "tile_kernel", True),
    (9, 63, 5000, 32, 8, "f32", "pass_kernel", None),       # fewer: pairs
    (1, 1100, 1030, 32, 8, "f32", "tile_kernel", True),     # few blocks: split rows
    (3, 1025, 577, 1, 1, "f32", "tile_kernel", False),
    (2, 1500, 1030, 32, 12, "f32", "tile_kernel", True),    # twelve plane words
    (150, 300, 320, 16, 9, "bf16", "tile_kernel", False),
    (2, 1030, 1500, 33, 8, "f32", "tile_kernel", True),     # two words per plane
    (270, 128, 130, 64, 6, "f32", "tile_kernel", False),
    (1, 2049, 4100, 64, 8, "bf16", "tile_kernel", True),
    (8, 63, 128, 32, 8, "f32", "dense_kernel", None),       # below the rule: the 16 x 16 form
    (1, 64, 64, 32, 8, "f32", "tile_kernel", False),        # a few heads: both sides in one launch
    (1, 512, 512, 32, 8, "f32", "tile_kernel", True),
    (2, 1023, 65, 16, 10, "bf16", "tile_kernel", True),
    (3, 300, 700, 32, 12, "f32", "tile_kernel", True),
    (31, 1024, 1024, 32, 8, "f32", "tile_kernel", False),   # 496 workgroups, one launch; 32 heads: two
    (32, 1024, 1024, 32, 8, "bf16", "tile_kernel", None),
    (1, 1100, 1100, 34, 9, "f32", "pass_kernel", None),     # no plane layout: pairs
    (32, 3000, 3000, 2, 10, "bf16", "pass_kernel", None),   # few hashes: pairs
    (32, 1200, 1200, 2, 10, "f32", "pass_kernel", None),
    (64, 1100, 1100, 4, 8, "f32", "pass_kernel", None),
    (4, 4000, 4000, 2, 10, "f32", "pass_kernel", None),     # (no scratch to split the rows)
    (1, 300, 8000, 4, 8, "f32", "pass_kernel", None),       # a short side beside a long one
    (4, 8000, 500, 2, 6, "bf16", "pass_kernel", None),
    (1024, 1, 512, 32, 8, "f32", "tile_kernel", False),     # many heads of a few rows: no pairs there
]


@pytest.mark.parametrize("bh,nq,nk,m,tau,dtype,form,split", BACKWARD)
def test_backward_tiles(bh, nq, nk, m, tau, dtype, form, split):
    (qc, kc), (q, k, v, dy) = inputs(bh, nq, nk, m, tau, dtype)
    out, ran = timed(FORMS, lambda: Y.backward(qc, kc, q, k, v, dy, m, tau))
    assert ran[form] >= 1 and sum(ran[f] for f in FORMS[:3]) == ran[form], ran
    if split is not None:
        assert (ran["dense_sum_kernel"] == 1) == split, ran
    again = Y.backward(qc, kc, q, k, v, dy, m, tau)
    assert all(torch.equal(a, b) for a, b in zip(out, again))
    sl = [0, bh - 1] if bh > 1 else [0]
    ref = oracle.backward(codes_np(qc[sl]), codes_np(kc[sl]), host(q[sl]), host(k[sl]), host(v[sl]), host(dy[sl]), m, tau)
    check_all(f"tiles bh{bh} {nq}x{nk} m{m} tau{tau} {dtype}",
              [(n, host(o[sl]), r) for n, o, r in zip(("dq", "dk", "dv"), out, ref)], TOL[dtype])


@pytest.mark.parametrize("bh,nq,nk,m,tau,dtype,tiles", [
    (1, 257, 300, 32, 8, "f32", True),
    (300, 130, 33, 5, 3, "bf16", True),
    (2, 1100, 600, 20, 12, "f32", True),
    (1, 500, 1030, 60, 8, "bf16", True),
    (1, 300, 290, 40, 12, "f32", False),     # no plane layout
    (1, 4000, 4000, 1, 4, "f32", False),     # one hash: few derived hashes
    (16, 100, 4000, 2, 10, "bf16", False),   # few and long workgroups of the tiles
    (4, 8000, 500, 4, 8, "bf16", False),
    (1, 300, 8000, 32, 8, "f32", True),
])
def test_star_tiles(bh, nq, nk, m, tau, dtype, tiles):
    (qc, kc), (q, k, v, dy) = inputs(bh, nq, nk, m, tau, dtype, "mixture")
    out, ran = timed(("tile_star_kernel", "pass_star_kernel"),
                     lambda: Y.backward_star(qc, kc, q, k, v, dy, m, tau))
    assert (ran["tile_star_kernel"], ran["pass_star_kernel"]) == ((1, 0) if tiles else (0, 1)), ran
    sl = [0, bh - 1] if bh > 1 else [0]
    ref = oracle.backward_star(codes_np(qc[sl]), codes_np(kc[sl]), host(q[sl]), host(k[sl]), host(v[sl]), host(dy[sl]),
                               m, tau)
    check_all(f"star tiles bh{bh} {nq}x{nk} m{m} tau{tau} {dtype}",
              [(n, host(o[sl]), r) for n, o, r in zip(("dq", "dk", "dv"), out, ref)], TOL[dtype])


@pytest.mark.parametrize("n,nk,m,tau,what", [
    (2048, 2048, 32, 8, "dy"), (2048, 2048, 32, 8, "v"), (700, 650, 32, 8, "dy"), (1500, 1200, 16, 11, "v"),
    (1200, 1500, 64, 8, "dy"),
])
def test_backward_one_large_row(n, nk, m, tau, what):
    """One row of dY (or V) 10^4 times the others: the rows of dK (or dQ) that it does not reach
    consist of weights 2^13 below the largest of their head.  A weight of one hash is at least
    about 2^8 in its fp16 pair's window, so then 2^-5, and ends at 2^-25: 2^-20 = 1e-6 of it,
    and less of a row's sum."""
    w = workloads.Workload("large", 1, 1, n, 64, tau, m, "f32", "gauss", 5100 + n + m)
    inp = make_inputs(w, n=n, n_k=nk)
    inp[what][:, inp[what].shape[1] // 2] *= 1e4
    q, k, v, dy = (to_dev(inp[s], "f32") for s in ("q", "k", "v", "dy"))
    qc, kc = Y.hash_qk(q, k, torch.from_numpy(inp["R"]).cuda(), m, tau)
    out, ran = timed(FORMS, lambda: Y.backward(qc, kc, q, k, v, dy, m, tau))
    assert ran["tile_kernel"] >= 1, ran
    ref = oracle.backward(codes_np(qc), codes_np(kc), host(q), host(k), host(v), host(dy), m, tau)
    got, want = (host(out[1])[0], ref[1][0]) if what == "dy" else (host(out[0])[0], ref[0][0])
    size = np.linalg.norm(want, axis=-1)
    err = (np.linalg.norm(got - want, axis=-1)[size > 0] / size[size > 0])
    print(f"[large row {n}x{nk} m{m} tau{tau} {what}] median row error {np.median(err):.2e}")
    assert np.median(err) < 1e-6, np.median(err)


@pytest.mark.parametrize("bh,nq,nk,m,tau,dtype", [
    (2, 2048, 1500, 32, 8, "f32"),        # maxima from the prep launch
    (1, 1200, 1100, 16, 9, "f32"),        # both sides in one launch
    (96, 1030, 600, 32, 10, "f32"),       # scanned by each workgroup; the forward in tiles as well
    (96, 1030, 600, 32, 10, "bf16"),
])
def test_tiles_resolve_every_feature_dim(bh, nq, nk, m, tau, dtype):
    """Feature dims of very different scales (10^-4 .. 10^4, and one of zeros): each dim has its own
    power of two, as in the bucket tables, so each column of Y and dV meets the bar on its
    own; dQ and dK, sums over all dims, meet it as a whole."""
    w = workloads.Workload("dims", 1, bh, nq, 64, tau, m, dtype, "gauss", 640 + nq)
    inp = make_inputs(w, n=nq, n_k=nk)
    g = np.random.default_rng(6)
    for key in ("v", "dy"):
        scales = 10.0 ** g.permutation(np.linspace(-4, 4, 64))
        scales[7] = 0.0
        inp[key] = inp[key] * scales
    q, k, v, dy = (to_dev(inp[s], dtype) for s in ("q", "k", "v", "dy"))
    qc, kc = Y.hash_qk(q, k, torch.from_numpy(inp["R"]).cuda(), m, tau)
    y = Y.forward(qc, kc, v, m, tau)
    (dq, dk, dv), ran = timed(FORMS, lambda: Y.backward(qc, kc, q, k, v, dy, m, tau))
    assert ran["tile_kernel"] >= 1, ran
    sl = [0]
    ry = oracle.forward(codes_np(qc[sl]), codes_np(kc[sl]), host(v[sl]), m, tau)
    rq, rk, rv = oracle.backward(codes_np(qc[sl]), codes_np(kc[sl]), host(q[sl]), host(k[sl]), host(v[sl]), host(dy[sl]),
                                 m, tau)
    for name, got, ref in (("y", host(y[sl])[0], ry[0]), ("dv", host(dv[sl])[0], rv[0])):
        size = np.linalg.norm(ref, axis=0)
        col = np.linalg.norm(got - ref, axis=0) / np.where(size > 0, size, 1.0)
        print(f"[dims {bh}x{nq}x{nk} {dtype}] {name}: worst column {col.max():.2e}")
        assert col.max() <= TOL[dtype], (name, col.max())
    check_all(f"dims {bh}x{nq}x{nk} {dtype}", [("dq", host(dq[sl]), rq), ("dk", host(dk[sl]), rk)], TOL[dtype])


@pytest.mark.parametrize("bh,nq,nk,m,tau,dtype", [
    (1, 1024, 1000, 32, 8, "f32"),    # both sides in one launch, split; 32-row tiles
    (1, 1024, 1000, 32, 8, "bf16"),
    (1, 900, 4000, 16, 9, "f32"),     # one side of few rows, one of many
    (64, 600, 1000, 48, 8, "f32"),    # a launch per side, scanned by each workgroup
    (96, 1000, 1000, 32, 8, "f32"),   # 64-row tiles; the forward in tiles as well
    (96, 1000, 1000, 32, 8, "bf16"),
])
@pytest.mark.parametrize("ratio", [1e-5, 1e-11])
def test_rows_far_apart(bh, nq, nk, m, tau, dtype, ratio):
    """Two opposite groups of rows that share no bucket, the first with dY, V, Q and K `ratio`
    times the second's (codes do not depend on a row's length): up to 1024 streamed rows, a tile far below
    its head has scales of its own, so the first group's outputs are as good as the second's."""
    g = np.random.default_rng(9300 + nq + m)
    unit = lambda a: a / np.linalg.norm(a, axis=-1, keepdims=True)
    u = unit(g.standard_normal((bh, 1, 64)))
    half = lambda n: n // 128 * 64
    first = lambda n: (np.arange(n) < half(n))[None, :, None]
    rows = lambda n: unit(np.where(first(n), 1.0, -1.0) * 3.0 * u + unit(g.standard_normal((bh, n, 64))))
    size = lambda n: np.where(first(n), ratio, 1.0)
    q, k = rows(nq) * size(nq), rows(nk) * size(nk)
    v, dy = g.standard_normal((bh, nk, 64)) * size(nk), g.standard_normal((bh, nq, 64)) * size(nq)
    q, k, v, dy = (to_dev(a, dtype) for a in (q, k, v, dy))
    qc, kc = Y.hash_qk(q, k, torch.from_numpy(g.standard_normal((64, m * tau)).astype(np.float32)).cuda(), m, tau)
    y, form = timed(("dense_fwd_kernel",), lambda: Y.forward(qc, kc, v, m, tau))
    assert (form["dense_fwd_kernel"] == 1) == (bh > 1), form
    (dq, dk, dv), ran = timed(FORMS, lambda: Y.backward(qc, kc, q, k, v, dy, m, tau))
    assert ran["tile_kernel"] >= 1, ran
    sl = [0, bh - 1] if bh > 1 else [0]
    c = (codes_np(qc[sl]), codes_np(kc[sl]))
    ry = oracle.forward(*c, host(v[sl]), m, tau)
    rq, rk, rv = oracle.backward(*c, host(q[sl]), host(k[sl]), host(v[sl]), host(dy[sl]), m, tau)
    # (dQ of a query streams the keys, dK and dV of a key the queries)
    outs = [("y", y, ry, nq, nk), ("dq", dq, rq, nq, nk), ("dk", dk, rk, nk, nq), ("dv", dv, rv, nk, nq)]
    for name, got, ref, n, streamed in outs:
        got = host(got[sl])
        for part in (slice(0, half(n)), slice(half(n), n)):
            if part.start == 0 and (streamed > 1024 or (name == "y" and form["dense_fwd_kernel"] == 0)):
                continue  # (one scale per head or bucket table)
            err = np.linalg.norm(got[:, part] - ref[:, part]) / np.linalg.norm(ref[:, part])
            print(f"[far apart {bh}x{nq}x{nk} m{m} {dtype} {ratio:g}] {name} from row {part.start}: {err:.2e}")
            assert err <= TOL[dtype], (name, part, err)


@pytest.mark.parametrize("m,bar", [(32, 2.5e-7), (48, 2.4e-7)])
def test_long_sums_of_one_sign(m, bar):
    """4096 clustered rows, not split: a running sum takes 128 additions of mostly one sign, each off by
    0.29 of the last place (2^-23.5) or so, together sqrt(128 / 3) times that or 1.6e-7; in parts of 2048
    rows 0.8e-7, beside 2.2e-7 of all else.  The bar is the error of the pair passes."""
    bh, n, tau = 16, 4096, 8
    (qc, kc), (q, k, v, dy) = inputs(bh, n, n, m, tau, "f32", "mixture")
    (dq, dk, dv), ran = timed(FORMS, lambda: Y.backward(qc, kc, q, k, v, dy, m, tau))
    assert ran["tile_kernel"] >= 1 and ran["dense_sum_kernel"] == 0, ran
    sl = [0, bh - 1]
    ref = oracle.backward(codes_np(qc[sl]), codes_np(kc[sl]), host(q[sl]), host(k[sl]), host(v[sl]), host(dy[sl]), m, tau)
    for name, got, r in zip(("dq", "dk"), (dq, dk), ref):
        err = np.linalg.norm(host(got[sl]) - r) / np.linalg.norm(r)
        print(f"[long sums m{m}] {name}: {err:.3e}")
        assert err <= bar, (name, err)


@pytest.mark.parametrize("bh,nq,nk,tau", [(1, 300, 5, 8), (2, 333, 290, 8), (300, 300, 130, 8), (1, 1000, 1500, 9)])
@pytest.mark.parametrize("ratio", [1e-7, 1e-4])
def test_expectation_rows_far_apart(bh, nq, nk, tau, ratio):
    """Two opposite groups of rows (cosines about -0.95 between them, P down to 1e-9), the first with
    dY and V `ratio` times the second's: a run of small rows has scales of its own (per tile of
    32 or 64 rows), so sums that the large ones hardly reach keep the bar."""
    g = np.random.default_rng(9100 + nq)
    unit = lambda a: a / np.linalg.norm(a, axis=-1, keepdims=True)
    u = unit(g.standard_normal((bh, 1, 64)))
    side = lambda n: np.where(np.arange(n) < n // 2, 1.0, -1.0)[None, :, None]
    rows = lambda n: unit(side(n) * np.sqrt(0.97) * u + np.sqrt(0.03) * unit(g.standard_normal((bh, n, 64))))
    size = lambda n: np.where(np.arange(n) < n // 2, ratio, 1.0)[None, :, None]
    q, k = rows(nq), rows(nk)
    v, dy = g.standard_normal((bh, nk, 64)) * size(nk), g.standard_normal((bh, nq, 64)) * size(nq)
    q, k, v, dy = (to_dev(a, "f32") for a in (q, k, v, dy))
    y, dq, dk, dv = torch.empty_like(q), torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
    Y.yoso_expectation_forward(q, k, v, tau, y)
    Y.yoso_expectation_backward(q, k, v, dy, tau, dq, dk, dv)
    sl = [0, bh - 1] if bh > 1 else [0]
    ey, edv, _, _ = oracle.expectation(host(q[sl]), host(k[sl]), host(v[sl]), host(dy[sl]), tau)
    # (each group's rows of Y and dV are mostly sums of their own group's)
    for name, got, ref, n in (("y", y, ey, nq), ("dv", dv, edv, nk)):
        d = np.linalg.norm(host(got[sl]) - ref, axis=-1)[:, :n // 2] / np.linalg.norm(ref, axis=-1)[:, :n // 2]
        print(f"[far apart {bh}x{nq}x{nk} tau{tau} {ratio:g}] {name}: worst small row {d.max(initial=0):.2e}")
        assert d.max(initial=0) < 1e-4, (name, d.max())


@pytest.mark.parametrize("what,scale", [("dy", 1e-25), ("v", 1e-25), ("dy", 1e-34), ("dy", 1e25), ("v", 1e30)])
@pytest.mark.parametrize("kind,n,m", [("backward", 300, 32), ("backward", 1500, 16), ("star", 300, 32),
                                      ("expectation", 300, 8)])
def test_tiles_any_magnitude(kind, n, m, what, scale):
    """dY or V of any finite size: the squares of such rows vanish or overflow, the rows' and
    heads' powers of two do not."""
    tau = 8
    w = workloads.Workload("magnitude", 1, 1, n, 64, tau, m, "f32", "gauss", 8300 + n + m)
    inp = make_inputs(w, n=n, n_k=n - 20)
    inp[what] *= scale
    q, k, v, dy = (to_dev(inp[s], "f32") for s in ("q", "k", "v", "dy"))
    if kind == "expectation":
        dq, dk, dv = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
        Y.yoso_expectation_backward(q, k, v, dy, tau, dq, dk, dv)
        _, rv, rq, rk = oracle.expectation(host(q), host(k), host(v), host(dy), tau)
    else:
        qc, kc = Y.hash_qk(q, k, torch.from_numpy(inp["R"]).cuda(), m, tau)
        call, ref = (Y.backward, oracle.backward) if kind == "backward" else (Y.backward_star, oracle.backward_star)
        (dq, dk, dv), ran = timed(("tile_kernel", "tile_star_kernel"), lambda: call(qc, kc, q, k, v, dy, m, tau))
        assert sum(ran.values()) >= 1, ran
        rq, rk, rv = ref(codes_np(qc), codes_np(kc), host(q), host(k), host(v), host(dy), m, tau)
    # (compared at the size of one: errors of values at 1e-34 square to nothing)
    f = 1.0 / scale
    check_all(f"magnitude {kind} {n} {what} {scale:g}",
              [("dq", host(dq) * f, rq * f), ("dk", host(dk) * f, rk * f)] +
              ([("dv", host(dv) * f, rv * f)] if what == "dy" and kind != "star" else []), TOL["f32"])


@pytest.mark.parametrize("m", [3, 15, 32, 63, 64])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("star", [False, True])
def test_largest_weights(star, dtype, m):
    """Every pair collides in every hash, V and dY rows of equal entries just below a power of
    two: the scalar products and the counts at their bounds, the last keys also beside
    pairs of a single hash."""
    n, nk, tau = 300, 270, 8
    g = np.random.default_rng(60 + m)
    u = g.standard_normal(64)
    q = np.tile(u / np.linalg.norm(u), (1, n, 1))
    k = np.tile(u / np.linalg.norm(u), (1, nk, 1))
    v, dy = np.full((1, nk, 64), 0.998), np.full((1, n, 64), -0.998)
    q, k, v, dy = (to_dev(a, dtype) for a in (q, k, v, dy))
    qc = torch.full((1, n, m), 5, dtype=torch.int16, device="cuda")
    kc = torch.full((1, nk, m), 5, dtype=torch.int16, device="cuda")
    kc[:, 200:, 1:] = 200
    call = Y.backward_star if star else Y.backward
    out, ran = timed(("tile_star_kernel", "tile_kernel"), lambda: call(qc, kc, q, k, v, dy, m, tau))
    assert sum(ran.values()) >= 1, ran
    ref = (oracle.backward_star if star else oracle.backward)(codes_np(qc), codes_np(kc), host(q), host(k), host(v),
                                                              host(dy), m, tau)
    check_all(f"largest weights {'star ' if star else ''}m{m} {dtype}",
              [(s, host(o), r) for s, o, r in zip(("dq", "dk", "dv"), out, ref)], TOL[dtype])


def test_bucket_tables_beside_the_tiles():
    """Clustered rows without a plane layout: the pair passes and the table form of the
    large buckets still serve them."""
    m, tau = 33, 9
    (qc, kc), (q, k, v, dy) = inputs(2, 2200, 2100, m, tau, "f32", "mixture")
    out, ran = timed(("bucket_kernel", "tile_kernel"), lambda: Y.backward(qc, kc, q, k, v, dy, m, tau))
    assert ran["bucket_kernel"] == 1 and ran["tile_kernel"] == 0, ran
    t = Y.yoso_backward_table_threshold()
    large = 0
    for h in range(m):
        bq, bk = (torch.bincount(c[0, :, h].long() & ((1 << tau) - 1), minlength=1 << tau) for c in (qc, kc))
        large += int(((bq * bk) > t * (bq + bk)).sum())
    assert large > 0
    ref = oracle.backward(codes_np(qc), codes_np(kc), host(q), host(k), host(v), host(dy), m, tau)
    check_all("buckets beside the tiles", [(n, host(o), r) for n, o, r in zip(("dq", "dk", "dv"), out, ref)], TOL["f32"])


@pytest.mark.parametrize("bh,nq,nk,tau,dtype", [
    (300, 33, 65, 8, "f32"),
    (3, 1030, 127, 12, "bf16"),
    (2, 255, 1500, 1, "f32"),
])
def test_expectation_tiles(bh, nq, nk, tau, dtype):
    """Clustered and opposite rows: both polynomials of the arccos and the switch between them."""
    (_, _), (q, k, v, dy) = inputs(bh, nq, nk, 1, tau, dtype, "mixture")
    k[:, ::3] *= -1.0
    y, dq, dk, dv = torch.empty_like(q), torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
    Y.yoso_expectation_forward(q, k, v, tau, y)
    Y.yoso_expectation_backward(q, k, v, dy, tau, dq, dk, dv)
    sl = [0, bh - 1]
    ey, edv, edq, edk = oracle.expectation(host(q[sl]), host(k[sl]), host(v[sl]), host(dy[sl]), tau)
    check_all(f"expectation tiles bh{bh} {nq}x{nk} tau{tau} {dtype}",
              [("y", host(y[sl]), ey), ("dq", host(dq[sl]), edq), ("dk", host(dk[sl]), edk), ("dv", host(dv[sl]), edv)],
              TOL[dtype])


@pytest.mark.parametrize("bh,nq,nk,m,tau,dtype,form", [
    (520, 64, 97, 8, 5, "f32", "16 x 16"),       # half of a workgroup of the tiles
    (520, 65, 97, 8, 5, "f32", "tiles"),
    (520, 64, 128, 32, 8, "bf16", "16 x 16"),
    (520, 20, 129, 32, 8, "bf16", "tiles"),
    (300, 20, 129, 32, 8, "f32", "tiles"),       # too few heads for the 16 x 16 form
    (520, 30, 200, 64, 8, "f32", "tiles"),       # two words per plane
    (520, 30, 200, 32, 10, "f32", "16 x 16"),
    (256, 100, 64, 12, 8, "f32", "16 x 16"),     # m not a multiple of 8
    (4, 1500, 1500, 32, 8, "f32", "tables"),     # few heads
])
def test_forward_rule(bh, nq, nk, m, tau, dtype, form):
    """The forward's three forms on either side of their rules.  (A launch of the tiles counts as
    dense_fwd_kernel, like one of the 16 x 16 form, and as tile_fwd_kernel.)"""
    (qc, kc), (q, k, v, dy) = inputs(bh, nq, nk, m, tau, dtype)
    names = ("dense_fwd_kernel", "tile_fwd_kernel", "table_kernel")
    y, ran = timed(names, lambda: Y.forward(qc, kc, v, m, tau, n_q=nq))
    assert ran == dict(zip(names, {"tiles": (1, 1, 0), "16 x 16": (1, 0, 0), "tables": (0, 0, 1)}[form])), ran
    sl = [0, bh - 1]
    ref = oracle.forward(codes_np(qc[sl]), codes_np(kc[sl]), host(v[sl]), m, tau)
    check_all(f"forward {form} bh{bh} {nq}x{nk} m{m} tau{tau} {dtype}", [("y", host(y[sl]), ref)], TOL[dtype])


@pytest.mark.parametrize("bh,nq,nk,m,tau,dtype,kernel", [
    (520, 65, 97, 8, 5, "f32", "tile"),        # 8 waves; a partial word of hashes
    (300, 130, 31, 32, 8, "bf16", "tile"),
    (260, 100, 64, 24, 12, "f32", "tile"),     # twelve plane words
    (270, 127, 129, 40, 8, "bf16", "tile"),    # two words per plane, the second partial
    (256, 257, 1, 64, 8, "f32", "tile"),       # one key
    (96, 1030, 600, 32, 10, "f32", "tile"),    # past the 16 x 16 form's lengths
    (256, 100, 64, 12, 8, "f32", "other"),     # m not a multiple of 8
    (4, 1500, 1500, 32, 8, "f32", "other"),    # few heads: tables
])
def test_forward_tiles(bh, nq, nk, m, tau, dtype, kernel):
    (qc, kc), (q, k, v, dy) = inputs(bh, nq, nk, m, tau, dtype)
    names = ("dense_fwd_kernel", "tile_fwd_kernel", "table_kernel")
    y, ran = timed(names, lambda: Y.forward(qc, kc, v, m, tau, n_q=nq))
    assert ran["tile_fwd_kernel"] == (1 if kernel == "tile" else 0), ran
    if kernel == "tile":
        assert ran == {"dense_fwd_kernel": 1, "tile_fwd_kernel": 1, "table_kernel": 0}, ran
    assert torch.equal(y, Y.forward(qc, kc, v, m, tau, n_q=nq))
    sl = [0, bh - 1]
    ref = oracle.forward(codes_np(qc[sl]), codes_np(kc[sl]), host(v[sl]), m, tau)
    check_all(f"forward tiles bh{bh} {nq}x{nk} m{m} tau{tau} {dtype}", [("y", host(y[sl]), ref)], TOL[dtype])
