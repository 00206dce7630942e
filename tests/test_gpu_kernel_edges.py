"""Kernels at the sizes where their tiling can go wrong (edges of tiles,
remainders, the smallest and largest of a range), against the FP64 oracle.
Bars as in the modules that cover the same calls at ordinary sizes."""
import sys

import numpy as np
import pytest

import oracle
from oracle import mlp as ref_mlp
from tests._util import normwise_rel, rand_irregular, status_agreement

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def torch():
    import torch as T
    assert T.cuda.is_available(), "GPU tests need a GPU"
    return T


@pytest.fixture(scope="module")
def F(torch):
    import paper_1510_04439_amd as F
    F.load_library()
    return F


@pytest.fixture(scope="module")
def h(F):
    hh = F.Handle(0)
    yield hh
    hh.close()


def dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("B", [1, 15, 16, 17, 64, 65, 300])
def test_mlp_batches(torch, F, h, B):
    """16 samples per workgroup, 4 per MFMA step, 16 shares of the batch."""
    _say(f"mlp batch {B}")
    rng = np.random.default_rng(40 + B)
    theta = (rng.standard_normal(ref_mlp.NPARAM) * 0.1).astype(np.float32)
    feat = rng.standard_normal((B, 32)).astype(np.float32) * 2 - 1
    fmu = rng.standard_normal(32).astype(np.float32)
    fsd = (rng.random(32) + 0.5).astype(np.float32)
    target = rng.standard_normal(B).astype(np.float32)
    X = (feat.astype(np.float64) - fmu) / fsd
    out_ref, _ = ref_mlp.forward(theta.astype(np.float64), X)
    _, g_ref = ref_mlp.loss_and_grad(theta.astype(np.float64), X, target.astype(np.float64))
    T = lambda a: dev(torch, a)
    prm, ft, mu_t, sd_t, tg = T(theta), T(feat), T(fmu), T(fsd), T(target)
    z = lambda *s: torch.full(s, float("nan"), dtype=torch.float32, device="cuda:0")
    out, z1, z2, work, grad = z(B), z(B, 128), z(B, 128), z(B * 257), z(ref_mlp.NPARAM)
    F.fpca_bw_mlp_forward(h, B, ft, mu_t, sd_t, prm, out, z1, z2)
    F.fpca_bw_mlp_backward(h, B, ft, mu_t, sd_t, prm, out, tg, z1, z2, work, grad)
    h.sync()
    assert np.abs(out.cpu().numpy() - out_ref).max() <= 1e-5 * max(1.0, np.abs(out_ref).max())
    assert normwise_rel(grad.cpu().numpy(), g_ref) < 1e-4


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("M,R", [((259, 326), (13, 14)), ((326, 257), (15, 16)), ((304, 264), (17, 18)),
                                 ((5001,), (403,)), ((61, 47, 66), (3, 5, 6))])
def test_smooth_mean_strips(torch, F, h, dt, M, R):
    """Strips of eight outputs: lines that end inside a strip, windows that
    leave one to seven taps after the blocks of eight, a line that fills a
    workgroup's LDS. A NaN sum reaches the windows that hold its node, and no
    others."""
    _say(f"strips M={M} R={R} {dt}")
    npdt = np.float64 if dt == "f64" else np.float32
    tdt = torch.float64 if dt == "f64" else torch.float32
    rng = np.random.default_rng(60 + sum(M))
    P = int(np.prod(M))
    w = (rng.integers(0, 6, P) * (rng.random(P) < 0.7)).astype(npdt)
    g = (w * (1.0 + 0.3 * rng.standard_normal(P))).astype(npdt)
    hb = [(r + 0.4) / (m - 1) for r, m in zip(R, M)]
    bad = int(np.ravel_multi_index([m // 2 for m in M], M))
    gn = g.copy()
    gn[bad] = np.nan
    code = F.FPCA_F64 if dt == "f64" else F.FPCA_F32
    res = []
    for sums in (g, gn):
        mu = torch.empty(P, dtype=tdt, device="cuda:0")
        st = torch.empty(P, dtype=torch.int8, device="cuda:0")
        F.fpca_smooth_mean(h, F.Grid(M), code, dev(torch, w), dev(torch, sums), F.FPCA_K_EPANECHNIKOV, hb, mu, st)
        h.sync()
        res.append((mu.cpu().numpy().astype(np.float64), st.cpu().numpy()))
    edge = [np.unique(np.clip([0, 1, 7, 8, m // 2, m - 9, m - 8, m - 2, m - 1], 0, m - 1)) for m in M]
    nodes = np.ravel_multi_index([a.reshape(-1) for a in np.meshgrid(*edge, indexing="ij")], M)
    nodes = np.unique(np.concatenate([nodes, rng.integers(0, P, 200)]))
    want, st_ref = oracle.smooth(M, hb, w.astype(np.float64), g.astype(np.float64), nodes)
    assert np.array_equal(res[0][1][nodes], st_ref)
    ok = st_ref == oracle.ST_OK
    assert normwise_rel(res[0][0][nodes], want, ok) < (1e-10 if dt == "f64" else 1e-5)
    x = np.stack(np.unravel_index(np.arange(P), M), 1) - np.array(np.unravel_index(bad, M))
    inside = np.all(np.abs(x) <= np.array(R), axis=1)
    assert np.array_equal(np.isnan(res[1][0]), inside | np.isnan(res[0][0]))


@pytest.mark.parametrize("M,R,n,r", [((5, 9, 13), (2, 3, 2), 230, 40), ((7, 6, 21), (3, 2, 1), 3, 17),
                                     ((13, 16, 14), (6, 1, 6), 104, 5), ((30, 33), (13, 14), 105, 33),
                                     ((70, 12), (28, 3), 9, 16)])
@pytest.mark.parametrize("mode", [0, 1])
def test_covop_blocks(torch, F, h, M, R, n, r, mode):
    """Blocks of 4 x 4 nodes cut by the grid, more curves than one LDS chunk and
    odd counts, one to three launches of 32 columns, windows that leave no node
    away from the border, the widest windows of d = 2 and 3: r columns of the
    covariance, products of unit vectors."""
    _say(f"covop blocks M={M} R={R} n={n} r={r} mode={mode}")
    rng = np.random.default_rng(80 + n)
    P = int(np.prod(M))
    Y = 1.0 + rng.standard_normal((n, 3)) @ rng.standard_normal((3, P)) + 0.3 * rng.standard_normal((n, P))
    mu = Y.mean(0)
    hb = [(k + 0.45) / (m - 1) for k, m in zip(R, M)]
    _, _, C, G = oracle.bin_common_grid(Y)
    cols = np.sort(rng.choice(P, r, replace=False))
    E = np.zeros((P, r))
    E[cols, np.arange(r)] = 1.0
    op = F.CovOp(h, F.Grid(M), dev(torch, Y), dev(torch, mu), hb, mode)
    try:
        out = torch.empty(P, r, dtype=torch.float64, device="cuda:0")
        op.apply(dev(torch, E), out)
        h.sync()
        got = out.cpu().numpy()
    finally:
        op.close()
    p = np.arange(P)
    check = range(r) if len(M) == 2 else range(0, r, max(1, r // 5))
    for j in check:
        q = int(cols[j])
        rb, _ = oracle.smooth_cov_raw(M, hb, C, G, np.concatenate([p * P + q, q * P + p]))
        ref = 0.5 * (rb[:P] + rb[P:]) - mu * mu[q]
        assert normwise_rel(got[:, j], ref) < 1e-10, j


@pytest.mark.parametrize("M,hb,dt", [((16, 17), 0.13, "f32"), ((24, 5), (0.1, 0.6), "f64"), ((25, 11), 0.12, "f32"),
                                     ((33, 7), (0.07, 0.4), "f32"), ((2, 40), (1.5, 0.06), "f64"),
                                     ((3, 16, 2), (0.6, 0.2, 1.2), "f32"), ((5, 2, 17), (0.5, 1.1, 0.14), "f64"),
                                     ((6, 5, 4), 0.45, "f32")])
def test_staged_smoother_and_cv(torch, F, h, M, hb, dt):
    """Lines at and beside the lengths the staged smoother rounds to, windows from
    one grid step to whole lines: the smoothed covariance with statuses, its
    complete-grid form, and masked cross-validation scores."""
    _say(f"staged M={M} h={hb} {dt}")
    rng = np.random.default_rng(120 + sum(M))
    d, P, nf = len(M), int(np.prod(M)), 3
    npdt, tdt = (np.float64, torch.float64) if dt == "f64" else (np.float32, torch.float32)
    code = F.FPCA_F64 if dt == "f64" else F.FPCA_F32
    off, t, y = rand_irregular(rng, d, 40, 1, 30, npdt)
    folds = np.arange(40, dtype=np.int32) % nf
    slabs = [oracle.bin_cov_pairs(M, off, t.astype(np.float64), y.astype(np.float64), folds, f, want_Q=True)
             for f in [-1] + list(range(nf))]
    C, G, Q = (np.stack([s[i] for s in slabs]).astype(npdt) for i in range(3))
    mask = (rng.random(P) < 0.8).astype(np.uint8)
    D = lambda a: dev(torch, a)
    tol = 1e-10 if dt == "f64" else 1e-5
    # smoother
    gam = torch.empty(P, P, dtype=tdt, device="cuda:0")
    st = torch.empty(P, P, dtype=torch.int8, device="cuda:0")
    F.fpca_smooth_cov(h, F.Grid(M), code, D(C[0]), 0.0, D(G[0]), None, F.FPCA_K_EPANECHNIKOV, hb, gam, st)
    h.sync()
    b, st_ref = oracle.smooth_cov_raw(M, hb, C[0].astype(np.float64), G[0].astype(np.float64))
    g, s_got = gam.cpu().numpy().astype(np.float64), st.cpu().numpy().reshape(-1)
    _, _, _, mp = oracle.smooth(M + M, np.tile(np.broadcast_to(hb, (d,)), 2), C[0].astype(np.float64),
                                G[0].astype(np.float64), want_moments=True)
    assert status_agreement(s_got, st_ref, mp)[0] == 0
    ok = ((s_got == 0) & (st_ref == 0)).reshape(P, P)
    ref = b.reshape(P, P)
    both = ok & ok.T
    assert normwise_rel(g, 0.5 * (ref + ref.T), both) < tol
    # a complete grid: weights c0 off the diagonal
    c0 = 0.01
    F.fpca_smooth_cov(h, F.Grid(M), F.FPCA_F64, None, c0, D(G[0].astype(np.float64)), None, F.FPCA_K_EPANECHNIKOV, hb,
                      g64 := torch.empty(P, P, dtype=torch.float64, device="cuda:0"), st)
    h.sync()
    W = np.full((P, P), c0)
    np.fill_diagonal(W, 0.0)
    b, st_ref = oracle.smooth_cov_raw(M, hb, W, G[0].astype(np.float64))
    ref = b.reshape(P, P)
    both = (st_ref == 0).reshape(P, P)
    assert normwise_rel(g64.cpu().numpy(), 0.5 * (ref + ref.T), both & both.T) < 1e-10
    # cross-validation, more jobs than one launch takes
    hs = np.outer([1.0, 1.2, 1.45, 0.9], np.broadcast_to(hb, (d,)))
    got = F.fpca_cv_batched(h, code, [(F.Grid(M, D(mask)), D(C), D(G), D(Q))], nf, hs)[0]
    want = np.zeros_like(got)
    for i, hv in enumerate(hs):
        for f in range(nf):
            bb, _ = oracle.smooth_cov_raw(M, hv, C[0].astype(np.float64) - C[f + 1], G[0].astype(np.float64) - G[f + 1])
            Gh = oracle.assemble_cov(bb.reshape(P, P), np.zeros(P), mask)
            want[i, f] = oracle.cv_score(Q[f + 1].astype(np.float64), G[f + 1].astype(np.float64),
                                         C[f + 1].astype(np.float64), Gh)
    np.testing.assert_allclose(got, want, rtol=1e-9 if dt == "f64" else 1e-5)


@pytest.mark.parametrize("dtype,n,M", [("f32", 1, 3), ("f32", 33, 64), ("f32", 200, 65), ("f32", 1000, 130),
                                       ("f32", 129, 260), ("f32", 17, 5764), ("f32", 16, 5761), ("f32", 1003, 5764),
                                       ("f64", 1, 3),
                                       ("f64", 17, 64), ("f64", 200, 101),
                                       ("f64", 1000, 128), ("f64", 65, 258)])
def test_gram_tiles(torch, F, h, dtype, n, M):
    """64-column tiles, 16- or 32-row stages, shares of the rows, columns in groups of four or not, and the
    128-column tiles of large FP32 products. The bar is
    the rounding bound of an n-term sum, (n + 4) u |Y|^T |Y|, entry by entry; the product is exactly symmetric."""
    _say(f"gram {dtype} n={n} M={M}")
    rng = np.random.default_rng(n + M)
    npt, tt, code, prec = ((np.float32, torch.float32, F.FPCA_F32, F.FPCA_PREC_F32) if dtype == "f32" else
                           (np.float64, torch.float64, F.FPCA_F64, F.FPCA_PREC_F64))
    y = (rng.standard_normal((n, M)) * 2 + 1).astype(npt)
    w = 1.0 / (M * (M - 1))
    S = torch.full((M, M), float("nan"), dtype=tt, device="cuda:0")
    F.fpca_bin(h, F.Grid((M,)), F.FPCA_BIN_COV, F.FPCA_COMMON_GRID, code, prec, n, None, None, dev(torch, y), None, 0,
               None, S)
    got = S.cpu().numpy().astype(np.float64)
    y64 = y.astype(np.float64)
    ref, amp = w * (y64.T @ y64), w * (np.abs(y64).T @ np.abs(y64))
    np.fill_diagonal(ref, 0.0)
    assert np.array_equal(got, got.T)
    assert np.all(np.abs(got - ref) <= (n + 4) * np.finfo(npt).eps * amp)


@pytest.mark.parametrize("P,k,p,q", [(9, 3, 5, 2), (16, 4, 8, 0), (17, 4, 8, 2), (51, 3, 10, 2), (65, 20, 10, 2),
                                     (113, 4, 12, 1), (127, 20, 10, 2), (128, 5, 11, 2), (129, 5, 11, 2),
                                     (190, 20, 12, 1)])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_eig_small_grids(torch, F, h, P, k, p, q, dt):
    """Up to 128 nodes and 32 basis columns the iteration runs in one workgroup: 1 to 8 blocks of 16 rows, the
    nodes in 2 to 16 shares; past that the split products, the last chunk of 129 nodes one node wide. Bars of the
    decompositions at ordinary sizes."""
    _say(f"eig small P={P} k={k} p={p} q={q} {dt}")
    rng = np.random.default_rng(P + k)
    V = np.linalg.qr(rng.standard_normal((P, P)))[0]
    npdt, tdt, code, prec = ((np.float64, torch.float64, F.FPCA_F64, F.FPCA_PREC_F64) if dt == "f64" else
                             (np.float32, torch.float32, F.FPCA_F32, F.FPCA_PREC_F32))
    Gam = (V * 1.5 ** -np.arange(P)) @ V.T
    Gam = ((Gam + Gam.T) / 2).astype(npdt)
    om = oracle.quad_weights((P,), rule="trapezoid")
    ef = torch.empty(k, P, dtype=tdt, device="cuda:0")
    ev, fve = F.fpca_eig_randomized(h, code, prec, F.Grid((P,)), dev(torch, Gam), dev(torch, om), k, p, q, 11, ef)
    rev, rphi, rfve = oracle.eig_randomized(Gam.astype(np.float64), om, k, p, q, 11)
    tol = 1e-10 if dt == "f64" else 1e-5
    assert np.abs(ev - rev).max() <= tol * np.abs(rev).max()
    assert np.abs(fve - rfve).max() <= tol
    phi = ef.cpu().numpy().astype(np.float64).T
    for j in range(k):
        gap = min(abs(rev[j] - rev[j - 1]) if j else np.inf, abs(rev[j] - rev[j + 1]) if j + 1 < k else np.inf)
        scale = max(1.0, 0.1 * rev[0] / gap) if np.isfinite(gap) else 1.0
        err = min(np.abs(phi[:, j] - rphi[:, j]).max(), np.abs(phi[:, j] + rphi[:, j]).max())
        assert err <= 100 * tol * scale * np.abs(rphi[:, j]).max(), (j, err)


@pytest.mark.parametrize("M,dt,q,Ns", [((3,), "f32", False, [2]), ((40, 41), "f32", True, [0, 300, 1, 2, 256, 257]),
                                       ((57, 57), "f32", False, [257, 3, 0, 90, 40]),
                                       ((58, 57), "f32", False, [2, 300]), ((74, 74), "f32", True, [300, 1, 7]),
                                       ((10, 10, 11), "f32", False, [60, 2, 100]),
                                       ((11, 11, 10), "f32", False, [60, 2, 100]), ((101,), "f64", True, [50] * 9),
                                       ((53, 52), "f64", False, [120, 30]), ((64, 43), "f64", True, [80, 11])])
def test_bin_cov_rows(torch, F, h, M, dt, q, Ns):
    """Rows of curves and the j = l terms in LDS: grids on both sides of what LDS holds of either, curves of no,
    one, two and more than one workgroup's observations, last groups of four curves not full. Bars as for the
    binning at ordinary sizes."""
    _say(f"bin cov rows M={M} {dt} Q={q}")
    rng = np.random.default_rng(len(Ns) + M[0])
    npdt, tdt, code, prec = ((np.float64, torch.float64, F.FPCA_F64, F.FPCA_PREC_F64) if dt == "f64" else
                             (np.float32, torch.float32, F.FPCA_F32, F.FPCA_PREC_F32))
    off = np.concatenate([[0], np.cumsum(Ns)]).astype(np.int64)
    t = rng.random((int(off[-1]), len(M))).astype(npdt)
    y = rng.standard_normal(int(off[-1])).astype(npdt)
    P = int(np.prod(M))
    out = [torch.full((P, P), float("nan"), dtype=tdt, device="cuda:0") for _ in range(3 if q else 2)]
    F.fpca_bin(h, F.Grid(M), F.FPCA_BIN_COV, F.FPCA_IRREGULAR, code, prec, len(Ns), dev(torch, off), dev(torch, t),
               dev(torch, y), None, 0, out[0], out[1], out[2] if q else None)
    ref = oracle.bin_cov_pairs(M, off, t.astype(np.float64), y.astype(np.float64), want_Q=q)
    for a, r in zip(out, ref):
        assert normwise_rel(a.cpu().numpy().astype(np.float64), r) < (1e-12 if dt == "f64" else 1e-5)


@pytest.mark.parametrize("M,k", [((7,), 1), ((30,), 15), ((9, 8), 4), ((9, 8), 8), ((9, 8), 16), ((20, 11), 31),
                                 ((12, 10), 32), ((5, 4, 6), 9), ((6, 5, 4), 17), ((6, 6, 4), 32)])
@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("common", [False, True])
def test_pace_runs_and_column_tiles(torch, F, h, M, k, dt, common):
    """1, 2 or 3 tiles of 16 columns (k components and the residual); curves of no, one, a run's and one more
    than a run's or a round's observations, or rows of the common grid with missing values. Bars of the scores at
    ordinary sizes."""
    _say(f"pace tiles M={M} k={k} {dt} common={common}")
    rng = np.random.default_rng(k + len(M))
    npdt, tdt, code = ((np.float64, torch.float64, F.FPCA_F64) if dt == "f64" else
                       (np.float32, torch.float32, F.FPCA_F32))
    P, d = int(np.prod(M)), len(M)
    mu = rng.standard_normal(P).astype(npdt)
    ef = (rng.standard_normal((k, P)) / np.sqrt(P)).astype(npdt)
    lam = np.linspace(2.0, 0.05, k)
    if common:
        n, off, t, design = 5, None, None, F.FPCA_COMMON_GRID
        y = rng.standard_normal((n, P)).astype(npdt)
        y[rng.random((n, P)) < 0.2] = np.nan
        y[2] = np.nan
    else:
        Ns = np.array([0, 1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 300])
        n, design = len(Ns), F.FPCA_IRREGULAR
        off = np.concatenate([[0], np.cumsum(Ns)]).astype(np.int64)
        t = rng.random((int(off[-1]), d)).astype(npdt)
        t[40, 0] = -0.5  # outside the domain: left out
        y = rng.standard_normal(int(off[-1])).astype(npdt)
    out = torch.full((n, k), float("nan"), dtype=tdt, device="cuda:0")
    D = lambda a: None if a is None else dev(torch, a)
    F.fpca_pace_scores(h, F.Grid(M), design, code, n, D(off), D(t), D(y), D(mu), D(ef), k, lam, 0.05, out)
    ref = oracle.pace_scores(M, off, None if t is None else t.astype(np.float64), y.astype(np.float64),
                             mu.astype(np.float64), ef.T.astype(np.float64), lam, 0.05)
    got = out.cpu().numpy().astype(np.float64)
    assert np.abs(got - ref).max() <= (1e-10 if dt == "f64" else 1e-5) * np.abs(ref).max()


def test_cv_batches_under_a_scratch_limit(torch, F, h, monkeypatch):
    """A scratch limit with room for some jobs of a staged batch takes fewer at a time, to the same scores."""
    _say("cv under a limit")
    rng = np.random.default_rng(5)
    M, P, nf = (8, 9), 72, 3
    off, t, y = rand_irregular(rng, 2, 40, 2, 12, np.float64)
    folds = (np.arange(40) % nf).astype(np.int32)
    slabs = [oracle.bin_cov_pairs(M, off, t, y, folds, f, want_Q=True) for f in [-1] + list(range(nf))]
    C, G, Q = (dev(torch, np.stack([s[i] for s in slabs])) for i in range(3))
    run = lambda hh: F.fpca_cv_batched(hh, F.FPCA_F64, [(F.Grid(M), C, G, Q)], nf, [0.3, 0.5])[0]
    full = run(h)
    # a job takes 14 P^2 doubles of moments and P^2 of fits, about 0.63 MB, the six jobs' partial sums less
    monkeypatch.setenv("FPCA_DEBUG_WS_LIMIT", str(2 << 20))
    lim = F.Handle(0)
    try:
        got = run(lim)
    finally:
        lim.close()
    np.testing.assert_allclose(got, full, rtol=1e-12)


def test_paths_without_scratch(torch, F, h, monkeypatch):
    """A handle whose scratch limit leaves no room for split sums, for the mirrored half of the operator's band and
    for the sums of the j = l terms takes the ways without them, to the same results."""
    _say("no scratch")
    rng = np.random.default_rng(3)
    M, n, r = (9, 8, 7), 11, 17
    P = int(np.prod(M))
    Y, X = rng.standard_normal((n, P)), rng.standard_normal((P, r))
    Yc = rng.standard_normal((300, 65))
    Ns, M2 = [40, 7, 12], (50, 52)
    off = np.concatenate([[0], np.cumsum(Ns)]).astype(np.int64)
    t, y = rng.random((int(off[-1]), 2)).astype(np.float32), rng.standard_normal(int(off[-1])).astype(np.float32)

    def run(hh):
        out = []
        op = F.CovOp(hh, F.Grid(M), dev(torch, Y), dev(torch, Y.mean(0)), [0.3, 0.3, 0.4], F.FPCA_COVOP_RECOMPUTE)
        o = torch.empty(P, r, dtype=torch.float64, device="cuda:0")
        op.apply(dev(torch, X), o)
        out.append(o.cpu().numpy())
        op.close()
        for tt, code, prec in ((torch.float32, F.FPCA_F32, F.FPCA_PREC_F32), (torch.float64, F.FPCA_F64, F.FPCA_PREC_F64)):
            S = torch.empty(65, 65, dtype=tt, device="cuda:0")
            F.fpca_bin(hh, F.Grid((65,)), F.FPCA_BIN_COV, F.FPCA_COMMON_GRID, code, prec, 300, None, None,
                       dev(torch, Yc).to(tt), None, 0, None, S)
            out.append(S.cpu().numpy().astype(np.float64))
        C, G = (torch.empty(2600, 2600, dtype=torch.float32, device="cuda:0") for _ in range(2))
        F.fpca_bin(hh, F.Grid(M2), F.FPCA_BIN_COV, F.FPCA_IRREGULAR, F.FPCA_F32, F.FPCA_PREC_F32, len(Ns),
                   dev(torch, off), dev(torch, t), dev(torch, y), None, 0, C, G)
        out += [C.cpu().numpy().astype(np.float64), G.cpu().numpy().astype(np.float64)]
        return out

    full = run(h)
    # rows of the three curves (2 x 31 KB) fit, their j = l sums (104 KB) and everything larger do not
    monkeypatch.setenv("FPCA_DEBUG_WS_LIMIT", str(66 * 1024))
    lim = F.Handle(0)
    try:
        small = run(lim)
    finally:
        lim.close()
    for a, b, tol in zip(full, small, (1e-12, 1e-5, 1e-12, 1e-5, 1e-5)):
        assert normwise_rel(b, a) < tol


@pytest.mark.parametrize("P", [5636, 6400])
def test_gram_both_sides_of_the_large_tiles(torch, F, h, P):
    """FP32 products of more than a thousand 128-column tiles: in whole rounds of the CUs (6400) and one tile past
    (5636, which 64-column tiles take). Entry by entry within the rounding bound of a sum of 1000 terms."""
    _say(f"gram large P={P}")
    n = 1000
    y = np.random.default_rng(P).standard_normal((n, P)).astype(np.float32)
    S = torch.full((P, P), float("nan"), dtype=torch.float32, device="cuda:0")
    F.fpca_bin(h, F.Grid((P,)), F.FPCA_BIN_COV, F.FPCA_COMMON_GRID, F.FPCA_F32, F.FPCA_PREC_F32, n, None, None,
               dev(torch, y), None, 0, None, S)
    h.sync()
    assert torch.equal(S, S.T)
    y64 = dev(torch, y).double()
    w = 1.0 / (P * (P - 1.0))
    ref, amp = w * (y64.T.contiguous() @ y64), w * (y64.abs().T.contiguous() @ y64.abs())
    ref.fill_diagonal_(0.0)
    assert bool(torch.all((S.double() - ref).abs() <= (n + 4) * np.finfo(np.float32).eps * amp))


@pytest.mark.parametrize("P,k,p", [(545, 5, 11), (1295, 20, 12), (2045, 36, 12), (1028, 50, 14)])
@pytest.mark.parametrize("prec", ["f32", "bf16x3"])
def test_eig_fp64_partials_of_fp32(torch, F, h, P, k, p, prec):
    """FP32 products whose partial sums are FP64 (shares of the nodes longer than the FP32 sums): node counts that are
    no multiple of four, of a tile or of a share, one to four blocks of 16 basis columns. Bars of the products at
    ordinary sizes: 1e-5 for FP32, 1e-4 for BF16x3."""
    _say(f"eig fp64 partials P={P} k={k} {prec}")
    rng = np.random.default_rng(P)
    V = np.linalg.qr(rng.standard_normal((P, P)))[0]
    Gam = ((V * 0.9 ** np.arange(P)) @ V.T).astype(np.float32)
    Gam = (Gam + Gam.T) / 2
    om = np.full(P, 1.0 / P)
    ef = torch.empty(k, P, dtype=torch.float32, device="cuda:0")
    ev, fve = F.fpca_eig_randomized(h, F.FPCA_F32, F.FPCA_PREC_F32 if prec == "f32" else F.FPCA_PREC_BF16X3,
                                    F.Grid((P,)), dev(torch, Gam), dev(torch, om), k, p, 2, 5, ef)
    rev, rphi, rfve = oracle.eig_randomized(Gam.astype(np.float64), om, k, p, 2, 5)
    tol = 1e-5 if prec == "f32" else 1e-4
    assert np.abs(ev - rev).max() <= tol * np.abs(rev).max()
    assert np.abs(fve - rfve).max() <= tol
    phi = ef.cpu().numpy().astype(np.float64).T
    for j in range(k):
        gap = min(abs(rev[j] - rev[j - 1]) if j else np.inf, abs(rev[j] - rev[j + 1]) if j + 1 < k else np.inf)
        scale = max(1.0, 0.1 * rev[0] / gap) if np.isfinite(gap) else 1.0
        err = min(np.abs(phi[:, j] - rphi[:, j]).max(), np.abs(phi[:, j] + rphi[:, j]).max())
        assert err <= 100 * tol * scale * np.abs(rphi[:, j]).max(), (j, err)
