"""What one call leaves on a handle (values in scratch memory, modes, limits)
must not show in the next one."""
import sys

import numpy as np
import pytest

import oracle
from tests._util import normwise_rel, rand_irregular

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


@pytest.fixture()
def h(F):
    hh = F.Handle(0)
    yield hh
    hh.close()


def dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def cv_slabs(M, npdt, seed, nf=3, n=40):
    rng = np.random.default_rng(seed)
    off, t, y = rand_irregular(rng, len(M), n, 2, 12, npdt)
    folds = (np.arange(n) % nf).astype(np.int32)
    slabs = [oracle.bin_cov_pairs(M, off, t.astype(np.float64), y.astype(np.float64), folds, f, want_Q=True)
             for f in [-1] + list(range(nf))]
    return [np.stack([s[i] for s in slabs]).astype(npdt) for i in range(3)]


@pytest.mark.parametrize("M", [(9, 7), (12, 5), (5, 4, 3)])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_cv_scores_after_other_data(torch, F, h, M, dt):
    """Cross-validation fits the nodes s_1 <= t_1 and leaves the rest of its scratch as it was. Scratch that holds
    infinities (the rows of a binning of infinite observations) must give the scores of a fresh handle, bit for bit."""
    _say(f"cv after other data M={M} {dt}")
    npdt, tdt, code, prec = ((np.float64, torch.float64, F.FPCA_F64, F.FPCA_PREC_F64) if dt == "f64" else
                             (np.float32, torch.float32, F.FPCA_F32, F.FPCA_PREC_F32))
    C, G, Q = (dev(torch, a) for a in cv_slabs(M, npdt, 5))
    run = lambda hh: F.fpca_cv_batched(hh, code, [(F.Grid(M), C, G, Q)], 3, [0.4])[0]
    fresh = F.Handle(0)
    try:
        want = run(fresh)
    finally:
        fresh.close()
    assert np.all(np.isfinite(want))
    # every curve meets every node: its row of sums is infinite throughout
    rng = np.random.default_rng(8)
    n, Ni, P = 8000, 300, int(np.prod(M))
    off = np.arange(n + 1, dtype=np.int64) * Ni
    t = (rng.random((n * Ni, len(M))) * 0.999 + 0.0005).astype(npdt)
    y = torch.full((n * Ni,), float("inf"), dtype=tdt, device="cuda:0")
    folds = dev(torch, np.zeros(n, np.int32))
    out = [torch.empty(2, P, P, dtype=tdt, device="cuda:0") for _ in range(2)]
    F.fpca_bin(h, F.Grid(M), F.FPCA_BIN_COV, F.FPCA_IRREGULAR, code, prec, n, dev(torch, off), dev(torch, t), y, folds,
               1, *out)
    h.sync()
    got = run(h)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("M", [(12, 10), (33, 7), (4, 17, 3)])
def test_conv_mode_reaches_the_covariance(torch, F, h, M):
    """With FFT passes asked for, the default engine's covariance and cross-validation are those of the pass engine
    with FFT passes, bit for bit (grids that the queue kernel does not take, and one below the pass engine's limit)."""
    _say(f"conv mode M={M}")
    rng = np.random.default_rng(3)
    P = int(np.prod(M))
    C = rng.random((P, P)) + 0.01
    C = (C + C.T) * 0.5
    G = C * rng.standard_normal((P, P))
    G = (G + G.T) * 0.5
    hb = [0.4] * len(M)
    slabs = [dev(torch, a) for a in cv_slabs(M, np.float64, 6)]
    F.fpca_set_conv(h, F.FPCA_CONV_FFT)
    res = {}
    for engine in (F.FPCA_ENGINE_PASSES, F.FPCA_ENGINE_AUTO):
        F.fpca_set_engine(h, engine)
        gam = torch.empty(P, P, dtype=torch.float64, device="cuda:0")
        st = torch.empty(P, P, dtype=torch.int8, device="cuda:0")
        F.fpca_smooth_cov(h, F.Grid(M), F.FPCA_F64, dev(torch, C), 0.0, dev(torch, G), None, F.FPCA_K_EPANECHNIKOV, hb,
                          gam, st)
        h.sync()
        sc = F.fpca_cv_batched(h, F.FPCA_F64, [(F.Grid(M), *slabs)], 3, [0.4])[0] if M != (12, 10) else None
        res[engine] = (gam.cpu().numpy(), st.cpu().numpy(), sc)
    a, b = res[F.FPCA_ENGINE_PASSES], res[F.FPCA_ENGINE_AUTO]
    assert np.array_equal(a[0], b[0], equal_nan=True)
    assert np.array_equal(a[1], b[1])
    assert a[2] is None or np.array_equal(a[2], b[2])


def test_many_cv_jobs_under_a_scratch_limit(torch, F, h, monkeypatch):
    """600 jobs on a small grid: their scores' partial sums are sized by the grid, so that a limit with room for one
    job's moments takes them all, to the same scores."""
    _say("many cv jobs under a limit")
    M = (8, 8)
    C, G, Q = (dev(torch, a) for a in cv_slabs(M, np.float64, 7))
    hs = np.geomspace(0.2, 0.6, 200)
    run = lambda hh: F.fpca_cv_batched(hh, F.FPCA_F64, [(F.Grid(M), C, G, Q)], 3, hs)[0]
    full = run(h)
    # one job: 14 P^2 doubles of moments and P^2 of fits, 0.5 MB
    monkeypatch.setenv("FPCA_DEBUG_WS_LIMIT", str(3 << 19))
    lim = F.Handle(0)
    try:
        got = run(lim)
    finally:
        lim.close()
    assert np.array_equal(got, full)


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_cv_datasets_of_several_grids(torch, F, h, dt):
    """Default engine, datasets of uneven size and one with a mask in one call: the scores of the separate calls."""
    _say(f"cv several grids {dt}")
    npdt, code = (np.float64, F.FPCA_F64) if dt == "f64" else (np.float32, F.FPCA_F32)
    data = []
    for i, M in enumerate([(9, 7), (16, 5), (9, 7), (17, 20), (4, 4)]):
        mask = dev(torch, (np.arange(M[0] * M[1]) % 5 > 0).astype(np.uint8)) if i == 2 else None
        data.append((F.Grid(M, mask), *(dev(torch, a) for a in cv_slabs(M, npdt, 20 + i))))
    hs = [0.35, 0.5, 0.7]
    got = F.fpca_cv_batched(h, code, data, 3, hs)
    for i, one in enumerate(data):
        assert np.array_equal(got[i], F.fpca_cv_batched(h, code, [one], 3, hs)[0]), i


def test_optional_scratch_that_does_not_fit(torch, F, monkeypatch):
    """Scratch that a call can do without and cannot have (the allocation fails) costs the handle neither the block it
    holds nor the message of its last error, and the results are those of a handle that got it."""
    _say("optional scratch")
    rng = np.random.default_rng(9)
    M, n = (40, 40), 1024
    P = M[0] * M[1]
    off = np.arange(n + 1, dtype=np.int64) * 5
    t, y = rng.random((5 * n, 2)), rng.standard_normal(5 * n)
    D = lambda a: dev(torch, a)
    d_off, d_t, d_y, folds = D(off), D(t), D(y), D(np.zeros(n, np.int32))
    Gam = rng.standard_normal((200, 200))
    Gam, om = D(Gam @ Gam.T), D(np.full(200, 1.0 / 200))
    z = lambda *s: torch.empty(*s, dtype=torch.float64, device="cuda:0")
    two, out, ef = [z(2, P, P) for _ in range(2)], [z(P, P) for _ in range(2)], z(4, 200)
    # 26 MB of rows (29.5 with the arena's margin), 32.8 MB of sums of the j = l terms
    monkeypatch.setenv("FPCA_DEBUG_ALLOC_LIMIT", str(31 << 20))
    lim = F.Handle(0)
    monkeypatch.delenv("FPCA_DEBUG_ALLOC_LIMIT")
    free = F.Handle(0)
    try:
        args = (F.Grid(M), F.FPCA_BIN_COV, F.FPCA_IRREGULAR, F.FPCA_F64, F.FPCA_PREC_F64, n, d_off, d_t, d_y)
        F.fpca_bin(lim, *args, folds, 1, *two)  # takes the rows' block
        lim.sync()
        with pytest.raises(F.FpcaError):
            F.fpca_set_conv(lim, 7)
        last = F.load_library().fpca_last_error()
        held = torch.cuda.mem_get_info()[0]
        res = []
        for hh in (lim, free):
            F.fpca_bin(hh, *args, None, 0, *out)
            hh.sync()
            if hh is lim:
                assert torch.cuda.mem_get_info()[0] == held
                assert F.load_library().fpca_last_error() == last
            res.append([o.cpu().numpy() for o in out])
        for a, b in zip(*res):
            assert normwise_rel(a, b) < 1e-13
    finally:
        lim.close()
        free.close()
    # the decomposition: 170 KB that it cannot do without, 324 KB with the shares of a split
    ev = []
    for cap in ("", str(300 << 10)):
        monkeypatch.setenv("FPCA_DEBUG_ALLOC_LIMIT", cap) if cap else None
        hh = F.Handle(0)
        try:
            ev.append(F.fpca_eig_randomized(hh, F.FPCA_F64, F.FPCA_PREC_F64, F.Grid((200,)), Gam, om, 4, 8, 2, 3, ef)[0])
        finally:
            hh.close()
    np.testing.assert_allclose(ev[0], ev[1], rtol=1e-12)


def gram_case(torch, F, npdt, n, P, seed):
    y = np.random.default_rng(seed).standard_normal((n, P)).astype(npdt)
    ref = (y.astype(np.float64).T @ y.astype(np.float64)) / (P * (P - 1.0))
    np.fill_diagonal(ref, 0.0)
    code, prec = (F.FPCA_F64, F.FPCA_PREC_F64) if npdt == np.float64 else (F.FPCA_F32, F.FPCA_PREC_F32)
    args = (F.Grid((P,)), F.FPCA_BIN_COV, F.FPCA_COMMON_GRID, code, prec, n, None, None, dev(torch, y), None, 0, None)
    S = torch.full((P, P), float("nan"), dtype=torch.float64 if npdt == np.float64 else torch.float32, device="cuda:0")
    return args, S, ref


@pytest.mark.parametrize("npdt", [np.float64, np.float32])
def test_captured_gram_after_the_scratch_moved(torch, F, h, npdt):
    """A captured binning of complete curves holds no address of the handle's scratch: replays are right after larger
    calls have replaced it."""
    _say(f"captured gram {npdt.__name__}")
    args, S, ref = gram_case(torch, F, npdt, 600, 96, 1)
    big, S2, ref2 = gram_case(torch, F, npdt, 4000, 300, 2)
    tol = 1e-13 if npdt == np.float64 else 1e-5
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        F.fpca_bin(h, *args, S)  # the handle has a block when the capture starts
    s.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        F.fpca_bin(h, *args, S)
    for _ in range(3):
        F.fpca_bin(h, *big, S2)
        F.fpca_bin(h, *args, S)
        h.sync()
        eager = S.cpu().numpy()
        S.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert normwise_rel(S.cpu().numpy().astype(np.float64), ref) < tol
        assert normwise_rel(eager.astype(np.float64), ref) < tol
        assert normwise_rel(S2.cpu().numpy().astype(np.float64), ref2) < tol


@pytest.mark.parametrize("npdt", [np.float64, np.float32])
@pytest.mark.parametrize("nstreams", [2, 11])
def test_gram_on_streams_in_turn(torch, F, h, npdt, nstreams):
    """One handle, products of complete curves queued on its streams in turn with nothing waited for between them: two, and
    more than it keeps blocks for."""
    _say(f"gram on {nstreams} streams {npdt.__name__}")
    tol = 1e-13 if npdt == np.float64 else 1e-5
    cases = [gram_case(torch, F, npdt, 3000 + 40 * i, 200 + 30 * (i % 3), 10 + i) for i in range(12)]
    streams = [torch.cuda.Stream() for _ in range(nstreams)]
    torch.cuda.synchronize()
    for _ in range(3):
        for i, (args, S, _) in enumerate(cases):
            with torch.cuda.stream(streams[i % nstreams]):
                F.fpca_bin(h, *args, S)
    torch.cuda.synchronize()
    for args, S, ref in cases:
        assert normwise_rel(S.cpu().numpy().astype(np.float64), ref) < tol


@pytest.mark.parametrize("M,bar", [(676, 3.4e-8), (1024, 3.2e-8), (1600, 3.7e-8)])
def test_eig_fp32_sums_stay_short(torch, F, h, M, bar):
    """FP32 products of a range where the nodes are split into many shares: the eigenfunctions' error against 64 bits,
    over six covariances, is no larger than with a separate FP32 partial product for every 32 (1600 nodes: 96) nodes,
    whose measured error and a tenth more is the bar (sums twice as long exceed it)."""
    _say(f"eig fp32 sums P={M}")
    err = []
    for seed in range(6):
        rng = np.random.default_rng(100 + seed)
        V = np.linalg.qr(rng.standard_normal((M, 30)))[0]
        Gam = ((V * 0.8 ** np.arange(30)) @ V.T).astype(np.float32)
        Gam = (Gam + Gam.T) / 2
        om = np.full(M, 1.0 / M)
        ef = torch.empty(6, M, dtype=torch.float32, device="cuda:0")
        F.fpca_eig_randomized(h, F.FPCA_F32, F.FPCA_PREC_F32, F.Grid((M,)), dev(torch, Gam), dev(torch, om), 6, 10, 2,
                              seed, ef)
        _, ref, _ = oracle.eig_randomized(Gam.astype(np.float64), om, 6, 10, 2, seed)
        got = ef.cpu().numpy().astype(np.float64)
        ref = ref.T * np.sign(np.sum(ref.T * got, axis=1, keepdims=True))
        err.append(np.linalg.norm(got - ref) / np.linalg.norm(ref))
    err = float(np.sqrt(np.mean(np.square(err))))
    _say(f"error {err:.3e} bar {bar:.1e}")
    assert err <= bar


@pytest.mark.parametrize("M,R,n,limit", [((9, 13, 11), (2, 3, 2), 20, 0), ((6, 60, 60), (2, 1, 1), 9, 10 << 20),
                                         ((200, 90), (3, 3), 9, 13 << 20), ((30, 21), (4, 5), 20, 0)])
def test_operator_products_repeat(torch, F, h, monkeypatch, M, R, n, limit):
    """Products of an operator repeat bit for bit, also replayed from a graph between other work of the handle; half
    of the pairs formed at once, in shares of the nodes (a limit on one allocation), and all pairs (a limit that leaves
    no room for the other half's blocks) agree to rounding. 40 columns: a launch of 32 and one of 8."""
    _say(f"operator products M={M} limit={limit}")
    rng = np.random.default_rng(len(M) + n)
    P, r = int(np.prod(M)), 40
    Y, X = dev(torch, 1.0 + rng.standard_normal((n, P))), dev(torch, rng.standard_normal((P, r)))
    mu = Y.mean(0)
    hb = [(k + 0.45) / (m - 1) for k, m in zip(R, M)]
    res = []
    for cap in (limit, 1):
        if cap:
            monkeypatch.setenv("FPCA_DEBUG_ALLOC_LIMIT", str(cap))
        hh = F.Handle(0)
        monkeypatch.delenv("FPCA_DEBUG_ALLOC_LIMIT", raising=False)
        op = F.CovOp(hh, F.Grid(M), Y, mu, hb, F.FPCA_COVOP_RECOMPUTE)
        try:
            outs = [torch.full((P, r), float("nan"), dtype=torch.float64, device="cuda:0") for _ in range(5)]
            for o in outs:
                op.apply(X, o)
            torch.cuda.synchronize()
            for o in outs[1:]:
                assert torch.equal(o, outs[0])
            s = torch.cuda.Stream()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=s):
                op.apply(X, outs[1])
            other = F.CovOp(hh, F.Grid(M), Y, mu, hb, F.FPCA_COVOP_RECOMPUTE)
            for _ in range(3):
                outs[1].fill_(float("nan"))
                other.apply(X, outs[2])
                torch.cuda.synchronize()
                graph.replay()
                torch.cuda.synchronize()
                assert torch.equal(outs[1], outs[0])
            other.close()
            res.append(outs[0].cpu().numpy())
        finally:
            op.close()
            hh.close()
    assert normwise_rel(res[0], res[1]) < 1e-13


@pytest.mark.parametrize("M,R,n,limit", [((64, 30, 28), (6, 2, 2), 6, 12 << 20), ((12, 30, 28), (5, 2, 2), 9, 1 << 20),
                                         ((70, 70), (28, 28), 5, 8 << 20)])
def test_operator_memory(torch, F, monkeypatch, M, R, n, limit):
    """The tables of an operator are held where they fit and dispensed with where they do not (a limit on one
    allocation): for some s_0 at a time, or solved pair by pair, to the same products; a stored band keeps none."""
    _say(f"operator memory M={M} limit={limit}")
    rng = np.random.default_rng(sum(M))
    d, P, r = len(M), int(np.prod(M)), 20
    Y, X = dev(torch, 1.0 + rng.standard_normal((n, P))), dev(torch, rng.standard_normal((P, r)))
    mu = Y.mean(0)
    hb = [(k + 0.45) / (m - 1) for k, m in zip(R, M)]
    # curves, their smooths and the low-rank sums, padded to blocks of four, and a block of each of the handle's
    curves = 8 * P * ((d + 1) * 1.4 * (n + 1) + 2 * n + 2 * n + 4) + (4 << 20)
    tb = {2: 8, 3: 4}[d]
    band = 8.0 * P * 64 * np.prod([(2 * -(-2 * k // tb) + 1) * (-(-m // tb) * tb) / m for k, m in zip(R, M)])
    res = []
    for cap, mode in ((0, F.FPCA_COVOP_RECOMPUTE), (limit, F.FPCA_COVOP_RECOMPUTE), (0, F.FPCA_COVOP_STORE_BAND),
                      (limit, F.FPCA_COVOP_STORE_BAND)):
        if cap:
            monkeypatch.setenv("FPCA_DEBUG_ALLOC_LIMIT", str(cap))
        hh = F.Handle(0)
        monkeypatch.delenv("FPCA_DEBUG_ALLOC_LIMIT", raising=False)
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        op = F.CovOp(hh, F.Grid(M), Y, mu, hb, mode)
        try:
            held = before - torch.cuda.mem_get_info()[0]
            _say(f"mode {mode} cap {cap}: held {held >> 20} MB")
            if mode == F.FPCA_COVOP_STORE_BAND:
                assert held <= band + curves + (8 << 20)
            elif cap:
                assert held <= 3 * cap + curves + (8 << 20)
            out = torch.full((P, r), float("nan"), dtype=torch.float64, device="cuda:0")
            op.apply(X, out)
            torch.cuda.synchronize()
            res.append(out.cpu().numpy())
        finally:
            op.close()
            hh.close()
    for a in res[1:]:
        assert normwise_rel(a, res[0]) < 1e-12


@pytest.mark.parametrize("npdt", [np.float64, np.float32])
def test_gram_after_its_stream_is_gone(torch, F, h, npdt):
    """A handle goes on to another stream after the one of its last product has been destroyed."""
    _say(f"gram after its stream {npdt.__name__}")
    tol = 1e-13 if npdt == np.float64 else 1e-5
    args, S, ref = gram_case(torch, F, npdt, 900, 150, 4)
    ncu = torch.cuda.get_device_properties(0).multi_processor_count
    for _ in range(2):
        raw = F.fpca_stream_create_cu_range(0, 0, ncu)
        with torch.cuda.stream(torch.cuda.ExternalStream(raw)):
            F.fpca_bin(h, *args, S)
        torch.cuda.synchronize()
        F.fpca_stream_destroy(raw)
        S.fill_(float("nan"))
        F.fpca_bin(h, *args, S)
        h.sync()
        assert normwise_rel(S.cpu().numpy().astype(np.float64), ref) < tol


def test_operator_on_a_full_card(torch, F, h):
    """On a card with little memory left an operator does without a table that would take more than half of it, and
    its products are those of one that had room."""
    _say("operator on a full card")
    rng = np.random.default_rng(12)
    M, R, n, r = (70, 70), (28, 28), 5, 8  # a table of 602 MB, blocks of 220 MB
    P = M[0] * M[1]
    Y, X = dev(torch, 1.0 + rng.standard_normal((n, P))), dev(torch, rng.standard_normal((P, r)))
    hb = [(k + 0.45) / (m - 1) for k, m in zip(R, M)]
    res = []
    for keep in (None, 400 << 20):
        torch.cuda.empty_cache()
        free = torch.cuda.mem_get_info()[0]
        filler = torch.empty(free - keep, dtype=torch.uint8, device="cuda:0") if keep else None
        before = torch.cuda.mem_get_info()[0]
        op = F.CovOp(h, F.Grid(M), Y, Y.mean(0), hb, F.FPCA_COVOP_RECOMPUTE)
        try:
            left = torch.cuda.mem_get_info()[0]
            _say(f"free {before >> 20} MB before, {left >> 20} after")
            if keep:
                assert left > before * 0.45
            del filler
            torch.cuda.empty_cache()
            out = torch.full((P, r), float("nan"), dtype=torch.float64, device="cuda:0")
            op.apply(X, out)
            h.sync()
            res.append(out.cpu().numpy())
        finally:
            op.close()
    assert normwise_rel(res[1], res[0]) < 1e-12


def test_two_threads_with_two_grids(torch, F):
    """Two host threads, a handle and a stream each, smooth covariances on grids whose kernels take different amounts
    of LDS at the same time: every call succeeds, with the results of a thread by itself."""
    _say("two threads")
    import threading
    jobs, want = [], []
    for i, M in enumerate([(5, 40), (5, 37)]):
        rng = np.random.default_rng(30 + i)
        P = int(np.prod(M))
        C = rng.random((P, P)) + 0.1
        G = C * rng.standard_normal((P, P))
        jobs.append((M, dev(torch, C + C.T), dev(torch, G + G.T)))

    def smooth(hh, job, times):
        M, C, G = job
        P = int(np.prod(M))
        gam = torch.empty(P, P, dtype=torch.float64, device="cuda:0")
        for _ in range(times):
            F.fpca_smooth_cov(hh, F.Grid(M), F.FPCA_F64, C, 0.0, G, None, F.FPCA_K_EPANECHNIKOV, 0.3, gam, None)
        hh.sync()
        return gam

    hs = [F.Handle(0), F.Handle(0)]
    try:
        want = [smooth(hs[i], jobs[i], 1).clone() for i in range(2)]
        torch.cuda.synchronize()
        got, errors = [None, None], []

        def work(i):
            try:
                with torch.cuda.stream(torch.cuda.Stream()):
                    got[i] = smooth(hs[i], jobs[i], 400)
            except Exception as e:  # reported by the main thread
                errors.append(e)

        threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        torch.cuda.synchronize()
        assert not errors, errors
        for a, b in zip(got, want):
            assert torch.equal(a, b)
    finally:
        for hh in hs:
            hh.close()
