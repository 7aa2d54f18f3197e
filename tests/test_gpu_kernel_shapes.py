"""GPU parity at the sizes where a kernel changes its launch shape or runs a
remainder: edges of tiles, row and particle counts on both sides of a rule.

Tolerances are stated per test and follow from the arithmetic: what a shape
cannot change is compared bit for bit, FP64 sums in another order within their
rounding, FP32 values against the FP64 oracle within the FP32 class (1e-5).
"""
import numpy as np
import pytest

import synthetic

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ppl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2010_08454_amd as p
    return p


# ------------------------------------------------- BLR on the matrix cores --
def _blr(ppl, X, y, n, seed):
    import torch
    d = X.shape[1]
    data = ppl.make_data(torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda(), dim=d)
    lw = torch.empty(n, dtype=torch.float64, device="cuda")
    lat = torch.empty((d, n), dtype=torch.float32, device="cuda")
    scal = torch.empty(8, dtype=torch.float64, device="cuda")
    ppl.ppl_importance(ppl.PPL_MODEL_BLR, data, n, seed, log_weights=lw, latents=lat, scalars=scal)
    return lw.cpu().numpy(), lat.cpu().numpy(), scal.cpu().numpy()


@pytest.mark.parametrize("D", [1, 31, 32, 33, 63, 64, 95, 100, 511, 512, 1023, 1024, 1087])
@pytest.mark.parametrize("dim", [4, 8, 12, 16])
def test_blr_shapes(ppl, orc, D, dim):
    """Row counts around the 64-row tiles, the 32-row blocks and the split
    rules; particle counts on both sides of each rule.  Residuals and their
    32-row sums do not depend on the shape; only the FP64 sum over the blocks
    (all of one sign) may be taken in another order, so each particle's
    log-weight agrees between shapes within (D / 32 + 16) 2^-52 of its
    likelihood sum (bounded by |lw| + D |log(2 pi var)| / 2)."""
    X, y, _ = synthetic.blr_data(D=D, d=dim, seed=70 + D)
    seed, big = 11, 524_289
    ref_lw, ref_lat, _ = _blr(ppl, X, y, big, seed)
    idx = np.array([0, 1, 63, 64, 255, 256, 8191, 8192, 131_071, 524_287, 524_288])
    rlw, _ = orc.particle_logweights(orc.MODEL_BLR, X, y, idx, seed, dim=dim)
    assert np.max(np.abs(ref_lw[idx] - rlw) / np.maximum(1.0, np.abs(rlw))) < 1e-5
    eps = (D / 32 + 16) * 2.0 ** -52
    for n in (1, 65, 8192, 8193, 32_768, 32_769, 131_072, 131_073):
        lw, lat, scal = _blr(ppl, X, y, n, seed)
        np.testing.assert_array_equal(lat, ref_lat[:, :n])
        assert np.all(np.abs(lw - ref_lw[:n]) <= eps * (np.abs(ref_lw[:n]) + D)), (n, D, dim)
        m = lw.max()
        assert abs(scal[0] - (m + np.log(np.exp(lw - m).sum()) - np.log(n))) <= 1e-10 * max(1.0, abs(scal[0]))


@pytest.mark.parametrize("n", [100, 20_000, 100_000, 200_000, 600_000])
@pytest.mark.parametrize("row", [0, 31, 700, 1050])
def test_blr_nonfinite_rows(ppl, n, row):
    """An infinite entry gives every particle zero weight and a NaN one makes
    every log-weight NaN, whichever part of the data loop holds the row."""
    X, y, _ = synthetic.blr_data(D=1060, d=16, seed=5)
    for value, status in ((np.inf, ppl.PPL_E_ZERO_WEIGHT), (np.nan, ppl.PPL_E_NONFINITE)):
        Xb = X.copy()
        Xb[row, 7] = value
        lw, _, scal = _blr(ppl, Xb, y, n, 3)
        assert scal[3] == status
        assert np.all(np.isneginf(lw)) if value == np.inf else np.all(np.isnan(lw))


@pytest.mark.parametrize("kind", ["ordinary", "subnormal", "huge", "infinite", "nan"])
@pytest.mark.parametrize("dim", [4, 8, 12, 16])
def test_blr_matrix_rows_equal_the_scalar_chain(ppl, dim, kind):
    """31 rows among rows of zeros (which add a square of zero): in either half of a
    64-row tile they run on the matrix cores, after the last 32 rows a lane forms the
    chain fma(-x_k, w_k, r) itself.  Every log-weight has the same bits wherever the
    rows lie, at each launch shape.  Subnormal entries meet latents of size 1e20 and a
    noise of 1e-20, which make them visible."""
    import torch
    D = 16 * 64 + 63
    g = np.random.default_rng(dim)
    rows = g.standard_normal((31, dim)).astype(np.float32)
    target = g.standard_normal(31).astype(np.float32)
    hyper = [1.0, 0.5]
    if kind == "subnormal":
        rows = (rows * np.float32(1e-20)) * np.float32(1e-20)
        assert np.all(np.abs(rows) < np.finfo(np.float32).tiny)
        target[:] = 0.0
        hyper = [1e20, 1e-20]
    elif kind == "huge":
        rows[::3] *= np.float32(1e18)
        rows[1::3] *= np.float32(1e-18)
    elif kind in ("infinite", "nan"):
        rows[5, dim - 2] = np.inf if kind == "infinite" else np.nan
    for n in (100, 20_000, 100_000, 400_000, 600_000):
        ref = None
        for at in (16 * 64 + 32, 0, 32, 15 * 64, 15 * 64 + 32, 16 * 64):     # the scalar chain, then the matrix cores
            X, y = np.zeros((D, dim), np.float32), np.zeros(D, np.float32)
            X[at:at + 31], y[at:at + 31] = rows, target
            data = ppl.make_data(torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda(), dim=dim, hyper=hyper)
            lw = torch.empty(n, dtype=torch.float64, device="cuda")
            ppl.ppl_importance(ppl.PPL_MODEL_BLR, data, n, 7, log_weights=lw)
            lw = lw.cpu().numpy()
            if ref is None:
                ref = lw
                if kind in ("ordinary", "subnormal"):
                    assert np.all(np.isfinite(lw))
                if kind in ("ordinary", "subnormal", "huge"):      # (a few huge squares exceed FP32)
                    assert np.unique(lw).size > 0.9 * n
            if kind == "nan":
                assert np.all(np.isnan(lw)) and np.all(np.isnan(ref))
            else:
                np.testing.assert_array_equal(lw.view(np.int64), ref.view(np.int64))


# ------------------------------------------------------ FP64 Box-Muller --
@pytest.mark.parametrize("seed", [1, 2 ** 63 + 5])
def test_poly_draws_64bit(ppl, seed):
    """Coefficient draws against numpy's extended precision.  In units of 2^-52
    relative: half of the logarithm's error 0.5, the root's rounding 0.5, the
    trigonometric value 1, the products with it and with the prior sd 0.5 each."""
    import torch
    n = 200_003
    data = ppl.make_data(torch.zeros(1, dtype=torch.float64, device="cuda"),
                         torch.zeros(1, dtype=torch.float64, device="cuda"))
    lat = torch.empty((6, n), dtype=torch.float64, device="cuda")
    ppl.ppl_importance(ppl.PPL_MODEL_POLY, data, n, seed, latents=lat)
    lat = lat.cpu().numpy()
    pi = np.longdouble("3.14159265358979323846264338327950288")
    for b in (1, 2, 3):
        w = ppl.ppl_philox(seed, b, 0, 0, n).cpu().numpy().view(np.uint32).astype(np.uint64)
        u = [(((w[:, 2 * h + 1] << np.uint64(32)) | w[:, 2 * h]) >> np.uint64(12)).astype(np.float64) + 0.5 for h in (0, 1)]
        u = [np.longdouble(v) * np.longdouble(2.0) ** -52 for v in u]
        r = np.sqrt(-2 * np.log(u[0]))
        q = np.rint(4 * u[1])
        t = pi * (2 * u[1] - q / 2)                    # exact reduction to a quarter turn
        q = q.astype(int) % 4
        c, s = np.cos(t), np.sin(t)
        cs = np.choose(q, [c, -s, -c, s]), np.choose(q, [s, c, -s, -c])
        for h in (0, 1):
            j = 2 * (b - 1) + h
            if j < 5:
                ref = 10 * r * cs[h]
                assert np.max(np.abs(lat[1 + j] - ref) / np.abs(ref)) <= 3 * 2.0 ** -52


# ---------------------------------------------- POLY, lanes per particle --
@pytest.mark.parametrize("D", [0, 1, 3, 4, 31, 33, 511, 512, 513, 1030])
@pytest.mark.parametrize("n_lo,n_hi", [(2, 5), (1, 3)])
def test_poly_shapes(ppl, orc, D, n_lo, n_hi):
    """Points around the quad's stride and the LDS chunk, particle counts on
    both sides of the launch rule (a quad, one lane, a quarter lane per
    particle), degree 1 in and out of the range.  The likelihood sums take
    another order per shape: D terms of one sign, within (D + 4) 2^-52."""
    import torch
    x, y = synthetic.poly_data(D=max(D, 1), seed=40 + D)
    x, y = x[:D], y[:D]
    dx, dy = (torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in (x, y))
    data = ppl.make_data(dx if D else None, dy if D else None, n_data=D, hyper=[10.0, n_lo, n_hi], dtype=ppl.PPL_F64) \
        if D else ppl.PplData(x=None, y=None, n_data=0, dim=0, dtype=ppl.PPL_F64, n_hyper=0)
    if not D:
        n_lo, n_hi = 2, 5
    seed, out = 9, {}
    for n in (262_145, 262_143, 32_769, 32_768, 65, 64, 1):
        lw = torch.empty(n, dtype=torch.float64, device="cuda")
        lat = torch.empty((6, n), dtype=torch.float64, device="cuda")
        summ = torch.empty(29, dtype=torch.float64, device="cuda")
        scal = torch.empty(8, dtype=torch.float64, device="cuda")
        ppl.ppl_importance(ppl.PPL_MODEL_POLY, data, n, seed, log_weights=lw, latents=lat, summaries=summ, scalars=scal)
        lw, lat, summ, scal = (t.cpu().numpy() for t in (lw, lat, summ, scal))
        if not out:
            out = dict(lw=lw, lat=lat)
            if D:
                ref = orc.importance(orc.MODEL_POLY, x, y, 300, seed, want_lw=True, hyper=[10.0, n_lo, n_hi])
                assert np.max(np.abs(lw[:300] - ref["lw"]) / np.maximum(1.0, np.abs(ref["lw"]))) < 1e-12
        np.testing.assert_array_equal(lat, out["lat"][:, :n])
        assert np.all(np.abs(lw - out["lw"][:n]) <= (D + 4) * 2.0 ** -52 * np.abs(out["lw"][:n]))
        # summaries and normaliser from the returned weights: sums of n terms
        w = np.exp(lw - lw.max())
        deg, c = lat[0].astype(int), lat[1:] * (np.arange(5)[:, None] < lat[0][None])
        tol = 1e-10
        assert abs(scal[0] - (lw.max() + np.log(w.sum()) - np.log(n))) <= tol * max(1.0, abs(scal[0]))
        for s in range(4):
            sel = w * (deg == s + 2)
            assert abs(summ[s] - sel.sum() / w.sum()) <= tol
            want = (sel * c).sum(1) / sel.sum() if sel.sum() > 0 else np.zeros(5)
            assert np.all(np.abs(summ[4 + 5 * s:9 + 5 * s] - want) <= tol * 100)
        assert np.all(np.abs(summ[24:] - (w * c).sum(1) / w.sum()) <= tol * 100)


# ----------------------------------------------- mixture-proposal kernels --
def _poly_q(seed=3):
    """A decoded polynomial proposal with spread means and scales of both sizes."""
    g = np.random.default_rng(seed)
    ls = lambda v: v - np.log(np.exp(v).sum())
    return np.concatenate([ls(g.standard_normal(4)), ls(g.standard_normal(8)), g.standard_normal(160),
                           g.uniform(-2.0, 1.0, 160)])


@pytest.mark.parametrize("D", [1, 7, 8, 63, 64, 511, 512, 513, 600])
def test_poly_mix_shapes(ppl, orc, D):
    """Points around the group's stride and the LDS chunk, particle counts on
    both sides of the rule for eight lanes per particle.  The likelihood is a sum
    of D terms of one sign and the proposal density one of eight, in another
    order: the log-weights agree within (D + 32) 2^-52 of the terms' size."""
    import torch
    from oracle import proposal
    x, y = synthetic.poly_data(D=D, seed=90 + D)
    data = ppl.make_data(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda())
    q = _poly_q()
    dq, seed, ref = torch.from_numpy(q).cuda(), 21, None
    for n in (16_385, 16_384, 4096, 33, 32, 1):
        lw = torch.empty(n, dtype=torch.float64, device="cuda")
        lat = torch.empty((6, n), dtype=torch.float64, device="cuda")
        summ = torch.empty(29, dtype=torch.float64, device="cuda")
        ppl.ppl_importance(ppl.PPL_MODEL_POLY, data, n, seed, q=dq, q_kind=ppl.PPL_Q_POLY_MIX, log_weights=lw,
                           latents=lat, summaries=summ)
        lw, lat, summ = (t.cpu().numpy() for t in (lw, lat, summ))
        if ref is None:
            ref = lw, lat
            rlw = proposal.propose_poly(seed, q, x, y, np.arange(200))[0]
            assert np.max(np.abs(lw[:200] - rlw) / np.maximum(1.0, np.abs(rlw))) < 1e-10
        np.testing.assert_array_equal(lat, ref[1][:, :n])
        assert np.all(np.abs(lw - ref[0][:n]) <= (D + 32) * 2.0 ** -52 * (np.abs(ref[0][:n]) + 100.0))
        w = np.exp(lw - lw.max())
        c = lat[1:]
        assert np.all(np.abs(summ[24:] - (w * c).sum(1) / w.sum()) <= 1e-9 * np.maximum(1.0, np.abs(summ[24:])))
        for s in range(4):
            assert abs(summ[s] - w[lat[0] == s + 2].sum() / w.sum()) <= 1e-10


@pytest.mark.parametrize("K", range(1, 9))
def test_gmm_proposal_components(ppl, orc, K):
    """Every component count's kernel against the oracle (FP32 likelihood: the
    1e-5 class), a data count with and without a remainder of the 16-point blocks."""
    import torch
    from oracle import proposal
    g = np.random.default_rng(K)
    d = 2 * K - 1
    mix = g.standard_normal(8)
    q = np.concatenate([mix - np.log(np.exp(mix).sum()), g.standard_normal(8 * d), g.uniform(-1.5, 0.5, 8 * d)])
    for D in (16, 37):
        y = synthetic.gmm_learn_data(K=K, D=D, seed=60 + K)
        data = ppl.make_data(None, torch.from_numpy(y).cuda(), dim=K, dtype=ppl.PPL_F32)
        n = 700
        lw = torch.empty(n, dtype=torch.float64, device="cuda")
        lat = torch.empty((2 * K, n), dtype=torch.float64, device="cuda")
        ppl.ppl_importance(ppl.PPL_MODEL_GMM, data, n, 5, q=torch.from_numpy(q).cuda(), q_kind=ppl.PPL_Q_GMM_MIX,
                           log_weights=lw, latents=lat)
        ref = proposal.propose_gmm(5, q, K, y, np.arange(n))[0]
        assert np.max(np.abs(lw.cpu().numpy() - ref) / np.maximum(1.0, np.abs(ref))) < 1e-5
        prior = torch.empty(n, dtype=torch.float64, device="cuda")
        ppl.ppl_importance(ppl.PPL_MODEL_GMM, data, n, 5, log_weights=prior)
        ref = proposal.gmm_prior_lw(5, K, y, np.arange(n))
        ref = ref[0] if isinstance(ref, tuple) else ref
        assert np.max(np.abs(prior.cpu().numpy() - ref) / np.maximum(1.0, np.abs(ref))) < 1e-5


# ------------------------------------------------------------ enumeration --
@pytest.mark.parametrize("K,T", [(2, 1), (2, 13), (3, 8), (4, 7), (5, 6), (6, 6), (7, 5), (8, 5)])
@pytest.mark.parametrize("gap", [0.0, 1e-14, 1e-10, 1e-3])
@pytest.mark.parametrize("far", [0.0, 1e4])
def test_enumerate_near_ties(ppl, orc, K, T, gap, far):
    """Two states whose means differ by `gap` make every path tie, or nearly,
    with the paths that swap them, across the prefixes too: the most probable
    path and its log joint are the oracle's whichever way the search goes
    (their tolerance: T additions of terms of size |lw|).  `far` puts one
    observation far out, so that the log-weights are large."""
    import torch
    pi0, A, mu, sigma, y, _ = synthetic.hmm_instance(K, T, seed=77)
    mu = mu.copy()
    mu[1] = mu[0] + gap
    A = A.copy()
    A[1] = A[0]
    A[:, 1] = A[:, 0]
    A /= A.sum(1, keepdims=True)
    pi0 = pi0.copy()
    pi0[1] = pi0[0]
    pi0 /= pi0.sum()
    y = y.copy()
    y[T // 2] += far
    o = orc.enumerate_hmm(y, orc.hmm_hyper(pi0, A, mu, sigma))
    data = ppl.hmm_data(torch.from_numpy(y).cuda(), pi0, A, mu, sigma)
    scal = torch.empty(4, dtype=torch.float64, device="cuda")
    marg = torch.empty((T, K), dtype=torch.float64, device="cuda")
    mp = torch.empty(T, dtype=torch.int32, device="cuda")
    ppl.ppl_enumerate(ppl.PPL_MODEL_HMM, data, scalars=scal, marginals=marg, map_path=mp)
    scal, marg, mp = scal.cpu().numpy(), marg.cpu().numpy(), mp.cpu().numpy()
    tol = (T + 2) * 2.0 ** -51 * max(1.0, abs(o["map_lw"]))
    assert scal[3] == 0 and abs(scal[2] - o["map_lw"]) <= tol and abs(scal[0] - o["log_z"]) <= tol + 2e-9

    def lw(z):
        r = (y - mu[z]) / sigma
        return (np.log(pi0[z[0]]) + np.log(A[z[:-1], z[1:]]).sum()
                + (-0.5 * np.log(2 * np.pi) - np.log(sigma) - 0.5 * r * r).sum())
    assert abs(lw(mp) - o["map_lw"]) <= 2 * tol
    if gap == 0.0:
        assert 1 not in mp                        # the lowest index among equals
    if far == 0.0:
        assert np.max(np.abs(marg - o["marginals"])) <= 2e-9


# ------------------------------------------------------ Metropolis-Hastings --
@pytest.mark.parametrize("D", [0, 1, 3, 5, 16, 20, 31, 32, 63, 64, 100, 2048, 2049])
@pytest.mark.parametrize("n_lo,n_hi", [(2, 5), (1, 4)])
def test_mcmc_shapes(ppl, D, n_lo, n_hi):
    """Chains on both sides of the rule for four lanes per chain, point counts
    around its stride and the scalar batches.  A chain depends only on its index:
    the same trace and state whichever kernel runs it (a likelihood sum in
    another order, D terms of one sign, moves log alpha by at most D 2^-52 |ll|;
    no decision here lies that close)."""
    import torch
    x, y = synthetic.poly_data(D=max(D, 1), seed=300 + D)
    dx, dy = torch.from_numpy(x[:D].copy()).cuda(), torch.from_numpy(y[:D].copy()).cuda()
    hyper = [10.0, n_lo, n_hi]
    data = ppl.make_data(dx, dy, n_data=D, hyper=hyper, dtype=ppl.PPL_F64)
    if D == 0:
        data.x = data.y = None
    T, burn, seed, ref = 20, 5, 13, None
    for C in (32_769, 32_768, 16_385, 16_384, 65, 64, 1):
        state = torch.empty((6, C), dtype=torch.float64, device="cuda")
        accepts = torch.empty(C, dtype=torch.int64, device="cuda")
        trace = torch.empty((T, C), dtype=torch.int8, device="cuda")
        la = torch.empty((T, C), dtype=torch.float64, device="cuda")
        summ = torch.empty(29, dtype=torch.float64, device="cuda")
        scal = torch.empty(4, dtype=torch.float64, device="cuda")
        ppl.ppl_mcmc(ppl.PPL_MODEL_POLY, data, C, T, seed, burn_in=burn, state=state, accepts=accepts, n_trace=trace,
                     log_alpha=la, summaries=summ, scalars=scal)
        state, accepts, trace, la, summ, scal = (v.cpu().numpy() for v in (state, accepts, trace, la, summ, scal))
        if ref is None:
            ref = state, accepts, trace, la
            # |ll| of the first state (importance sampling's execution c) and of every state and proposal after it
            lw = torch.empty(C, dtype=torch.float64, device="cuda")
            ppl.ppl_importance(ppl.PPL_MODEL_POLY, data, C, seed, log_weights=lw)
            size = np.abs(lw.cpu().numpy()) + np.cumsum(np.abs(la) + 4.0, axis=0)
        np.testing.assert_array_equal(state, ref[0][:, :C])
        np.testing.assert_array_equal(accepts, ref[1][:C])
        np.testing.assert_array_equal(trace, ref[2][:, :C])
        assert np.all(np.abs(la - ref[3][:, :C]) <= (D + 4) * 2.0 ** -52 * size[:, :C])
        kept = trace[burn:]
        counts = [(kept == m).sum() for m in range(2, 6)]
        assert scal[1] == sum(counts) and scal[2] == C and abs(scal[0] - accepts.mean() / T) < 1e-15 * T * C
        for m in range(4):
            assert abs(summ[m] - (counts[m] / max(1, sum(counts)))) < 1e-12
        if n_lo == 2:
            assert np.allclose(summ[24:], sum(summ[m] * summ[4 + 5 * m:9 + 5 * m] for m in range(4)), rtol=1e-9, atol=1e-9)


# --------------------------------------------- resampling of persistent SMC --
@pytest.mark.parametrize("n,far", [(1, 0.0), (2, 0.0), (511, 4.0), (513, 0.0), (2561, 8.0), (3072, 4.0), (33_000, 12.0),
                                   ((1 << 17) - 1, 12.0), ((1 << 17) + 1, 6.0), ((1 << 18) + 513, 12.0),
                                   ((1 << 19) + 4097, 6.0)])
def test_smc_ancestors_with_far_observations(ppl, orc, n, far):
    """Every third observation lies `far` away, so an event may leave a handful of
    particles with weight: a block's ancestors then lie in one tile, in neighbouring
    tiles or in many, and it finds them by marks or by searches.  Every ancestor
    follows from the event's own log-weights (the oracle resamples those)."""
    from forced_check import check_forced
    from test_gpu_smc import ESS_BAND, run_gpu
    T, seed = 24, 19
    y = synthetic.lgssm_data(T=T, seed=43)
    y[2::3] += np.float32(far)
    g = run_gpu(ppl, ppl.PPL_MODEL_LGSSM, y, n, seed, ess_frac=0.9, max_events=T, records=True)
    E = g["n_resample"]
    f = orc.smc_forced(orc.MODEL_LGSSM, y.astype(np.float64), n, seed, g["resampled"], g["ancestors"][:max(E, 1)],
                       g["event_lw"][:max(E, 1)], ess_frac=0.9, ess_band=ESS_BAND, want_state=True)
    print(check_forced(g, f, n, full=True, min_events=0 if n < 3 else 8))


# --------------------------------------------------------- batched mixtures --
@pytest.mark.parametrize("moves", [0, 1])
@pytest.mark.parametrize("K", range(1, 9))
def test_batched_every_instantiation(ppl, K, moves):
    """Every component count at 1, 2, 4 and 8 particles per lane and blocks of 1
    and 64 factors, with slots beyond the last particle (700, 4097) and without
    (4096), a far observation (the shifted form of the factor) and a length that
    leaves a remainder of the moves' side by side data.  The particles and the
    normaliser are the same bits for every launch shape, and log Z-hat is the sum
    of its trace (D additions of values up to |log Z-hat| in another order)."""
    from test_gpu_batched import run_batch
    rng = np.random.default_rng(1000 + K)
    batch = []
    for D, N in ((67, 700), (50, 4097), (90, 4096)):
        y = (rng.normal(size=K) * 10.0)[rng.integers(0, K, D)] + rng.normal(size=D)
        y[D // 2] += 80.0
        batch.append((K, y.astype(np.float32), N))
    ref = None
    for tune in ((4, 0, 64, 0), (1, 0, 64, 0), (2, 0, 64, 0), (8, 0, 64, 0), (8, 0, 1, 0)):
        g = run_batch(ppl, batch, 5, tune=tune, max_events=90, move_steps=moves)
        for i, gi in enumerate(g):
            D = batch[i][1].size
            assert gi["status"] == 0
            assert abs(np.nansum(gi["logz_trace"]) - gi["log_z"]) <= D * 2.0 ** -52 * (abs(gi["log_z"]) + 1.0)
            if ref is not None:
                for key in ("log_z", "n_resample", "lw", "state", "ancestors"):
                    np.testing.assert_array_equal(np.asarray(gi[key]), np.asarray(ref[i][key]))
        ref = g if ref is None else ref


# ------------------------------------------------------ standalone resampling --
@pytest.mark.parametrize("n", [1, 2, 63, 1023, 1025, 2048, 2049, 8192, 8193, 20_000, 2048 * 256, 2048 * 256 + 1])
@pytest.mark.parametrize("kind", ["even", "one", "ends", "zero"])
def test_resample_launch_shapes(ppl, orc, n, kind):
    """Entry counts on both sides of the rules for own maxima and local tile
    prefixes.  The weights are 0 or 1 (log-weights 0 or -inf), which quantise
    exactly, so every ancestor is the oracle's."""
    import torch
    lw = np.full(n, -np.inf, dtype=np.float32)
    if kind == "even":
        lw[::2] = 0.0
    elif kind == "one":
        lw[n // 3] = 0.0
    elif kind == "ends":
        lw[0] = lw[-1] = 0.0
    state = np.arange(5 * n, dtype=np.float32).reshape(5, n)
    anc = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    out = ppl.ppl_resample_gather(torch.from_numpy(lw).cuda(), torch.from_numpy(state).cuda(), seed=6, step=2, inst=1,
                                  anc=anc).cpu().numpy()
    got = anc.cpu().numpy()
    if kind == "zero":
        assert np.all(got == -1) and np.all(np.isnan(out))
        return
    ref, _ = orc.resample(lw.astype(np.float64), seed=6, step=2, inst=1, band=0.0)
    np.testing.assert_array_equal(got, ref)
    np.testing.assert_array_equal(out, state[:, ref])
