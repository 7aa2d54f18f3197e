"""GPU parity of lightweight Metropolis-Hastings (many independent chains of
the polynomial model) against the CPU oracle, through the C ABI.

Both sides run FP64 from the same Philox words.  The oracle runs beside the
GPU's chains: where its log acceptance ratio and the GPU's straddle log v
within twice their difference (plus 1e-9 relative), the decision is a tie and
the GPU's is taken; every other decision must agree.  Then: traces of n
bit-exact, log acceptance ratios within 1e-10 (mixed), final coefficients
within 1e-12, accepted counts exact, summaries within 1e-10."""
import math

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


def mixed_err(a, b):
    a, b = np.asarray(a, np.float64), np.asarray(b, np.float64)
    return float(np.max(np.abs(a - b) / np.maximum(1.0, np.abs(b)))) if a.size else 0.0


def run_gpu(ppl, x, y, C, T, seed, burn=0, trace=True):
    import torch
    dev = torch.device("cuda:0")
    dx = torch.from_numpy(np.ascontiguousarray(x, np.float64)).to(dev) if x.size else torch.zeros(1, dtype=torch.float64, device=dev)
    dy = torch.from_numpy(np.ascontiguousarray(y, np.float64)).to(dev) if y.size else torch.zeros(1, dtype=torch.float64, device=dev)
    data = ppl.make_data(dx, dy, n_data=y.size, dtype=ppl.PPL_F64)
    st = torch.empty((6, C), dtype=torch.float64, device=dev)
    acc = torch.empty(C, dtype=torch.int64, device=dev)
    summ = torch.empty(29, dtype=torch.float64, device=dev)
    scal = torch.empty(4, dtype=torch.float64, device=dev)
    ntr = torch.empty((max(T, 1), C), dtype=torch.int8, device=dev) if trace else None
    la = torch.empty((max(T, 1), C), dtype=torch.float64, device=dev) if trace else None
    r = ppl.ppl_mcmc(ppl.PPL_MODEL_POLY, data, C, T, seed, burn_in=burn, state=st, accepts=acc, summaries=summ,
                     scalars=scal, n_trace=ntr, log_alpha=la, sync=True)
    out = dict(rate=r.accept_rate, state=st.cpu().numpy(), accepts=acc.cpu().numpy(), summaries=summ.cpu().numpy(),
               scalars=scal.cpu().numpy())
    if trace:
        out["n_trace"] = ntr.cpu().numpy()[:T]
        out["la"] = la.cpu().numpy()[:T]
    return out


@pytest.mark.parametrize("C,T,burn,D", [(3000, 200, 50, 100), ((1 << 16) + 5, 40, 10, 100), (257, 500, 0, 12),
                                         (1, 30, 30, 5)])
def test_mcmc_matches_oracle(ppl, orc, C, T, burn, D):
    x, y = synthetic.poly_data(D=D)
    seed = 19
    g = run_gpu(ppl, x, y, C, T, seed, burn)
    o = orc.mcmc_poly(x, y, C, T, seed, burn_in=burn, want_trace=True, given_la=g["la"])
    assert o["nontie_diff"] == 0, o["nontie_diff"]
    assert o["ties"] <= 2 + 1e-6 * C * T
    assert np.array_equal(g["n_trace"], o["n_trace"])
    assert mixed_err(g["la"], o["la_trace"]) < 1e-10
    assert mixed_err(g["state"], o["state"]) < 1e-12
    assert np.array_equal(g["accepts"], o["accepts"])
    assert mixed_err(g["summaries"], o["summaries"]) < 1e-10
    assert abs(g["rate"] - o["accepts"].sum() / (C * T)) < 1e-12
    assert g["scalars"][1] == C * (T - burn) and g["scalars"][2] == C and g["scalars"][3] == 0


def test_mcmc_without_data_samples_the_prior(ppl):
    """No data: the chains' n is uniform on {2..5} (the site-count factor at work)."""
    g = run_gpu(ppl, np.zeros(0), np.zeros(0), 1 << 18, 200, 3, burn=50, trace=False)
    p = g["summaries"][:4]
    assert np.all(np.abs(p - 0.25) < 0.01), p
    assert 0.0 < g["rate"] <= 1.0


def test_mcmc_zero_iterations_is_the_prior_draw(ppl, orc):
    x, y = synthetic.poly_data()
    g = run_gpu(ppl, x, y, 1000, 0, 7, trace=False)
    o = orc.mcmc_poly(x, y, 1000, 0, 7)
    assert mixed_err(g["state"], o["state"]) < 1e-12
    assert np.all(g["accepts"] == 0) and np.all(g["summaries"] == 0.0) and g["rate"] == 0.0


def test_mcmc_rejects_bad_arguments(ppl):
    import torch
    dev = torch.device("cuda:0")
    x, y = synthetic.poly_data()
    data = ppl.make_data(torch.from_numpy(x).to(dev), torch.from_numpy(y).to(dev))
    for kw in (dict(n_chains=0, n_iters=10, burn_in=0), dict(n_chains=10, n_iters=10, burn_in=11),
               dict(n_chains=10, n_iters=-1, burn_in=0)):
        with pytest.raises(ppl.PplError) as e:
            ppl.ppl_mcmc(ppl.PPL_MODEL_POLY, data, kw["n_chains"], kw["n_iters"], 1, burn_in=kw["burn_in"],
                         ws=ppl.workspace(1 << 20))
        assert e.value.code == ppl.PPL_E_ARG
    with pytest.raises(ppl.PplError) as e:
        ppl.ppl_mcmc(ppl.PPL_MODEL_BLR, data, 10, 10, 1, ws=ppl.workspace(1 << 20))
    assert e.value.code == ppl.PPL_E_MODEL


@pytest.mark.parametrize("C,D", [(65, 5), (1000, 20), (4097, 100), (16384, 33), (32768, 100)])
def test_mcmc_least_workspace(ppl, C, D):
    """A workspace of 256 + 240 ceil(C / 256) bytes, rounded up to 256, takes every
    call, with the same chains; one byte less is refused.  A likelihood sum in
    another order (D terms of one sign) moves log alpha by at most D 2^-52 of
    the log-likelihoods' size, a summary (sums of C (T - burn) terms) by 1e-10."""
    import torch
    x, y = synthetic.poly_data(D=D)
    data = ppl.make_data(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda())
    least = 256 + (-(-C // 256) * 240 + 255) // 256 * 256
    full = ppl.ppl_workspace_size(ppl.PPL_MODEL_POLY, data, C, ppl.PPL_ALGO_MCMC)
    T, got = 25, []
    for size in (full, least):
        out = dict(state=torch.empty((6, C), dtype=torch.float64, device="cuda"),
                   accepts=torch.empty(C, dtype=torch.int64, device="cuda"),
                   summaries=torch.empty(29, dtype=torch.float64, device="cuda"),
                   scalars=torch.empty(4, dtype=torch.float64, device="cuda"),
                   n_trace=torch.empty((T, C), dtype=torch.int8, device="cuda"),
                   log_alpha=torch.empty((T, C), dtype=torch.float64, device="cuda"))
        block = ppl.workspace(size + 256).fill_(0x5A)
        ppl.ppl_mcmc(ppl.PPL_MODEL_POLY, data, C, T, 23, burn_in=5, ws=block[:size], **out)
        assert torch.all(block[size:] == 0x5A)             # nothing written past the end
        got.append({k: v.cpu().numpy() for k, v in out.items()})
    for key in ("state", "accepts", "n_trace"):
        np.testing.assert_array_equal(got[0][key], got[1][key], err_msg=key)
    lw = torch.empty(C, dtype=torch.float64, device="cuda")
    ppl.ppl_importance(ppl.PPL_MODEL_POLY, data, C, 23, log_weights=lw)      # chain c starts at execution c
    size = np.abs(lw.cpu().numpy()) + np.cumsum(np.abs(got[0]["log_alpha"]) + 4.0, axis=0)
    assert np.all(np.abs(got[0]["log_alpha"] - got[1]["log_alpha"]) <= (D + 4) * 2.0 ** -52 * size)
    for key in ("summaries", "scalars"):
        assert mixed_err(got[0][key], got[1][key]) < 1e-10, key
    with pytest.raises(ppl.PplError) as e:
        ppl.ppl_mcmc(ppl.PPL_MODEL_POLY, data, C, T, 23, ws=ppl.workspace(least)[:least - 1])
    assert e.value.code == ppl.PPL_E_WORKSPACE
