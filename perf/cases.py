"""The work a user has this library do, as a list of timed cases.

Every case goes through the binding's public functions with the outputs and the
workspace allocated beforehand, as ``bench.py`` does.  Sizes are those of the
repository's benchmark configurations and tests, with ragged ones beside them.

  poly      importance sampling of the polynomial fit (FP64), prior proposal
  blr       importance sampling of the linear regression (FP32 likelihood), row by
            row or from sufficient statistics, prior or Gaussian proposal
  resample  systematic resampling with the gather of particle state
  lgssm     sequential Monte Carlo over the linear-Gaussian state space
  gmm       sequential Monte Carlo over one mixture, plain or resample-move
  batch     sequential Monte Carlo over many mixtures in one launch
  enum      enumeration of every path of a hidden Markov model
  mcmc      lightweight Metropolis-Hastings chains over the polynomial fit
  train     training of the learned proposal (forward, backward, Adam)
  infer     importance sampling with the learned proposal
"""
import math

import numpy as np
import torch

import paper_2010_08454_amd as ppl

F64, F32 = torch.float64, torch.float32
LOG_2PI = math.log(2.0 * math.pi)


def listed():
    return [
        # one small posterior query: a serving call, where launches and latency count
        dict(name="poly-10k", path="poly", n=10_000, d=100),
        # the particle count of the method's published importance-sampling runs
        dict(name="poly-2m", path="poly", n=2_000_000, d=100),
        # the headline workload: every particle against every row
        dict(name="blr-1m", path="blr", n=1 << 20, d=10_000, dim=16, stats=False, q=False),
        # the resampling step of a large filter kept outside the library: 1 GiB of state
        dict(name="resample-16m", path="resample", n=1 << 24, fields=16, f64=False),
        # a long filter over a million particles, resampling at most steps
        dict(name="lgssm-1m", path="lgssm", n=1 << 20, d=1000),
        # one mixture with a ragged, modest particle count and rejuvenation moves
        dict(name="gmm-move-20011", path="gmm", n=20_011, d=500, k=4, moves=1),
        # many datasets of very different lengths filtered at once
        dict(name="batch-64", path="batch", inst=64, n=1 << 16, lo=2.0, hi=4.5, moves=0),
        # exact inference by brute force: 2^40 executions
        dict(name="enum-4x20", path="enum", k=4, t=20),
        # many chains over a small dataset
        dict(name="mcmc-64k", path="mcmc", n=1 << 16, d=100, iters=1000, burn=200),
        # proposal training at the batch size that trains best
        dict(name="train-poly-512", path="train", model="poly", k=0, batch=512, steps=512, d=1000),
        # amortised inference, a launch-bound call
        dict(name="infer-poly-4k", path="infer", model="poly", k=0, n=1 << 12, d=1000),
        # amortised inference at a throughput size
        dict(name="infer-gmm-1m", path="infer", model="gmm", k=5, n=1 << 20, d=100),
    ]


def _log_int(rng, lo, hi):
    """A whole number spread over the logarithm of [lo, hi]; now and then a power of two."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    if rng.random() < 0.2:
        v = 2.0 ** round(math.log2(v))
    return int(min(max(round(v), lo), hi))


def draw(rng):
    path = rng.choice(["poly", "poly", "blr", "blr", "resample", "resample", "lgssm", "gmm", "batch", "enum", "mcmc",
                       "train", "infer", "infer"])
    if path == "poly":
        d = _log_int(rng, 10, 1000)
        return dict(path=path, n=_log_int(rng, 1000, min(2_000_000, 400_000_000 // d)), d=d)
    if path == "blr":
        return dict(path=path, n=_log_int(rng, 1000, 1 << 20), d=_log_int(rng, 100, 10_000),
                    dim=rng.choice([4, 8, 12, 16]), stats=rng.random() < 0.4, q=rng.random() < 0.4)
    if path == "resample":
        fields = rng.randint(1, 16)
        return dict(path=path, n=_log_int(rng, 1000, (1 << 28) // fields if fields > 15 else 1 << 24), fields=fields,
                    f64=rng.random() < 0.25)
    if path == "lgssm":
        return dict(path=path, n=_log_int(rng, 1000, 1 << 20), d=_log_int(rng, 50, 1000))
    if path == "gmm":
        return dict(path=path, n=_log_int(rng, 1000, 1 << 17), d=_log_int(rng, 50, 1000), k=rng.randint(2, 8),
                    moves=rng.choice([0, 0, 1, 2]))
    if path == "batch":
        return dict(path=path, inst=rng.randint(8, 64), n=_log_int(rng, 1000, 1 << 16), lo=2.0,
                    hi=round(rng.uniform(3.0, 4.5), 2), moves=rng.choice([0, 0, 0, 1]))
    if path == "enum":
        k = rng.randint(2, 8)
        top = min(int(38 / math.log2(k)), 40, 1024 // (k * k))
        return dict(path=path, k=k, t=rng.randint(max(2, int(10 / math.log2(k))), top))
    if path == "mcmc":
        iters = _log_int(rng, 100, 1000)
        return dict(path=path, n=_log_int(rng, 1000, 1 << 16), d=_log_int(rng, 20, 200), iters=iters, burn=iters // 5)
    if path == "train":
        poly = rng.random() < 0.5
        return dict(path=path, model="poly" if poly else "gmm", k=0 if poly else rng.randint(2, 8),
                    batch=64 * _log_int(rng, 1, 64), steps=_log_int(rng, 16, 128),
                    d=_log_int(rng, 50, 1000) if poly else _log_int(rng, 50, 500))
    poly = rng.random() < 0.5
    return dict(path=path, model="poly" if poly else "gmm", k=0 if poly else rng.randint(2, 8),
                n=_log_int(rng, 1000, 1 << 20), d=_log_int(rng, 50, 1000))


# ----------------------------------------------------------------- inputs --
def _gpu(a, dtype=None):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dtype).cuda()


def _poly_host(g, d):
    x = g.uniform(-1.0, 1.0, d)
    return x, 0.5 - 1.2 * x + 0.8 * x ** 3 + 0.1 * g.standard_normal(d)


def _gmm_host(g, k, d):
    z = g.choice(k, size=d, p=g.dirichlet(np.ones(k)))
    return ((5.0 * g.standard_normal(k))[z] + g.standard_normal(d)).astype(np.float32)


def _blr_host(case, seed):
    """X, y and the Gaussian proposal {mean, Cholesky factor} of the linear regression (its posterior)."""
    g = np.random.default_rng(seed)
    d, dim = case["d"], case["dim"]
    X = g.standard_normal((d, dim)).astype(np.float32)
    y = (X.astype(np.float64) @ g.standard_normal(dim) + 0.5 * g.standard_normal(d)).astype(np.float32)
    cov = np.linalg.inv(X.T.astype(np.float64) @ X / 0.25 + np.eye(dim))
    mean = cov @ (X.T.astype(np.float64) @ y) / 0.25
    return X, y, np.concatenate([mean, np.linalg.cholesky(cov).ravel()]).astype(np.float32)


def _hmm_host(case, seed):
    """pi0, A, mu, sigma, y of a sticky chain with Gaussian emissions."""
    g = np.random.default_rng(seed)
    k, t = case["k"], case["t"]
    pi0 = g.dirichlet(np.ones(k))
    A = g.dirichlet(np.ones(k), size=k) + 3.0 * np.eye(k)
    A /= A.sum(1, keepdims=True)
    mu = 2.0 * (np.arange(k) - (k - 1) / 2.0) + 0.3 * g.standard_normal(k)
    z = [g.choice(k, p=pi0)]
    for _ in range(t - 1):
        z.append(g.choice(k, p=A[z[-1]]))
    return pi0, A, mu, 1.0, mu[z] + g.standard_normal(t)


def _lgssm_host(g, d):
    x, y = 0.0, np.empty(d)
    for t in range(d):
        x = 0.9 * x + g.standard_normal()
        y[t] = x + 0.5 * g.standard_normal()
    return y.astype(np.float32)


def _empty(*shape, dtype=F64):
    return torch.zeros(shape, dtype=dtype, device="cuda")


def prepare(case, seed):
    g = np.random.default_rng(seed)
    path, s = case["path"], dict(case=case, seed=seed)
    if path == "poly":
        x, y = _poly_host(g, case["d"])
        s["data"] = ppl.make_data(_gpu(x), _gpu(y))
        s["model"] = ppl.PPL_MODEL_POLY
        s["out"] = dict(scalars=_empty(8), summaries=_empty(29), log_weights=_empty(case["n"]), latents=_empty(6, case["n"]))
        s["ws"] = ppl.workspace(ppl.ppl_workspace_size(s["model"], s["data"], case["n"], ppl.PPL_ALGO_IS))
    elif path == "blr":
        X, y, q = _blr_host(case, seed)
        s["data"] = ppl.make_data(_gpu(X), _gpu(y), dim=case["dim"])
        s["model"] = ppl.PPL_MODEL_BLR_STATS if case["stats"] else ppl.PPL_MODEL_BLR
        s["q"] = _gpu(q) if case["q"] else None
        s["out"] = dict(scalars=_empty(8), summaries=_empty(case["dim"]), log_weights=_empty(case["n"]))
        s["ws"] = ppl.workspace(ppl.ppl_workspace_size(s["model"], s["data"], case["n"], ppl.PPL_ALGO_IS))
    elif path == "resample":
        r = torch.Generator("cuda").manual_seed(seed)
        s["lw"] = torch.randn(case["n"], dtype=F64 if case["f64"] else F32, device="cuda", generator=r)
        s["state"] = torch.randn(case["fields"], case["n"], device="cuda", generator=r)
        s["out"] = dict(state=torch.empty_like(s["state"]), ancestors=_empty(case["n"], dtype=torch.int32))
        s["ws"] = ppl.workspace(ppl.ppl_workspace_size(0, None, case["n"], ppl.PPL_ALGO_RESAMPLE))
    elif path in ("lgssm", "gmm"):
        y = _lgssm_host(g, case["d"]) if path == "lgssm" else _gmm_host(g, case["k"], case["d"])
        s["model"] = ppl.PPL_MODEL_LGSSM if path == "lgssm" else ppl.PPL_MODEL_GMM
        s["data"] = ppl.make_data(None, _gpu(y), dim=case.get("k", 0), dtype=ppl.PPL_F32)
        width = 1 if path == "lgssm" else 2 * case["k"]
        s["out"] = dict(scalars=_empty(8), latents=_empty(width, case["n"], dtype=F32),
                        log_weights=_empty(case["n"], dtype=F32), ess_trace=_empty(case["d"]),
                        resampled=_empty(case["d"], dtype=torch.uint8))
        s["ws"] = ppl.workspace(ppl.ppl_workspace_size(s["model"], s["data"], case["n"], ppl.PPL_ALGO_SMC))
    elif path == "batch":
        ks = [int(g.integers(3, 9)) for _ in range(case["inst"])]
        ys = [_gpu(_gmm_host(g, k, int(10.0 ** g.uniform(case["lo"], case["hi"])))) for k in ks]
        s["table"] = ppl.InstanceTable(ys, ks, case["n"], move_steps=case["moves"])
        # the configuration the autotuner settles on for such batches
        s["tune"] = (8, -(-case["n"] // 4096), 256, 0)
        total = case["inst"] * case["n"]
        s["out"] = dict(out=_empty(case["inst"], 4), log_weights=_empty(total, dtype=F32), latents=_empty(16 * total, dtype=F32))
        s["ws"] = ppl.workspace(ppl.ppl_smc_batched_workspace_size(ppl.PPL_MODEL_GMM, s["table"], s["tune"]))
    elif path == "enum":
        pi0, A, mu, sigma, y = _hmm_host(case, seed)
        s["data"] = ppl.hmm_data(_gpu(y), pi0, A, mu, sigma)
        s["out"] = dict(scalars=_empty(4), marginals=_empty(case["t"], case["k"]), map_path=_empty(case["t"], dtype=torch.int32))
        s["ws"] = ppl.workspace(ppl.ppl_workspace_size(ppl.PPL_MODEL_HMM, s["data"], 1, ppl.PPL_ALGO_ENUM))
    elif path == "mcmc":
        x, y = _poly_host(g, case["d"])
        s["data"] = ppl.make_data(_gpu(x), _gpu(y))
        s["out"] = dict(scalars=_empty(4), summaries=_empty(29), state=_empty(6, case["n"]),
                        accepts=_empty(case["n"], dtype=torch.int64))
        s["ws"] = ppl.workspace(ppl.ppl_workspace_size(ppl.PPL_MODEL_POLY, s["data"], case["n"], ppl.PPL_ALGO_MCMC))
    else:
        s["model"] = ppl.PPL_MODEL_POLY if case["model"] == "poly" else ppl.PPL_MODEL_GMM
        s["weights"] = ppl.ppl_proposal_init(seed)
        batch, steps = (case["batch"], case["steps"]) if path == "train" else (512, 64)
        s["cfg"] = ppl.train_config(batch * steps, batch, case["d"], dim=case["k"], use_graph=True)
        s["train_ws"] = ppl.workspace(ppl.ppl_proposal_train_workspace_size(s["model"], s["cfg"]))
        if path == "train":
            block, count = s["weights"][: 12 * ppl.N_PARAMS].view(F32), ppl.N_PARAMS
            s["out"] = dict(loss=_empty(steps), master=block[:count], moment1=block[count:2 * count],
                            moment2=block[2 * count:])
        else:
            # a proposal that has seen some training, and the data it is asked about
            ppl.ppl_proposal_train(s["model"], s["cfg"], seed, s["weights"], ws=s["train_ws"])
            poly = case["model"] == "poly"
            if poly:
                x, y = _poly_host(g, case["d"])
                s["data"] = ppl.make_data(_gpu(x), _gpu(y))
            else:
                s["data"] = ppl.make_data(None, _gpu(_gmm_host(g, case["k"], case["d"])), dim=case["k"], dtype=ppl.PPL_F32)
            nq = 332 if poly else 8 + 16 * (2 * case["k"] - 1)
            s["out"] = dict(scalars=_empty(8), summaries=_empty(29 if poly else 8), log_weights=_empty(case["n"]),
                            q_params=_empty(nq), data_summaries=_empty(64))
            s["ws"] = ppl.workspace(ppl.ppl_proposal_infer_workspace_size(s["model"], s["data"], case["n"]))
    return s


def run(s):
    case, seed, out = s["case"], s["seed"], s["out"]
    path = case["path"]
    if path == "poly":
        ppl.ppl_importance(s["model"], s["data"], case["n"], seed, ws=s["ws"], **out)
    elif path == "blr":
        ppl.ppl_importance(s["model"], s["data"], case["n"], seed, q=s["q"], ws=s["ws"], **out)
    elif path == "resample":
        ppl.ppl_resample_gather(s["lw"], s["state"], seed, step=3, out=out["state"], anc=out["ancestors"], ws=s["ws"])
    elif path in ("lgssm", "gmm"):
        ppl.ppl_smc(s["model"], s["data"], case["n"], seed, 0.5, ws=s["ws"], move_steps=case.get("moves", 0), **out)
    elif path == "batch":
        ppl.ppl_smc_batched(ppl.PPL_MODEL_GMM, s["table"], seed, 0.5, tune=s["tune"], ws=s["ws"], **out)
    elif path == "enum":
        ppl.ppl_enumerate(ppl.PPL_MODEL_HMM, s["data"], ws=s["ws"], **out)
    elif path == "mcmc":
        ppl.ppl_mcmc(ppl.PPL_MODEL_POLY, s["data"], case["n"], case["iters"], seed, burn_in=case["burn"], ws=s["ws"], **out)
    elif path == "train":
        ppl.ppl_proposal_train(s["model"], s["cfg"], seed, s["weights"], loss_trace=out["loss"], ws=s["train_ws"])
    else:
        ppl.ppl_proposal_infer(s["model"], s["data"], s["weights"], case["n"], seed, ws=s["ws"], **out)
    return out


# ------------------------------------------------------------------- work --
def work(case):
    path, n, d = case["path"], case.get("n", 0), case.get("d", 0)
    if path == "poly":       # Horner (4 FMA), difference, square; coefficients and weights written once
        return {"flops": 10.0 * n * d, "bytes": 16.0 * d + 56.0 * n}
    if path == "blr":
        dim = case["dim"]
        if case["stats"]:
            return {"flops": 2.0 * (dim * dim + dim) * (n + d), "bytes": 4.0 * d * (dim + 1) + 8.0 * n}
        return {"flops": (2.0 * dim + 2.0) * n * d, "bytes": 4.0 * d * (dim + 1) + 8.0 * n}
    if path == "resample":   # weights read, state read and written, ancestors written
        return {"flops": 10.0 * n, "bytes": n * ((8.0 if case["f64"] else 4.0) + 8.0 * case["fields"] + 4.0)}
    if path == "lgssm":      # a quarter Philox block, half a Box-Muller pair, dynamics, density, trigger
        return {"flops": 42.0 * n * d, "bytes": 8.0 * n + 4.0 * d}
    if path == "gmm":
        return {"flops": (7.0 * case["k"] + 9.0) * n * d, "bytes": 4.0 * n * (2 * case["k"] + 1) + 4.0 * d}
    if path == "batch":      # mean data count of the log-uniform lengths, mean component count 5.5
        span = math.log(10.0) * (case["hi"] - case["lo"])
        mean = (10.0 ** case["hi"] - 10.0 ** case["lo"]) / span if span > 0 else 10.0 ** case["lo"]
        return {"flops": (7.0 * 5.5 + 9.0) * case["inst"] * n * mean, "bytes": 4.0 * case["inst"] * (12.0 * n + mean)}
    if path == "enum":
        return {"flops": (2.0 + 4.0 / case["k"]) * float(case["k"]) ** case["t"], "bytes": 8.0 * case["t"] * (case["k"] + 1)}
    if path == "mcmc":
        return {"flops": 10.0 * n * d * case["iters"], "bytes": 56.0 * n + 16.0 * d}
    if path == "train":      # network products, the simulated data, and the update of weights and moments
        pairs = float(case["batch"] * case["steps"])
        return {"flops": pairs * (851_968.0 + 45.0 * d), "bytes": case["steps"] * 6.0 * 4.0 * ppl.N_PARAMS}
    per = 10.0 if case["model"] == "poly" else 7.0 * case["k"] + 4.0
    return {"flops": per * n * d, "bytes": 8.0 * n + 2.0 * 147_456 + 16.0 * d}


# ------------------------------------------------------------------ exact --
def _philox(i, c1, c2, c3, seed):
    """The four words of Philox4x32-10 blocks (i, c1, c2, c3) under key `seed`, as int64 tensors."""
    mask = 0xFFFFFFFF
    c = [i & mask] + [torch.full_like(i, v) for v in (c1, c2, c3)]
    k0, k1 = seed & mask, (seed >> 32) & mask
    for _ in range(10):
        a, b = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((b >> 32) & mask) ^ c[1] ^ k0, b & mask, ((a >> 32) & mask) ^ c[3] ^ k1, a & mask]
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return c


def _u32(w):
    return ((w >> 9).to(F64) + 0.5) * 2.0 ** -23


def _u64(lo, hi):
    return (((hi << 20) | (lo >> 12)).to(F64) + 0.5) * 2.0 ** -52


def _box_muller(u1, u2):
    r = torch.sqrt(-2.0 * torch.log(u1))
    return r * torch.cos(2.0 * math.pi * u2), r * torch.sin(2.0 * math.pi * u2)


def _pair64(w):
    return _box_muller(_u64(w[0], w[1]), _u64(w[2], w[3]))


def _scalars(lw):
    m = lw.max()
    e = torch.exp(lw - m)
    s1, s2, n = e.sum(), (e * e).sum(), float(lw.numel())
    vals = [float(m + torch.log(s1)) - math.log(n), float(s1 * s1 / s2), 0.0, 0.0, float(m), float(s1), float(s2), n]
    return torch.tensor(vals, dtype=F64), e


def _poly_summaries(n, c, w):
    """P(n), E[c | n] and E[c] of weighted draws (c zero past the degree)."""
    out = []
    mass = [float((w * (n == k)).sum()) for k in range(2, 6)]
    total = sum(mass)
    out += [v / total for v in mass]
    for k in range(2, 6):
        sel = w * (n == k)
        out += [float((sel * c[j]).sum()) / mass[k - 2] if mass[k - 2] > 0 else 0.0 for j in range(5)]
    return torch.tensor(out + [float((w * c[j]).sum()) / total for j in range(5)], dtype=F64)


def _poly_draw(i, seed):
    n = 2 + ((_philox(i, 0, 0, 0, seed)[0] * 4) >> 32)
    z = [v for b in (1, 2, 3) for v in _pair64(_philox(i, b, 0, 0, seed))]
    return n, [10.0 * v for v in z[:5]]


def _poly_loglik(c, x, y):
    acc = torch.zeros_like(c[0])
    for xv, yv in zip(x, y):
        p = (((c[4] * xv + c[3]) * xv + c[2]) * xv + c[1]) * xv + c[0]
        acc += (yv - p) ** 2
    return -0.5 * acc


def _exact_poly(case, seed):
    x, y = _poly_host(np.random.default_rng(seed), case["d"])
    n, c = _poly_draw(torch.arange(case["n"], device="cuda"), seed)
    kept = [torch.where(n > j, c[j], torch.zeros_like(c[j])) for j in range(5)]
    lw = _poly_loglik(kept, x.tolist(), y.tolist())
    scal, e = _scalars(lw)
    return dict(scalars=scal, summaries=_poly_summaries(n, kept, e), log_weights=lw, latents=torch.stack([n.to(F64)] + c))


def _exact_blr(case, seed):
    X, y, q = _blr_host(case, seed)
    n, d, dim = case["n"], case["d"], case["dim"]
    X, y, q = _gpu(X, F64), _gpu(y, F64), _gpu(q, F64)
    i, z = torch.arange(n, device="cuda"), []
    for b in range(dim // 4):
        w = _philox(i, b, 0, 1 if case["q"] else 0, seed)
        z += _box_muller(_u32(w[0]), _u32(w[1])) + _box_muller(_u32(w[2]), _u32(w[3]))
    z = torch.stack(z[:dim])
    extra = torch.zeros(n, dtype=F64, device="cuda")
    if case["q"]:
        L = torch.tril(q[dim:].reshape(dim, dim))
        w = q[:dim, None] + L @ z
        extra = -0.5 * (w * w).sum(0) + 0.5 * (z * z).sum(0) + torch.log(torch.diagonal(L)).sum()
    else:
        w = z
    lw, step = torch.empty(n, dtype=F64, device="cuda"), max(1, (1 << 27) // d)
    for a in range(0, n, step):
        lw[a:a + step] = ((y[:, None] - X @ w[:, a:a + step]) ** 2).sum(0)
    lw = -0.5 * d * math.log(2.0 * math.pi * 0.25) - lw / 0.5 + extra
    scal, e = _scalars(lw)
    return dict(scalars=scal, summaries=(w * e).sum(1) / e.sum(), log_weights=lw)


def _exact_enum(case, seed):
    pi0, A, mu, sigma, y = _hmm_host(case, seed)
    k, t = case["k"], case["t"]
    le = -0.5 * LOG_2PI - math.log(sigma) - 0.5 * ((y[:, None] - mu) / sigma) ** 2
    lA, f, b, v = np.log(A), np.empty((t, k)), np.zeros((t, k)), np.empty((t, k))
    f[0] = v[0] = np.log(pi0) + le[0]
    back = np.zeros((t, k), dtype=np.int64)
    for s in range(1, t):
        f[s] = np.logaddexp.reduce(f[s - 1][:, None] + lA, axis=0) + le[s]
        back[s] = np.argmax(v[s - 1][:, None] + lA, axis=0)
        v[s] = np.max(v[s - 1][:, None] + lA, axis=0) + le[s]
    for s in range(t - 2, -1, -1):
        b[s] = np.logaddexp.reduce(lA + (le[s + 1] + b[s + 1])[None], axis=1)
    log_z = np.logaddexp.reduce(f[-1])
    path = [int(np.argmax(v[-1]))]
    for s in range(t - 1, 0, -1):
        path.append(int(back[s][path[-1]]))
    return dict(scalars=np.array([log_z, float(k) ** t, v[-1].max(), 0.0]), marginals=np.exp(f + b - log_z),
                map_path=np.array(path[::-1], dtype=np.int32))


def _exact_mcmc(case, seed):
    x, y = (v.tolist() for v in _poly_host(np.random.default_rng(seed), case["d"]))
    i = torch.arange(case["n"], device="cuda")
    zero = torch.zeros(case["n"], dtype=F64, device="cuda")
    n, c = _poly_draw(i, seed)
    c = [torch.where(n > j, c[j], zero) for j in range(5)]
    xs, ys = torch.tensor(x, dtype=F64, device="cuda")[:, None], torch.tensor(y, dtype=F64, device="cuda")[:, None]

    def loglik(v):
        return -0.5 * ((ys - ((((v[4] * xs + v[3]) * xs + v[2]) * xs + v[1]) * xs + v[0])) ** 2).sum(0)

    ll, accepts = loglik(c), torch.zeros_like(i)
    mass, sums, total = [zero.clone() for _ in range(4)], [[zero.clone() for _ in range(5)] for _ in range(4)], 0
    for t in range(case["iters"]):
        w = _philox(i, 3 * t, 0, 8, seed)
        z = _pair64(_philox(i, 3 * t + 1, 0, 8, seed)) + _pair64(_philox(i, 3 * t + 2, 0, 8, seed))
        site = (w[0] * (n + 1)) >> 32
        n2 = torch.where(site == 0, 2 + ((w[1] * 4) >> 32), n)
        c2 = []
        for j in range(5):
            fresh = 10.0 * torch.where(n == j, z[1], torch.where(n == j - 1, z[2], z[3]))
            moved = torch.where(n2 <= j, zero, torch.where(n > j, c[j], fresh))
            c2.append(torch.where(site == 0, moved, torch.where(site == j + 1, 10.0 * z[0], c[j])))
        ll2 = loglik(c2)
        ok = torch.log(_u32(w[2])) < (ll2 - ll) + torch.log((n + 1).to(F64)) - torch.log((n2 + 1).to(F64))
        n, ll, accepts = torch.where(ok, n2, n), torch.where(ok, ll2, ll), accepts + ok
        c = [torch.where(ok, c2[j], c[j]) for j in range(5)]
        if t >= case["burn"]:
            total += case["n"]
            for m in range(4):
                here = (n == m + 2).to(F64)
                mass[m] += here
                for j in range(5):
                    sums[m][j] += here * c[j]
    mass = [float(v.sum()) for v in mass]
    sums = [[float(v.sum()) for v in row] for row in sums]
    summ = [v / total for v in mass] + [sums[m][j] / mass[m] if mass[m] else 0.0 for m in range(4) for j in range(5)]
    summ += [sum(sums[m][j] for m in range(4)) / total for j in range(5)]
    rate = float(accepts.sum()) / (case["n"] * case["iters"])
    return dict(scalars=torch.tensor([rate, float(total), float(case["n"]), 0.0], dtype=F64),
                summaries=torch.tensor(summ, dtype=F64), state=torch.stack([n.to(F64)] + c), accepts=accepts)


def _exact_infer(case, seed):
    """The summary statistics of the observed data; the network's products are defined by their
    16-bit storage points, so what follows from them has no 64-bit value."""
    g, d, s = np.random.default_rng(seed), case["d"], np.zeros(64)
    if case["model"] == "poly":
        x, y = _poly_host(g, d)
        s[:8] = [np.mean(x ** j * y) / 10.0 for j in range(8)]
        s[8:22] = [np.mean(x ** k) for k in range(1, 15)]
        s[22] = np.mean(y * y) / 100.0
        at, rss = 23, []
        for n in range(2, 6):
            V = x[:, None] ** np.arange(n)
            c = np.linalg.lstsq(V, y, rcond=None)[0]
            s[at:at + n] = c / 10.0
            rss.append(np.sum((y - V @ c) ** 2))
            at += n
        s[37:41] = [np.log1p(max(0.0, r - rss[3]) / 2.0) / 10.0 for r in rss]
        s[41] = math.log(d) / 10.0
    else:
        y = np.sort(_gmm_host(g, case["k"], d).astype(np.float64))
        s[:16] = [y[int((q + 0.5) * d / 16.0)] / 10.0 for q in range(16)]
        s[16:48] = np.bincount(np.clip(np.floor(y + 16.0), 0, 31).astype(int), minlength=32) / d
        c = y - y.mean()
        sd = math.sqrt(np.mean(c * c))
        s[48:53] = [y.mean() / 10.0, sd / 10.0, np.mean(c ** 3) / sd ** 3, (np.mean(c ** 4) / sd ** 4 - 3.0) / 10.0,
                    math.log(d) / 10.0]
    return dict(scalars=None, summaries=None, log_weights=None, q_params=None, data_summaries=s)


def exact(case, seed):
    """The outputs in 64 bits from plain torch and numpy, without the library.  Resampling only moves
    values; the filters resample on 32-bit weights, so their particles follow from 32-bit rounding; the
    network trains through 16-bit storage points."""
    made = dict(poly=_exact_poly, blr=_exact_blr, enum=_exact_enum, mcmc=_exact_mcmc, infer=_exact_infer)
    return made[case["path"]](case, seed) if case["path"] in made else None
