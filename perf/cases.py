"""The calls that a user of the library makes, over the sizes it is used at.

Every case goes through the package's public entry points: the likelihood of
one theta (what a likelihood search calls again and again), batches of small
likelihoods, the p-variate, tile-low-rank and mixed-precision likelihoods,
data simulation and prediction.  Locations are a jittered grid on the unit
square in Morton order, and Z is a draw of the model itself (random Fourier
features of its spectral density), as a fitted model meets it.
"""
import math

import numpy as np
import torch

import paper_2008_07437_amd as mvg

PRECISION = {"fp64": mvg.MVG_FP64, "tlr": mvg.MVG_TLR, "bf16x3": mvg.MVG_MIXED_BF16X3}
THETA = {"a": 0.1, "nu1": 0.5, "nu2": 1.0, "beta": 0.5}


def listed():
    return [
        # the objective of a likelihood search on a few hundred stations: one theta, latency
        {"name": "loglik_200", "kind": "loglik", "n": 200, "nb": 0, "precision": "fp64", **THETA},
        # the same on an odd size, at smoothnesses between the closed forms, as an optimiser visits them
        {"name": "loglik_1537", "kind": "loglik", "n": 1537, "nb": 0, "precision": "fp64",
         "a": 0.17, "nu1": 0.73, "nu2": 1.21, "beta": 0.35},
        # an ordinary dataset at the default tile size
        {"name": "loglik_6400", "kind": "loglik", "n": 6400, "nb": 0, "precision": "fp64", **THETA},
        # the dense exact workload at its usual size and tile size
        {"name": "loglik_25600", "kind": "loglik", "n": 25600, "nb": 1024, "precision": "fp64", **THETA},
        # many theta on one small dataset (profiles, bootstrap, grid searches)
        {"name": "batch_400x1024", "kind": "batch", "n": 400, "k": 1024, **THETA},
        # small requests of uneven size waiting together in a server
        {"name": "many_ragged_192", "kind": "many", "lo": 20, "hi": 512, "k": 192, **THETA},
        # the trivariate model
        {"name": "trivariate_2500", "kind": "loglik_p", "n": 2500, "p": 3, "nb": 0, "a": 0.1,
         "nu1": 0.5, "nu2": 1.0, "beta": 0.4},
        # tile low rank at its default tile size and accuracy
        {"name": "tlr_25600", "kind": "loglik", "n": 25600, "nb": 0, "precision": "tlr", "acc": 1e-7, **THETA},
        # mixed precision on a rough field, where it holds 1e-6
        {"name": "mixed_25600", "kind": "loglik", "n": 25600, "nb": 1024, "precision": "bf16x3",
         "a": 0.1, "nu1": 0.5, "nu2": 0.5, "beta": 0.5},
        # a synthetic field from the model: generate Sigma, factor it, Z = L eps
        {"name": "simulate_3200", "kind": "simulate", "n": 3200, "nb": 0, **THETA},
        # a prediction request on a resident factor
        {"name": "predict_5000x100", "kind": "predict", "n": 5000, "m": 100, "mse": False, "nb": 0, **THETA},
        # a map of predictions with its mean squared errors
        {"name": "predict_mse_5000x1000", "kind": "predict", "n": 5000, "m": 1000, "mse": True, "nb": 0, **THETA},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["loglik", "loglik", "loglik", "batch", "many", "loglik_p", "tlr", "mixed", "simulate",
                       "predict", "predict"])
    th = {"a": round(math.exp(rng.uniform(math.log(0.03), math.log(0.2))), 4),
          "nu1": rng.choice([0.5, round(rng.uniform(0.4, 0.9), 3)]),
          "nu2": rng.choice([1.0, round(rng.uniform(0.5, 1.3), 3)]), "beta": round(rng.uniform(0.0, 0.6), 3)}
    if kind == "loglik":
        n = _log_uniform(rng, 100, 16000)
        return {"kind": "loglik", "n": n, "nb": rng.choice([0, 0, 256, 768, 1024] if n > 2000 else [0, 0, 128, 256]),
                "precision": "fp64", **th}
    if kind == "batch":
        return {"kind": "batch", "n": rng.randint(30, 512), "k": _log_uniform(rng, 8, 768), **th}
    if kind == "many":
        lo = rng.randint(1, 100)
        return {"kind": "many", "lo": lo, "hi": rng.randint(lo + 20, 512), "k": _log_uniform(rng, 2, 400), **th}
    if kind == "loglik_p":
        return {"kind": "loglik_p", "n": _log_uniform(rng, 100, 5000), "p": rng.choice([1, 3, 4]), "nb": rng.choice([0, 256]),
                **{**th, "beta": round(rng.uniform(0.0, 0.45), 3)}}
    if kind == "tlr":
        return {"kind": "loglik", "n": _log_uniform(rng, 3000, 20000), "nb": 0, "precision": "tlr",
                "acc": rng.choice([1e-5, 1e-7]), **THETA, "a": th["a"], "beta": th["beta"]}
    if kind == "mixed":
        return {"kind": "loglik", "n": _log_uniform(rng, 4000, 20000), "nb": rng.choice([512, 1024]), "precision": "bf16x3",
                **THETA, "nu2": 0.5, "a": round(rng.uniform(0.05, 0.1), 4), "beta": th["beta"]}
    if kind == "simulate":
        return {"kind": "simulate", "n": _log_uniform(rng, 100, 9000), "nb": rng.choice([0, 256]), **th}
    return {"kind": "predict", "n": _log_uniform(rng, 100, 9000), "m": _log_uniform(rng, 5, 1500), "mse": rng.random() < 0.5,
            "nb": rng.choice([0, 256]), **th}


# ------------------------------------------------------------------- inputs


def _spread16(q):
    q = q.astype(np.uint64)
    for s, m in ((8, 0x00FF00FF), (4, 0x0F0F0F0F), (2, 0x33333333), (1, 0x55555555)):
        q = (q | (q << np.uint64(s))) & np.uint64(m)
    return q


def _locations(n, g):
    """A jittered grid on the unit square, n points kept, in Morton order."""
    k = math.isqrt(n - 1) + 1 if n > 1 else 1
    cell = np.sort(g.permutation(k * k)[:n])
    x = (cell // k + 0.5 + g.uniform(-0.4, 0.4, n)) / k
    y = (cell % k + 0.5 + g.uniform(-0.4, 0.4, n)) / k
    key = _spread16((x * 65536).astype(np.uint32)) | (_spread16((y * 65536).astype(np.uint32)) << np.uint64(1))
    order = np.argsort(key, kind="stable")
    return x[order], y[order]


def _model(case, p=2):
    """sigma^2, a, nu and the matrix of latent correlations of the case's model."""
    nu = [case["nu1"], case["nu2"], 0.5 * (case["nu1"] + case["nu2"]), 1.5][:p]
    beta = [[1.0 if i == j else case["beta"] for j in range(p)] for i in range(p)]
    return {"sigma_sq": [1.0, 1.2, 0.8, 1.0][:p], "a": case["a"], "nu": nu, "beta": beta}


def _six(t):
    return (t["sigma_sq"][0], t["sigma_sq"][1], t["a"], t["nu"][0], t["nu"][1], t["beta"][0][1])


def _dev(v):
    return torch.as_tensor(np.ascontiguousarray(v), dtype=torch.float64, device="cuda")


def _draw_z(x, y, t, g, terms=1024):
    """Z of the p-variate model t at (x, y), interleaved: random frequencies of
    the rougher and smoother variables' spectral densities, each weighted so
    that the covariance of Z is Sigma(t)."""
    p, a = len(t["nu"]), t["a"]
    own = np.asarray(t["nu"])[g.integers(0, p, terms)]
    w = g.standard_normal((2, terms)) / np.sqrt(g.chisquare(2.0 * own)) / a
    u = 1.0 + (a * w[0]) ** 2 + (a * w[1]) ** 2
    dens = np.stack([v * u ** -(v + 1.0) for v in t["nu"]])
    amp = np.sqrt(np.asarray(t["sigma_sq"])[:, None] * dens / dens.mean(0) / terms)
    low = np.linalg.cholesky(np.asarray(t["beta"]))
    c, s = (_dev((amp * (low @ g.standard_normal((p, terms)))).T) for _ in range(2))
    ang = x[:, None] * _dev(w[0])[None, :] + y[:, None] * _dev(w[1])[None, :]
    return (torch.cos(ang) @ c + torch.sin(ang) @ s).reshape(-1).contiguous()


def _inputs(case, seed):
    """Everything that a call reads, from the seed alone."""
    g = np.random.Generator(np.random.Philox(key=[seed, 7]))
    kind = case["kind"]
    if kind == "many":
        tasks = []
        for n in g.integers(case["lo"], case["hi"] + 1, case["k"]):
            x, y = (_dev(v) for v in _locations(int(n), g))
            t = _model(case)
            t["a"] *= float(g.uniform(0.8, 1.25))
            tasks.append((x, y, _draw_z(x, y, t, g, 64), t))
        return {"tasks": tasks}
    x, y = (_dev(v) for v in _locations(case["n"], g))
    t = _model(case, case.get("p", 2))
    d = {"x": x, "y": y, "theta": t}
    if kind == "simulate":
        d["eps"] = _dev(g.standard_normal(2 * case["n"]))
        return d
    d["z"] = _draw_z(x, y, t, g)
    if kind == "batch":
        six = np.asarray(_six(t))
        scale = g.uniform(0.8, 1.2, (case["k"], 6))
        d["thetas"] = np.clip(six * scale, None, [9.0, 9.0, 9.0, 4.9, 4.9, 0.9])
    if kind == "predict":
        d["x0"], d["y0"] = (_dev(v) for v in g.uniform(0.0, 1.0, (2, case["m"])))
    return d


def _options(case):
    o = {"precision": PRECISION[case.get("precision", "fp64")], "nb": case["nb"]}
    if "acc" in case:
        o["tlr_acc"] = case["acc"]
    return o


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    if case["kind"] == "many":
        s["tasks"] = [(x, y, z, _six(t)) for x, y, z, t in s["tasks"]]
    elif case["kind"] == "predict":
        _, s["factor"] = mvg.loglik(s["x"], s["y"], s["z"], _six(s["theta"]), _options(case), keep=True)
    return s


def run(state):
    s, case = state, state["case"]
    kind = case["kind"]
    if kind == "loglik":
        return mvg.loglik(s["x"], s["y"], s["z"], _six(s["theta"]), _options(case))
    if kind == "batch":
        return mvg.loglik(s["x"], s["y"], s["z"], s["thetas"])
    if kind == "many":
        return mvg.loglik_many(s["tasks"])
    if kind == "loglik_p":
        return mvg.loglik_p(s["x"], s["y"], s["z"], s["theta"], _options(case))
    if kind == "simulate":
        sigma = mvg.cov_generate(s["x"], s["y"], _six(s["theta"]), _options(case))
        info = mvg.potrf_tiled(sigma, _options(case))
        return {"info": info, "z": mvg.mvg_trmv(sigma, s["eps"])}
    out = mvg.cokrige_predict(s["factor"], s["x0"], s["y0"], with_mse=case["mse"])
    return {"zhat": out[0], "mse": out[1]} if case["mse"] else {"zhat": out}


# --------------------------------------------------------------------- work


def _rows(case):
    return case.get("p", 2) * case["n"]


def work(case):
    kind = case["kind"]
    if kind == "many":
        mean = 0.5 * (case["lo"] + case["hi"])
        cube = (case["lo"] + case["hi"]) * (case["lo"] ** 2 + case["hi"] ** 2) / 4  # mean of n^3
        return {"bytes": case["k"] * 8 * (4 * mean + 3), "flops": case["k"] * 8 * cube / 3}
    rows = _rows(case)
    if kind == "batch":
        return {"bytes": 8 * (4 * case["n"] + 9 * case["k"]), "flops": case["k"] * rows ** 3 / 3}
    if kind == "predict":
        # weights and locations once; with the errors, the factor once and its solve for two columns a target
        b, f = 8 * (2 * rows + 4 * case["m"]), 2.0 * rows * 2 * case["m"]
        return {"bytes": b + 4 * rows * rows, "flops": f + 2.0 * rows * rows * case["m"]} if case["mse"] else {"bytes": b, "flops": f}
    if case.get("precision") == "tlr":
        # each pair of locations generated once; the diagonal tiles' factors; one product of
        # rank 30 (the usual mean) for each pair of tiles and each earlier column
        nb = case["nb"] or 1200
        t = rows / nb
        return {"bytes": 8 * 2 * rows, "flops": 8.0 * rows * rows + t * nb ** 3 / 3 + t ** 3 / 6 * 2 * nb * nb * 30}
    return {"bytes": 8 * 2 * rows, "flops": rows ** 3 / 3}


# -------------------------------------------------------------------- exact


def _matern(h, a, nus):
    """Matern correlations of the distances h for every smoothness of nus:
    x^nu K_nu(x) / (2^(nu-1) Gamma(nu)), K_nu by the trapezoidal rule on
    int_0^inf exp(-x cosh t) cosh(nu t) dt."""
    step = 0.08
    t = torch.arange(0, 360, dtype=torch.float64, device=h.device) * step
    nu = torch.tensor(nus, dtype=torch.float64, device=h.device)[:, None]
    weight = torch.cosh(nu * t[None, :]) * step
    weight[:, 0] *= 0.5
    ch = torch.cosh(t)[:, None]
    norm = torch.tensor([-(v - 1.0) * math.log(2.0) - math.lgamma(v) for v in nus], dtype=torch.float64, device=h.device)[:, None]
    x = (h / a).reshape(-1)
    out = torch.empty((len(nus), x.numel()), dtype=torch.float64, device=h.device)
    for lo in range(0, x.numel(), 1 << 21):
        part = x[lo:lo + (1 << 21)]
        near = part.clamp_min(1e-12)
        k = weight @ torch.exp(-near[None, :] * ch)
        v = torch.exp(norm + nu * torch.log(near)[None, :]) * k
        out[:, lo:lo + (1 << 21)] = torch.where(part[None, :] > 0, v, torch.ones_like(v))
    return out.reshape(len(nus), *h.shape)


def _cov(x, y, x0, y0, t):
    """C_ij(|s - s0|) of the model t as a (p n) x (p m) matrix, interleaved."""
    p, nu, b = len(t["nu"]), t["nu"], t["beta"]
    pairs = [(i, j) for i in range(p) for j in range(i, p)]
    h = torch.sqrt((x[:, None] - x0[None, :]) ** 2 + (y[:, None] - y0[None, :]) ** 2)
    m = _matern(h, t["a"], [0.5 * (nu[i] + nu[j]) for i, j in pairs])
    out = torch.empty((x.numel(), p, x0.numel(), p), dtype=torch.float64, device=x.device)
    for k, (i, j) in enumerate(pairs):
        rho = b[i][j] * math.sqrt(nu[i] * nu[j]) / (0.5 * (nu[i] + nu[j]))
        out[:, i, :, j] = out[:, j, :, i] = rho * math.sqrt(t["sigma_sq"][i] * t["sigma_sq"][j]) * m[k]
    return out.reshape(p * x.numel(), p * x0.numel())


def _exact_loglik(tasks):
    out = {"loglik": [], "logdet": [], "quad": []}
    for x, y, z, t in tasks:
        low = torch.linalg.cholesky(_cov(x, y, x, y, t))
        logdet = 2.0 * float(torch.log(torch.diagonal(low)).sum())
        quad = float(torch.linalg.solve_triangular(low, z[:, None], upper=False).square().sum())
        out["logdet"].append(logdet)
        out["quad"].append(quad)
        out["loglik"].append(-0.5 * z.numel() * math.log(2.0 * math.pi) - 0.5 * logdet - 0.5 * quad)
    return {**{k: np.asarray(v) for k, v in out.items()}, "status": None}


def exact(case, seed):
    kind = case["kind"]
    if kind != "many" and _rows(case) > 20000:
        return None
    s = _inputs(case, seed)
    if kind == "many":
        return _exact_loglik(s["tasks"])
    x, y, t = s["x"], s["y"], s["theta"]
    if kind in ("loglik", "loglik_p"):
        return _exact_loglik([(x, y, s["z"], t)])
    if kind == "batch":
        each = [{"sigma_sq": list(v[:2]), "a": v[2], "nu": list(v[3:5]), "beta": [[1.0, v[5]], [v[5], 1.0]]}
                for v in s["thetas"].tolist()]
        return _exact_loglik([(x, y, s["z"], v) for v in each])
    low = torch.linalg.cholesky(_cov(x, y, x, y, t))
    if kind == "simulate":
        return {"info": None, "z": (low @ s["eps"][:, None])[:, 0]}
    # some columns at a time: the library's solve of very many at once does not find its workspace
    c0 = torch.cat([torch.linalg.solve_triangular(low, _cov(x, y, s["x0"][k:k + 128], s["y0"][k:k + 128], t), upper=False)
                    for k in range(0, case["m"], 128)], dim=1)
    v = torch.linalg.solve_triangular(low, s["z"][:, None], upper=False)
    zhat = (c0.T @ v).reshape(-1, 2)
    if not case["mse"]:
        return {"zhat": zhat}
    return {"zhat": zhat, "mse": sum(t["sigma_sq"]) - c0.square().sum(0).reshape(-1, 2).sum(1)}
