"""Timed cases of the dispersion-curve library, through its public calls.

A case is one pass of work as a user's program would ask for it: a curve, a
batch of models, a step of inversion chains, a sign map, a classification of
picks, a burst of served requests.  The listed sizes are those of the
library's own workloads (the two-layer case, a 40-wavelength curve on 1000
velocities, the 20-layer fine-scale curve, the 4096-model batch, the
256-chain inversion step, the served chains); draw() spreads over the same
ranges, odd sizes among them.

Inputs are synthetic velocity-increasing profiles, some with one slower
layer.  Sizes (layers and wavelengths of each model) follow from the case
alone and values from the seed, so that passes on other seeds have outputs
of the same shapes.
"""
import math
import weakref

import numpy as np
import torch

import paper_2003_02256_amd as M

# How a pick is searched: (precision, flags) of the calls.
SEARCH = {
    "walk": (M.MASW_PREC_FP64, 0),                          # Algorithm 1's scan in FP64
    "split": (M.MASW_PREC_SPLIT, 0),                        # FP32 sweep, FP64 check and refinement
    "inertia": (M.MASW_PREC_FP64, M.MASW_SEARCH_INERTIA),   # search on FP64 inertia counts
}


def listed():
    return [
        # the smallest call: a worked example's curve, one launch, buffers on the device
        dict(name="curve_two_layer", kind="curve", search="walk", host=False, layers=2, lambdas=30,
             lam_hi=40.0, c_lo=50.0, c_hi=450.0, n_c=801),
        # an experimental curve's length and grid, host arrays in and out
        dict(name="curve_host_40", kind="curve", search="walk", host=True, layers=10, lambdas=40,
             lam_hi=60.0, c_lo=50.0, c_hi=1049.0, n_c=1000),
        # one site at fine scale, by each of the three searches
        dict(name="curve_fine_walk", kind="curve", search="walk", host=False, layers=20, lambdas=1000,
             lam_hi=100.0, c_lo=50.0, c_hi=1200.0, n_c=115001),
        dict(name="curve_fine_split", kind="curve", search="split", host=False, layers=20, lambdas=1000,
             lam_hi=100.0, c_lo=50.0, c_hi=1200.0, n_c=115001),
        dict(name="curve_fine_inertia", kind="curve", search="inertia", host=False, layers=20, lambdas=1000,
             lam_hi=100.0, c_lo=50.0, c_hi=1200.0, n_c=115001),
        # many models of uneven sizes in one launch, by each of the three searches
        dict(name="batch_walk", kind="batch", search="walk", models=4096, n_c=19001),
        dict(name="batch_split", kind="batch", search="split", models=4096, n_c=19001),
        dict(name="batch_inertia", kind="batch", search="inertia", models=4096, n_c=19001),
        # one step of a population of inversion chains: curves and misfits, no refinement
        dict(name="chains_step", kind="chains", search="split", chains=256, layers=15, lambdas=151, n_c=9501),
        # the whole (wavelength, velocity) plane of a site, signs and log-determinants
        dict(name="sign_map", kind="sign_map", layers=20, lambdas=300, n_c=11501),
        # modes and poles among a batch's picks
        dict(name="classify_picks", kind="classify", models=512, n_c=19001),
        # requests that arrive together at the server, to the last result
        dict(name="serve_burst", kind="serve", search="split", requests=64, n_c=9501),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["curve", "curve", "curve", "batch", "batch", "chains", "sign_map", "classify", "serve"])
    search = rng.choice(sorted(SEARCH))
    if kind == "curve":
        return dict(kind=kind, search=search, host=rng.random() < 0.25, layers=_log_int(rng, 1, 30),
                    lambdas=_log_int(rng, 10, 1000), lam_hi=round(rng.uniform(30.0, 100.0), 1), c_lo=50.0,
                    c_hi=1200.0, n_c=_log_int(rng, 301, 115001))
    if kind == "batch":
        return dict(kind=kind, search=search, models=_log_int(rng, 16, 2048), n_c=_log_int(rng, 1901, 19001))
    if kind == "chains":
        return dict(kind=kind, search=search, chains=_log_int(rng, 16, 400), layers=rng.randint(3, 25),
                    lambdas=rng.randint(30, 300), n_c=_log_int(rng, 1901, 9501))
    if kind == "sign_map":
        return dict(kind=kind, layers=_log_int(rng, 2, 30), lambdas=_log_int(rng, 40, 500),
                    n_c=_log_int(rng, 501, 11501))
    if kind == "classify":
        return dict(kind=kind, models=_log_int(rng, 8, 512), n_c=_log_int(rng, 1901, 19001))
    return dict(kind=kind, search=search, requests=rng.randint(2, 64), n_c=_log_int(rng, 1901, 9501))


# ---------------------------------------------------------------- inputs --
def _profiles(rng, n_layers, slower=0.15, poisson=True):
    """Velocity-increasing profiles, flattened as the batch call takes them:
    h ~ U(0.5, 3) m, beta from U(100, 200) m/s by U(5, 40) a layer, the
    half-space 100 m/s above the last layer, about `slower` of the models
    with one layer at 0.6 to 0.9 of the one above it."""
    n_layers = np.asarray(n_layers)
    m, n_max = len(n_layers), int(n_layers.max())
    j = np.arange(n_max + 1)
    finite = j[None, :n_max] < n_layers[:, None]
    record = j[None, :] <= n_layers[:, None]
    h = rng.uniform(0.5, 3.0, (m, n_max))
    step = np.where(j[None, :] == n_layers[:, None], 100.0, rng.uniform(5.0, 40.0, (m, n_max + 1)))
    step[:, 0] = np.where(n_layers == 0, 100.0, 0.0)
    beta = rng.uniform(100.0, 200.0, (m, 1)) + np.cumsum(step, axis=1)
    ratio = np.full((m, n_max + 1), math.sqrt(3.0))
    if poisson:
        nu = rng.uniform(0.25, 0.4, (m, n_max + 1))
        ratio = np.sqrt((2.0 - 2.0 * nu) / (1.0 - 2.0 * nu))
    u, v, f = rng.uniform(size=m), rng.uniform(size=m), rng.uniform(0.6, 0.9, m)
    for i in np.nonzero((u < slower) & (n_layers > 1))[0]:
        k = 1 + int(v[i] * (n_layers[i] - 1))
        beta[i, k] = beta[i, k - 1] * f[i]
    rho = rng.uniform(1700.0, 2200.0, (m, n_max + 1))
    off = np.zeros(m + 1, np.int32)
    off[1:] = np.cumsum(n_layers)
    return off, h[finite], (ratio * beta)[record], beta[record], rho[record]


def _wavelengths(counts, lo, hi):
    """Log-spaced wavelengths lo..hi of every model, flattened."""
    counts = np.asarray(counts)
    off = np.zeros(len(counts) + 1, np.int32)
    off[1:] = np.cumsum(counts)
    i = np.arange(off[-1]) - np.repeat(off[:-1], counts)
    return off, lo * (hi / lo) ** (i / np.repeat(np.maximum(counts - 1, 1), counts))


def _arrays(case, seed):
    """Host arrays of a case: c_test and the flattened models and wavelengths."""
    kind = case["kind"]
    sizes = np.random.default_rng([7, case["n_c"], case.get("models", 0), case.get("requests", 0)])
    rng = np.random.default_rng([11, int(seed)])
    c_lo, c_hi = case.get("c_lo", 50.0), case.get("c_hi", 1000.0)
    c = c_lo + (c_hi - c_lo) / (case["n_c"] - 1) * np.arange(case["n_c"])
    if kind in ("curve", "sign_map"):
        models = _profiles(rng, [case["layers"]], slower=0.0)
        lams = _wavelengths([case["lambdas"]], 1.0, case.get("lam_hi", 100.0))
    elif kind in ("batch", "classify"):
        n = case["models"]
        models = _profiles(rng, sizes.integers(3, 31, n))
        lams = _wavelengths(sizes.integers(50, 501, n), 1.0, 80.0)
    elif kind == "chains":
        # perturbed copies of one site
        n, N = case["chains"], case["layers"]
        _, h, _, beta, rho = _profiles(rng, [N], slower=0.0, poisson=False)
        h = (h * (1.0 + 0.02 * rng.standard_normal((n, N)))).ravel()
        beta = (beta * (1.0 + 0.02 * rng.standard_normal((n, N + 1)))).ravel()
        models = (np.arange(n + 1, dtype=np.int32) * N, h, math.sqrt(3.0) * beta, beta, np.tile(rho, n))
        lams = _wavelengths([case["lambdas"]] * n, 1.0, 40.0)
    else:  # serve
        n = case["requests"]
        models = _profiles(rng, sizes.integers(5, 26, n), slower=0.0, poisson=False)
        lams = _wavelengths(sizes.integers(30, 301, n), 1.0, 40.0)
    return (c,) + models + lams


class _Session:
    """A context that is given back with its last user (and any server on it stopped)."""

    def __init__(self, budget):
        self.ctx = M.masw_create(0, budget)
        self._close = weakref.finalize(self, M.masw_destroy, self.ctx)


def _dev(x):
    return torch.as_tensor(x, device="cuda")


def _outputs(w, c_ref=True):
    e = lambda t: torch.empty(w, dtype=t, device="cuda")
    return {"c_t": e(torch.float64), "idx": e(torch.int32), "status": e(torch.int32),
            "c_ref": e(torch.float64) if c_ref else None}


def prepare(case, seed):
    kind = case["kind"]
    c, layer_off, h, alpha, beta, rho, lambda_off, lam = _arrays(case, seed)
    prec, flags = SEARCH[case.get("search", "walk")]
    w = len(lam)
    s = {"kind": kind, "session": _Session((96 << 20) + 256 * w + 64 * case["n_c"])}
    ctx = s["session"].ctx
    if kind == "curve" and case["host"]:
        s["args"] = (c, lam, h, alpha, beta, rho, prec, flags, None)
        s["w"] = w
        return s
    if kind == "serve":
        s["out"] = {"c_t": np.empty(w), "idx": np.empty(w, np.int32), "status": np.empty(w, np.int32),
                    "c_ref": np.empty(w)}
        s["requests"] = []
        for i in range(case["requests"]):
            lo, hi, a, b = layer_off[i], layer_off[i + 1], lambda_off[i], lambda_off[i + 1]
            r = slice(lo + i, hi + i + 1)
            s["requests"].append(((c, lam[a:b], h[lo:hi], alpha[r], beta[r], rho[r], prec),
                                  tuple(v[a:b] for v in s["out"].values())))
        M.masw_server_start(ctx, search_inertia=int(case["search"] == "inertia"), pool_bytes=48 << 20)
        return s
    c, layer_off, h, alpha, beta, rho, lambda_off, lam = map(_dev, (c, layer_off, h, alpha, beta, rho, lambda_off, lam))
    batch = (c, layer_off, h, alpha, beta, rho, lambda_off, lam)
    if kind == "curve":
        s["out"] = _outputs(w)
        s["call"] = M.PreparedCurve(ctx, c, lam, h, alpha, beta, rho, prec, flags, None, *s["out"].values())
    elif kind == "sign_map":
        cells = w * case["n_c"]
        s["out"] = {"sigma": torch.empty(cells, dtype=torch.int8, device="cuda"),
                    "log_abs_det": torch.empty(cells, dtype=torch.float64, device="cuda")}
        s["call"] = M.PreparedSignMap(ctx, c, lam, h, alpha, beta, rho, prec, 0, None, *s["out"].values())
    elif kind == "classify":
        # the picks to be classified, as the program that found them holds them
        found = _outputs(w, c_ref=False)
        M.masw_dispersion_batch(ctx, *batch, M.MASW_PREC_FP64, M.MASW_SEARCH_INERTIA | M.MASW_NO_REFINE, None,
                                *found.values())
        s["out"] = {"pick_class": torch.empty(w, dtype=torch.int32, device="cuda"),
                    "c_sec": torch.empty(w, dtype=torch.float64, device="cuda")}
        s["args"] = batch + (found["idx"], 0, None)
    elif kind == "chains":
        s["out"] = _outputs(w, c_ref=False)
        s["out"]["misfit"] = torch.empty(case["chains"], dtype=torch.float64, device="cuda")
        measured = 150.0 + 2.0 * lam  # an experimental curve of the same wavelengths
        s["args"] = batch + (prec, flags | M.MASW_NO_REFINE, None)
        s["measured"] = measured
    else:
        s["out"] = _outputs(w)
        s["args"] = batch + (prec, flags, None)
    return s


def run(s):
    kind, ctx = s["kind"], s["session"].ctx
    if kind in ("curve", "sign_map"):
        if "call" in s:
            s["call"]()
        else:
            w = s["w"]
            out = {"c_t": np.empty(w), "idx": np.empty(w, np.int32), "status": np.empty(w, np.int32),
                   "c_ref": np.empty(w)}
            M.masw_dispersion_curve(ctx, *s["args"], *out.values())
            return out
    elif kind == "batch":
        M.masw_dispersion_batch(ctx, *s["args"], *s["out"].values())
    elif kind == "chains":
        o = s["out"]
        M.masw_dispersion_batch_misfit(ctx, *s["args"], o["c_t"], o["idx"], o["status"], None, s["measured"],
                                       o["misfit"])
    elif kind == "classify":
        M.masw_classify_picks(ctx, *s["args"], *s["out"].values())
    else:
        tickets = [M.masw_submit(ctx, *args) for args, _ in s["requests"]]
        for t, (_, out) in zip(tickets, s["requests"]):
            M.masw_wait(ctx, t, -1, *out)
    return s["out"]


# ------------------------------------------------------------------ work --
def _depth(c, layer_off, beta, h, lambda_off, lam):
    """Grid points up to each pick, taking it at 0.9 beta of the layer at a third of a wavelength."""
    w = np.diff(lambda_off)
    n = np.diff(layer_off)
    out = np.empty(len(lam))
    for m in range(len(n)):
        z = np.cumsum(h[layer_off[m]:layer_off[m + 1]])
        b = beta[layer_off[m] + m:layer_off[m + 1] + m + 1]
        l = slice(lambda_off[m], lambda_off[m] + w[m])
        out[l] = np.searchsorted(c, 0.9 * b[np.searchsorted(z, lam[l] / 3.0)])
    return np.minimum(out + 1, len(c))


def work(case):
    """Inputs read once and outputs written once; determinant evaluations at
    101 operations a layer and 48 for the half-space, every grid point up to
    the pick where the search walks, else one bisection's worth of them."""
    kind = case["kind"]
    c, layer_off, h, alpha, beta, rho, lambda_off, lam = _arrays(case, 0)
    n, w = np.diff(layer_off), len(lam)
    per_eval = np.repeat(101.0 * n + 48.0, np.diff(lambda_off))
    read = 8.0 * (len(c) + len(h) + 3 * len(alpha) + w) + 4.0 * 2 * len(layer_off)
    if kind == "sign_map":
        cells = float(w) * len(c)
        return {"bytes": read + 9.0 * cells, "flops": float(per_eval[0]) * cells}
    if kind == "classify":
        # both ends of the bracket, and a root to 1e-12 of a grid step's 1e-3 by a third-order method
        return {"bytes": read + 4.0 * w + 12.0 * w, "flops": 6.0 * float(per_eval.sum())}
    refine = 0.0 if kind == "chains" else 4.0
    if case["search"] == "inertia":
        evals = np.full(w, math.log2(len(c)) + refine)
    else:
        evals = _depth(c, layer_off, beta, h, lambda_off, lam) + refine
    written = 16.0 * w + (8.0 * w if refine else 8.0 * len(n))
    return {"bytes": read + written, "flops": float((evals * per_eval).sum())}


# ----------------------------------------------------------------- exact --
# Plain torch in 64 bits: the element matrices of the stiffness method and
# the determinant by eliminating 2x2 blocks from the top layer down, one
# (model, wavelength, velocity) an entry of every tensor.
class _Plain:
    def __init__(self, layer_off, h, alpha, beta, rho):
        dev = "cuda" if torch.cuda.is_available() else "cpu"
        self.dev = dev
        n = np.diff(layer_off)
        m, n_max = len(n), int(n.max())
        pad = lambda: np.ones((n_max + 1, m))
        H, A, B, R = pad(), pad(), pad(), pad()
        for i in range(m):
            lo, hi = layer_off[i], layer_off[i + 1]
            H[:n[i], i] = h[lo:hi]
            r = slice(lo + i, hi + i + 1)
            A[:n[i] + 1, i], B[:n[i] + 1, i], R[:n[i] + 1, i] = alpha[r], beta[r], rho[r]
        t = lambda x: torch.as_tensor(x, dtype=torch.float64, device=dev)
        self.h, self.a, self.b, self.r, self.n = t(H), t(A), t(B), t(R), torch.as_tensor(n, device=dev)
        self.n_max, self.uniform = n_max, bool((n == n[0]).all())

    def det(self, model, k, c):
        """sign(Re det K), ln|det K| and the sign of the product of the layers'
        denominators at wavenumbers k and velocities c of `model`."""
        c2 = c * c
        n = self.n[model]
        last = (n, model)
        mu_ref = self.r[last] * self.b[last] ** 2
        s11 = s12 = s22 = torch.zeros_like(c)
        sign, poles, log = torch.ones_like(c), torch.ones_like(c), 2.0 * (n + 1) * torch.log(k * mu_ref)
        for j in range(self.n_max):
            a, b, rho = self.a[j, model], self.b[j, model], self.r[j, model]
            t = k * self.h[j, model]
            xr, xs = 1.0 - c2 / (a * a), 1.0 - c2 / (b * b)
            Er, ar, Sr, Rr = self.terms(xr, t)
            Es, as_, Ss, Rs = self.terms(xs, t)
            Cr, Cs = Er + ar, Es + as_
            u = Er * as_ + ar * Es + ar * as_
            D = Sr * Ss + Rr * Rs - 2.0 * u
            F = rho * c2 / mu_ref / D
            m = rho * b * b / mu_ref
            k11, k22 = F * (Cr * Ss - Rr * Cs), F * (Sr * Cs - Rs * Cr)
            k12 = F * (u - Rr * Rs) - m * (1.0 + xs)
            k13, k14, k24 = F * (Rr * Es - Ss * Er), F * (as_ * Er - ar * Es), F * (Rs * Er - Sr * Es)
            p11, p12, p22 = s11 + k11, s12 + k12, s22 + k22
            d = p11 * p22 - p12 * p12
            w11, w12 = p22 * k13 + p12 * k14, p22 * k14 - p12 * k24
            w21, w22 = -p11 * k14 - p12 * k13, p11 * k24 - p12 * k14
            q11 = k11 - (k13 * w11 - k14 * w21) / d
            q12 = -k12 - (k13 * w12 - k14 * w22) / d
            q22 = k22 - (k14 * w12 + k24 * w22) / d
            dl = torch.log(d.abs())
            if self.uniform:
                s11, s12, s22 = q11, q12, q22
                sign, poles, log = sign * torch.sign(d), poles * torch.sign(D), log + dl
            else:
                on = j < n
                s11, s12, s22 = (torch.where(on, q, s) for q, s in ((q11, s11), (q12, s12), (q22, s22)))
                sign = torch.where(on, sign * torch.sign(d), sign)
                poles = torch.where(on, poles * torch.sign(D), poles)
                log = torch.where(on, log + dl, log)
        xr = (1.0 - c2 / self.a[last] ** 2).to(torch.complex128)
        xs = (1.0 - c2 / self.b[last] ** 2).to(torch.complex128)
        r, s = torch.sqrt(xr), torch.sqrt(xs)
        z = (c2 / self.b[last] ** 2) / (1.0 - r * s)
        det = (s11 + z * r) * (s22 + z * s) - (s12 + z - 2.0) ** 2
        return sign * torch.sign(det.real), log + torch.log(det.abs()), poles

    @staticmethod
    def terms(x, t):
        """E, E (cosh tq - 1), E sinh(tq)/q, E q sinh(tq) for q = sqrt(x), with E = exp(-t Re q)."""
        q = torch.sqrt(x.abs())
        tq = t * q
        em = torch.expm1(-tq)
        sh = -0.5 * em * (2.0 + em)
        half = torch.sin(0.5 * tq)
        up = x > 0
        E = torch.where(up, 1.0 + em, 1.0)
        a = torch.where(up, 0.5 * em * em, -2.0 * half * half)
        sn = torch.where(up, sh, torch.sin(tq))
        S = torch.where(q > 0, sn / torch.where(q > 0, q, 1.0), t)
        return E, a, S, x * S

    def first_change(self, model, k, c, cells=1 << 21):
        """Index of the first sign change along c of every wavelength (-1: none)."""
        found = torch.full_like(model, -1)
        left = torch.arange(len(model), device=self.dev)
        at, carry = 0, None
        while at < len(c) and len(left):
            n = max(2, min(len(c) - at, cells // len(left)))
            cc = c[at:at + n]
            g = self.det(model[left].repeat_interleave(len(cc)), k[left].repeat_interleave(len(cc)),
                         cc.repeat(len(left)))[0].reshape(len(left), -1)
            prev = torch.cat([g[:, :1] if carry is None else carry[:, None], g[:, :-1]], 1)
            change = g != prev
            hit = change.any(1)
            found[left[hit]] = (at + change.to(torch.int8).argmax(1))[hit]
            left, carry = left[~hit], g[~hit, -1]
            at += len(cc)
        return found

    def root(self, model, k, lo, hi):
        """The sign change of det K in [lo, hi], bisected to the last bits."""
        s = self.det(model, k, lo)[0]
        for _ in range(46):
            mid = 0.5 * (lo + hi)
            same = self.det(model, k, mid)[0] == s
            lo, hi = torch.where(same, mid, lo), torch.where(same, hi, mid)
        return 0.5 * (lo + hi)


def exact(case, seed):
    kind = case["kind"]
    c, layer_off, h, alpha, beta, rho, lambda_off, lam = _arrays(case, seed)
    p = _Plain(layer_off, h, alpha, beta, rho)
    t = lambda x: torch.as_tensor(x, device=p.dev)
    model = t(np.repeat(np.arange(len(layer_off) - 1), np.diff(lambda_off)))
    k, c = 2.0 * math.pi / t(lam), t(c)
    if kind == "sign_map":
        log = torch.empty(len(lam) * len(c), dtype=torch.float64, device=p.dev)
        rows = max(1, (1 << 21) // len(c))
        for i in range(0, len(lam), rows):
            m = model[i:i + rows]
            log[i * len(c):(i + len(m)) * len(c)] = p.det(m.repeat_interleave(len(c)),
                                                         k[i:i + rows].repeat_interleave(len(c)), c.repeat(len(m)))[1]
        return {"sigma": None, "log_abs_det": log}
    depth = float(_depth(c.cpu().numpy(), layer_off, beta, h, lambda_off, lam).sum())
    if depth * p.n_max > 1.5e10:
        return None
    idx = p.first_change(model, k, c)
    ok = idx > 0
    nan = torch.full((len(lam),), math.nan, dtype=torch.float64, device=p.dev)
    i, mo, kk = idx[ok], model[ok], k[ok]
    c_t = nan.clone()
    c_t[ok] = c[i]
    if kind == "chains":
        e = 150.0 + 2.0 * t(lam)
        mis = torch.zeros(case["chains"], dtype=torch.float64, device=p.dev)
        mis.index_add_(0, model, (c_t - e).abs() / e)
        return {"c_t": c_t, "idx": idx.to(torch.int32), "status": None, "c_ref": None,
                "misfit": mis / case["lambdas"]}
    c_ref = nan.clone()
    c_ref[ok] = p.root(mo, kk, c[i - 1], c[i])
    if kind == "classify":
        # no root where a pole changes the sign, nor at or above the half-space's beta
        lo, hi = p.det(mo, kk, c[i - 1]), p.det(mo, kk, c[i])
        mode = (lo[0] * lo[2] != hi[0] * hi[2]) & (c[i] < p.b[p.n[mo], mo])
        c_ref[ok] = torch.where(mode, c_ref[ok], nan[ok])
        return {"pick_class": None, "c_sec": c_ref}
    return {"c_t": c_t, "idx": idx.to(torch.int32), "status": None, "c_ref": c_ref}
