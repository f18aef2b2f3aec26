"""The calls that a user of this library makes, as measurable cases.

Each case is one pass through the public Python entry points on data that is
already on the GPU.  The shapes are the library's own workloads (10,000 x 16,
K = 8; 1e5 to 1e8 points of 128 dimensions, K = 1024; unit-normalised vectors
of 768 dimensions, K = 4096) and sizes around them: widths that are no
multiple of the kernels' tiles, the 96 and 100 dimensions of common embedding
sets, a width between the two screening layouts, and the small batches in
which an index takes in new vectors.

Data: a seeded mixture of diagonal Gaussians (means ~ N(0, 4), per-dimension
standard deviations ~ U[0.5, 1.5], Dirichlet(1) weights), drawn on the GPU;
"norm" scales every row to unit length, as embeddings are.  Parameters:
"stage" 0 is the random-point initialisation (distinct rows as means, the
data's variance per dimension, equal weights), where the components are broad
and a point meets many of them; stage t > 0 are the parameters after t EM
iterations on the first `fit_rows` rows, done here in plain torch in fp64, so
that some components are split, some merged and some sit on few points, as in
a fit.
"""
from __future__ import annotations

import math

import torch

import paper_2606_10896_amd as gmm

DEV = "cuda"
FLOOR = 1e-6

# ops: "em"      one E-step into fp64 statistics (diagonal model)
#      "em_iso"  the same for the isotropic model
#      "fit"     gmm_fit, "fit_iso" gmm_fit_iso: `iters` EM iterations
#      "assign"  gmm_assign_topk with m ranks and the threshold tau = 1 / k
#      "kmeans"  gmm_kmeans, `iters` Lloyd iterations (the warm start)
#      "kmeanspp" gmm_kmeanspp, k centres


def _case(op, n, d, k, k_true, stage=0, fit_rows=0, iters=0, m=0, norm=False, name=None):
    c = {"op": op, "n": n, "d": d, "k": k, "k_true": k_true, "stage": stage,
         "fit_rows": fit_rows, "iters": iters, "m": m, "norm": norm}
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # new vectors taken into an index of 1024 cells, a small batch at a time: latency
        _case("assign", 1000, 128, 1024, 1024, stage=5, fit_rows=131072, m=2,
              name="assign_batch"),
        # the tiny workload whole: ten iterations of almost nothing but launches
        _case("fit", 10_000, 16, 8, 8, iters=10, name="fit_tiny"),
        # the small workload's fit from its initialisation, first iterations
        _case("fit", 100_000, 128, 1024, 1024, iters=6, name="fit_small"),
        # the paper's own model on 96-dimensional vectors, a fit's first iterations
        _case("fit_iso", 1_000_000, 96, 1024, 1024, iters=6, name="fit_iso"),
        # first E-step of a fit on a 100-dimensional embedding set of odd size: broad components
        _case("em", 1_183_514, 100, 1024, 1024, name="em_first"),
        # an E-step of the mid workload in the course of its fit
        _case("em", 1_000_000, 128, 1024, 1024, stage=6, fit_rows=262144, name="em_mid"),
        # an E-step of the large workload in the course of its fit
        _case("em", 100_000_000, 128, 1024, 1024, stage=6, fit_rows=1048576, name="em_large"),
        # a width between the two screening layouts, not a multiple of 64
        _case("em", 500_000, 200, 512, 512, stage=4, fit_rows=131072, name="em_d200"),
        # the coarse-quantizer shape: unit vectors, twice as many true clusters as cells
        _case("em", 1_000_000, 768, 4096, 8192, stage=3, fit_rows=262144, norm=True,
              name="em_ivf"),
        # multi-assignment of every vector of that index after its fit
        _case("assign", 1_000_000, 768, 4096, 8192, stage=3, fit_rows=262144, m=2, norm=True,
              name="assign_ivf"),
        # the k-means warm start of the mid workload
        _case("kmeans", 1_000_000, 128, 1024, 1024, iters=4, name="kmeans_mid"),
        # k-means++ seeding of the mid workload, a quarter of its centres
        _case("kmeanspp", 1_000_000, 128, 256, 1024, name="kmeanspp_mid"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any of the listed calls, sizes between and around the listed ones."""
    op = rng.choice(["assign", "assign", "fit", "fit", "fit_iso", "em", "em", "em", "em_iso",
                     "kmeans", "kmeanspp"])
    wide = op in ("em", "assign") and rng.random() < 0.3
    if wide:
        d, k, n = rng.randint(257, 800), _log(rng, 200, 4096), _log(rng, 2000, 600_000)
    else:
        d, k = rng.choice([rng.randint(8, 64), rng.randint(65, 128), 128, 96, 100,
                           rng.randint(129, 256)]), _log(rng, 8, 2048)
        n = {"assign": _log(rng, 100, 4_000_000), "fit": _log(rng, 5000, 500_000),
             "fit_iso": _log(rng, 5000, 1_000_000), "em": _log(rng, 5000, 10_000_000),
             "em_iso": _log(rng, 5000, 4_000_000), "kmeans": _log(rng, 5000, 2_000_000),
             "kmeanspp": _log(rng, 20_000, 2_000_000)}[op]
    iters = rng.randint(2, 6) if op in ("fit", "fit_iso", "kmeans") else 0
    # no larger a job than the largest listed one
    n = min(n, int(1e12 / (k * max(d, 64) * max(1, iters))))
    norm = wide and rng.random() < 0.7
    kt = k if rng.random() < 0.7 else 2 * k
    stage = rng.choice([0, 2, 5]) if op == "em" else 4 if op in ("assign", "em_iso") else 0
    rows = min(262144 if k <= 2048 and not wide else 131072, max(64 * k, 8192)) if stage else 0
    if op in ("fit", "fit_iso", "kmeans", "kmeanspp", "em"):
        n = max(n, 8 * k)
    return _case(op, n, d, k, kt, stage=stage, fit_rows=rows,
                 iters=iters, m=min(k, rng.choice([1, 2, 2, 4, 8])) if op == "assign" else 0,
                 norm=norm)


# ------------------------------------------------------------------ inputs

def _rows(g, n, d, mix, norm):
    """n rows of the mixture (means, stds, cumulative weights), fp32."""
    mu, sd, cum = mix
    x = torch.empty(n, d, dtype=torch.float32, device=DEV)
    step = max(1, (1 << 27) // d)
    for a in range(0, n, step):
        b = min(n, a + step)
        comp = torch.searchsorted(cum, torch.rand(b - a, generator=g, device=DEV))
        comp.clamp_(max=cum.numel() - 1)
        v = x[a:b]
        v.normal_(generator=g)
        v.mul_(sd.index_select(0, comp)).add_(mu.index_select(0, comp))
        if norm:
            v.div_(torch.linalg.vector_norm(v, dim=1, keepdim=True))
    return x


def _logd(x, w, mu, var):
    """log pi_k + log N(x | mu_k, diag var_k), every argument fp64."""
    iv = 1.0 / var
    c = torch.log(w) - 0.5 * (mu * mu * iv + torch.log(2.0 * math.pi * var)).sum(1)
    return torch.addmm(torch.addmm(c, x, (mu * iv).t()), x * x, (-0.5 * iv).t())


def _estep(x, w, mu, var):
    """Statistics and log-likelihood of x at (w, mu, var), plain fp64."""
    k, d = mu.shape
    w, mu, var = w.double(), mu.double(), var.double()
    nk = torch.zeros(k, dtype=torch.float64, device=DEV)
    s, q = (torch.zeros(k, d, dtype=torch.float64, device=DEV) for _ in range(2))
    ll = torch.zeros(1, dtype=torch.float64, device=DEV)
    step = max(1, min(x.shape[0], (1 << 28) // k))
    for a in range(0, x.shape[0], step):
        xx = x[a:a + step].double()
        l = _logd(xx, w, mu, var)
        z = torch.logsumexp(l, 1, keepdim=True)
        r = l.sub_(z).exp_()
        ll += z.sum()
        nk += r.sum(0)
        s += r.t() @ xx
        q += r.t() @ (xx * xx)
    return nk, s, q, ll


def _mstep(nk, s, q, n, w, mu, var):
    m = s / nk[:, None]
    v = (q / nk[:, None] - m * m).clamp_(min=FLOOR)
    dead = (nk == 0)[:, None]
    return ((nk / n).float(), torch.where(dead, mu.double(), m).float(),
            torch.where(dead, var.double(), v).float())


def _mstep_iso(nk, s, q, n, w, mu, var):
    m = s / nk[:, None]
    v = ((q.sum(1) / nk - (m * m).sum(1)) / mu.shape[1]).clamp_(min=FLOOR)
    dead = nk == 0
    return ((nk / n).float(), torch.where(dead[:, None], mu.double(), m).float(),
            torch.where(dead, var.double(), v).float())


def _inputs(case, seed):
    """(x, weights, means, vars, u): the data, the parameters before the call (isotropic
    calls: one variance per component) and k uniforms, from the seed alone."""
    n, d, k, kt = case["n"], case["d"], case["k"], case["k_true"]
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1000003 + n * 31 + d * 7 + k)
    mix = (2.0 * torch.randn(kt, d, generator=g, device=DEV),
           0.5 + torch.rand(kt, d, generator=g, device=DEV),
           torch.cumsum(torch.empty(kt, device=DEV).exponential_(generator=g).double(), 0))
    mix = (mix[0], mix[1], (mix[2] / mix[2][-1]).float())
    rows = case["fit_rows"]
    iso = case["op"] in ("em_iso", "fit_iso")
    x = _rows(g, n, d, mix, case["norm"])
    # the rows the parameters come from: the data's first ones, or, for calls with little
    # data of their own (a batch to assign), rows of the same mixture
    xf = x[:max(rows, min(n, 131072))] if n >= max(rows, 8 * k) else _rows(
        g, max(rows, 8 * k), d, mix, case["norm"])
    pick = torch.randperm(xf.shape[0], generator=g, device=DEV)[:k]
    w = torch.full((k,), 1.0 / k, device=DEV)
    mu = xf[pick].clone()
    var = xf.double().var(0, unbiased=False).float()
    var = var.mean().repeat(k) if iso else var.expand(k, d).contiguous()
    for _ in range(case["stage"]):
        full = var[:, None].expand(k, d) if iso else var
        nk, s, q, _ = _estep(xf, w, mu, full)
        w, mu, var = (_mstep_iso if iso else _mstep)(nk, s, q, xf.shape[0], w, mu, var)
    u = torch.rand(k, generator=g, device=DEV, dtype=torch.float64)
    return x, w, mu, var, u


def prepare(case, seed):
    n, d, k, op = case["n"], case["d"], case["k"], case["op"]
    x, w, mu, var, u = _inputs(case, seed)
    st = {"case": case, "x": x, "w": w, "mu": mu, "var": var}
    f64 = dict(dtype=torch.float64, device=DEV)
    if op == "kmeanspp":
        st.update(u=u, idx=torch.empty(k, dtype=torch.int64, device=DEV),
                  centers=torch.empty(k, d, device=DEV),
                  ws=torch.empty(gmm.load_library().gmm_kmeanspp_workspace_bytes(n),
                                 dtype=torch.uint8, device=DEV))
        return st
    st["ws"] = gmm.workspace(n, d, k, {"assign": case["m"], "kmeans": 1}.get(op, 0))
    if op in ("em", "em_iso"):
        st.update(nk=torch.empty(k, **f64), s=torch.empty(k, d, **f64),
                  q=torch.empty((k,) if op == "em_iso" else (k, d), **f64),
                  ll=torch.empty(1, **f64))
    elif op == "assign":
        st.update(idx=torch.empty(n, case["m"], dtype=torch.int32, device=DEV),
                  resp=torch.empty(n, case["m"], device=DEV))
    else:
        # the parameters that the call updates in place
        st.update(w1=w.clone(), mu1=mu.clone(), var1=var.clone())
        if op == "kmeans":
            st["assign"] = torch.empty(n, dtype=torch.int32, device=DEV)
        else:
            st["hist"] = torch.empty(case["iters"], **f64)
    return st


# ------------------------------------------------------------------ one pass

def run(st):
    case, x = st["case"], st["x"]
    op = case["op"]
    if op in ("em", "em_iso"):
        for t in (st["nk"], st["s"], st["q"], st["ll"]):
            t.zero_()
        fn = gmm.gmm_estep_accumulate if op == "em" else gmm.gmm_estep_accumulate_iso
        fn(x, st["w"], st["mu"], st["var"], st["nk"], st["s"], st["q"], st["ll"], st["ws"])
        return {"nk": st["nk"], "s": st["s"], "q": st["q"], "ll": st["ll"]}
    if op == "assign":
        gmm.gmm_assign_topk(x, st["w"], st["mu"], st["var"], case["m"], 1.0 / case["k"],
                            st["idx"], st["resp"], st["ws"])
        return {"idx": st["idx"], "resp": st["resp"]}
    if op == "kmeanspp":
        gmm.gmm_kmeanspp(x, st["u"], st["idx"], st["centers"], st["ws"])
        return {"idx": st["idx"], "centers": st["centers"]}
    # the call starts from the same parameters each time
    st["w1"].copy_(st["w"])
    st["mu1"].copy_(st["mu"])
    st["var1"].copy_(st["var"])
    if op == "kmeans":
        gmm.gmm_kmeans(x, st["w1"], st["mu1"], st["var1"], case["iters"], st["assign"], st["ws"],
                       var_floor=FLOOR)
        return {"w": st["w1"], "mu": st["mu1"], "var": st["var1"], "assign": st["assign"]}
    fn = gmm.gmm_fit if op == "fit" else gmm.gmm_fit_iso
    fn(x, st["w1"], st["mu1"], st["var1"], case["iters"], st["hist"], st["ws"], var_floor=FLOOR)
    return {"w": st["w1"], "mu": st["mu1"], "var": st["var1"], "hist": st["hist"]}


# ------------------------------------------------------------------ what a pass needs

def work(case):
    """Every point meets every component once (the log-densities; for k-means the inner
    products) and enters the statistics of at least one; the data is read once per scan that
    has to follow another's result."""
    n, d, k, op = case["n"], case["d"], case["k"], case["op"]
    x, par = 4.0 * n * d, 4.0 * k * (2 * d + 1)
    if op == "kmeanspp":
        return {"bytes": x * (k - 1) + 4.0 * k * d, "flops": 3.0 * n * d * (k - 1)}
    if op == "assign":
        return {"bytes": x + par + 8.0 * n * case["m"], "flops": 4.0 * n * k * d}
    if op == "kmeans":
        scans = case["iters"] + 1
        return {"bytes": scans * x + 2 * par + 4.0 * n,
                "flops": scans * (2.0 * n * k * d + 2.0 * n * d)}
    it = case["iters"] if op.startswith("fit") else 1
    per = 2.0 * n * k * (d + 1) if op.endswith("iso") else 4.0 * n * k * d
    return {"bytes": it * (x + 3 * par), "flops": it * (per + 4.0 * n * d)}


def tolerance(case):
    """Against fp64 the calls were measured at: statistics 2e-12 (log-likelihood) to 5e-8,
    fits 4e-7 after six iterations (an iteration's rounding moves the next one's
    responsibilities), responsibilities 3e-7, k-means and k-means++ equal.  A rank whose
    responsibility meets tau to rounding may come or go ("max", "differ"), as may a
    point halfway between two centres."""
    op = case["op"]
    if op == "assign":
        return {"rel": 2e-6, "max": 5e-3, "differ": 5e-5}
    if op == "kmeans":
        return {"rel": 1e-5, "differ": 1e-4}
    if op == "kmeanspp":
        return {"rel": 1e-6, "differ": 0.0}
    if op.startswith("fit"):
        return {"rel": 2e-5}
    return {"rel": 1e-6}


# ------------------------------------------------------------------ 64-bit results

def _kmeanspp64(x, u, k):
    xs = [x[a:a + 200_000].double() for a in range(0, x.shape[0], 200_000)]
    n = x.shape[0]
    d2 = torch.full((n,), math.inf, dtype=torch.float64, device=DEV)
    idx = torch.empty(k, dtype=torch.int64, device=DEV)
    idx[0] = (u[0] * n).long().clamp(0, n - 1)
    for t in range(1, k):
        c = x[idx[t - 1]].double()
        d2 = torch.minimum(d2, torch.cat([((b - c) ** 2).sum(1) for b in xs]))
        cum = torch.cumsum(d2, 0)
        idx[t] = torch.searchsorted(cum, (u[t] * cum[-1]).reshape(1), right=True)[0].clamp(max=n - 1)
    return {"idx": idx, "centers": x[idx].double()}


def _kmeans64(x, mu, var, k, iters):
    n, d = x.shape
    for it in range(iters + 1):
        c = mu.double()
        cc = 0.5 * (c * c).sum(1)
        assign = torch.cat([(x[a:a + 100_000].double() @ c.t() - cc).argmax(1)
                            for a in range(0, n, 100_000)])
        nk = torch.bincount(assign, minlength=k).double()
        s, q = (torch.zeros(k, d, dtype=torch.float64, device=DEV) for _ in range(2))
        for a in range(0, n, 100_000):
            xx = x[a:a + 100_000].double()
            s.index_add_(0, assign[a:a + 100_000], xx)
            q.index_add_(0, assign[a:a + 100_000], xx * xx)
        if it < iters:
            mu = torch.where((nk == 0)[:, None], c, s / nk[:, None]).float()
    w, mu, var = _mstep(nk, s, q, n, None, mu, var)
    return {"w": w.double(), "mu": mu.double(), "var": var.double(), "assign": assign.int()}


def exact(case, seed):
    n, d, k, op = case["n"], case["d"], case["k"], case["op"]
    cost = 8.0 * n * k * d * max(1, case["iters"])
    if cost > 4e13:
        return None
    x, w, mu, var, u = _inputs(case, seed)
    if op == "kmeanspp":
        return _kmeanspp64(x, u, k)
    if op == "kmeans":
        return _kmeans64(x, mu, var, k, case["iters"])
    if op == "assign":
        m, idx, resp = case["m"], [], []
        step = max(1, (1 << 27) // k)
        for a in range(0, n, step):
            l = _logd(x[a:a + step].double(), w.double(), mu.double(), var.double())
            z = torch.logsumexp(l, 1, keepdim=True)
            t, i = torch.topk(l, m, dim=1)
            r = (t - z).exp_()
            keep = r > 1.0 / k
            keep[:, 0] = True
            idx.append(torch.where(keep, i, -1).int())
            resp.append(torch.where(keep, r, 0.0))
        return {"idx": torch.cat(idx), "resp": torch.cat(resp)}
    if op in ("em", "em_iso"):
        iso = op == "em_iso"
        nk, s, q, ll = _estep(x, w, mu, var[:, None].expand(k, d) if iso else var)
        return {"nk": nk, "s": s, "q": q.sum(1) if iso else q, "ll": ll}
    iso = op == "fit_iso"
    hist = []
    for _ in range(case["iters"]):
        nk, s, q, ll = _estep(x, w, mu, var[:, None].expand(k, d) if iso else var)
        hist.append(ll)
        w, mu, var = (_mstep_iso if iso else _mstep)(nk, s, q, n, w, mu, var)
    return {"w": w.double(), "mu": mu.double(), "var": var.double(), "hist": torch.cat(hist)}
