"""The one-product screening of the E-step and of the assignment (k_coarse, k_refine,
k_assign_refine and the points they hand to the two- or three-product passes) against the fp64
checker, at the edges of its tiles and of its rules: workgroups of 64 to 256 points, blocks of 16 to 64 components, widths
with and without a remainder, points with more components in reach than a list or a lane state
holds, the sample that switches the pass off, and weights near the end of the float range.  The
workspace starts as garbage, so a point that no kernel wrote would show."""
import numpy as np
import pytest

import gmm_synth as g
import gmmcheck
import oracle
from gmmcheck import (check_assign, check_params, check_params_iso, check_stats, gpu_assign,
                      gpu_estep, gpu_estep_iso, gpu_mstep, gpu_mstep_iso)

pytestmark = pytest.mark.gpu


def _dirty_ws(n, d, k):
    import torch
    import paper_2606_10896_amd as gmm
    ws = gmm.workspace(n, d, k)
    ws.fill_(0xEE)
    torch.cuda.synchronize()
    return ws


def _dirty_ws_m(n, d, k, m=1):
    import torch
    import paper_2606_10896_amd as gmm
    ws = gmm.workspace(n, d, k, m)
    ws.fill_(0xEE)
    torch.cuda.synchronize()
    return ws


def _check(x, th, label):
    n, d = x.shape
    ref = oracle.iterate(x, *th)
    st = gpu_estep(x, *th, ws=_dirty_ws(n, d, th[0].shape[0]))
    r = check_stats(st, ref, label)
    r2 = check_params(*gpu_mstep(st, float(n), *th), ref, n, label)
    print(f"  {label}: {r} {r2}", flush=True)
    return st, ref


@pytest.mark.parametrize("n,d,k", [
    (255, 64, 31), (256, 63, 32), (257, 65, 33), (513, 128, 64), (700, 127, 97),
    (128, 129, 32), (129, 192, 65), (385, 193, 40), (300, 256, 33), (1000, 7, 130),
    (300, 2, 9), (64, 1, 3), (2000, 100, 257), (129, 257, 33), (200, 384, 40), (130, 512, 17),
    (65, 640, 33), (129, 768, 64), (90, 895, 20), (70, 1024, 33),
    # whole workgroups of points (n >= 65536) instead of shared ones
    (65613, 20, 40), (65536, 128, 70), (65600, 130, 33), (65700, 250, 20), (65599, 385, 9),
    (65601, 700, 7), (65600, 1000, 5)])
def test_tile_edges(n, d, k):
    w = g.custom(f"c{n}_{d}_{k}", n, d, max(2, k // 2), k, data_seed=n * 3 + d, init_seed=k)
    x, th0 = g.make(w)
    for t, th in enumerate(oracle.fit(x, *th0, 3, keep_thetas=True)["thetas"]):
        _check(x, th, f"n{n} d{d} k{k} t{t}")


@pytest.mark.parametrize("n,d,k", [(300, 128, 1024), (300, 127, 1030), (65, 700, 300), (90, 300, 500)])
def test_many_outputs_of_few_partial_sums(n, d, k):
    """The reduction with one thread an output, outputs in a last workgroup in part."""
    w = g.custom(f"cr{n}_{d}_{k}", max(n, k), d, k // 2, k, data_seed=n + d, init_seed=k)
    x, th0 = g.make(w)
    _check(x[:n], th0, f"outputs n{n} d{d} k{k}")


@pytest.mark.parametrize("n,d,k", [(65600, 770, 97), (65573, 896, 96), (65601, 960, 33),
                                   (65536, 1024, 130)])
def test_blocks_of_the_widest_rows(n, d, k):
    """Whole workgroups above 768 dimensions through an odd and an even number of blocks of 16
    components, a last one in part."""
    w = g.custom(f"cb{n}_{d}_{k}", n, d, max(2, k // 2), k, data_seed=n * 7 + d, init_seed=k)
    x, th0 = g.make(w)
    for t, th in enumerate(oracle.fit(x, *th0, 1, keep_thetas=True)["thetas"]):
        _check(x, th, f"n{n} d{d} k{k} t{t}")
    _check_assign(x, th, 2, 1.0 / k, f"assign n{n} d{d} k{k}")


@pytest.mark.parametrize("n,d,k", [(255, 64, 33), (257, 100, 64), (700, 128, 97),
                                   (300, 190, 40), (129, 250, 32), (70, 500, 20), (40, 800, 9),
                                   (65601, 30, 20), (65600, 200, 9), (65537, 600, 5),
                                   (65540, 1000, 4)])
def test_tile_edges_isotropic(n, d, k):
    w = g.custom(f"ci{n}_{d}_{k}", n, d, max(2, k // 2), k, data_seed=n * 5 + d, init_seed=k)
    x, (wt, mu, var) = g.make(w)
    v = var.mean(axis=1).astype(np.float32)
    for t in range(3):
        ref = oracle.iso_iterate(x, wt, mu, v)
        st = gpu_estep_iso(x, wt, mu, v, ws=_dirty_ws(n, d, k))
        check_stats(st, ref, f"iso n{n} d{d} k{k} t{t}")
        check_params_iso(*gpu_mstep_iso(st, float(n), wt, mu, v), ref, n, f"iso n{n} t{t}")
        wt, mu, v = (ref[a].astype(np.float32) for a in ("weights", "means", "vars"))


def _reach(d, seed, n):
    """Clusters of 1 to 14 near-identical components, scattered over the slots."""
    rng = np.random.default_rng(seed)
    sizes = np.tile(np.arange(1, 15), 6)
    k = int(sizes.sum())
    cl = np.repeat(np.arange(sizes.size), sizes)
    order = rng.permutation(k)
    centre = rng.normal(0.0, 4.0, (sizes.size, d))
    mu = (centre[cl] + rng.normal(0.0, 0.02, (k, d)))[order].astype(np.float32)
    var = np.ones((k, d), np.float32)
    wt = rng.dirichlet(np.full(k, 5.0)).astype(np.float32)
    x = (centre[rng.integers(0, sizes.size, n)] + rng.normal(0.0, 1.0, (n, d))).astype(np.float32)
    return x, (wt, mu, var)


@pytest.mark.parametrize("d,seed", [(16, 1), (96, 2), (128, 3), (200, 4), (300, 5), (770, 6)])
def test_many_components_in_reach(d, seed):
    """Points whose candidates overflow the list, or one lane state of one lane group only."""
    x, th = _reach(d, seed, 6000)
    _check(x, th, f"reach d{d}")


def _check_assign(x, th, m, tau, label, min_checked=0.9):
    import torch
    import paper_2606_10896_amd as gmm
    n, d = x.shape
    k = th[0].shape[0]
    ws = gmm.workspace(n, d, k, m)
    ws.fill_(0xEE)
    torch.cuda.synchronize()
    ref = oracle.assign_topk(x, *th, m, tau, mr=m + 1)
    gidx, gresp = gpu_assign(x, *th, m, tau, ws=ws)
    print(f"  {label}: {check_assign(gidx, gresp, ref, m, tau, label, min_checked):.4f}", flush=True)


@pytest.mark.parametrize("n,d,k,m,tau", [
    (300, 24, 40, 2, 1 / 40), (65600, 24, 40, 3, 1 / 40), (65537, 130, 20, 8, 1e-6),
    (2000, 24, 40, 2, 1e-13), (2000, 24, 40, 1, 0.0), (65600, 260, 9, 2, 0.1),
    (700, 900, 33, 4, 1e-3), (1, 128, 9, 2, 0.1)])
def test_assignment_routes(n, d, k, m, tau):
    """Shared and whole workgroups, tau below the candidate window (2^-40), m = 1."""
    w = g.custom(f"ca{n}_{d}_{k}", max(n, k), d, k, k, data_seed=n + d, init_seed=k + 1)
    x, th0 = g.make(w)
    th = oracle.fit(x, *th0, 2, keep_thetas=True)["thetas"][-1]
    _check_assign(x[:n], th, m, tau, f"assign n{n} d{d} k{k} m{m} tau{tau}")


@pytest.mark.parametrize("n,d", [(400, 64), (6000, 64), (6000, 200), (500, 400)])
def test_assignment_of_heavy_points(n, d, monkeypatch):
    """Few heavy points (every component in fp64) and many (the two-pass screening).  There
    the normaliser keeps the screening error of the components that are no candidates, and
    with 14 near-identical ones they carry most of it: a screened responsibility is within
    2^-21 (S + d) relative, S = sum mu^2 / var of the components (the bound stated for the
    split-bf16 screening)."""
    x, th = _reach(d, 11, n)
    s = float((th[1].astype(np.float64) ** 2 / th[2]).sum(1).max())
    monkeypatch.setattr(gmmcheck, "TOL_RESP", max(gmmcheck.TOL_RESP, 2.0 ** -21 * (s + d)))
    _check_assign(x, th, 4, 1e-4, f"assign heavy n{n} d{d}", min_checked=0.5)


def _heavy(ws):
    import torch
    return int(ws[:64].view(torch.int32)[6])


@pytest.mark.parametrize("n,d,m,lo,hi", [
    (1050, 64, 2, 257, 512),          # a workgroup a point
    (2403, 64, 8, 513, 2048),       # four points a workgroup, a last one in part
    (2402, 100, 1, 513, 1536),
    (5001, 200, 3, 1537, 4096),     # more groups of four than workgroups
    (2501, 400, 2, 513, 2048),
    (9001, 64, 2, 3300, 9001),      # more than that: the two-pass screening
    (11003, 200, 2, 4097, 11003)])
def test_heavy_points_over_all_components(n, d, m, lo, hi, monkeypatch):
    """Heavy points in fp64 over every component, up to where the two passes take them.  A
    responsibility is then the fp32 rounding of an fp64 value (that of a light point: below
    k 2^-40 off); the passes keep a screening error of 2^-21 (S + d)."""
    import torch
    import paper_2606_10896_amd as gmm
    x, th = _reach(d, 23, n)
    k = th[0].shape[0]
    s = float((th[1].astype(np.float64) ** 2 / th[2]).sum(1).max())
    passes = hi == n
    monkeypatch.setattr(gmmcheck, "TOL_RESP",
                        max(gmmcheck.TOL_RESP, 2.0 ** -21 * (s + d)) if passes else 1e-6)
    ws = gmm.workspace(n, d, k, m)
    ws.fill_(0xEE)
    torch.cuda.synchronize()
    ref = oracle.assign_topk(x, *th, m, 1e-4, mr=m + 1)
    gidx, gresp = gpu_assign(x, *th, m, 1e-4, ws=ws)
    heavy = _heavy(ws)
    print(f"  heavy over all n{n} d{d} m{m}: {heavy} heavy, "
          f"{check_assign(gidx, gresp, ref, m, 1e-4, f'n{n} d{d}', 0.5):.4f}", flush=True)
    assert lo <= heavy <= hi


@pytest.mark.parametrize("n,d", [(70, 64), (601, 300), (3001, 200), (40000, 64)])
def test_heavy_points_spread_over_workgroups(n, d):
    """From one heavy point a workgroup of the passes over them to as many as it has room for."""
    x, th = _reach(d, 31, n)
    _check(x, th, f"spread n{n} d{d}")
    if n > 10000:                           # more than are done over all components
        s = float((th[1].astype(np.float64) ** 2 / th[2]).sum(1).max())
        tol = gmmcheck.TOL_RESP
        try:
            gmmcheck.TOL_RESP = max(tol, 2.0 ** -21 * (s + d))
            _check_assign(x, th, 2, 1e-4, f"spread assign n{n} d{d}", min_checked=0.5)
        finally:
            gmmcheck.TOL_RESP = tol


@pytest.mark.parametrize("n", [300, 3000])
def test_assignment_with_weights_near_the_end_of_the_float_range(n):
    w = g.custom("cx", 3000, 24, 10, 40, data_seed=8, init_seed=9)
    x, (wt, mu, var) = g.make(w)
    var = var.copy()
    var[7] = 1e-29
    _check_assign(x[:n], (wt, mu, var), 2, 1 / 40, f"assign wild n{n}")


@pytest.mark.parametrize("d,n", [(20, 32768), (128, 32768), (190, 24576), (250, 16384),
                                 (300, 16384), (500, 16384), (640, 16384), (760, 16384),
                                 (800, 8192), (1000, 8192)])
def test_shared_and_whole_workgroups_agree(d, n):
    """One row below the number from which on a workgroup's waves have points of their own, and
    that number: the same rows but one, listed by either form."""
    k = 21
    w = g.custom(f"cs{d}", n, d, 10, k, data_seed=d, init_seed=d + 1)
    x, th0 = g.make(w)
    th = oracle.fit(x[:4000], *th0, 2, keep_thetas=True)["thetas"][-1]
    a, ra = gpu_assign(x[:-1], *th, 2, 0.01, ws=_dirty_ws_m(n - 1, d, k, 2))
    b, rb = gpu_assign(x, *th, 2, 0.01, ws=_dirty_ws_m(n, d, k, 2))
    same = a == b[:-1]
    assert same.mean() > 0.9999
    # two fp32 roundings of fp64 responsibilities, normalisers k 2^-40 apart at most
    assert np.abs(ra - rb[:-1])[same].max() <= 1e-6
    _check(x[-300:], th, f"split d{d}")
    _check_assign(x[-300:], th, 2, 0.01, f"split assign d{d}")


@pytest.mark.parametrize("d,n", [(100, 32768), (190, 24576), (250, 16384), (300, 24576),
                                 (900, 24576), (1000, 8192)])
def test_shared_and_whole_workgroups_agree_isotropic(d, n):
    import torch
    import paper_2606_10896_amd as gmm
    k = 37
    w = g.custom(f"ct{d}", n, d, k, k, data_seed=d, init_seed=d + 1)
    x, (_, mu, _) = g.make(w)
    xd, md = torch.from_numpy(x).cuda(), torch.from_numpy(mu).cuda()
    m64 = mu.astype(np.float64)
    score = x.astype(np.float64) @ m64.T - 0.5 * (m64 ** 2).sum(1)
    for rows in (n - 1, n):
        wd, vd = torch.full((k,), 1.0 / k, device="cuda"), torch.ones(k, d, device="cuda")
        assign = torch.empty(rows, dtype=torch.int32, device="cuda")
        gmm.gmm_kmeans(xd[:rows], wd, md.clone(), vd, 0, assign, _dirty_ws_m(rows, d, k))
        assert (assign.cpu().numpy() == score[:rows].argmax(1)).all(), rows


@pytest.mark.parametrize("n,d,k", [(65600, 20, 33), (900, 300, 20)])
def test_kmeans_through_the_screening(n, d, k):
    import torch
    import paper_2606_10896_amd as gmm
    w = g.custom(f"ck{n}", n, d, k, k, data_seed=n, init_seed=k)
    x, (wt, mu, var) = g.make(w)
    ref = oracle.kmeans(x, mu, var, 3)
    xd, wd, md, vd = (torch.from_numpy(a.copy()).cuda() for a in (x, wt, mu, var))
    assign = torch.empty(n, dtype=torch.int32, device="cuda")
    gmm.gmm_kmeans(xd, wd, md, vd, 3, assign, _dirty_ws_m(n, d, k))
    same = (assign.cpu().numpy() == ref["assign"]).mean()
    print(f"  k-means n{n}: assignment equal {same:.6f}", flush=True)
    assert same >= 0.9999
    np.testing.assert_allclose(md.cpu().numpy(), ref["means"], rtol=1e-4, atol=1e-4)
    np.testing.assert_allclose(wd.cpu().numpy(), ref["weights"], rtol=1e-3, atol=2.0 / n)


@pytest.mark.parametrize("scale", [1e-3, 0.05, 1.0])
def test_kmeans_of_rows_of_any_scale(scale):
    """Wide rows whose squared distances (8e-3 between centres at scale 1e-3) are small beside
    the constant that all centres share, 0.5 d log(2 pi) + log k: the bound that dismisses a
    centre may not be made of that constant.  Every assignment is the fp64 nearest centre, and
    no point is left to the passes for points with many candidates (their number is the seventh
    counter at the workspace's start)."""
    import torch
    import paper_2606_10896_amd as gmm
    rng = np.random.default_rng(17)
    n, d, k = 4000, 1000, 64
    c = rng.normal(0.0, 2.0, (k, d))
    x = (scale * (c[rng.integers(0, k, n)] + rng.normal(0.0, 1.0, (n, d)))).astype(np.float32)
    mu = (scale * (c + rng.normal(0.0, 0.2, (k, d)))).astype(np.float32)
    xd, md = (torch.from_numpy(a).cuda() for a in (x, mu))
    wd, vd = torch.full((k,), 1.0 / k, device="cuda"), torch.ones(k, d, device="cuda")
    assign, ws = torch.empty(n, dtype=torch.int32, device="cuda"), _dirty_ws_m(n, d, k)
    gmm.gmm_kmeans(xd, wd, md, vd, 0, assign, ws)
    torch.cuda.synchronize()
    m64 = mu.astype(np.float64)
    near = (x.astype(np.float64) @ m64.T - 0.5 * (m64 ** 2).sum(1)).argmax(1)
    assert (assign.cpu().numpy() == near).all()
    heavy = int(ws[:64].view(torch.int32)[6])
    print(f"  k-means scale {scale}: {heavy} of {n} points with many candidates", flush=True)
    assert heavy == 0


@pytest.mark.parametrize("spread", [0.0, 1.0])
def test_sample_switches_the_pass(spread):
    """n beyond the sample's threshold: one mixture whose components all overlap (the sample
    finds every point heavy), one of separate components."""
    rng = np.random.default_rng(5)
    n, d, k = (1 << 18) + 77, 8, 24
    mu = rng.normal(0.0, 0.05 + 8.0 * spread, (k, d)).astype(np.float32)
    var = rng.uniform(0.8, 1.2, (k, d)).astype(np.float32)
    wt = np.full(k, 1.0 / k, np.float32)
    x = (mu[rng.integers(0, k, n)] + rng.normal(0.0, 1.0, (n, d))).astype(np.float32)
    _check(x, (wt, mu, var), f"sample spread {spread}")


def test_weights_near_the_end_of_the_float_range():
    """A component of variance 1e-29 (its expanded-form weights pass 1e28) and a dead one."""
    w = g.custom("cw", 3000, 24, 10, 40, data_seed=8, init_seed=9)
    x, (wt, mu, var) = g.make(w)
    var = var.copy()
    var[7] = 1e-29
    wt = wt.copy()
    wt[11] = 0.0
    ref = oracle.iterate(x, wt, mu, var)
    st = gpu_estep(x, wt, mu, var, ws=_dirty_ws(3000, 24, 40))
    check_stats(st, ref, "wild")
    assert st["nk"][11] == 0.0


@pytest.mark.parametrize("weight", [0.0, np.nan])
@pytest.mark.parametrize("n", [300, 65600, (1 << 18) + 5])
def test_no_component_left(n, weight):
    """Every weight 0, or NaN as after an iteration on NaN rows: no component, so nothing to
    screen, at shared and whole workgroups and with the sample.  No point reaches a component:
    statistics 0, log-likelihood -inf, every rank empty."""
    import torch
    import paper_2606_10896_amd as gmm
    rng = np.random.default_rng(3)
    d, k, m = 20, 70, 2
    x, mu = (rng.normal(0.0, 1.0, s).astype(np.float32) for s in ((n, d), (k, d)))
    wt, var = np.full(k, weight, np.float32), np.ones((k, d), np.float32)
    st = gpu_estep(x, wt, mu, var, ws=_dirty_ws(n, d, k))
    assert st["loglik"] == -np.inf
    for a in ("nk", "s", "q"):
        assert (st[a] == 0.0).all(), a
    ws = gmm.workspace(n, d, k, m)
    ws.fill_(0xEE)
    torch.cuda.synchronize()
    idx, resp = gpu_assign(x, wt, mu, var, m, 0.1, ws=ws)
    assert (idx == -1).all() and (resp == 0.0).all()
