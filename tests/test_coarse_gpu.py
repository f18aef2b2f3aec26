"""The one-product screening of the E-step (k_coarse, k_refine and the points it hands to
k_logz) against the fp64 checker, at the edges of its tiles and of its rules: workgroups of
128 and 256 points, blocks of 32 components, widths with and without a remainder, points with
more components in reach than a list or a lane state holds, the sample that switches the pass
off, and weights near the end of the float range.  The workspace starts as garbage, so a point
that no kernel wrote would show."""
import numpy as np
import pytest

import gmm_synth as g
import oracle
from gmmcheck import (check_params, check_params_iso, check_stats, gpu_estep, gpu_estep_iso,
                      gpu_mstep, gpu_mstep_iso)

pytestmark = pytest.mark.gpu


def _dirty_ws(n, d, k):
    import torch
    import paper_2606_10896_amd as gmm
    ws = gmm.workspace(n, d, k)
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
    (300, 2, 9), (64, 1, 3), (2000, 100, 257)])
def test_tile_edges(n, d, k):
    w = g.custom(f"c{n}_{d}_{k}", n, d, max(2, k // 2), k, data_seed=n * 3 + d, init_seed=k)
    x, th0 = g.make(w)
    for t, th in enumerate(oracle.fit(x, *th0, 3, keep_thetas=True)["thetas"]):
        _check(x, th, f"n{n} d{d} k{k} t{t}")


@pytest.mark.parametrize("n,d,k", [(255, 64, 33), (257, 100, 64), (700, 128, 97),
                                   (300, 190, 40), (129, 250, 32)])
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


@pytest.mark.parametrize("d,seed", [(16, 1), (96, 2), (128, 3), (200, 4)])
def test_many_components_in_reach(d, seed):
    """Clusters of 1 to 14 near-identical components, scattered over the slots: points whose
    candidates overflow the list, or one lane state of either lane half only."""
    rng = np.random.default_rng(seed)
    sizes = np.tile(np.arange(1, 15), 6)
    k = int(sizes.sum())
    cl = np.repeat(np.arange(sizes.size), sizes)
    order = rng.permutation(k)
    centre = rng.normal(0.0, 4.0, (sizes.size, d))
    mu = (centre[cl] + rng.normal(0.0, 0.02, (k, d)))[order].astype(np.float32)
    var = rng.uniform(0.5, 1.5, (k, d)).astype(np.float32) * 0 + np.float32(1.0)
    wt = rng.dirichlet(np.full(k, 5.0)).astype(np.float32)
    n = 6000
    x = (centre[rng.integers(0, sizes.size, n)] + rng.normal(0.0, 1.0, (n, d))).astype(np.float32)
    _check(x, (wt, mu, var), f"reach d{d}")


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
