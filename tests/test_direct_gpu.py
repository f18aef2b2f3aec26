"""Statistics of the routed components in the direct form up to 128 dimensions
(k_stats_direct: tiles of 128 points by 32 components, fp64 MFMA) against fp64 sums, at the
edges of its tiles: points, components, dimensions, unaligned rows, tiles without any mass."""
import numpy as np
import pytest

from gmmcheck import gpu_estep

pytestmark = pytest.mark.gpu


def _exact(x, w, mu, var):
    x, w, mu, var = (a.astype(np.float64) for a in (x, w, mu, var))
    ld = np.stack([np.log(w[c]) - 0.5 * (np.log(2 * np.pi * var[c]).sum()
                                         + ((x - mu[c]) ** 2 / var[c]).sum(1))
                   for c in range(len(w))], 1)
    m = ld.max(1, keepdims=True)
    r = np.exp(ld - m)
    r /= r.sum(1, keepdims=True)
    return r


@pytest.mark.parametrize("n,d,k,routed", [
    (1, 128, 2, 1), (127, 128, 33, 31), (128, 127, 40, 32), (129, 64, 70, 33), (257, 63, 70, 65),
    (1000, 65, 9, 9), (1023, 2, 35, 33), (5000, 16, 12, 5), (4097, 100, 40, 1)])
def test_routed_components(n, d, k, routed):
    rng = np.random.default_rng(n + d + k)
    centre = rng.normal(0.0, 8.0, (4, d))
    mu = (centre[rng.integers(0, 4, k)] + rng.normal(0.0, 2e-2 / np.sqrt(d), (k, d)))
    var = np.full((k, d), 0.5)
    ill = rng.permutation(k)[:routed]
    var[ill] = rng.uniform(0.5, 2.0, (routed, 1)) * 1e-4
    mu, var = mu.astype(np.float32), var.astype(np.float32)
    w = rng.dirichlet(np.full(k, 5.0)).astype(np.float32)
    # points near the routed components (several of them hold a share), the rest far away
    x = rng.normal(0.0, 30.0, (n, d))
    near = rng.random(n) < 0.6
    x[near] = mu[ill[rng.integers(0, routed, int(near.sum()))]] + rng.normal(
        0.0, 1e-2, (int(near.sum()), d))
    x = x.astype(np.float32)
    e = (mu.astype(np.float64) ** 2 / var).sum(1)
    assert (e[ill] > 2.0e5).all() or d < 8
    r = _exact(x, w, mu, var)
    st = gpu_estep(x, w, mu, var)
    xd = x.astype(np.float64)
    # r is rounded to fp32 from log2 r, itself rounded to fp32: relative error at most
    # ln 2 * 2^-24 * 150 + 2^-22 < 2^-16 for the smallest r kept, 2^-18 from r = 2^-40 on
    tol = 2.0 ** -18
    for c in ill:
        nk, s, q = r[:, c].sum(), r[:, c] @ xd, r[:, c] @ (xd * xd)
        sa = r[:, c] @ np.abs(xd)
        floor = n * 2.0 ** -60                   # what holds less than 2^-60 may be left out
        assert abs(st["nk"][c] - nk) <= tol * nk + floor, (c, st["nk"][c], nk)
        top = np.abs(xd).max()
        assert (np.abs(st["s"][c] - s) <= tol * sa + floor * top).all(), c
        assert (np.abs(st["q"][c] - q) <= tol * q + floor * top * top).all(), c
    print(f"  routed n{n} d{d} k{k}: {routed} components, "
          f"N_k {r[:, ill].sum():.3f}", flush=True)


@pytest.mark.parametrize("d", [16, 128, 200, 300])
@pytest.mark.parametrize("place", [0, 15, 16, 38])
def test_one_light_component(d, place):
    """One component with little mass among heavy ones that overlap everywhere: its statistics are
    those of the points that the dense pass flags, once for the sixteen components of a group
    whichever of them is the light one."""
    rng = np.random.default_rng(100 * d + place)
    n, k = 4000, 39
    mu = rng.normal(0.0, 2.0 / np.sqrt(d), (k, d)).astype(np.float32)
    var = rng.uniform(0.9, 1.1, (k, d)).astype(np.float32)
    w = np.full(k, 1.0)
    w[place] = 0.02
    w = (w / w.sum()).astype(np.float32)
    x = (mu[rng.integers(0, k, n)] + rng.normal(0.0, 1.0, (n, d))).astype(np.float32)
    r = _exact(x, w, mu, var)
    mass = r.sum(0)
    assert mass[place] < 64.0 < np.delete(mass, place).min()
    st = gpu_estep(x, w, mu, var)
    xd = x.astype(np.float64)
    # log Z keeps the screening error of what is below 2^-20 of it, r is as above
    tol = 2.0 ** -16
    c = place
    assert abs(st["nk"][c] - mass[c]) <= tol * mass[c], (st["nk"][c], mass[c])
    assert (np.abs(st["s"][c] - r[:, c] @ xd) <= tol * (r[:, c] @ np.abs(xd))).all()
    assert (np.abs(st["q"][c] - r[:, c] @ (xd * xd)) <= tol * (r[:, c] @ (xd * xd))).all()
