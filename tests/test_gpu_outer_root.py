"""The FP64 fluctuation from one refined root per node (fluct64) on the MI355X, at the edges of its
cases: flow one way, the other, changing sign along the path, at rest at one end; close to coalescing
roots (on both sides of the band left to the general path); past abs(Fr) = 3, where the arccos argument
changes sign; depths beyond the range of its FP32 estimate.

Per edge, relative to the edge's own fluctuations, against the oracle.  Tolerance 1e-12: FP64 rounding
(2^-53) of a root grows with its sensitivity, at most 1 / (1 - x) = 400 here (A_g >= 1e-4), in the
kernel and in the oracle: 1e-13, times ten for the few roundings each takes.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

TOL = 1e-12
KINDS = ["up", "down", "turning", "one end at rest", "near critical", "fast", "tiny", "huge"]


@pytest.fixture(scope="module")
def dsve():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1912_04791_amd import dsve as d
    return d


def edges(kind, n, seed):
    rng = np.random.default_rng(seed)
    h = rng.uniform(0.3, 3.0, n)
    fr = rng.uniform(0.02, 0.9, n)
    sign = rng.choice([-1.0, 1.0], n)
    if kind == "up":
        sign[:] = 1.0
    elif kind == "down":
        sign[:] = -1.0
    elif kind == "near critical":
        fr = rng.uniform(0.9, 1.1, n)
    elif kind == "fast":
        fr = rng.uniform(2.0, 9.0, n)
    elif kind == "tiny":
        h *= 1e-30
    elif kind == "huge":
        h *= 1e30
    c = np.sqrt(9.81 * h)
    u = sign * fr * c
    hR = h * (1 + 0.05 * rng.uniform(-1, 1, n))
    uR = u * (1 + 0.05 * rng.uniform(-1, 1, n))
    if kind == "turning":
        uR = -u * rng.uniform(0.01, 3.0, n)
    elif kind == "one end at rest":
        swap = rng.random(n) < 0.5
        u, uR = np.where(swap, 0.0, u), np.where(swap, u, 0.0)
    z = 0.1 * h * rng.uniform(-1, 1, n)
    zR = z + 0.02 * h * rng.uniform(-1, 1, n)
    return (h, h * u, z), (hR, hR * uR, zR)


def fluct(dsve, WL, WR, A_g, G):
    import torch
    n = WL[0].size
    ctx = dsve.Context.single(16, porosity=0.4, A_g=A_g, n_gauss=G, dx=1.0)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (*WL, *WR)]
    Dm = torch.zeros(3, n, dtype=torch.float64, device="cuda")
    Dp = torch.zeros_like(Dm)
    ctx.dot_edge_fluct(*dev, Dm, Dp)
    ctx.sync()
    ctx.close()
    return Dm.cpu().numpy(), Dp.cpu().numpy()


@pytest.mark.parametrize("G", [1, 2, 3, 5])
@pytest.mark.parametrize("A_g", [0.05, 1e-4])
def test_every_kind_of_edge_alone_and_mixed(dsve, G, A_g):
    # each kind in waves of its own, then all kinds shuffled into the same waves: the same bits
    n = 64 * 40
    parts = [edges(k, n, 10 * G + i) for i, k in enumerate(KINDS)]
    WL = tuple(np.concatenate([p[0][r] for p in parts]) for r in range(3))
    WR = tuple(np.concatenate([p[1][r] for p in parts]) for r in range(3))
    gm, gp = fluct(dsve, WL, WR, A_g, G)
    perm = np.random.default_rng(G).permutation(n * len(KINDS))
    sm, sp = fluct(dsve, tuple(a[perm] for a in WL), tuple(a[perm] for a in WR), A_g, G)
    assert np.array_equal(sm, gm[:, perm]) and np.array_equal(sp, gp[:, perm])
    # the Grass law scales with the depth: the oracle takes tiny and huge edges at (h, z) / s, q / s^1.5
    for i, kind in enumerate(KINDS):
        s = slice(i * n, (i + 1) * n)
        sc = {"tiny": 1e-30, "huge": 1e30}.get(kind, 1.0)
        f = np.array([1.0, np.sqrt(sc), 1.0])[:, None] * np.sqrt(sc) * sc
        L, R = (tuple(a[s] / (sc, sc * np.sqrt(sc), sc)[r] for r, a in enumerate(W)) for W in (WL, WR))
        rm, rp = oracle.fluct(L, R, 9.81, 1.0 / 0.6, A_g, G=G)
        size = np.abs(rm).max(axis=0) + np.abs(rp).max(axis=0)
        for got, ref in ((gm[:, s] / f, rm), (gp[:, s] / f, rp)):
            assert (np.abs(got - ref).max(axis=0) / size).max() <= TOL, kind


@pytest.mark.parametrize("G", [1, 3, 5])
def test_an_end_below_the_range_of_the_estimate(dsve, G):
    # the nodes are within the range, one end of the path is not (a dry side): the same bound
    rng = np.random.default_rng(G)
    n = 64 * 5
    h = rng.uniform(0.3, 3.0, n)
    q = rng.uniform(0.02, 0.25, n) * np.sqrt(9.81 * h) * h
    wet, dry = (h, q, 0.1 * h), (np.full(n, 1e-25), np.zeros(n), 0.2 * h)
    flip = rng.random(n) < 0.5
    WL = tuple(np.where(flip, a, b) for a, b in zip(wet, dry))
    WR = tuple(np.where(flip, b, a) for a, b in zip(wet, dry))
    gm, gp = fluct(dsve, WL, WR, 0.05, G)
    rm, rp = oracle.fluct(WL, WR, 9.81, 1.0 / 0.6, 0.05, G=G)
    size = np.abs(rm).max(axis=0) + np.abs(rp).max(axis=0)
    for got, ref in ((gm, rm), (gp, rp)):
        assert (np.abs(got - ref).max(axis=0) / size).max() <= TOL
