"""Runs of few channels in one launch (k_parts) on the MI355X: channels of one workgroup and channels
cut into parts, at the lengths where the number of waves or parts changes, every kind of end, every
number of quadrature nodes; bitwise the per-step kernels, and the oracle to the FP64 and mixed bars
(relative L1 1e-12 and 1e-5).
"""
import numpy as np
import pytest

from paper_1912_04791_amd import inputs

from common import oracle_run, per_channel_rel_l1
from test_gpu_segments import channels

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dsve():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1912_04791_amd import dsve as d
    return d


def run(dsve, wl, precision="fp64", solver="adot", per_step=False, splits=None, noalloc=False):
    ctx = dsve.Context.from_workload(wl, precision=precision, solver=solver)
    if per_step:
        ctx.set_resident(1)
    h, q, z, t = dsve.upload(wl)
    for n in splits or [wl.steps]:
        (ctx.adot_step_noalloc if noalloc else ctx.adot_step)(h, q, z, n, t)
        ctx.sync()
        if not per_step:
            assert ctx.last_run() == (0, 0, 1)
    out = tuple(x.cpu().numpy() for x in (h, q, z, t))
    ctx.close()
    return out


def same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("mixed", 1e-5)])
@pytest.mark.parametrize("lengths", [
    [1, 2, 62, 63, 64, 65, 125, 126] * 3,               # one workgroup each
    [127, 128, 219, 220, 221, 256, 330, 511],           # parts of short channels
    [512, 1, 63, 700, 126, 127, 880],                   # both, longer than 511 cells among them
])
def test_lengths_and_ends(dsve, lengths, precision, tol):
    wl = channels(lengths, seed=sum(lengths), steps=27)
    got = run(dsve, wl, precision)
    assert same(got, run(dsve, wl, precision, per_step=True))
    assert same(got, run(dsve, wl, precision, splits=[1, 8, 7, 11]))
    assert same(got, run(dsve, wl, precision, noalloc=True))
    want = oracle_run(wl)
    assert per_channel_rel_l1(got, want, wl.offsets).max() <= tol
    np.testing.assert_allclose(got[3], want[3], rtol=1e-12 if precision == "fp64" else 1e-6)


@pytest.mark.parametrize("G", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("precision,solver", [("fp64", "adot"), ("mixed", "adot"), ("fp64", "dot")])
def test_quadrature_nodes_and_solvers(dsve, G, precision, solver):
    # each G has its own number of waves per role and cells per part
    for n_cells in (40, 700):
        wl = inputs.make_c1(n_cells=n_cells, steps=21)
        wl.n_gauss = G
        assert same(run(dsve, wl, precision, solver), run(dsve, wl, precision, solver, per_step=True))


@pytest.mark.parametrize("name,n_cells", [("soni", 1500), ("mpm", 900), ("vanrijn", 300), ("thr", 64), ("c3", 3000)])
def test_laws_friction_and_turning_flow(dsve, name, n_cells):
    wl = (inputs.make_soni(n_channels=1, n_cells=n_cells, steps=30) if name == "soni"
          else inputs.make_c3(n_cells=n_cells, steps=30) if name == "c3"
          else inputs.make_bellal(name, n_channels=1, n_cells=n_cells, steps=30))
    wl.q[n_cells // 2:] *= -0.5      # flow towards one another: edges where it changes direction
    got = run(dsve, wl, "fp64")
    assert same(got, run(dsve, wl, "fp64", per_step=True))
    assert per_channel_rel_l1(got, oracle_run(wl), wl.offsets).max() <= 1e-12


def test_largest_context_in_parts_and_the_next(dsve):
    # 64 parts of 110 cells; one cell more goes to the per-step kernels
    for n_cells, one in ((64 * 110, True), (64 * 110 + 1, False)):
        wl = inputs.make_c2(n_cells=n_cells, steps=19, length=1000.0 * n_cells / (1 << 20), max_mode=8)
        ctx = dsve.Context.from_workload(wl)
        h, q, z, t = dsve.upload(wl)
        ctx.adot_step(h, q, z, wl.steps, t)
        ctx.sync()
        assert (ctx.last_run() == (0, 0, 1)) == one
        got = tuple(x.cpu().numpy() for x in (h, q, z, t))
        ctx.close()
        assert same(got, run(dsve, wl, per_step=True))


def test_two_streams_at_once(dsve):
    # runs in parts on two streams, enqueued together, each as if alone
    import torch
    wl = inputs.make_c1(n_cells=2000, steps=60)
    ref = run(dsve, wl, per_step=True)
    streams = [torch.cuda.Stream() for _ in range(2)]
    ctxs = [dsve.Context.from_workload(wl, stream=s) for s in streams]
    states = [dsve.upload(wl) for _ in streams]
    torch.cuda.synchronize()
    for c, (h, q, z, t) in zip(ctxs, states):
        c.adot_step(h, q, z, wl.steps, t)
    for c, st in zip(ctxs, states):
        c.sync()
        assert same(tuple(x.cpu().numpy() for x in st), ref)
        c.close()
