"""Runs in parts (k_parts) whose parts are not on the device together, forced from the host: one part
comes late, and another takes its channel over, bitwise the run of all parts; or one leaves between two
steps, and the run ends with an error, its arrays as they were.
"""
import ctypes

import pytest

from paper_1912_04791_amd import inputs

from test_gpu_parts import run, same
from test_gpu_segments import channels

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dsve():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1912_04791_amd import dsve as d
    return d


def hold(dsve, ctx, part, step=0, wait_us=2000):
    f = dsve.lib.dsve_test_hold_part
    f.argtypes = [ctypes.c_void_p] + [ctypes.c_int] * 3
    assert f(ctx._h, part, step, wait_us) == 0


def held_run(dsve, wl, part, n_steps, precision="fp64", solver="adot"):
    ctx = dsve.Context.from_workload(wl, precision=precision, solver=solver)
    h, q, z, t = dsve.upload(wl)
    hold(dsve, ctx, part)
    for n in n_steps:
        ctx.adot_step(h, q, z, n, t)
        ctx.sync()
        assert ctx.last_run() == (0, 0, 1)
    out = tuple(x.cpu().numpy() for x in (h, q, z, t))
    ctx.close()
    return out


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("part", [0, 1])
@pytest.mark.parametrize("lengths", [
    [256, 504, 511, 330, 505],            # every kind of end; 8 waves of 63 cells and one cell more
    [512, 1, 63, 700, 126, 880, 1009],    # with channels of one workgroup, which never wait
])
def test_a_late_part(dsve, lengths, part, precision):
    wl = channels(lengths, seed=sum(lengths), steps=27)
    ref = run(dsve, wl, precision, per_step=True)
    assert same(held_run(dsve, wl, part, [27], precision), ref)
    assert same(held_run(dsve, wl, part, [1, 2, 24], precision), ref)


@pytest.mark.parametrize("G", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("solver", ["adot", "dot"])
def test_a_late_part_of_each_kernel(dsve, G, solver):
    wl = inputs.make_c1(n_cells=700, steps=12)
    wl.n_gauss = G
    assert same(held_run(dsve, wl, 1, [5, 7], solver=solver), run(dsve, wl, solver=solver, per_step=True))


@pytest.mark.parametrize("name,n_cells", [("soni", 1500), ("mpm", 900), ("vanrijn", 300), ("c3", 7040)])
def test_a_late_part_with_laws_and_friction(dsve, name, n_cells):
    wl = (inputs.make_soni(n_channels=1, n_cells=n_cells, steps=15) if name == "soni"
          else inputs.make_c3(n_cells=n_cells, steps=15) if name == "c3"
          else inputs.make_bellal(name, n_channels=1, n_cells=n_cells, steps=15))
    assert same(held_run(dsve, wl, 2, [8, 7]), run(dsve, wl, per_step=True))


def test_more_launches_than_the_device_takes_whole(dsve):
    # twelve streams with a run of 64 parts each: none waits for ever, each as if alone
    import torch
    wl = inputs.make_c1(n_cells=64 * 110, steps=40)
    ref = run(dsve, wl, per_step=True)
    streams = [torch.cuda.Stream() for _ in range(12)]
    ctxs = [dsve.Context.from_workload(wl, stream=s) for s in streams]
    states = [dsve.upload(wl) for _ in streams]
    torch.cuda.synchronize()
    for c, (h, q, z, t) in zip(ctxs, states):
        c.adot_step(h, q, z, wl.steps, t)
    for c, st in zip(ctxs, states):
        c.sync()
        assert same(tuple(x.cpu().numpy() for x in st), ref)
        c.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("step", [1, 7, 8, 16, 19])     # before a maximum, and (8, 16) before cells of a neighbour
def test_a_part_that_stops_answering(dsve, step, precision):
    import numpy as np
    wl = channels([700, 100, 880], seed=3, steps=20)
    ctx = dsve.Context.from_workload(wl, precision=precision)
    h, q, z, t = dsve.upload(wl)
    before = [x.cpu().numpy() for x in (h, q, z, t)]
    hold(dsve, ctx, 1, step)
    ctx.adot_step(h, q, z, wl.steps, t)
    with pytest.raises(dsve.DsveError) as ex:
        ctx.sync()
    assert ex.value.status == dsve.E_HIP and "did not answer" in str(ex.value)
    after = [x.cpu().numpy() for x in (h, q, z, t)]
    # the channel of one workgroup has run, the others are as they were
    ref = run(dsve, wl, precision, per_step=True)
    for a, b, r in zip(after[:3], before[:3], ref[:3]):
        want = b.copy()
        want[700:800] = r[700:800]
        assert np.array_equal(a, want)
    assert np.array_equal(after[3], [before[3][0], ref[3][1], before[3][2]])
    # and the context goes on when the error is cleared
    hold(dsve, ctx, -1)
    ctx.clear_error()
    h, q, z, t = dsve.upload(wl)
    ctx.adot_step(h, q, z, wl.steps, t)
    ctx.sync()
    assert same([x.cpu().numpy() for x in (h, q, z, t)], ref)
    ctx.close()
