"""Runs in parts (k_parts) whose parts are not on the device together, forced from the host: one part
comes late, and another takes its channel over; bitwise the run of all parts.
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
