"""A run that the caller captured into a graph, replayed after the context was given another launch, with
eager runs of the context in between: bitwise the eager run each time (MI355X).
"""
import numpy as np
import pytest

from paper_1912_04791_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dsve():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1912_04791_amd import dsve as d
    return d


@pytest.mark.parametrize("shape", [dict(n_channels=9, len_lo=600, len_hi=9000),      # segments
                                   dict(n_channels=400, len_lo=8, len_hi=120)])      # the packed kernel's tiles
def test_replays_after_another_launch(dsve, shape):
    import torch
    wl = inputs.make_c4(steps=14, **shape)
    stream = torch.cuda.Stream()
    ctx = dsve.Context.from_workload(wl, stream=stream)
    ctx.set_resident(1)
    first = dsve.upload(wl)
    state = [x.clone() for x in first]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        ctx.adot_step_noalloc(*state[:3], wl.steps, state[3])

    def eager():
        with torch.cuda.stream(stream):
            own = [x.clone() for x in first]
            ctx.adot_step(*own[:3], wl.steps, own[3])
        ctx.sync()
        return [x.cpu().numpy() for x in own]

    want = eager()
    for launch in [(64, 1, 6), (128, 3, 0), (256, 2, 60)]:
        ctx.set_launch(*launch)
        assert all(np.array_equal(a, b) for a, b in zip(eager(), want))
        for s, f in zip(state, first):
            s.copy_(f)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(np.array_equal(s.cpu().numpy(), w) for s, w in zip(state, want)), launch
    ctx.close()


def test_a_long_first_run_under_capture(dsve):
    # 330 steps: a first run of that length replays graphs of its own, but for under capture
    import torch
    wl = inputs.make_c2(n_cells=9000, steps=330, length=1000.0 * 9000 / (1 << 20))
    stream = torch.cuda.Stream()
    ctx = dsve.Context.from_workload(wl, stream=stream)
    first = dsve.upload(wl)
    state = [x.clone() for x in first]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        ctx.adot_step(*state[:3], wl.steps, state[3])
    assert ctx.last_run() == (0, 0, wl.steps)
    for _ in range(3):
        with torch.cuda.stream(stream):
            own = [x.clone() for x in first]
            ctx.adot_step(*own[:3], wl.steps, own[3])
        ctx.sync()
        for s, f in zip(state, first):
            s.copy_(f)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(s, o) for s, o in zip(state, own))
    ctx.close()
