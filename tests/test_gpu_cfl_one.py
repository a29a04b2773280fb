"""cfl_reduce in one launch (k_cfl_one) on the MI355X: sizes at the edges of a lane's cells, of a
workgroup's and of the full grid; a second call on the same context.  The maximum is exact, so it equals
the larger of the maxima of two parts of the channel bit for bit; dt = CFL dx / amax, one division.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dsve():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1912_04791_amd import dsve as d
    return d


def amax_dt(ctx, h, q):
    import torch
    out = torch.zeros(2, dtype=torch.float64, device="cuda")
    ctx.cfl_reduce(h, q, torch.zeros_like(h), out[:1], out[1:])
    ctx.sync()
    return tuple(float(v) for v in out)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 256, 257, 2047, 2048, 2049, 512 * 2048 - 1, 512 * 2048 + 1,
                               3_000_001])
def test_maximum_of_the_parts(dsve, n, precision):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(n)
    h = 0.5 + 2.0 * torch.rand(n, generator=gen, device="cuda", dtype=torch.float64)
    q = h * (2.0 * torch.rand(n, generator=gen, device="cuda", dtype=torch.float64) - 1.0)
    kw = dict(porosity=0.4, A_g=0.01, dx=0.5, cfl=0.8, precision=precision)
    ctx = dsve.Context.single(n, **kw)
    got = amax_dt(ctx, h, q)
    assert got[1] == 0.8 * 0.5 / got[0]
    if n > 1:
        parts = []
        for a, b in ((0, n // 2), (n // 2, n)):
            sub = dsve.Context.single(b - a, **kw)
            parts.append(amax_dt(sub, h[a:b].contiguous(), q[a:b].contiguous())[0])
            sub.close()
        assert got[0] == max(parts)
    # the fastest cell last, then a slower state: nothing of the call before stays behind
    q2 = q.clone()
    q2[n - 1] = 9.0 * h[n - 1]
    assert amax_dt(ctx, h, q2)[0] > 9.0
    assert amax_dt(ctx, h, q) == got
    ctx.close()
