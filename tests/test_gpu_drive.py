"""Models driven together against one at a time, bit for bit: one and more
tables of models, frames and slices that differ between them, the MLP sizes
that hold their weights in registers and one that does not."""
import numpy as np
import pytest

from paper_2503_12886_amd import gbr
from gpu_util import dev, host, make_ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_in,hidden", [(56, 256), (100, 40)])
@pytest.mark.parametrize("count", [1, 2, 16, 17, 35])
def test_drive(count, d_in, hidden):
    import torch
    rng = np.random.default_rng(count + d_in)
    ctx = make_ctx()
    groups, refs = [], []
    for i in range(count):
        K, B, N = [1, 7, 20, 40, 63][i % 5], 1 + i % 3, [1, 15, 16, 17, 1000, 33][i % 6]
        n = hidden * d_in + hidden + hidden * hidden + hidden + K * hidden + K
        mlp = dev(rng.normal(size=n).astype(np.float32) * 0.1)
        theta = dev(rng.normal(size=(B, d_in)).astype(np.float32))
        bases = dev(rng.normal(size=(K + 1, N, 16)).astype(np.float32))
        psi, raw = torch.full((B, K), np.nan, device="cuda"), torch.full((B, N, 16), np.nan, device="cuda")
        gbr.gbr_mlp_forward(ctx, mlp, theta, d_in, hidden, K, psi)
        gbr.gbr_blend(ctx, bases, psi, raw)
        refs.append((host(psi), host(raw)))
        groups.append((mlp, theta, bases, torch.full_like(psi, np.nan), torch.full_like(raw, np.nan)))
    gbr.gbr_drive(ctx, groups, d_in, hidden)
    for i, ((_, _, _, psi, raw), (p, r)) in enumerate(zip(groups, refs)):
        assert (host(psi) == p).all() and (host(raw) == r).all(), i
    ctx.close()


def test_refused():
    import torch
    ctx = make_ctx(max_frames=2)
    f = lambda *s: torch.zeros(*s, device="cuda")
    n = 8 * 4 + 8 + 8 * 8 + 8 + 2 * 8 + 2
    ok = (f(n), f(1, 4), f(3, 5, 16), f(1, 2), f(1, 5, 16))
    gbr.gbr_drive(ctx, [ok], 4, 8)
    with pytest.raises(ValueError):
        gbr.gbr_drive(ctx, [ok, (f(n), f(1, 4), f(3, 5, 16), f(1, 3), f(1, 5, 16))], 4, 8)
    with pytest.raises(gbr.GbrError):
        gbr.gbr_drive(ctx, [], 4, 8)
    with pytest.raises(gbr.GbrError):
        gbr.gbr_drive(ctx, [(f(n), f(3, 4), f(3, 5, 16), f(3, 2), f(3, 5, 16))], 4, 8)   # more frames than the context's
    ctx.close()
