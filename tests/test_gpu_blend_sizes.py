"""The blend, its adjoint and the fused update at the edges of their slice and
frame tiles, and a size whose dweights waves take several spans, against
float64 sums.  Bounds: the blend is the float64 sum rounded once; dbases and
dweights meet at most 17 + ceil(B / 16) and 290 roundings per term, so they
are within gamma_d of their terms' magnitudes (Higham, section 3.1)."""
import numpy as np
import pytest

from paper_2503_12886_amd import gbr
from paper_2503_12886_amd.trainer import bases_lr_table
from gpu_util import U32, make_ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,B,N", [(1, 1, 1), (7, 2, 33), (8, 16, 65), (15, 17, 64), (16, 3, 100), (23, 32, 50),
                                   (24, 33, 31), (31, 5, 77), (32, 48, 20), (39, 49, 33), (40, 64, 17), (47, 7, 40),
                                   (48, 1, 50), (63, 64, 70), (20, 2, 66_001)])
def test_sizes(K, B, N):
    import torch
    g = torch.Generator(device="cuda").manual_seed(K * 100 + B)
    bases = torch.randn(K + 1, N, 16, generator=g, device="cuda")
    bases[..., 14:] = 0.0
    w = torch.rand(B, K, generator=g, device="cuda") * 2 - 0.5
    draw = torch.randn(B, N, 16, generator=g, device="cuda")
    draw[..., 14:] = 0.0
    ctx = make_ctx()
    W = torch.cat([torch.ones(B, 1, device="cuda"), w], 1).double()
    b64, d64 = bases.double().reshape(K + 1, -1), draw.double().reshape(B, -1)

    raw = torch.full((B, N, 16), float("nan"), device="cuda")
    gbr.gbr_blend(ctx, bases, w, raw)
    ref = (W @ b64).reshape(B, N, 16)
    lo = torch.nextafter(ref.float(), torch.full_like(raw, -torch.inf))
    hi = torch.nextafter(ref.float(), torch.full_like(raw, torch.inf))
    assert bool(((raw >= lo) & (raw <= hi)).all())
    assert float((raw != ref.float()).double().mean()) < 1e-4 + 2.0 / raw.numel()

    dbases = torch.full_like(bases, float("nan"))
    dw = torch.full((B, K), float("nan"), device="cuda")
    gbr.gbr_blend_backward(ctx, draw, bases, w, dbases, dw)
    gam = lambda d: d * U32 / (1 - d * U32)
    db_ref, db_mag = (W.t() @ d64).reshape(bases.shape), (W.abs().t() @ d64.abs()).reshape(bases.shape)
    assert bool(((dbases - db_ref).abs() <= gam(17 + -(-B // 16)) * db_mag).all())
    dw_ref, dw_mag = d64 @ b64[1:].t(), d64.abs() @ b64[1:].abs().t()
    assert bool(((dw - dw_ref).abs() <= gam(290) * dw_mag).all())

    # the fused update is the two-step one, bit for bit
    lr = bases_lr_table()
    states = [[bases.clone(), torch.rand(bases.shape, generator=g, device="cuda")] for _ in range(2)]
    m, v = states[0][1] * 1e-3, states[0][1] * 1e-4
    one = [bases.clone(), m.clone(), v.clone()]
    two = [bases.clone(), m.clone(), v.clone()]
    gbr.gbr_blend_adam_step(ctx, 0, draw, w, *one, lr)
    gbr.gbr_adam_step(ctx, 1, two[0], dbases, two[1], two[2], N * 16, lr)
    assert all(np.array_equal(a.cpu().numpy(), b.cpu().numpy()) for a, b in zip(one, two))
    ctx.close()
