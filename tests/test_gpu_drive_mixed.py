"""Models of very different numbers of slices driven together: each is blended as
on its own.  An infinite value in a model's last slice shows it: blended among
more slices than the model has, it would meet weights of 0 and turn to NaN."""
import numpy as np
import pytest

from paper_2503_12886_amd import gbr
from gpu_util import dev, host, make_ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("slices", [(7, 63), (63, 7, 15, 7, 31), (1, 8, 16, 24, 32, 40, 48, 56, 63, 7, 15, 23, 31, 39, 47, 55, 7)])
def test_mixed(slices):
    import torch
    rng = np.random.default_rng(len(slices))
    ctx = make_ctx()
    groups, refs = [], []
    for i, K in enumerate(slices):
        B, N = 1 + i % 2, [100, 17, 1000][i % 3]
        mlp = dev(rng.normal(size=gbr.mlp_params(56, 256, K)).astype(np.float32) * 0.1)
        theta = dev(rng.normal(size=(B, 56)).astype(np.float32))
        bases = rng.normal(size=(K + 1, N, 16)).astype(np.float32)
        bases[K, N // 2, :7] = np.inf
        bases = dev(bases)
        psi, raw = torch.full((B, K), np.nan, device="cuda"), torch.full((B, N, 16), np.nan, device="cuda")
        gbr.gbr_mlp_forward(ctx, mlp, theta, 56, 256, K, psi)
        gbr.gbr_blend(ctx, bases, psi, raw)
        refs.append((host(psi), host(raw)))
        assert np.isinf(refs[-1][1]).any() or K % 8 != 7
        groups.append((mlp, theta, bases, torch.full_like(psi, np.nan), torch.full_like(raw, np.nan)))
    gbr.gbr_drive(ctx, groups, 56, 256)
    for i, ((_, _, _, psi, raw), (p, r)) in enumerate(zip(groups, refs)):
        assert np.array_equal(host(psi), p) and np.array_equal(host(raw), r, equal_nan=True), (i, slices[i])
    ctx.close()


@pytest.mark.parametrize("N", [1 << 36, (1 << 37) + 1, 1 << 40, (1 << 62) + 5])
def test_sizes_beyond_a_grid_are_refused(N):
    """More workgroups than a grid has: an error before anything is launched."""
    import torch
    ctx = make_ctx(max_frames=2)
    t = torch.zeros(1 << 17, device="cuda")
    p = t.data_ptr()
    g = (gbr.gbr_drive_group * 2)(gbr.gbr_drive_group(p, p, p, p, p, 5, 1, 2), gbr.gbr_drive_group(p, p, p, p, p, N, 1, 2))
    with pytest.raises(gbr.GbrError) as e:
        gbr.gbr_drive(ctx, g, 4, 8)
    assert e.value.code == -1
    ctx.close()
