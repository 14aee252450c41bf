"""The compositing of few tiles by three waves a quadrant against the one-wave
form, bit for bit: the same frames rendered one at a time (few tiles) and in a
batch with a frame of many tiles.  Lists around a step's 32 and a batch's 64
candidates, quadrants that stop inside a step, frames that leave part of their
tiles empty, frames without a visible splat."""
import numpy as np
import pytest

from paper_2503_12886_amd import gbr, synth
from gpu_util import dev, host, make_ctx, render
from test_gpu_list_stream import faint_pile

pytestmark = pytest.mark.gpu


def frames():
    out = []
    for n in (8, 31, 32, 33, 63, 64, 65, 97, 700):
        out.append((16, 16, faint_pile(n, n)))
    dense = faint_pile(300, 1)
    dense[:, 10] += 4.0                              # stops inside the first steps
    out.append((21, 13, dense))
    mixed = faint_pile(500, 2)
    mixed[:, 0:2] *= 60.0
    mixed[:, 7:10] -= 2.0
    mixed[:, 10] += np.where(np.arange(500) % 5 == 0, 4.0, 0.0).astype(np.float32)
    out.append((50, 34, mixed))
    behind = faint_pile(64, 3)
    behind[:, 2] -= 2.0
    out.append((16, 16, behind))
    out.append((100, 70, synth.make_scene(3000, 0, seed=4)[0]))
    return out


def run(ctx, fs):
    """Images, per-pixel stop positions and gradients of the frames in one batch."""
    import torch
    cams = [synth.fixed_camera(w, h, 1.17 * w, 0.5, bg=(0.2, 0.3, 0.4)) for w, h, _ in fs]
    off = np.concatenate([[0], np.cumsum([r.shape[0] for _, _, r in fs])]).tolist()
    imgs, kept, images = render(ctx, np.concatenate([r for _, _, r in fs]), cams, off)
    nit = gbr.gbr_inspect(ctx, "n_iter", sum(w * h for w, h, _ in fs))
    dimg = [np.random.default_rng(w + r.shape[0]).normal(size=3 * w * h).astype(np.float32) for w, h, r in fs]
    draw = torch.empty(off[-1] * 16, device="cuda")
    gbr.gbr_render_backward(ctx, dev(np.concatenate(dimg)), draw)
    d = host(draw).reshape(-1, 16)
    del kept, images
    return imgs, nit, [d[off[i]:off[i + 1]] for i in range(len(fs))]


def test_same_bits():
    fs = frames()
    ctx = make_ctx(max_pixels=1 << 19, max_entries=1 << 22)
    many = (592, 592, synth.make_scene(50, 0, seed=9)[0])     # 37 x 37 tiles
    imgs, nit, draws = run(ctx, fs + [many])
    p = 0
    for i, f in enumerate(fs):
        one, n1, d1 = run(ctx, [f])
        assert (one[0] == imgs[i]).all(), i
        assert (n1 == nit[p:p + f[0] * f[1]]).all(), i
        assert (d1[0] == draws[i]).all(), i
        p += f[0] * f[1]
    assert (imgs[8] != imgs[8][:, :1, :1]).any()              # something was drawn
    ctx.close()
