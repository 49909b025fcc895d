"""The single-block list building for few entries and the single-block tile order
against the general path (a large on-device capacity takes it): the same image,
state and gradients to the last bit, at the edges of both rules."""
import pytest
import torch

import workloads as W
from tests.gpu_helpers import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,w,h", [(1, 16, 16), (3, 17, 1), (64, 40, 40), (257, 128, 128), (300, 250, 260),
                                   (900, 256, 256), (900, 272, 256), (2500, 128, 128), (1500, 720, 728),
                                   (300, 1024, 512), (300, 1040, 512)])
def test_small_lists_equal_the_general_path(n, w, h):
    """One tile, ragged tiles, 256 and 272 tiles (one or two digits), 2048 and 2080
    tiles, and entry counts on both sides of 16384; the count from the host and,
    with the smallest capacity that holds it, from the device."""
    import paper_2512_11800_amd as M
    g = M.Gaussians.from_scene(W.uniform_scene(n, seed=n, extent=0.3, log_scale_mean=-3.0))
    cams, opts = [W.camera_on_axis(2.0, w, h)], W.Options()
    img, saved, st = M.render_forward(g, cams, opts, ws=M.Workspace())
    log(f"[lists] n {n} {w}x{h}: {st.n_entries} entries")
    gi = torch.randn(img.shape, generator=torch.Generator().manual_seed(n)).cuda()
    grads = M.render_backward(g, cams, opts, st, saved, gi)
    for cap in (1, 200_000):
        ws = M.Workspace()
        ws.capacity = max(cap, st.n_entries)
        img2, saved2, st2 = M.render_forward(g, cams, opts, ws=ws, on_device=True)
        assert torch.equal(img, img2) and torch.equal(saved, saved2)
        grads2 = M.render_backward(g, cams, opts, st2, saved2, gi)
        st2.check()
        assert all(torch.equal(grads[k], grads2[k]) for k in grads)


@pytest.mark.parametrize("w,h", [(2048, 2048), (2064, 2048)])
def test_every_tile_is_rendered_once(w, h):
    """16384 and 16512 tiles: with full coverage each pixel counts every Gaussian."""
    import paper_2512_11800_amd as M
    g = M.Gaussians.from_scene(W.uniform_scene(3, seed=5, extent=0.3))
    _, saved, _ = M.render_forward(g, [W.camera_on_axis(2.0, w, h)], W.Options(full_coverage=True))
    c = saved[..., 7]
    assert torch.equal(torch.where(c < 0, -c - 1, c), torch.full_like(c, 3.0))
